// bf16 MFMA GEMM for the block's linear layers (App. B: the projection and MLP terms):
//   out[m, n] = epilogue( sum_k A[m, k] * W[n, k] + bias[n] ),  fp32 accumulation.
// A is the activation matrix [M, K] (row-major, bf16); W is a linear weight stored
// [out_features, in_features] inside the block's weight blob, so both operands are
// K-contiguous and one launch can cover any panel [n0, n1) of output features -- the unit
// in which streamed weights become usable chunk by chunk (Sec. 3.2).
//
// Tiling: a workgroup of 4 waves owns a BM x BN output tile; each wave owns a
// (BM/2) x (BN/2) quadrant built from 32x32x16 bf16 MFMAs.  The MFMA "A" operand is the
// weight fragment and the "B" operand the activation fragment, so an accumulator lane holds
// one token row and 4 consecutive output features per register quad: epilogues then load
// bias/gate and store results 4 features at a time.  K is consumed in slabs of 64 that are
// copied global -> LDS directly (no register staging) into two stages; 16-byte chunks of each
// 128-byte LDS row are XOR-swizzled so that the fragment reads of consecutive rows spread over
// all banks.
//
// What bounds the loop is the rate at which a CU's L1 takes in the operands (32 bytes per clock at the
// matrix cores' full rate on the 256 x 256 tile, against some 38 that the path moves with nothing else to
// do), so the copies have to be on their way all the time and evenly.  A slab is therefore worked off
// in four quadrant phases, (activation half, weight half) = (0,0) (0,1) (1,1) (1,0) (six where the
// activations go in thirds): each phase needs one half-tile that the one before did not, reads it into
// registers a phase ahead, and the half-tile's LDS space is refilled for the slab after next as soon as all
// waves have read it.  Two hand-overs per slab
// (barriers that leave the four youngest half-tiles in flight) instead of one that waits for everything:
// 8192-cubed 837 -> 762 us, 13640 x 9216 x 3072 651 -> 603 us, 13640 x 3072 x 14336 1169 -> 971 us
// (the time per slab of a full chip 1.52 -> 1.33 us).
#pragma once
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "heads.h"
#include "kernels.h"

namespace {

constexpr int EPI_SPLIT_GELU_ERF = 2;  // kernel variant of EPI_SPLIT_GELU with the erf form of the activation
constexpr int EPI_PARTIAL = 3;         // kernel variant of EPI_GATE_RESID that stores the sums of one part of K, nothing added
constexpr int EPI_LAST_PART = 4;       // kernel variant of EPI_GATE_RESID for the last part of K, which adds the ones before it from memory
constexpr int EPI_HEADS = 5;           // kernel variant of EPI_SPLIT_GELU whose plain features are heads (HeadsOut)
constexpr int EPI_HEADS_ERF = 6;       // and with the erf form of the activation
constexpr int EPI_MEET = 7;            // kernel variant of EPI_GATE_RESID for all parts of K, whose workgroups put the sum together (gemm_meet)
constexpr bool cut_sum(int epi) { return epi == EPI_PARTIAL || epi == EPI_MEET; }      // a launch's workgroups: tiles, part by part
constexpr int BK = 64;                 // K slab (bf16 elements) = 128 bytes per LDS row
constexpr int STAGES = 2;              // slabs resident in LDS: one being multiplied, one in flight
constexpr int ROWB = BK * 2;           // bytes per LDS row
constexpr int CHUNKS = BK / 8;         // 16-byte chunks per LDS row
constexpr int KSTEPS = BK / 16;        // MFMA k-steps per slab

// slot of chunk c in row `row` is c ^ swz(row): conflict-free for 16-byte fragment reads of
// consecutive rows on a 32-bank (8 lanes per phase) as well as a 64-bank (16 lanes) LDS
__device__ __forceinline__ int swz(int row) { return ((row >> 1) & 7) ^ ((row & 1) << 2); }

// 16 bytes per lane from global memory straight into LDS: lane l's data lands at lds + 16*l
// (`lds` must be wave-uniform).
__device__ __forceinline__ void lds_load16(const void* gptr, void* lds) {
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)gptr,
                                     (void __attribute__((address_space(3)))*)lds, 16, 0, 0);
}

// The same through a buffer resource: the address is base + voff (per lane) + soff (uniform), and
// lanes whose offset lies past the resource's size fetch zeros, which takes care of ragged tile
// edges.  The memory pipeline takes these a little faster than loads with a 64-bit address per lane.
__device__ __forceinline__ void lds_bload16(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, uint32_t soff, void* lds) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (void __attribute__((address_space(3)))*)lds, 16, voff, soff, 0, 0);
}
__device__ __forceinline__ uint32_t rsrc_bytes(uint64_t bytes) { return bytes > 0xffffffffull ? 0xffffffffu : (uint32_t)bytes; }
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
}

// Slab hand-over: this wave's global->LDS loads (the next slab) have landed and its LDS reads
// (the last fragments of the current slab) have returned; after the barrier that holds for the
// whole workgroup, so the next slab may be read and the current one overwritten.
__device__ __forceinline__ void slab_handover() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The same where the N youngest of this wave's loads may still be in flight.
typedef __attribute__((address_space(3))) const bf16x8 lds_frag;
template <int N>
__device__ __forceinline__ void handover() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The lane's number, computed here: the compiler does not keep the register from where it was asked for before.
__device__ __forceinline__ int lane_here() {
    uint32_t zero = 0u;
    asm volatile("" : "+v"(zero));
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// The epilogue's staging: a wave passes its quadrant through a slice of LDS of its own, ROWS tokens (and of fp32 results 64
// features) at a time, so that global stores are 16 bytes per lane with the lanes of a row on one contiguous segment.
// 16-byte chunks of the slice's rows are XOR-swizzled like those of the slabs.
template <int NT, int ELT, int ROWS>
struct Stage {
    static constexpr int FP = NT * 32 * ELT <= 256 ? NT * 32 : 256 / ELT;      // features per pass
    static constexpr int PASSES = NT * 32 / FP, NTP = FP / 32;
    static constexpr int RB = FP * ELT, CPR = RB / 16;         // bytes and chunks of a staged row
    static constexpr int RPI = 64 / CPR, ST = ROWS / RPI;      // rows per store, stores per slice
    static constexpr int BYTES = ROWS * RB;
    static __device__ __forceinline__ int at(int row, int chunk) { return row * RB + ((chunk ^ (row & (CPR - 1))) << 4); }
};
// Activations go out 32 tokens at a time (gemm_epilogue), fp32 results half a quadrant at a time: with nothing to compute between
// the slices, smaller ones would only add waits.  Where heads are placed (EPI_HEADS) on tiles of 64 and 128 features, the two waves of the
// same tokens share a slice of all of them, which has the heads whole (elsewhere the barrier costs 0.4 us of a launch).
constexpr bool heads_out(int epi) { return epi == EPI_HEADS || epi == EPI_HEADS_ERF; }
// the arguments of a variant's kernels
template <int EPI>
using KernelArgs = std::conditional_t<heads_out(EPI), GemmArgs, GemmCore>;
static_assert(sizeof(GemmCore) <= 216, "what only some variants read goes to those alone");
constexpr bool bf16_out(int epi) { return epi == EPI_SPLIT_GELU || epi == EPI_SPLIT_GELU_ERF || heads_out(epi); }
constexpr bool joint_slices(int bn, int epi) { return heads_out(epi) && bn < 256; }
template <int BM, int BN, int EPI>
constexpr int slice_rows() { return bf16_out(EPI) && !joint_slices(BN, EPI) ? 32 : BM / 2; }
template <int BM, int BN, int EPI>
using StageOf = Stage<joint_slices(BN, EPI) ? BN / 32 : BN / 64, bf16_out(EPI) ? 2 : 4, slice_rows<BM, BN, EPI>()>;
// orders a wave's LDS accesses before and after it, for the compiler (the LDS itself takes a wave's accesses in order)
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// In the accumulators a lane owns one token row and 4 consecutive features per register quad.  Bias and GELU are applied there,
// slice by slice, so that the stores of one slice are on their way while the next is computed; bias, gate and residual of fp32
// results at the write-out, where they need a few registers per lane instead of one per feature, which leaves room to fetch
// residual rows a batch ahead.  Bound, on a full chip of 256 x 256 tiles, by the VALU (GELU: 9.5 us, 46 operations of 256 values
// per lane and some) or by the memory that all CUs turn to at once (33 MB of bf16 in 5.2 us, 5.8 before; residual and result,
// 134 MB, in 21 us, 26.8 with a batch fetched when it was needed).  A Wan-like share of 1320 rows, whose three gated layers end in
// it: 607 -> 598 us.
template <int BM, int BN, int EPI>
__device__ __forceinline__ void gemm_epilogue(const KernelArgs<EPI>& g, floatx16 (&acc)[BN / 64][BM / 64], int m0, int n0, int part, int uw, char* smem) {
    constexpr int WM = BM / 2, WN = BN / 2;        // wave quadrant
    constexpr int MT = WM / 32, NT = WN / 32;      // 32x32 MFMA tiles per wave
    constexpr bool OUT_BF16 = bf16_out(EPI), JOINT = joint_slices(BN, EPI);
    constexpr bool ACT_ERF = (EPI == EPI_SPLIT_GELU_ERF || EPI == EPI_HEADS_ERF);
    constexpr int ELT = OUT_BF16 ? 2 : 4;
    constexpr int SJ = slice_rows<BM, BN, EPI>() / 32;     // MFMA tiles of tokens per slice
    using St = StageOf<BM, BN, EPI>;
    constexpr int ST = St::ST, RPI = St::RPI, CPR = St::CPR;
    // the same value, of which the compiler knows nothing: what is made from it is made where it is used, and not ahead of the
    // main loop (lane coordinates) or of the write-out (all its addresses at once), where it would fill the registers
    auto opaque = [](int v) { asm volatile("" : "+v"(v)); return v; };
    const int lane = lane_here(), wave = uw;
    const int wm0 = (wave & 1) * WM, wn0 = (wave >> 1) * WN;
    const int li = lane & 31, lg = lane >> 5;
    // Bias of the wave's features where the activation needs it, in accumulator order: 4 consecutive features per (feature tile, register
    // quad).  Fetched in one go: taken one by one in the epilogue, each would cost a memory round trip.
    uint32x2 bias_raw[NT][4];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int vb = 0; vb < 4; ++vb) bias_raw[i][vb] = uint32x2{0u, 0u};
    if (OUT_BF16 && g.has_bias) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int vb = 0; vb < 4; ++vb) {
                const int n = min(n0 + wn0 + i * 32 + vb * 8 + lg * 4, g.N - 4);
                bias_raw[i][vb] = *(const uint32x2*)wv_ptr(g.W, g.bias_off + 2ull * n);
            }
    }
    char* const stg = smem + (JOINT ? wave & 1 : wave) * St::BYTES;
    const int cofs = JOINT ? (wave >> 1) * NT * 4 : 0;     // the wave's first chunk of a staged row
    // slice (p, j): tokens j*32.. and features p*FP.. of the quadrant, computed and written to LDS.  Whether a quadrant's features are
    // activated is decided once (n_split falls inside at most one column of quadrants): a decision per quad is a branch per quad,
    // between which nothing overlaps
    enum { PLAIN, ACTIVATED, MIXED };
    auto stage = [&](auto act, int p, int j, int row0, char* stg) __attribute__((always_inline)) {
        wave_lds_order();
#pragma unroll
        for (int ii = 0; ii < (JOINT ? NT : St::NTP); ++ii) {
            const int i = p * St::NTP + ii;
            floatx16 sums = acc[i][j];
            if constexpr (SJ == 1) asm volatile("" : "+v"(sums));      // from the accumulation registers now, not all tiles' ahead of the first store
#pragma unroll
            for (int vb = 0; vb < 4; ++vb) {
                const uint32x2 bb = bias_raw[i][vb];
                const float b[4] = {__uint_as_float(bb.x << 16), __uint_as_float(bb.x & 0xffff0000u),
                                    __uint_as_float(bb.y << 16), __uint_as_float(bb.y & 0xffff0000u)};
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = OUT_BF16 ? sums[vb * 4 + e] + b[e] : sums[vb * 4 + e];
                if constexpr (OUT_BF16) {
                    if constexpr (decltype(act)::value != PLAIN) {
                        const bool here = decltype(act)::value == ACTIVATED || n0 + wn0 + i * 32 + vb * 8 + lg * 4 >= g.n_split;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float a = ACT_ERF ? gelu_erf_f32(v[e]) : gelu_tanh_f32(v[e]);
                            v[e] = here ? a : v[e];
                        }
                    }
                    bf16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = (bf16)v[e];
                    *(bf16x4*)(stg + St::at(row0 + li, cofs + ii * 4 + vb) + lg * 8) = o;
                } else {
                    *(floatx4*)(stg + St::at(row0 + li, ii * 8 + vb * 2 + lg)) = floatx4{v[0], v[1], v[2], v[3]};
                }
            }
        }
        wave_lds_order();
    };
    const int row_l = lane / CPR, chunk_l = lane % CPR;        // a store's row (of RPI) and chunk of this lane
    if constexpr (OUT_BF16 || EPI == EPI_PARTIAL) {
        slab_handover();                       // every wave is done reading the slabs; the bias loads flew meanwhile
        // the staged rows that the wave writes out, and the first feature of a staged row
        constexpr int RW = JOINT ? WM / 2 : SJ * 32, STW = RW / RPI;
        const int r0 = JOINT ? (wave >> 1) * RW : 0, nb = n0 + (JOINT ? 0 : wn0);
        if constexpr (heads_out(EPI)) {
            if (nb < g.n_split) {              // (whole tiles of either sort: gemm_check)
                // Heads of q, k or v (a tile lies in one of the three), a vector in hd / 8 neighbouring lanes, to where attention reads them.  The
                // whole quadrant is staged first: its registers are free then for a loop over the slices in which nothing waits for memory
                // but the first rows of the rotary tables.  Bound by the VALU: the norm and the rotation are some 8 operations per value, 0.9 us of a
                // slice.  What it replaces, a pass over rows in memory: toy 45 -> 41 us a block, Wan-like 1320 rows 603 -> 588 (two passes), Flux-like
                // 2304 rows 620 -> 607.
                const HeadsOut& h = g.heads;
                const RelayoutArgs& r = h.r;
                const int lsh = r.hd == 128 ? 4 : 3, D = r.n_heads * r.hd, sec = nb / D, tns = h.first + sec;
                const bool norm = r.has_norm && tns < 2, turn = r.rope_cos && tns < 2;
                uint32x4 w_raw = {0u, 0u, 0u, 0u};
                if (norm) w_raw = *(const uint32x4*)wv_ptr(g.W, (tns ? r.kn_off : r.qn_off) + ((nb / 8 + lane_here() % CPR) & ((1 << lsh) - 1)) * 16);
                // slices of RW tokens: of the wave's quadrant, one after the other, or (JOINT) its share of one
                constexpr int SLICES = JOINT ? 1 : MT, NEXT = JOINT ? 32 * St::RB : 4 * St::BYTES;
                const int m_first = m0 + wm0 + r0;
#pragma unroll
                for (int j = 0; j < MT; ++j) { __builtin_amdgcn_sched_barrier(0); stage(std::integral_constant<int, PLAIN>{}, 0, j, 0, stg + j * NEXT); }
                if (JOINT) __syncthreads();
                const int here = lane_here(), chunk = here % CPR, row = here / CPR, hh_c = nb - sec * D + chunk * 8, hh = hh_c >> (lsh + 3), sub = (hh_c >> 3) & ((1 << lsh) - 1);
                const bool own = hh >= r.h0 && hh < r.h0 + r.h_local;
                // sample of the token o tokens behind token i of sample b (o < 32, and samples are no shorter: gemm_check); its number there
                auto sample = [&](int b, int i, int o, int& io) __attribute__((always_inline)) {
                    io = i + o;
                    const bool next = h.rps && io >= h.rps;
                    io -= next ? h.rps : 0;
                    return b + next;
                };
                // Most slices lie in one sample and one segment of the joint sequence: then a lane's addresses are one offset from a scalar
                // base, and its rows a constant apart.  (With an address made for each row the slices took twice as long.)
                struct Slice { bool whole; int b, i, pos; };       // sample, its token, position of the first token
                auto slice = [&](int m) __attribute__((always_inline)) {
                    const int b = h.rps ? m / h.rps : 0, i = m - b * h.rps, last = i + RW - 1, lrow = r.row0 + i;
                    const bool whole = m + RW <= g.M && (!h.rps || last < h.rps) && ((lrow < r.map.len0) == (r.row0 + last < r.map.len0));
                    return Slice{whole, b, i, local_pos(r.map, lrow)};
                };
                auto vectors = [&](auto norm_c, auto turn_c) __attribute__((always_inline)) {
                    constexpr bool NORM = decltype(norm_c)::value, TURN = decltype(turn_c)::value;
                    bf16* const send = tns == 0 ? r.send_q : tns == 1 ? r.send_k : r.send_v;
                    bf16* const to_own = tns ? r.K : r.Q;
                    const bool store = own ? tns < 2 : send != nullptr;
                    float w[8];
                    unpack8(w_raw, w);
                    const int rows = own ? r.map.n_total : r.map.n_local, head = own ? hh - r.h0 : hh < r.h0 ? hh : hh - r.h_local;
                    const uint32_t off = ((uint32_t)(head * rows + row) * r.hd + sub * 8) * 2u;
                    floatx4 cs[TURN ? STW : 1], sn[TURN ? STW : 1], cs1[TURN ? STW : 1], sn1[TURN ? STW : 1];
                    auto tables = [&](int m_in, auto& c, auto& s) __attribute__((always_inline)) {
                        if constexpr (TURN) {
                            const int m = m_in < g.M ? m_in : 0;           // (of a slice behind the end: some rows)
                            const Slice first = slice(m);
#pragma unroll
                            for (int u = 0; u < STW; ++u) {
                                int i;
                                sample(first.b, first.i, m + u * RPI + row < g.M ? u * RPI + row : 0, i);
                                const uint32_t at = (uint32_t)(r.row0 + i) * (r.hd / 2) + sub * 4;
                                c[u] = *(const floatx4*)(r.rope_cos + at);
                                s[u] = *(const floatx4*)(r.rope_sin + at);
                            }
                        }
                    };
                    tables(m_first, cs, sn);
#pragma unroll 1
                    for (int j = 0; j < SLICES; ++j) {
                        const int mw = m_first + j * 32;
                        if (SLICES > 1) tables(mw + 32, cs1, sn1);
                        uint32x4 val[STW];
#pragma unroll
                        for (int u = 0; u < STW; ++u) val[u] = *(const uint32x4*)(stg + j * NEXT + St::at(r0 + u * RPI + row, chunk));
                        if constexpr (NORM || TURN)
#pragma unroll
                            for (int u = 0; u < STW; ++u) val[u] = head_piece<true>(val[u], r.hd, NORM, w, TURN, cs[TURN ? u : 0], sn[TURN ? u : 0]);
                        const Slice at = slice(mw);
                        if (at.whole) {
                            auto put = [&](bf16* to) __attribute__((always_inline)) {
#pragma unroll
                                for (int u = 0; u < STW; ++u) *(uint32x4*)((char*)to + off + u * RPI * r.hd * 2) = val[u];
                            };
                            if (own && tns < 2) put(to_own + at.b * h.op_bs + (size_t)at.pos * r.hd);
                            if (!own && send) put(send + at.b * h.send_bs + (size_t)(r.row0 + at.i) * r.hd);
                        } else if (store) {
                            bf16* const base = (own ? to_own : send) + (size_t)(head * (long)rows) * r.hd + sub * 8;
#pragma unroll
                            for (int u = 0; u < STW; ++u) {
                                int i;
                                const int b = sample(at.b, at.i, u * RPI + row, i);
                                if (mw + u * RPI + row < g.M) *(uint32x4*)(base + b * (own ? h.op_bs : h.send_bs) + (size_t)(own ? local_pos(r.map, r.row0 + i) : r.row0 + i) * r.hd) = val[u];
                            }
                        }
                        if constexpr (TURN && SLICES > 1)
#pragma unroll
                            for (int u = 0; u < STW; ++u) cs[u] = cs1[u], sn[u] = sn1[u];
                    }
                };
                using Yes = std::true_type;
                using No = std::false_type;
                if (norm && turn) vectors(Yes{}, Yes{});
                else if (norm) vectors(Yes{}, No{});
                else if (turn) vectors(No{}, Yes{});
                else if (tns < 2 || __any(!own)) vectors(No{}, No{});
                if (tns < 2) return;
                // own v: a lane has 8 tokens of one chunk, neighbouring lanes the 8 tokens that follow
                constexpr int TG = RW / 8;
                static_assert(TG * CPR <= 64, "a lane per 8 tokens of a chunk");
                const int grp = here % TG, c = here / TG;
                const int vc = nb - sec * D + c * 8, vh = vc >> (lsh + 3);
                const uint32_t v_row = (uint32_t)((vh - r.h0) * r.hd + (vc & (r.hd - 1))) * r.n_pad;
                if (c < CPR && vh >= r.h0 && vh < r.h0 + r.h_local) {
#pragma unroll 1
                    for (int j = 0; j < SLICES; ++j) {
                        const int mw = m_first + j * 32, cnt = min(8, g.M - mw - grp * 8);
                        uint32x4 u[8];
#pragma unroll
                        for (int k = 0; k < 8; ++k) u[k] = *(const uint32x4*)(stg + j * NEXT + St::at(r0 + grp * 8 + k, c));
                        const Slice at = slice(mw);
                        if (at.whole && (at.pos & 7) == 0) {
                            v_turned_line(u, (char*)(r.Vt + at.b * h.vt_bs + at.pos), (v_row + grp * 8) * 2u, r.n_pad);
                        } else if (cnt > 0) {
                            v_turned(u, cnt, r.n_pad, [&](int k) __attribute__((always_inline)) {
                                int i;
                                const int b = sample(at.b, at.i, grp * 8 + k, i);
                                return (uint16_t*)r.Vt + b * h.vt_bs + v_row + local_pos(r.map, r.row0 + i);
                            });
                        }
                    }
                }
                // The columns of Vt behind the last position, a lane per row of it: by the wave that has local row 0 of the sample.
                if (r.row0 == 0 && r.n_pad > r.map.n_total) {
                    const int rps = h.rps ? h.rps : g.M, end = min(m_first + (SLICES - 1) * 32 + RW, g.M);
                    for (int b = (m_first + rps - 1) / rps; b * rps < end; ++b)
                        for (int f = here; f < St::FP; f += 64) {
                            const int vc = nb - sec * D + f - r.h0 * r.hd;
                            if (vc < 0 || vc >= r.h_local * r.hd) continue;
                            uint16_t* const col = (uint16_t*)r.Vt + b * h.vt_bs + (size_t)vc * r.n_pad;
                            int p = r.map.n_total;
                            for (; p & 7; ++p) col[p] = 0;
                            for (; p < r.n_pad; p += 8) *(uint32x4*)(col + p) = uint32x4{0u, 0u, 0u, 0u};
                        }
                }
                return;
            }
        }
        auto write_out = [&](auto act) __attribute__((always_inline)) {
            constexpr int ACT = decltype(act)::value;
#pragma unroll
            for (int p = 0; p < St::PASSES; ++p) {
                const int n = nb + p * St::FP + chunk_l * (16 / ELT);          // first column of the lane's chunk
#pragma unroll
                for (int j0 = 0; j0 < MT; j0 += SJ) {
#pragma unroll
                    for (int j = 0; j < SJ; ++j) stage(act, p, j0 + j, j * 32, stg);
                    if (JOINT) __syncthreads();
                    const int r = opaque(row_l);
                    constexpr int UB = STW > 4 && MT == 3 ? 4 : STW;   // (as the register allocator has it without spills)
#pragma unroll
                    for (int u0 = 0; u0 < STW; u0 += UB) {
                        uint32x4 val[UB];
#pragma unroll
                        for (int u = 0; u < UB; ++u) val[u] = *(const uint32x4*)(stg + St::at(r0 + (u0 + u) * RPI + row_l, chunk_l));
#pragma unroll
                        for (int u = 0; u < UB; ++u) {
                            const int m = m0 + wm0 + j0 * 32 + r0 + (u0 + u) * RPI + r;
                            if (m < g.M && n < g.n1) {
                                if constexpr (OUT_BF16) {
                                    bf16* const dst = ACT == PLAIN || (ACT == MIXED && n < g.n_split) ? g.out0 + (size_t)m * g.ld0 + n
                                                                                                      : g.out1 + (size_t)m * g.ld1 + g.col1_off + (n - g.n_split);
                                    *(uint32x4*)dst = val[u];
                                } else {
                                    *(uint32x4*)(g.part + (size_t)part * g.M * g.N + (size_t)m * g.N + n) = val[u];
                                }
                            }
                        }
                    }
                }
            }
        };
        using Plain = std::integral_constant<int, PLAIN>;
        if constexpr (!OUT_BF16) {
            write_out(Plain{});
        } else if constexpr (heads_out(EPI)) {
            write_out(std::integral_constant<int, ACTIVATED>{});
        } else {
            if (nb >= g.n_split) write_out(std::integral_constant<int, ACTIVATED>{});
            else if (min(nb + St::FP, g.n1) <= g.n_split) write_out(Plain{});
            else write_out(std::integral_constant<int, MIXED>{});
        }
    } else {
        // y = resid + gate * (...), the product rounded before the sum; the gate belongs to the row's
        // sample.  The residual rows of UB stores are fetched together and a batch ahead: taken one by one, each store
        // would wait out a memory round trip of its own.  Lanes outside the problem read a valid
        // address (row M-1, column 0) and store nothing.
        const bool has_gate = g.gate != nullptr;
        const float* const gate_p = has_gate ? g.gate : g.resid;       // a readable address either way
        const long gate_bs = has_gate ? g.gate_bs : 0;
        auto write_out = [&](auto per_sample) {
            constexpr bool PS = decltype(per_sample)::value;
            constexpr bool LAST = EPI == EPI_LAST_PART;
            constexpr int AHEAD = LAST ? 0 : 1, UB = BM * BN <= 128 * 128 ? 4 : 8;        // (two workgroups per CU: 256 registers)
            static_assert(ST % UB == 0, "write-out batches");
            constexpr int HB = ST / UB, NB = St::PASSES * HB;          // batches of a slice (a pass), of the quadrant
            floatx4 rr[1 + AHEAD][UB], gt[1 + AHEAD][PS ? UB : 1], sum[LAST ? UB : 1];      // native vectors: arrays of them stay in registers
            floatx4 gate_c = {1.f, 1.f, 1.f, 1.f}, bias_c = {0.f, 0.f, 0.f, 0.f};
            auto col = [&](int p) { return n0 + wn0 + p * St::FP + chunk_l * 4; };
            auto token = [&](int b, int u, int r) { return m0 + wm0 + (b % HB * UB + u) * RPI + r; };
            auto fetch = [&](int b, int buf) __attribute__((always_inline)) {
                const int nc = col(b / HB) < g.n1 ? col(b / HB) : 0, r = opaque(row_l);
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    const int mm = min(token(b, u, r), g.M - 1);
                    int sm = 0, i = mm;
                    if (PS) { sm = mm / g.rows_per_sample; i = mm - sm * g.rows_per_sample; }
                    rr[buf][u] = *(const floatx4*)(g.resid + (size_t)sm * g.resid_bs + (size_t)i * g.ldy + nc);
                    if constexpr (PS) gt[buf][u] = *(const floatx4*)(gate_p + (size_t)sm * gate_bs + nc);
                    if constexpr (LAST) sum[u] = *(const floatx4*)(g.part + (size_t)mm * g.N + nc);       // of the parts before, in order
                }
            };
            if (AHEAD) fetch(0, 0);
            slab_handover();                   // every wave is done reading the slabs; these loads flew meanwhile
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int p = b / HB, buf = AHEAD ? b & 1 : 0, r = opaque(row_l);
                const int n = col(p), nc = n < g.n1 ? n : 0;
                __builtin_amdgcn_sched_barrier(0);         // (batches kept apart, for the registers' sake)
                if (b + AHEAD < NB) fetch(b + AHEAD, AHEAD ? buf ^ 1 : 0);
                if (b % HB == 0) {
                    if (!PS && has_gate) gate_c = *(const floatx4*)(gate_p + nc);
                    if (g.has_bias) {
                        const uint32x2 bb = *(const uint32x2*)wv_ptr(g.W, g.bias_off + 2ull * nc);
                        bias_c = floatx4{__uint_as_float(bb.x << 16), __uint_as_float(bb.x & 0xffff0000u), __uint_as_float(bb.y << 16),
                                         __uint_as_float(bb.y & 0xffff0000u)};
                    }
                }
                if (b % HB == 0) {
#pragma unroll
                    for (int j = 0; j < MT; ++j) stage(std::integral_constant<int, PLAIN>{}, p, j, j * 32, stg);
                }
                if constexpr (LAST) {
                    for (int q = 1; q < part; ++q)
#pragma unroll
                        for (int u = 0; u < UB; ++u) {
                            const floatx4 t = *(const floatx4*)(g.part + ((size_t)q * g.M + min(token(b, u, r), g.M - 1)) * g.N + nc);
#pragma unroll
                            for (int e = 0; e < 4; ++e) sum[u][e] += t[e];
                        }
                }
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    const int m = token(b, u, r);
                    floatx4 val = *(const floatx4*)(stg + St::at((b % HB * UB + u) * RPI + row_l, chunk_l)), o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) val[e] = (LAST ? sum[LAST ? u : 0][e] + val[e] : val[e]) + bias_c[e];
                    const floatx4 gq = PS && has_gate ? gt[buf][PS ? u : 0] : gate_c;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = __fadd_rn(rr[buf][u][e], __fmul_rn(gq[e], val[e]));
                    if (m < g.M && n < g.n1) {
                        int sm = 0, i = m;
                        if (PS) { sm = m / g.rows_per_sample; i = m - sm * g.rows_per_sample; }
                        *(floatx4*)(g.y + (size_t)sm * g.y_bs + (size_t)i * g.ldy + n) = o;
                    }
                }
            }
        };
        if (g.rows_per_sample) write_out(std::true_type{}); else write_out(std::false_type{});
    }
}

// The parts of a cut sum, put together by the workgroups that computed them: each sends the others what it does not finish itself
// and finishes its share of the tile, in units of 32 tokens x 64 (32) features that the parts of a wave's quadrant take turns in.  A
// wave deals with the waves of the same quadrant only; a word of memory per tile and wave has their state.  Nobody waits for a workgroup
// that may not be running: each counts itself in when it begins, and the one that is done first looks whether all are there.  If so, they
// exchange; if not (the grid is more than the chip holds, or another stream's work is on it), all send everything, and the one
// that is done last, which is then waiting for others' stores at most, finishes the tile alone.  The sum is in the order of the parts either way.
// Data and words go past the XCDs' L2 (stores and loads of agent scope), so that no cache has to be written back or cleared.
// Bound by the memory the chip turns to at once: two thirds of what the parts and a kernel that adds them up moved.  2304 x 3072 x 15360 in two
// parts 202.7 -> 189.4 us, 1320 x 3072 x 14336 in three 113.6 -> 108.3, 512 + 64 rows x 3072 x 12288 in two 77.8 -> 76.1 (their blocks: 614 -> 599,
// 588 -> 569 with the heads above, 329 -> 324 us).
enum : uint32_t { MEET_DONE_FIRST = 1u << 8, MEET_EXCHANGE = 1u << 16, MEET_ALONE = 1u << 17, MEET_SENT = 1u << 24 };   // low byte: begun
constexpr int AGENT_SCOPE = 16;                // cache policy of a buffer access: sc1
template <int BM, int BN>
struct Meet {
    using St = Stage<BN / 64, 4, 32>;
    static constexpr int MT = BM / 64, UNITS = St::PASSES * MT, SLOTS = (UNITS + 1) / 2;       // units of a quadrant, at most so many its own
    static constexpr int QUADS = St::NTP * 4;                                                  // 16-byte pieces of a lane in a unit
    static constexpr int BYTES = 4 * SLOTS * St::BYTES;
};
__device__ __forceinline__ uint32_t meet_word(const uint32_t* w) { return __builtin_amdgcn_readfirstlane(__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)); }
template <int BM, int BN>
__device__ __forceinline__ void gemm_meet(const GemmCore& g, floatx16 (&acc)[BN / 64][BM / 64], int m0, int n0, int part, uint32_t tile, int uw, char* smem) {
    using Mt = Meet<BM, BN>;
    using St = typename Mt::St;
    constexpr int MT = Mt::MT, UNITS = Mt::UNITS, QUADS = Mt::QUADS, ST = St::ST, RPI = St::RPI, CPR = St::CPR;
    const int lane = lane_here(), wave = uw, P = g.ksplits;
    const int m_q = m0 + (wave & 1) * (BM / 2), n_q = n0 + (wave >> 1) * (BN / 2);             // of the wave's quadrant
    const int li = lane & 31, lg = lane >> 5;
    uint32_t* const word = g.words + tile * 4 + wave;
    char* const slots = smem + wave * (Mt::SLOTS * St::BYTES);
    const __amdgpu_buffer_rsrc_t sums = make_rsrc(g.part + (size_t)tile * P * (BM * BN), (uint32_t)P * (BM * BN * 4));
    auto sum_at = [&](int q, int u) { return (uint32_t)__builtin_amdgcn_readfirstlane(((q * 4 + wave) * UNITS + u) * St::BYTES); };
    auto inside = [&](int u) { return m_q + u % MT * 32 < g.M && n_q + u / MT * St::FP < g.n1; };
    const int first = __builtin_amdgcn_readfirstlane((part + P - wave % P) % P);       // the wave's own units: first, first + P, ...

    slab_handover();                           // every wave is done reading the slabs
    uint32_t seen = 0;
    if (lane == 0) seen = __hip_atomic_fetch_add(word, MEET_DONE_FIRST, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int next = first, slot = 0;
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const int p = u / MT, j = u % MT;
        const bool own = u == next;
        if (own) next += P;
        if (own || inside(u)) {
#pragma unroll
            for (int t = 0; t < QUADS; ++t) {
                const floatx16& a = acc[p * St::NTP + t / 4][j];
                const floatx4 v = {a[t % 4 * 4], a[t % 4 * 4 + 1], a[t % 4 * 4 + 2], a[t % 4 * 4 + 3]};
                if (own) *(floatx4*)(slots + slot * St::BYTES + t * 1024 + lane * 16) = v;
                else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint32x4, v), sums, t * 1024 + lane * 16, sum_at(part, u), AGENT_SCOPE);
            }
        }
        if (own) ++slot;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // what was sent is there for all to see
    seen = __builtin_amdgcn_readfirstlane(seen);
    const int rank = (seen >> 8) & 0xff;                       // parts that were done before
    uint32_t say = MEET_SENT;
    if (rank == 0) {
        seen = (int)(seen & 0xff) == P ? MEET_EXCHANGE : MEET_ALONE;
        say += seen;
    } else {
        while (!(seen & (MEET_EXCHANGE | MEET_ALONE))) {
            __builtin_amdgcn_s_sleep(1);
            seen = meet_word(word);
        }
    }
    const bool exchange = seen & MEET_EXCHANGE;
    wave_lds_order();
    if (!exchange) {
        for (int u = first, k = 0; u < UNITS; u += P, ++k)
#pragma unroll
            for (int t = 0; t < QUADS; ++t)
                __builtin_amdgcn_raw_buffer_store_b128(*(const uint32x4*)(slots + k * St::BYTES + t * 1024 + lane * 16), sums, t * 1024 + lane * 16, sum_at(part, u), AGENT_SCOPE);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    if (lane == 0) __hip_atomic_fetch_add(word, say, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!exchange && rank != P - 1) return;

    // the units this wave finishes: its own, or all of the quadrant
    const int u0 = exchange ? first : 0, step = exchange ? P : 1;
    const int r_l = lane / CPR, c_l = lane % CPR;              // a store's row (of RPI) and chunk of this lane
    const int other1 = part == 0 ? 1 : 0, other2 = part == 2 ? 1 : 2;      // the other parts, in order (the second: P = 3)
    const bool has_gate = g.gate != nullptr;
    const float* const gate_p = has_gate ? g.gate : g.resid;   // a readable address either way
    const long gate_bs = has_gate ? g.gate_bs : 0;
    struct Rows { floatx4 resid[ST], gate[ST], bias; };
    struct Sums { floatx4 a[QUADS], b[QUADS], own[QUADS]; };
    auto finish = [&](auto per_sample, auto three) __attribute__((always_inline)) {
        constexpr bool PS = decltype(per_sample)::value, THREE = decltype(three)::value;
        // (lanes outside the problem read a valid address, row M-1 or column 0, and store nothing)
        auto place = [&](int u, int s, int& sm, int& i) {
            i = min(m_q + u % MT * 32 + s * RPI + r_l, g.M - 1);
            sm = 0;
            if (PS) { sm = i / g.rows_per_sample; i -= sm * g.rows_per_sample; }
        };
        auto column = [&](int u) { return n_q + u / MT * St::FP + c_l * 4; };
        auto fetch_rows = [&](int u, Rows& r) __attribute__((always_inline)) {
            const int n = column(u), nc = n < g.n1 ? n : 0;
            r.gate[0] = floatx4{1.f, 1.f, 1.f, 1.f};
            if (!PS && has_gate) r.gate[0] = *(const floatx4*)(gate_p + nc);
            r.bias = floatx4{0.f, 0.f, 0.f, 0.f};
            if (g.has_bias) {
                const uint32x2 bb = *(const uint32x2*)wv_ptr(g.W, g.bias_off + 2ull * nc);
                r.bias = floatx4{__uint_as_float(bb.x << 16), __uint_as_float(bb.x & 0xffff0000u), __uint_as_float(bb.y << 16), __uint_as_float(bb.y & 0xffff0000u)};
            }
#pragma unroll
            for (int s = 0; s < ST; ++s) {
                int sm, i;
                place(u, s, sm, i);
                r.resid[s] = *(const floatx4*)(g.resid + (size_t)sm * g.resid_bs + (size_t)i * g.ldy + nc);
                if constexpr (PS) r.gate[s] = *(const floatx4*)(gate_p + (size_t)sm * gate_bs + nc);
            }
        };
        auto fetch_sums = [&](int u, Sums& x) __attribute__((always_inline)) {
            auto get = [&](int q, floatx4 (&to)[QUADS]) __attribute__((always_inline)) {
#pragma unroll
                for (int t = 0; t < QUADS; ++t) to[t] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(sums, t * 1024 + lane * 16, sum_at(q, u), AGENT_SCOPE));
            };
            get(other1, x.a);
            if (THREE) get(other2, x.b);
            if (!exchange) get(part, x.own);
        };
        auto put_out = [&](int u, int k, const Sums& x, const Rows& r) __attribute__((always_inline)) {
            char* const stg = slots + k * St::BYTES;
            floatx4 v[QUADS];
#pragma unroll
            for (int t = 0; t < QUADS; ++t) {
                const floatx4 own = exchange ? *(const floatx4*)(stg + t * 1024 + lane * 16) : x.own[t];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (THREE) v[t][e] = part == 2 ? (x.a[t][e] + x.b[t][e]) + own[e] : (x.a[t][e] + own[e]) + x.b[t][e];
                    else v[t][e] = x.a[t][e] + own[e];
                }
            }
            wave_lds_order();
#pragma unroll
            for (int t = 0; t < QUADS; ++t) *(floatx4*)(stg + St::at(li, t / 4 * 8 + t % 4 * 2 + lg)) = v[t];
            wave_lds_order();
            const int n = column(u);
#pragma unroll
            for (int s = 0; s < ST; ++s) {
                const floatx4 val = *(const floatx4*)(stg + St::at(s * RPI + r_l, c_l)), gq = PS && !has_gate ? floatx4{1.f, 1.f, 1.f, 1.f} : r.gate[PS ? s : 0];
                floatx4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = __fadd_rn(r.resid[s][e], __fmul_rn(gq[e], val[e] + r.bias[e]));
                if (m_q + u % MT * 32 + s * RPI + r_l < g.M && n < g.n1) {
                    int sm, i;
                    place(u, s, sm, i);
                    *(floatx4*)(g.y + (size_t)sm * g.y_bs + (size_t)i * g.ldy + n) = o;
                }
            }
            wave_lds_order();
        };
        Rows rows;
        Sums sums_of;
        // rows are the caller's and come while the others are waited for; a unit that is not there (its quadrant ends before) reads row M-1
        if (u0 < UNITS) fetch_rows(u0, rows);
        while ((int)(meet_word(word) >> 24) < P) __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory");
        if (u0 >= UNITS) return;
        fetch_sums(u0, sums_of);
#pragma unroll 1
        for (int u = u0, k = 0; u < UNITS; u += step, k += exchange) {
            if constexpr (UNITS > 2) {         // the next unit's operands ahead
                Rows rows1;
                Sums sums1;
                const int un = u + step < UNITS ? u + step : u;
                fetch_rows(un, rows1);
                fetch_sums(un, sums1);
                if (inside(u)) put_out(u, k, sums_of, rows);
                rows = rows1;
                sums_of = sums1;
            } else {
                if (inside(u)) put_out(u, k, sums_of, rows);
                if (u + step < UNITS) { fetch_rows(u + step, rows); fetch_sums(u + step, sums_of); }
            }
        }
    };
    using Yes = std::true_type;
    using No = std::false_type;
    if (g.rows_per_sample) { if (P == 3) finish(Yes{}, Yes{}); else finish(Yes{}, No{}); }
    else { if (P == 3) finish(No{}, Yes{}); else finish(No{}, No{}); }
}

// One tile of one problem: tokens m0.., features n0...  STRADDLE: the byte where the blob switches buffers falls
// inside the tile's weight rows (at most one tile column of a launch), so each lane picks its base.
template <int BM, int BN, int EPI, bool STRADDLE>
__device__ __forceinline__ void gemm_tile_run(const KernelArgs<EPI>& g, int m0, int n0, int part, uint32_t tile, int uw) {
    constexpr int WM = BM / 2, WN = BN / 2;        // wave quadrant
    constexpr int MT = WM / 32, NT = WN / 32;      // 32x32 MFMA tiles per wave
    constexpr int PA = MT % 2 ? 3 : 2;             // the activations go in thirds or halves, the weights in halves
    constexpr int MH = MT / PA, NH = NT / 2;       // MFMA tiles of a part
    constexpr int GA = WM / PA / 8, GW = WN / 2 / 8;           // 8-row units of a part per wave row (column)
    constexpr int LA = GA / 2, LW = GW / 2;        // wave-loads (1 KiB = one unit each) per wave and part
    constexpr int L = PA * LA + 2 * LW;            // and per slab
    constexpr int A_STAGE = BM * ROWB, W_STAGE = BN * ROWB;

    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const sA = smem;                         // [STAGES][BM][ROWB] activations
    char* const sW = smem + STAGES * A_STAGE;      // [STAGES][BN][ROWB] weights

    // (the lane made here, the wave's number in a scalar register: of two variants of this in a kernel, the first would otherwise
    // keep registers for the second)
    const int lane = lane_here();
    const int wm0 = (uw & 1) * WM, wn0 = (uw >> 1) * WN;
    const int li = lane & 31, lg = lane >> 5;

    // Slab copies go global -> LDS directly (no register staging).  One such load writes the
    // wave's 64 x 16 bytes to consecutive LDS addresses, i.e. 8 rows (a unit); which 16-byte chunk of
    // its row a lane fetches is chosen so that the chunk lands in its swizzled slot.  Part h of an operand is the
    // rows that the h-th parts of the waves' quadrants cover: unit (j*4 + wave) of it is unit `unit(..)` of the tile.
    auto unit = [](int G, int parts, int h, int idx) { return (idx / G) * parts * G + h * G + idx % G; };
    uint32_t a_voff[PA][LA], w_voff[2][LW];        // byte offsets from the tile's first row
#pragma unroll
    for (int h = 0; h < PA; ++h)
#pragma unroll
        for (int j = 0; j < LA; ++j) {
            const int row = unit(GA, PA, h, j * 4 + uw) * 8 + lane / CHUNKS;
            a_voff[h][j] = (uint32_t)row * (uint32_t)g.lda * 2u + ((lane % CHUNKS) ^ swz(row)) * 16;
        }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < LW; ++j) {
            const int row = unit(GW, 2, h, j * 4 + uw) * 8 + lane / CHUNKS;
            w_voff[h][j] = (uint32_t)row * (uint32_t)g.K * 2u + ((lane % CHUNKS) ^ swz(row)) * 16;
        }
    const uint64_t t_begin = g.w_off + (uint64_t)n0 * g.K * 2, t_end = g.w_off + (uint64_t)min(n0 + BN, g.N) * g.K * 2;
    // resources that end with the tile's last valid row: the rows of a ragged tile beyond it read zeros
    const void* const a_base = g.A + (size_t)m0 * g.lda;
    const void* const w_base = wv_ptr(g.W, t_begin);
    const uint32_t a_bytes = rsrc_bytes(((uint64_t)(g.M - 1 - m0) * g.lda + g.K) * 2), w_bytes = rsrc_bytes(t_end - t_begin);

    floatx16 acc[NT][MT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // LDS address of this lane's fragment of k-step kk in row 0 of its quadrant; rows 32 apart share the swizzle
    lds_frag *a_frag[KSTEPS], *w_frag[KSTEPS];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
        const int c = ((kk * 2 + lg) ^ swz(li)) << 4;
        a_frag[kk] = (lds_frag*)(sA + (wm0 + li) * ROWB + c);
        w_frag[kk] = (lds_frag*)(sW + (wn0 + li) * ROWB + c);
    }

    // slabs of this workgroup: all, or those of its part
    constexpr bool CUT = cut_sum(EPI) || EPI == EPI_LAST_PART;
    const int kt0 = CUT ? part * g.part_slabs : 0;
    const int KT = CUT ? min(g.part_slabs, g.K / BK - kt0) : g.K / BK;
    bf16x8 fa[2][MH][KSTEPS], fw[2][NH][KSTEPS];

    // Slab kt's copies into stage st.  Past the last slab the resources are empty: the copies of the two slabs that do
    // not exist fetch nothing, so the loop needs no tail and its wait counts never change.
    struct Src { __amdgpu_buffer_rsrc_t a, w; uint32_t k0; bool on; };
    auto source = [&](int kt) {
        const bool on = kt < KT;
        return Src{make_rsrc(a_base, on ? a_bytes : 0u), make_rsrc(w_base, on ? w_bytes : 0u), on ? (uint32_t)(kt0 + kt) * (BK * 2) : 0u, on};
    };
    auto issue_a = [&](auto st, int h, const Src& src, int q) {
        lds_bload16(src.a, a_voff[h][q], src.k0, sA + st.value * A_STAGE + unit(GA, PA, h, q * 4 + uw) * 1024);
    };
    auto issue_w = [&](auto st, int h, const Src& src, int q) {
        char* const dst = sW + st.value * W_STAGE + unit(GW, 2, h, q * 4 + uw) * 1024;
        if (STRADDLE && src.on) {                  // rows past the matrix read the tile's first bytes; they are never stored
            const uint64_t o = (uint64_t)w_voff[h][q] + src.k0;
            lds_load16(wv_ptr(g.W, t_begin + (o < t_end - t_begin ? o : 0)), dst);
        } else {
            lds_bload16(src.w, w_voff[h][q], src.k0, dst);
        }
    };
    // The copies of a slab in two groups: parts a0 w0, whose stage is free a slab and a half before, then w1 a1 (a2).
    auto issue_first = [&](auto st, const Src& src, int q) {
        if (q < LA) issue_a(st, 0, src, q); else issue_w(st, 0, src, q - LA);
    };
    auto issue_second = [&](auto st, const Src& src, int q) {
        if (q < LW) issue_w(st, 1, src, q); else issue_a(st, 1 + (q - LW) / LA, src, (q - LW) % LA);
    };
    constexpr int L1 = LA + LW, L2 = L - L1;
    // r-th of the MH (NH) * KSTEPS fragments of a part
    auto read_a = [&](auto st, auto h, auto buf, int r) {
        fa[buf.value][r / KSTEPS][r % KSTEPS] =
            a_frag[r % KSTEPS][(st.value * A_STAGE + (h.value * MH + r / KSTEPS) * 32 * ROWB) / 16];
    };
    auto read_w = [&](auto st, auto h, auto buf, int r) {
        fw[buf.value][r / KSTEPS][r % KSTEPS] =
            w_frag[r % KSTEPS][(st.value * W_STAGE + (h.value * NH + r / KSTEPS) * 32 * ROWB) / 16];
    };
    // One phase: the MFMAs of activation part ha (held in fa[ba]) with weight half hb (in fw[bw]), with fragment reads for
    // the phases to come between the first of them and the copies [u0, u1) of a group spread over them
    auto phase = [&](auto ha, auto ba, auto hb, auto bw, int n_reads, auto read, int u0, int u1, auto issue) __attribute__((always_inline)) {
        constexpr int NM = KSTEPS * NH * MH;
        int r = 0, u = u0;
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            const int kk = q / (NH * MH), i = (q / MH) % NH, j = q % MH;
            acc[hb.value * NH + i][ha.value * MH + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                fw[bw.value][i][kk], fa[ba.value][j][kk], acc[hb.value * NH + i][ha.value * MH + j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            for (; r * NM < n_reads * 2 * (q + 1) && r < n_reads; ++r) read(r);
            for (; (u - u0) * NM < (u1 - u0) * (q + 1) && u < u1; ++u) issue(u);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    // One slab of stage (and parity) st, as the serpentine of its quadrant phases.  At each hand-over every wave's loads of
    // the parts about to be read have landed and its reads of the ones before have returned, so those are refilled.  What
    // may still be in flight there: one slab's worth of copies issued after them.
    // Activation part a is in fragment buffer (parity * PA + a) & 1; weight half 0 in buffer `parity` where it is used to
    // the slab's end (PA = 2), else in 0.
    auto slab = [&](auto st, int kt) __attribute__((always_inline)) {
        constexpr int P = decltype(st)::value;
        using SN = std::integral_constant<int, P ^ 1>;
        using A0 = std::integral_constant<int, (P * PA) & 1>;
        using A1 = std::integral_constant<int, (P * PA + 1) & 1>;
        using NA = std::integral_constant<int, ((P ^ 1) * PA) & 1>;       // a0 of the next slab
        using W0 = std::integral_constant<int, PA == 2 ? P : 0>;
        using W1 = std::integral_constant<int, W0::value ^ 1>;
        using NW = std::integral_constant<int, PA == 2 ? P ^ 1 : 0>;      // w0 of the next slab
        const Src src = source(kt + 2);
        auto first = [&](int u) { issue_first(st, src, u); };
        auto second = [&](int u) { issue_second(st, src, u); };
        handover<L>();
        if constexpr (PA == 2) {
            phase(I0{}, A0{}, I0{}, W0{}, NH * KSTEPS, [&](int r) { read_w(st, I1{}, W1{}, r); }, 0, L1 / 2, first);
            phase(I0{}, A0{}, I1{}, W1{}, MH * KSTEPS, [&](int r) { read_a(st, I1{}, A1{}, r); }, L1 / 2, L1, first);
            handover<L>();
            phase(I1{}, A1{}, I1{}, W1{}, MH * KSTEPS, [&](int r) { read_a(SN{}, I0{}, NA{}, r); }, 0, L2 / 2, second);
            phase(I1{}, A1{}, I0{}, W0{}, NH * KSTEPS, [&](int r) { read_w(SN{}, I0{}, NW{}, r); }, L2 / 2, L2, second);
        } else {
            phase(I0{}, A0{}, I0{}, W0{}, NH * KSTEPS, [&](int r) { read_w(st, I1{}, W1{}, r); }, 0, L1 / 3, first);
            phase(I0{}, A0{}, I1{}, W1{}, MH * KSTEPS, [&](int r) { read_a(st, I1{}, A1{}, r); }, L1 / 3, 2 * L1 / 3, first);
            phase(I1{}, A1{}, I1{}, W1{}, MH * KSTEPS, [&](int r) { read_a(st, I2{}, A0{}, r); }, 2 * L1 / 3, L1, first);
            handover<L>();
            phase(I1{}, A1{}, I0{}, W0{}, 0, [](int) {}, 0, L2 / 3, second);
            phase(I2{}, A0{}, I0{}, W0{}, MH * KSTEPS, [&](int r) { read_a(SN{}, I0{}, NA{}, r); }, L2 / 3, 2 * L2 / 3, second);
            phase(I2{}, A0{}, I1{}, W1{}, NH * KSTEPS, [&](int r) { read_w(SN{}, I0{}, NW{}, r); }, 2 * L2 / 3, L2, second);
        }
    };
    auto issue_slab = [&](auto st, int kt) {
        const Src src = source(kt);
#pragma unroll
        for (int q = 0; q < L1; ++q) issue_first(st, src, q);
#pragma unroll
        for (int q = 0; q < L2; ++q) issue_second(st, src, q);
    };
    issue_slab(I0{}, 0);
    issue_slab(I1{}, 1);
    handover<2 * L - L1>();
#pragma unroll
    for (int r = 0; r < MH * KSTEPS; ++r) read_a(I0{}, I0{}, I0{}, r);
#pragma unroll
    for (int r = 0; r < NH * KSTEPS; ++r) read_w(I0{}, I0{}, I0{}, r);
    for (int kt = 0; kt < KT; kt += 2) {           // an odd last slab is followed by one of zeros
        slab(I0{}, kt);
        slab(I1{}, kt + 1);
    }

    if constexpr (EPI == EPI_MEET) gemm_meet<BM, BN>(g, acc, m0, n0, part, tile, uw, smem);
    else gemm_epilogue<BM, BN, EPI>(g, acc, m0, n0, part, uw, smem);
}

// The same for small tiles, which are for layers with too few large ones to give every CU a workgroup: there the time is
// the serial walk over K, slab by slab.  A wave holds all fragments of a slab, double-buffered in registers, so a slab's
// stage is free as soon as it has been read and S stages keep S - 1 slabs on their way, which covers the latency of
// weights read cold; one hand-over per slab.  A lone 64x64 workgroup takes 0.30 us per slab (LDS traffic and the
// hand-over; six more stages change nothing, two fewer cost a fifth), 128x64 0.43, against 0.55 of the 128x128 tile.
// 576 x 3072 x 12288: 164 us with the former loop, 111 with the 128x128 tile above, 85 with 128x64 (240 workgroups);
// 64 x 3072 x 12288: 166, 102, 63 with 64x64; 512 x 512 x 2560: 31.4, 20.5, 12.2.
template <int BM, int BN, int S, int EPI>
__device__ __forceinline__ void gemm_ring_run(const KernelArgs<EPI>& g, int m0, int n0, int part, uint32_t tile, int uw) {
    constexpr int WM = BM / 2, WN = BN / 2;        // wave quadrant
    constexpr int MT = WM / 32, NT = WN / 32;      // 32x32 MFMA tiles per wave
    constexpr int LA = BM / 32, LW = BN / 32, L = LA + LW;     // wave-loads (8 rows each) per wave and slab
    constexpr int STAGE = (BM + BN) * ROWB;

    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int li = lane & 31, lg = lane >> 5;
    const int wm0 = (uw & 1) * WM, wn0 = (uw >> 1) * WN;

    uint32_t a_voff[LA], w_voff[LW];               // byte offsets from the tile's first row
#pragma unroll
    for (int j = 0; j < LA; ++j) {
        const int row = (j * 4 + uw) * 8 + lane / CHUNKS;
        a_voff[j] = (uint32_t)row * (uint32_t)g.lda * 2u + ((lane % CHUNKS) ^ swz(row)) * 16;
    }
#pragma unroll
    for (int j = 0; j < LW; ++j) {
        const int row = (j * 4 + uw) * 8 + lane / CHUNKS;
        w_voff[j] = (uint32_t)row * (uint32_t)g.K * 2u + ((lane % CHUNKS) ^ swz(row)) * 16;
    }
    const uint64_t t_begin = g.w_off + (uint64_t)n0 * g.K * 2, t_end = g.w_off + (uint64_t)min(n0 + BN, g.N) * g.K * 2;
    const bool straddle = g.W.split > t_begin && g.W.split < t_end;
    const void* const a_base = g.A + (size_t)m0 * g.lda;
    const void* const w_base = wv_ptr(g.W, t_begin);
    const uint32_t a_bytes = rsrc_bytes(((uint64_t)(g.M - 1 - m0) * g.lda + g.K) * 2), w_bytes = rsrc_bytes(t_end - t_begin);

    floatx16 acc[NT][MT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    lds_frag *a_frag[KSTEPS], *w_frag[KSTEPS];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
        const int c = ((kk * 2 + lg) ^ swz(li)) << 4;
        a_frag[kk] = (lds_frag*)(smem + (wm0 + li) * ROWB + c);
        w_frag[kk] = (lds_frag*)(smem + BM * ROWB + (wn0 + li) * ROWB + c);
    }
    // slabs of this workgroup: all, or those of its part
    constexpr bool CUT = cut_sum(EPI) || EPI == EPI_LAST_PART;
    const int kt0 = CUT ? part * g.part_slabs : 0;
    const int KT = CUT ? min(g.part_slabs, g.K / BK - kt0) : g.K / BK;
    bf16x8 fa[2][MT][KSTEPS], fw[2][NT][KSTEPS];

    struct Src { __amdgpu_buffer_rsrc_t a, w; uint32_t k0; bool on; };
    auto source = [&](int kt) {
        const bool on = kt < KT;
        return Src{make_rsrc(a_base, on ? a_bytes : 0u), make_rsrc(w_base, on ? w_bytes : 0u), on ? (uint32_t)(kt0 + kt) * (BK * 2) : 0u, on};
    };
    auto issue = [&](const Src& src, int stage, int q) {       // q-th of L copies of a slab into the stage at byte `stage`
        char* const dst = smem + stage + uw * 1024 + q * 4096;
        if (q < LA) {
            lds_bload16(src.a, a_voff[q < LA ? q : 0], src.k0, dst);
        } else {
            const uint32_t vo = w_voff[q < LA ? 0 : q - LA];
            if (straddle && src.on) {              // rows past the matrix read the tile's first bytes; they are never stored
                const uint64_t o = (uint64_t)vo + src.k0;
                lds_load16(wv_ptr(g.W, t_begin + (o < t_end - t_begin ? o : 0)), dst);
            } else {
                lds_bload16(src.w, vo, src.k0, dst);
            }
        }
    };
    auto read = [&](auto buf, int stage, int r) {              // r-th of (MT + NT) * KSTEPS fragments, k-step by k-step
        const int kk = r / (MT + NT), t = r % (MT + NT);
        if (t < MT) fa[buf.value][t][kk] = a_frag[kk][(stage + t * 32 * ROWB) / 16];
        else fw[buf.value][t - MT][kk] = w_frag[kk][(stage + (t - MT) * 32 * ROWB) / 16];
    };
    auto slab = [&](auto buf, int kt, int here, int next) __attribute__((always_inline)) {
        using Other = std::integral_constant<int, decltype(buf)::value ^ 1>;
        constexpr int NM = KSTEPS * NT * MT, NR = KSTEPS * (MT + NT);
        const Src src = source(kt + S);
        handover<(S - 2) * L>();               // slab kt + 1 has landed; slab kt is in every wave's registers
        int r = 0, u = 0;
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            const int kk = q / (NT * MT), i = (q / MT) % NT, j = q % MT;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[buf.value][i][kk], fa[buf.value][j][kk], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            for (; u * NM < L * (q + 1) && u < L; ++u) issue(src, here, u);
            for (; r * NM < NR * (q + 1) && r < NR; ++r) read(Other{}, next, r);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
#pragma unroll
    for (int st = 0; st < S; ++st) {
        const Src src = source(st);
#pragma unroll
        for (int q = 0; q < L; ++q) issue(src, st * STAGE, q);
    }
    handover<(S - 1) * L>();
#pragma unroll
    for (int r = 0; r < KSTEPS * (MT + NT); ++r) read(I0{}, 0, r);
    int here = 0;
    auto after = [&](int st) { return st == (S - 1) * STAGE ? 0 : st + STAGE; };
    for (int kt = 0; kt < KT; kt += 2) {           // an odd last slab is followed by one of zeros
        int next = after(here);
        slab(I0{}, kt, here, next);
        here = next;
        next = after(here);
        slab(I1{}, kt + 1, here, next);
        here = next;
    }
    if constexpr (EPI == EPI_MEET) gemm_meet<BM, BN>(g, acc, m0, n0, part, tile, uw, smem);
    else gemm_epilogue<BM, BN, EPI>(g, acc, m0, n0, part, uw, smem);
}

// A problem's tiles in the order of their logical ids: groups of about 8 row-tiles, all of one size (a short last group would walk
// every weight tile once more), walked feature-tile-major.
template <int BM, int BN>
struct TileWalk {
    int tiles_m, tiles_n, GM;
    __host__ __device__ __forceinline__ explicit TileWalk(const GemmCore& g) {
        tiles_m = (g.M + BM - 1) / BM;
        tiles_n = (g.n1 - g.n0 + BN - 1) / BN;
        const int n_groups = std::max(1, (tiles_m + 4) / 8);
        GM = (tiles_m + n_groups - 1) / n_groups;
    }
    struct Tile { int m0, n0, above, gsz; };       // first token and feature; row-tiles of its group before it, in all
    __host__ __device__ __forceinline__ Tile at(const GemmCore& g, uint32_t lid, int col_step = 1) const {
        const int group = lid / (GM * tiles_n), in = lid % (GM * tiles_n);
        const int first_m = group * GM;
        const int gsz = std::min(tiles_m - first_m, GM);
        int col = in / gsz;
        if (col_step > 1) col = col * col_step % tiles_n;
        return Tile{(first_m + in % gsz) * BM, g.n0 + col * BN, in % gsz, gsz};
    }
};

// Workgroup `bid` of the `nblk` that problem owns.  S: stages of the ring loop, 0 = the quadrant-phase loop (two stages).
template <int BM, int BN, int S, int EPI>
__device__ __forceinline__ void gemm_tile_body(const KernelArgs<EPI>& g, uint32_t bid, uint32_t nblk, int uw) {
    // logical tile: XCD-contiguous id, then (part of K by part of K) the walk over the tiles
    const TileWalk<BM, BN> walk(g);
    const int tiles_m = walk.tiles_m, tiles_n = walk.tiles_n;
    uint32_t lid = xcd_contiguous_id(bid, nblk);
    int part = cut_sum(EPI) ? lid / (tiles_m * tiles_n) : 0;
    lid -= part * (tiles_m * tiles_n);
    if (EPI == EPI_LAST_PART) part = g.ksplits - 1;
    if (EPI == EPI_MEET && lane_here() == 0) __hip_atomic_fetch_add(g.words + lid * 4 + uw, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int step = 1;
    if constexpr (heads_out(EPI)) step = g.col_step;
    const auto tile = walk.at(g, lid, step);
    int m0 = tile.m0, n0 = tile.n0;
    if constexpr (EPI == EPI_MEET) {           // scalars that the compiler would keep in vector registers, and loop over at every copy
        m0 = __builtin_amdgcn_readfirstlane(m0);
        n0 = __builtin_amdgcn_readfirstlane(n0);
        part = __builtin_amdgcn_readfirstlane(part);
        lid = __builtin_amdgcn_readfirstlane(lid);
    }
    if constexpr (S > 0) {
        gemm_ring_run<BM, BN, S, EPI>(g, m0, n0, part, lid, uw);
    } else {
        const uint64_t t_begin = g.w_off + (uint64_t)n0 * g.K * 2, t_end = g.w_off + (uint64_t)min(n0 + BN, g.N) * g.K * 2;
        if (g.W.split > t_begin && g.W.split < t_end) gemm_tile_run<BM, BN, EPI, true>(g, m0, n0, part, lid, uw);
        else gemm_tile_run<BM, BN, EPI, false>(g, m0, n0, part, lid, uw);
    }
}

// two workgroups per CU: 256 registers
template <int BM, int BN>
constexpr int min_waves() { return BM * BN <= 128 * 128 ? 2 : 1; }

// Two independent problems of one tile shape and epilogue in one launch (the text and image streams
// of a double-stream block, App. B): a small problem's workgroups ride along with the large one's
// instead of holding the chip for the length of their K loop.  The first problem's share of the grid
// is padded to a multiple of 8 so that both keep the block-index-to-XCD correspondence.
template <int EPI>
struct GemmPair {
    KernelArgs<EPI> g[2];
    uint32_t tiles0, tiles0_pad, tiles;        // workgroups of the first problem, with padding, of both
};

// The last round of workgroups leaves CUs without a tile.  There the grid goes on with workgroups that fetch, for the tiles of that
// round, what their CU's copies are about to ask for, into the L2 of the XCD they share (`IdleFetch` is their number and pace).
// A CU's loads return in order, so that a copy that misses L2 holds up all behind it; waves of its own workgroup or of its CU
// fetching ahead wait in the same queue and gain nothing.  No result depends on it: a workgroup that is late, or on another XCD
// than thought, only fetches in vain.
// Operands that come from HBM (sets in turn, 1.2 GB; none / fetching): 2304 x 3072 x 12288 (216 tiles of 128x256) 176.6 / 167.1 us, 1531 x
// 12288 x 3072 (384 of 192x256) 122.9 / 117.1, 512 x 12288 x 3072 52.5 / 50.3.  The same few operands again and again, which the last-level
// cache holds: 149.4 / 151.6, 118.1 / 120.8, 43.6 / 44.0.  A pace 0.8 to 1.75 times this one gives the same within 2 %.
constexpr uint32_t IDLE_MOST = 224;            // tiles of a last round beside which fetching still pays
constexpr int FETCH_SLABS = 4, FETCH_LEAD = 2; // a chunk is 512 bytes of a row; the first ones are asked for before a fetch could help

// What a fetching workgroup reads of the tiles on its XCD in the last round, of which `lane` is one and lane0 the first of its problem:
// in each problem their logical ids follow one another, so a weight panel begins with every walk over a group's row-tiles, and
// the row-tiles of the first walk are all there are.
template <int BM, int BN>
struct TilePanels {
    typename TileWalk<BM, BN>::Tile t;
    uint64_t k0, w_begin, w_bytes, a_begin, a_bytes;   // first byte of the part of K; panels in bytes of the weight blob (before k0) and of A (behind it)
    __host__ __device__ __forceinline__ TilePanels(const GemmCore& g, bool cut, uint32_t lid) {
        const TileWalk<BM, BN> walk(g);
        const uint32_t whole = walk.tiles_m * walk.tiles_n, part = cut ? lid / whole : 0;
        t = walk.at(g, lid - part * whole);
        k0 = cut ? (uint64_t)part * g.part_slabs * (BK * 2) : 0;
        w_begin = g.w_off + (uint64_t)t.n0 * g.K * 2;
        const uint64_t w_end = g.w_off + (uint64_t)std::min(t.n0 + BN, g.n1) * g.K * 2;
        const uint64_t w1 = g.W.split > w_begin && g.W.split < w_end ? g.W.split : w_end;      // what lies in one buffer
        w_bytes = w1 > w_begin + k0 ? w1 - w_begin - k0 : 0;
        a_begin = (uint64_t)t.m0 * g.lda * 2 + k0;
        a_bytes = ((uint64_t)(std::min(g.M - t.m0, BM) - 1) * g.lda + g.K) * 2 - k0;
    }
    __host__ __device__ __forceinline__ bool lists_w(int lane, int lane0) const { return lane == lane0 || t.above == 0; }
    __host__ __device__ __forceinline__ bool lists_a(int lane, int lane0) const { return lane - lane0 < t.gsz; }
};

struct Panel { uint64_t base; uint32_t bytes, row_bytes; };
// The panels of one problem's tiles among them, the lane's tile (if any) being `lid`.  -> panels listed so far
template <int BM, int BN, int EPI>
__device__ __forceinline__ int list_panels(const GemmCore& g, Panel* panels, int n, bool on, uint32_t lid, bool with_a) {
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const TilePanels<BM, BN> p(g, cut_sum(EPI), on ? lid : 0);
    const int lane0 = __ffsll((unsigned long long)__ballot(on)) - 1;
    const bool new_w = on && p.lists_w(lane, lane0), new_a = on && with_a && p.lists_a(lane, lane0);
    const uint64_t wm = __ballot(new_w), am = __ballot(new_a), below = (1ull << lane) - 1;
    if (new_w) panels[n + __popcll(wm & below)] = Panel{(uint64_t)(uintptr_t)wv_ptr(g.W, p.w_begin) + p.k0, rsrc_bytes(p.w_bytes), (uint32_t)g.K * 2u};
    n += __popcll(wm);
    if (new_a) panels[n + __popcll(am & below)] = Panel{(uint64_t)(uintptr_t)g.A + p.a_begin, rsrc_bytes(p.a_bytes), (uint32_t)g.lda * 2u};
    return n + __popcll(am);
}
// tiles0, tiles0_pad, tiles: as in GemmPair; one problem: all three alike
template <int BM, int BN, int EPI>
__device__ __forceinline__ void gemm_idle_fetch(const GemmCore& g0, const GemmCore& g1, uint32_t tiles0, uint32_t tiles0_pad, uint32_t tiles, const IdleFetch& f, uint32_t bid, int uw) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    Panel* const panels = (Panel*)smem;                        // at most 2 x 32
    int* const count = (int*)(smem + 64 * sizeof(Panel));
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    if (uw == 0) {
        const uint32_t b = (tiles & ~255u) + (bid & 7u) + 8u * lane;       // a lane per tile of the round on this XCD
        int n = list_panels<BM, BN, EPI>(g0, panels, 0, b < tiles0, xcd_contiguous_id(b, tiles0), f.with_a);
        if (tiles > tiles0_pad) n = list_panels<BM, BN, EPI>(g1, panels, n, b >= tiles0_pad && b < tiles, xcd_contiguous_id(b - tiles0_pad, tiles - tiles0_pad), f.with_a);
        if (lane == 0) *count = n;
    }
    __syncthreads();
    // the waves of all fetching workgroups of this XCD, two rows of a chunk each at a time
    const uint32_t before = (tiles + 7u - (bid & 7u)) >> 3, helpers = ((tiles + f.workgroups + 7u - (bid & 7u)) >> 3) - before;
    const uint32_t waves = helpers * 4, mine = ((bid >> 3) - before) * 4 + uw;
    constexpr uint32_t PAIRS = (BN > BM ? BN : BM) / 2;
    const uint32_t slabs = cut_sum(EPI) ? g0.part_slabs : g0.K / BK, pairs = (uint32_t)*count * PAIRS, chunks = (slabs + FETCH_SLABS - 1) / FETCH_SLABS;
    const unsigned long long begin = __builtin_amdgcn_s_memrealtime();
    for (uint32_t c = FETCH_LEAD; c < chunks; c += f.stride) {
        unsigned long long t;
        while ((t = __builtin_amdgcn_s_memrealtime() - begin) < (c - FETCH_LEAD) * f.ticks_per_chunk) __builtin_amdgcn_s_sleep(2);
        if (t > f.deadline) break;
        for (uint32_t i = mine; i < pairs; i += waves) {
            const Panel q = panels[i / PAIRS];
            const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)q.base), hi = __builtin_amdgcn_readfirstlane((uint32_t)(q.base >> 32));
            const __amdgpu_buffer_rsrc_t rs = make_rsrc((const void*)(uintptr_t)((uint64_t)hi << 32 | lo), __builtin_amdgcn_readfirstlane(q.bytes));
            const uint32_t row = (i % PAIRS) * 2 + (lane >> 5);
            lds_bload16(rs, row * q.row_bytes + c * (FETCH_SLABS * ROWB) + (lane & 31) * 16, 0, smem + 2048 + uw * 1024);      // kept nowhere
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // before the LDS is another workgroup's
}
// Tiles with one workgroup per CU; two problems of the largest take all registers as it is, and the last part of a cut sum has a
// launch of its own only where a batch fills the chip (gemm_plan).
constexpr bool can_idle_fetch(int bm, int bn, int epi, bool pair) { return bm * bn > 128 * 128 && epi != EPI_LAST_PART && !(pair && bm * bn == 256 * 256); }

template <int BM, int BN, int S, int EPI>
__global__ __launch_bounds__(256, (min_waves<BM, BN>())) void gemm_bf16_kernel(KernelArgs<EPI> g, uint32_t tiles, IdleFetch f) {
    const int uw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (!can_idle_fetch(BM, BN, EPI, false) || blockIdx.x < tiles) gemm_tile_body<BM, BN, S, EPI>(g, blockIdx.x, tiles, uw);
    else gemm_idle_fetch<BM, BN, EPI>(g, g, tiles, tiles, tiles, f, blockIdx.x, uw);
}
template <int BM, int BN, int S, int EPI>
__global__ __launch_bounds__(256, (min_waves<BM, BN>())) void gemm_pair_kernel(GemmPair<EPI> p, IdleFetch f) {
    const int uw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (can_idle_fetch(BM, BN, EPI, true)) {
        if (blockIdx.x >= p.tiles) { gemm_idle_fetch<BM, BN, EPI>(p.g[0], p.g[1], p.tiles0, p.tiles0_pad, p.tiles, f, blockIdx.x, uw); return; }
    }
    const uint32_t tiles1 = p.tiles - p.tiles0_pad;
    if constexpr (heads_out(EPI) || EPI == EPI_MEET) {         // one body for both problems: two of them cost registers across each other
        const uint32_t second = blockIdx.x >= p.tiles0_pad;
        if (second || blockIdx.x < p.tiles0)
            gemm_tile_body<BM, BN, S, EPI>(p.g[second], blockIdx.x - (second ? p.tiles0_pad : 0), second ? tiles1 : p.tiles0, uw);
    } else {
        if (blockIdx.x < p.tiles0) gemm_tile_body<BM, BN, S, EPI>(p.g[0], blockIdx.x, p.tiles0, uw);
        else if (blockIdx.x >= p.tiles0_pad) gemm_tile_body<BM, BN, S, EPI>(p.g[1], blockIdx.x - p.tiles0_pad, tiles1, uw);
    }
}

template <int BM, int BN, int S, int EPI>
constexpr size_t gemm_smem() {
    constexpr size_t loop = (size_t)(S > 0 ? S : STAGES) * (BM + BN) * ROWB;
    static_assert(!heads_out(EPI) || (size_t)BM * BN * 2 <= loop, "a tile of heads is staged whole");
    constexpr size_t epi = EPI == EPI_MEET ? Meet<BM, BN>::BYTES : (joint_slices(BN, EPI) ? 2 : 4) * StageOf<BM, BN, EPI>::BYTES;
    return loop > epi ? loop : epi;
}

template <class Kernel>
hipError_t allow_smem(Kernel kernel, size_t smem) {
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
}

// workgroups that the tiles of one problem take
inline uint32_t tile_count(const GemmArgs& g, int bm, int bn, bool cut) {
    return (uint32_t)(((g.M + bm - 1) / bm) * ((g.n1 - g.n0 + bn - 1) / bn)) * (cut ? g.ksplits : 1);
}

// the first problem's share of a launch of two
inline uint32_t pad_tiles(uint32_t tiles) { return (tiles + 7u) & ~7u; }

// The order in which the feature-tiles of a launch whose tiles are not alike (heads, activated) are walked, so that each XCD, which has a
// range of them, gets its share of either sort: every step-th, a golden section of them.  For launches of more than two rounds: single-stream
// blocks in order / in steps 943.6 / 935.2 us (2900 x 22592 x 3072, erf), 1371 / 1363 and 1190.5 / 1179.3 (4500 and 4608 x 21504 x 3072), others
// 0.1 % faster, 8800 x 13376 x 2048 1367 / 1375; of 756 tiles (2304 x 21504 x 3072) it depends on the chip: the launch 260 / 264, 264 / 260 us.
inline int even_step(int tiles_n) {
    int step = std::max(1, (int)(0.618 * tiles_n + 0.5));
    auto common = [&](int a, int b) { while (b) { const int t = a % b; a = b; b = t; } return a; };
    while (common(step, tiles_n) != 1) ++step;
    return step;
}

template <int BM, int BN, int S, int EPI>
hipError_t launch(const GemmArgs& g_in, const GemmArgs* second, hipStream_t s) {
    constexpr bool cut = cut_sum(EPI);
    GemmArgs g = g_in;
    if (heads_out(EPI) && !second && tile_count(g, BM, BN, cut) > 512) g.col_step = even_step((g.n1 - g.n0 + BN - 1) / BN);
    const uint32_t tiles = tile_count(g, BM, BN, cut);
    constexpr size_t smem = gemm_smem<BM, BN, S, EPI>();
    if (!second) {
        static const hipError_t allowed = allow_smem(gemm_bf16_kernel<BM, BN, S, EPI>, smem);
        if (allowed != hipSuccess) return allowed;
        const IdleFetch f = can_idle_fetch(BM, BN, EPI, false) ? gemm_idle_fetch_plan(BM, BN, cut, g, nullptr, tiles, 0) : IdleFetch{};
        hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, S, EPI>), dim3(tiles + f.workgroups), dim3(256), smem, s, (const KernelArgs<EPI>&)g, tiles, f);
    } else if constexpr ((BM * BN == 65536 && cut_sum(EPI)) || (BN < 128 && EPI == EPI_MEET)) {
        return hipErrorInvalidValue;               // does not fit the registers; gemm_plan never asks for it
    } else {
        static const hipError_t allowed = allow_smem(gemm_pair_kernel<BM, BN, S, EPI>, smem);
        if (allowed != hipSuccess) return allowed;
        GemmPair<EPI> p;
        p.g[0] = g;
        p.g[1] = *second;
        p.tiles0 = tiles;
        p.tiles0_pad = pad_tiles(p.tiles0);
        p.tiles = p.tiles0_pad + tile_count(*second, BM, BN, cut);
        const IdleFetch f = can_idle_fetch(BM, BN, EPI, true) ? gemm_idle_fetch_plan(BM, BN, cut, g, second, p.tiles, p.tiles - p.tiles0_pad) : IdleFetch{};
        hipLaunchKernelGGL((gemm_pair_kernel<BM, BN, S, EPI>), dim3(p.tiles + f.workgroups), dim3(256), smem, s, p, f);
    }
    return hipGetLastError();
}

// one problem, or two in one launch, with the given tile shape
template <int EPI>
hipError_t launch_tile(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s) {
    switch (tile) {
        case GEMM_256x256: return launch<256, 256, 0, EPI>(g, second, s);
        case GEMM_128x128: return launch<128, 128, 0, EPI>(g, second, s);
        case GEMM_128x256: return launch<128, 256, 0, EPI>(g, second, s);
        case GEMM_192x256: return launch<192, 256, 0, EPI>(g, second, s);
        case GEMM_128x64: return launch<128, 64, 3, EPI>(g, second, s);        // 72 and 80 KB of LDS: two workgroups per CU
        case GEMM_64x64: return launch<64, 64, 5, EPI>(g, second, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace
