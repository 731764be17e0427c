// Full (non-causal, unmasked) softmax attention for the heads this rank owns, over the whole
// joint sequence (App. B: the 4*B*S^2*d term; Sec. 2.1: under Ulysses each rank attends over all
// N tokens for H/P heads).  Flash-style: the nq x nk score matrix is never materialised; keys
// and values stream through LDS in tiles of 64 keys with an online softmax.
//
// The kernel works on the transposed problem so that no data ever changes lanes between the
// two contractions:
//   S^T[key, query] = K . Q^T      (MFMA A = key rows from LDS,   B = query fragment in registers)
//   O^T[d,   query] = V^T . P^T    (MFMA A = V^T rows from LDS,   B = P^T built from S^T registers)
// With 32x32x16 MFMAs a lane owns ONE query column, so the softmax reference and the row sum are
// per-lane scalars and a rescale of O^T is a lane-uniform multiply.  The 32 key rows of each S^T tile
// are fed in an order that swaps bits 2 and 3 of the row index; the accumulator registers
// v=8a..8a+7 of lane group g then hold keys 16a+8g .. 16a+8g+7 in order, which is exactly the
// B-operand layout of the second contraction (8 consecutive k per lane), so P^T is a pure
// register repack.  V is kept transposed in HBM ([head, d, key]) so that its A-operand rows
// are contiguous 16-byte reads as well.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "modvec.h"

namespace {

// One wave-load: 64 lanes x 16 bytes from global memory straight into 1 KiB of consecutive LDS.
// The address is base + voff (per lane) + soff (uniform, advanced per tile); lanes whose offset
// lies past the resource's size fetch zeros, which takes care of the ragged last K tile.
__device__ __forceinline__ void lds_bload16(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, uint32_t soff, void* lds) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (void __attribute__((address_space(3)))*)lds, 16, voff, soff, 0, 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)(bytes > 0xffffffffull ? 0xffffffffu : (uint32_t)bytes), 0x00020000);
}

constexpr int BKV = 64;    // keys per tile
constexpr float kNoRef = -3.402823466e38f;     // reference of a query before its first score: finite, so that a tile, and with it
                                               // a whole part of the keys, may hold nothing but -inf scores (weights of zero)

__device__ __forceinline__ float max3f(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }

// Where the output row of query q of head h goes, or NULL.
template <int HD>
__device__ __forceinline__ bf16* out_row(const AttnArgs& a, int h, int q) {
    if (q >= a.nq) return nullptr;
    const int hps = a.hps ? a.hps : a.H;            // heads per sample of a batch
    const int b = h / hps, hh = h % hps;
    if (!a.scatter) return a.O + (size_t)b * a.o_bs + (size_t)hh * a.o_hs + (size_t)q * a.o_qs;
    // the second exchange by the stores themselves: this rank's positions go to the projection operand,
    // the others to the send buffer (in ascending position order, as the receiver expects them)
    const TokenMap& m = a.map;
    if (q >= m.pos0 && q < m.pos0 + m.len0) return a.dst0 + (size_t)b * a.bs0 + (size_t)(q - m.pos0) * a.ld + (a.h0 + hh) * HD;
    if (q >= m.pos1 && q < m.pos1 + m.len1) return a.dst1 + (size_t)b * a.bs1 + (size_t)(q - m.pos1) * a.ld + (a.h0 + hh) * HD;
    const int ri = q - (q >= m.pos0 + m.len0 ? m.len0 : 0) - (q >= m.pos1 + m.len1 ? m.len1 : 0);
    return a.send ? a.send + (size_t)b * a.send_bs + ((size_t)hh * (m.n_total - m.n_local) + ri) * HD : nullptr;
}

// Output row of query q of head h, times inv: lane = query, value(d, 4*vb + e) = column d*32 + vb*8 + lg*4 + e.
template <int HD, class Value>
__device__ __forceinline__ void store_rows(const AttnArgs& a, int h, int q, int lg, Value&& value, float inv) {
    bf16* const op = out_row<HD>(a, h, q);
    if (!op) return;
#pragma unroll
    for (int d = 0; d < HD / 32; ++d)
#pragma unroll
        for (int vb = 0; vb < 4; ++vb) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (bf16)(value(d, vb * 4 + e) * inv);
            *(bf16x4*)(op + d * 32 + vb * 8 + lg * 4) = w;
        }
}

// What a sweep holds after some of its tiles, as it lies in registers: O^T a KiB per store and wave, then reference and
// row sum of every lane.  A workgroup's state is state_floats<HD, NW>() long.
template <int HD>
__device__ __forceinline__ void store_state(float* to, int wave, int lane, const floatx16 (&o)[HD / 32], float mc, float l_run) {
    float* const p = to + wave * (64 * (HD / 2 + 2));
#pragma unroll
    for (int i = 0; i < HD / 8; ++i) {
        const floatx4 v = {o[i / 4][i % 4 * 4], o[i / 4][i % 4 * 4 + 1], o[i / 4][i % 4 * 4 + 2], o[i / 4][i % 4 * 4 + 3]};
        *(floatx4*)(p + i * 256 + lane * 4) = v;
    }
    *(float2*)(p + HD / 8 * 256 + lane * 2) = make_float2(mc, l_run);
}
template <int HD>
__device__ __forceinline__ void load_state(const float* from, int wave, int lane, floatx16 (&o)[HD / 32], float& mc, float& l_run) {
    const float* const p = from + wave * (64 * (HD / 2 + 2));
#pragma unroll
    for (int i = 0; i < HD / 8; ++i) {
        const floatx4 v = *(const floatx4*)(p + i * 256 + lane * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[i / 4][i % 4 * 4 + e] = v[e];
    }
    const float2 ml = *(const float2*)(p + HD / 8 * 256 + lane * 2);
    mc = ml.x;
    l_run = ml.y;
}

// A part of the keys joined to the ones before it, (m, l) and (mc, l_part) the references and row sums: both brought to the higher
// reference.  One order and one rounding for the workgroup that has all parts and for the kernel that reads them.
struct Joint {
    float before, part;                        // factors
    __device__ __forceinline__ float join(float sum, float o) const { return fmaf(o, part, __fmul_rn(sum, before)); }
};
__device__ __forceinline__ Joint join_part(float& m, float& l, float mc, float l_part) {
    const float hi = fmaxf(m, mc);
    const Joint f = {__builtin_amdgcn_exp2f(m - hi), __builtin_amdgcn_exp2f(mc - hi)};
    l = f.join(l, l_part);
    m = hi;
    return f;
}

// One sweep of a workgroup (NW waves of 32 queries each, the wave's first at q0) over the key tiles [T0, T1) of head h.
// `from`: not NULL = go on from the state another workgroup left there after the tiles before T0 (store_state).
// repeat() is asked where a tile was out of the fast softmax's range: whether the sweep is to be repeated here; if not, finish
// is not called.  In a repeated sweep the waves that were in range compute what they did before: a query's bits depend on the 32
// queries of its wave, and not on how many waves a workgroup has or whose keys are in parts.  finish(o, mc, l) gets O^T, the reference it is taken against and the lane's row sum.
// ALL_PARTS: the tiles are parts of a.part_tiles (an even number) one after the other, each swept as by a workgroup of its own
// and joined to the ones before (join_part) in registers; the copies run on from part to part.
enum { FIRST, FAST, REPEATED };                 // tiles: of a sweep's beginning, of its rest, of the rest of a repeated one
template <int HD, int NW, bool ALL_PARTS, class Repeat, class Finish>
__device__ __forceinline__ void attn_sweep(const AttnArgs& a, int h, int q0, int T0, int T1, const float* from, Repeat&& repeat, Finish&& finish) {
    constexpr int KCH = HD / 8;                 // 16-byte chunks per K row
    constexpr int KROW = HD * 2;                // bytes per K row in LDS
    constexpr int KL = BKV * KCH / 64, VL = HD * 8 / 64;   // wave-loads (1 KiB each) per K / V^T tile
    constexpr int LPW = (KL + VL + NW - 1) / NW;           // wave-loads per wave per tile (round robin)
    constexpr int K_TILE = BKV * KROW, V_TILE = HD * 128;
    constexpr int DT = HD / 32;                 // 32-row tiles of O^T
    constexpr int KS = HD / 16;                 // k-steps of the first contraction

    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const sK = smem;                      // [2][BKV][KROW]
    char* const sV = smem + 2 * K_TILE;         // [2][HD][128]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lj = lane & 31, lg = lane >> 5;

    // K swizzle: 256-byte rows (HD=128) rotate over 16 chunk slots, 128-byte rows over 8
    auto kswz = [](int key) { return HD == 128 ? (key & 15) : (((key >> 1) & 7) ^ ((key & 1) << 2)); };
    auto vswz = [](int row) { return ((row >> 1) & 7) ^ ((row & 1) << 2); };

    // ---- query fragments (B operand), resident in registers for the whole sweep
    bf16x8 qf[KS];
    {
        const int qr = min(q0 + lj, a.nq - 1);
        const bf16* qp = a.Q + ((size_t)h * a.nq + qr) * HD + lg * 8;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) qf[kk] = *(const bf16x8*)(qp + kk * 16);
    }

    // ---- tile copies go global -> LDS directly: one load writes the wave's 64 x 16 bytes to
    // consecutive LDS addresses (1 KiB = 1024/KROW key rows, or 8 V^T rows); the 16-byte chunk a
    // lane fetches is the one whose swizzled slot it fills.  Per-lane offsets are computed once; a
    // tile only advances the uniform offset, so the copies cost no vector instructions per tile.
    // Key rows past nk read zeros (their scores are masked below); V^T rows are padded to nk_pad.
    const int uw = __builtin_amdgcn_readfirstlane(wave);
    constexpr int K_RPL = 1024 / KROW;          // key rows per wave-load
    const __amdgpu_buffer_rsrc_t k_rsrc = make_rsrc(a.K + (size_t)h * a.nk * HD, (uint64_t)a.nk * KROW);
    const __amdgpu_buffer_rsrc_t v_rsrc = make_rsrc(a.Vt + (size_t)h * HD * a.nk_pad, (uint64_t)HD * a.nk_pad * 2);
    uint32_t t_voff[LPW];                       // wave-load j = jj * NW + wave: K loads first, then V^T
#pragma unroll
    for (int jj = 0; jj < LPW; ++jj) {
        const int j = jj * NW + uw;
        if (j < KL) {
            const int key = j * K_RPL + lane / KCH;
            t_voff[jj] = (uint32_t)key * KROW + (((lane % KCH) ^ kswz(key)) << 4);
        } else {
            const int row = min(j - KL, VL - 1) * 8 + (lane >> 3);
            t_voff[jj] = (uint32_t)row * (uint32_t)a.nk_pad * 2 + (((lane & 7) ^ vswz(row)) << 4);
        }
    }
    auto issue_tile = [&](int t, int buf) {
        const uint32_t k_soff = (uint32_t)t * (BKV * KROW), v_soff = (uint32_t)t * (BKV * 2);
#pragma unroll
        for (int jj = 0; jj < LPW; ++jj) {
            // with KL a multiple of NW a wave-load's role is known at compile time
            constexpr bool kStatic = KL % NW == 0;
            const int j = jj * NW + uw;         // wave-uniform
            const bool is_k = kStatic ? jj < KL / NW : j < KL;
            if (is_k)
                lds_bload16(k_rsrc, t_voff[jj], k_soff, sK + buf * K_TILE + j * 1024);
            else if (kStatic || j < KL + VL)
                lds_bload16(v_rsrc, t_voff[jj], v_soff, sV + buf * V_TILE + (j - KL) * 1024);
        }
    };

    floatx16 o[DT];
    float mc, l_run;                            // reference of the exponentials (base-2 units), row sum
    const float c2 = a.scale * 1.4426950408889634f;   // logits in base-2 units

    // key row fed to MFMA row i: swap bits 2 and 3 of i
    const int krow = (lj & 0x13) | ((lj & 4) << 1) | ((lj & 8) >> 1);

    int out_of_range = 0;                       // wave-uniform: a fast tile met scores it could not take
    __shared__ int any_out_of_range;            // ... of any wave of the workgroup: written before a tile's barrier, read after it
    if (tid == 0) any_out_of_range = 0;
    bool tracks = false;                        // of a repeated sweep, wave-uniform: tiles past the first track, too
    const int T_end = T1;                       // of the copies

    // One tile.  The LDS buffer is a compile-time constant so that fragment addresses are a per-lane
    // register plus an immediate.
    //
    // Softmax is invariant to the reference its exponentials are taken against, as long as numerator and
    // denominator share it; magnitudes only have to stay inside the fp32 / bf16 range, whose relative
    // precision does not depend on scale.  A tracking tile does what online softmax usually does: take
    // the tile's maximum, move the reference there, rescale O^T and the row sum (of the first tile, which always tracks, there is
    // nothing to rescale).  A fast tile takes no
    // maximum: it forms P^T = exp2(s * c2 - mc) against the reference it inherits (one FMA, one exp2 and
    // half a conversion per score) and looks at the row sums afterwards.  A query whose 64 values add
    // up to 2^20 or more has its reference, O^T and row sum shifted by a whole power of two (exact); if
    // they add up to 2^64 or more, or to no number (exp2 overflowed), the tile is declared out of range:
    // nothing is repaired on the spot, the workgroup repeats the whole sweep, and this wave its own with tracking tiles.
    auto tile = [&](int t, auto buf_c, auto mode_c) __attribute__((always_inline)) {
        constexpr int buf = decltype(buf_c)::value, mode = decltype(mode_c)::value;
        if (t + 1 < T_end) issue_tile(t + 1, buf ^ 1);
        const char* cK = sK + buf * K_TILE;
        const char* cV = sV + buf * V_TILE;

        // ---- S^T = K . Q^T for 2 x 32 keys.  MFMA i handles key half (i & 1) and k-step (i >> 1), so
        // consecutive MFMAs hit different accumulators; K fragments run 4 reads ahead in a ring.
        // Register v of tile mt is key k0 + mt*32 + 16*(v/8) + 8*lg + v%8; keys past nk score -inf.
        floatx16 s[2];
        const int k0 = t * BKV;
        {
            bf16x8 kf[4];
            auto kfrag = [&](int i) {
                const int key = (i & 1) * 32 + krow, c = (i >> 1) * 2 + lg;
                return *(const bf16x8*)(cK + key * KROW + ((c ^ kswz(key)) << 4));
            };
#pragma unroll
            for (int i = 0; i < 4; ++i) kf[i] = kfrag(i);
#pragma unroll
            for (int i = 0; i < 2 * KS; ++i) {
                if (i < 2) {
                    floatx16 z;
#pragma unroll
                    for (int v = 0; v < 16; ++v) z[v] = 0.f;
                    s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i & 3], qf[i >> 1], z, 0, 0, 0);
                } else {
                    s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i & 3], qf[i >> 1], s[i & 1], 0, 0, 0);
                }
                if (i + 4 < 2 * KS) kf[i & 3] = kfrag(i + 4);
            }
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
            for (int i = 0; i < 2 * KS - 4; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
        }
        if (k0 + BKV > a.nk) {
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int key = k0 + mt * 32 + 16 * (v >> 3) + 8 * lg + (v & 7);
                    if (key >= a.nk) s[mt][v] = -INFINITY;
                }
        }
        // first V^T fragments: issued now so that they land while the softmax runs
        bf16x8 vf[4];
        auto vfrag = [&](int i) {                   // i = ks * DT + d
            const int row = (i % DT) * 32 + lj, c = (i / DT) * 2 + lg;
            return *(const bf16x8*)(cV + row * 128 + ((c ^ vswz(row)) << 4));
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) vf[i] = vfrag(i);
        // The softmax stays between two scheduling fences: in one region with the second contraction the
        // compiler threads the exponentials between its MFMAs, which measured 5 % slower than keeping
        // the three phases apart and leaving the overlap to the SIMD's other wave.
        __builtin_amdgcn_sched_barrier(0);

        float alpha = 1.f;
        if (mode == FIRST || (mode == REPEATED && tracks)) {
            float mx;                                   // the lane's 32 scores: a tree of three-input maxima
            {
                float m3[11];
#pragma unroll
                for (int i = 0; i < 10; ++i) m3[i] = max3f(s[(3 * i) >> 4][(3 * i) & 15], s[(3 * i + 1) >> 4][(3 * i + 1) & 15], s[(3 * i + 2) >> 4][(3 * i + 2) & 15]);
                m3[10] = fmaxf(s[1][14], s[1][15]);
                const float a0 = max3f(m3[0], m3[1], m3[2]), a1 = max3f(m3[3], m3[4], m3[5]), a2 = max3f(m3[6], m3[7], m3[8]);
                mx = max3f(max3f(a0, a1, a2), m3[9], m3[10]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float mc_new = fmaxf(mc, mx * c2);                             // -inf where all scores are: mc stays
            if constexpr (mode == REPEATED) {
                alpha = __builtin_amdgcn_exp2f(mc - mc_new);                     // 0 from kNoRef
#pragma unroll
                for (int d = 0; d < DT; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[d][v] *= alpha;
            }
            mc = mc_new;
        }

        // ---- P^T in bf16, in the B-operand layout of the second contraction (fragment ks = registers
        // 8*(ks&1).. of half ks>>1).  The row sum adds the rounded values in pairs (bf16 dot product with
        // (1, 1), fp32 accumulate): the weights the second contraction really applies to V.
        bf16x8 pf[4];
        float psum;
        {
            float ps[4] = {0.f, 0.f, 0.f, 0.f};           // four chains: a row sum is not one long dependency
            bf16x2 ones;
            ones[0] = (bf16)1.0f;
            ones[1] = (bf16)1.0f;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    bf16x2 pp;
                    pp[0] = (bf16)__builtin_amdgcn_exp2f(fmaf(s[ks >> 1][8 * (ks & 1) + e], c2, -mc));
                    pp[1] = (bf16)__builtin_amdgcn_exp2f(fmaf(s[ks >> 1][8 * (ks & 1) + e + 1], c2, -mc));
                    pf[ks][e] = pp[0];
                    pf[ks][e + 1] = pp[1];
                    ps[(e >> 1) & 3] = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, ps[(e >> 1) & 3], false);
                }
            psum = (ps[0] + ps[1]) + (ps[2] + ps[3]);
        }
        l_run = mode == REPEATED ? fmaf(l_run, alpha, psum) : l_run + psum;
        __builtin_amdgcn_sched_barrier(0);

        // ---- O^T += V^T . P^T: MFMA i handles k-step (i / DT) of 16 keys and d-tile (i % DT);
        // V^T fragments keep running 4 reads ahead
        {
#pragma unroll
            for (int i = 0; i < 4 * DT; ++i) {
                o[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i & 3], pf[i / DT], o[i % DT], 0, 0, 0);
                if (i + 4 < 4 * DT) vf[i & 3] = vfrag(i + 4);
            }
#pragma unroll
            for (int i = 0; i < 4 * DT - 4; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 1);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 1);
        }

        if (mode == FAST || (mode == REPEATED && !tracks)) {
            const float row = psum + __shfl_xor(psum, 32);
            if (__any(!(row < 1048576.0f))) {
                if (__any(!(row < 18446744073709551616.0f))) {
                    out_of_range = 1;
                    any_out_of_range = 1;
                } else {
                    // queries at or past 2^20: divide by 2^e, e = the sum's binary exponent; the others keep e = 0
                    const int e = row < 1048576.0f ? 0 : (int)(__float_as_uint(row) >> 23) - 127;
                    const float alpha = __uint_as_float((uint32_t)(127 - e) << 23);
                    mc += (float)e;
                    l_run *= alpha;
#pragma unroll
                    for (int d = 0; d < DT; ++d)
#pragma unroll
                        for (int v = 0; v < 16; ++v) o[d][v] *= alpha;
                }
            }
        }

        __syncthreads();                        // tile t+1 has landed, tile t may be overwritten
    };
    // One sweep: the first tile tracks (it sets the reference) unless the state is inherited, the others go in pairs.
    auto sweep = [&](auto mode_c, bool landed) __attribute__((always_inline)) {
        int t = T0;
        if (from) {
            load_state<HD>(from, wave, lane, o, mc, l_run);
            issue_tile(t, 1);
            __syncthreads();                    // (waits for the LDS-DMA, then the barrier)
        } else {
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[d][v] = 0.f;
            mc = kNoRef;
            l_run = 0.f;
            if (!landed) {
                issue_tile(t, 0);
                __syncthreads();
            }
            tile(t, std::integral_constant<int, 0>{}, std::integral_constant<int, FIRST>{});
            ++t;
        }
        for (; t < T1; t += 2) {
            tile(t, std::integral_constant<int, 1>{}, mode_c);
            if (t + 1 < T1) tile(t + 1, std::integral_constant<int, 0>{}, mode_c);
        }
    };
    // the K/V tiles are the workgroup's: if any wave met a tile out of range, all of them go again
    auto again = [&] {
        if (!__builtin_amdgcn_readfirstlane(any_out_of_range)) return false;
        __syncthreads();                        // every wave has read it
        if (tid == 0) any_out_of_range = 0;
        return true;
    };
    if constexpr (ALL_PARTS) {
        floatx16 sum[DT];                       // the parts so far
        float m_sum = kNoRef, l_sum = 0.f;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[d][v] = 0.f;
        for (T0 = 0; T0 < T_end; T0 += a.part_tiles) {
            T1 = min(T_end, T0 + a.part_tiles);
            sweep(std::integral_constant<int, FAST>{}, T0 > 0);
            if (again()) {
                tracks = out_of_range != 0;
                sweep(std::integral_constant<int, REPEATED>{}, false);
                out_of_range = 0;
            }
            const Joint f = join_part(m_sum, l_sum, mc, l_run + __shfl_xor(l_run, 32));
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[d][v] = f.join(sum[d][v], o[d][v]);
        }
        finish(sum, m_sum, l_sum);
    } else {
        sweep(std::integral_constant<int, FAST>{}, false);
        if (again()) {
            if (!repeat()) return;
            tracks = out_of_range != 0;
            sweep(std::integral_constant<int, REPEATED>{}, false);
        }
        finish(o, mc, l_run);
    }
}

// The workgroups behind the sweeps: modulation rows that nothing needs before attention is over.  They stream weights while the matrix
// cores work, on CUs without a sweep or beside one that leaves half of its CU free.
// What remains of their time is what they slow the sweeps by (their own loads in flight, and whether they go past L2 or behind the sweeps'
// waves in the issue order, changed nothing): double-stream block at degree 8, 27 of 40 us of the product gone for 11 us of attention, 326 -> 311 us;
// Wan-like short clip 569 -> 564.
template <int NW>
__device__ __forceinline__ void attn_mod_rows(const AttnArgs& a, uint32_t b) {
    const uint32_t per = (a.mod.n1 - a.mod.n0 + NW * MV_ROWS - 1) / (NW * MV_ROWS), of = b / per;
    modvec_rows<3>(a.mod, of % a.mod.mats, of / a.mod.mats, a.mod.n0 + ((b - of * per) * NW + (threadIdx.x >> 6)) * MV_ROWS);
}

// NW waves of 32 queries each per workgroup: 4 (two workgroups per CU), 7 or 8 (one per CU); for 64-wide heads twice as many,
// held to the 128 registers that takes: at 129 a CU has one 7-wave workgroup and 8 heads x 20892 take 1.11 ms instead of 0.90.
// PARTS: the keys are cut (a.splits > 1), each part for a workgroup of its own, the results go to scratch.  ALL_PARTS: cut alike,
// and a workgroup has all parts of its queries, for which it holds a second O^T: 247 to 251 registers with 128-wide heads; 163 with
// 64-wide ones, where three 4-wave workgroups then share a CU, which costs no time (32 heads x 4696: 198.4 us whole, 198.6).
enum { WHOLE, PARTS, ALL_PARTS };
template <int HD, int NW, int FORM>
__global__ __launch_bounds__(64 * NW, HD == 64 ? (FORM == ALL_PARTS ? 3 : 4) : 2) void attn_fwd_kernel(AttnArgs a) {
    constexpr int BQ = 32 * NW, DT = HD / 32;
    const uint32_t sweeps = gridDim.x - a.mod_blocks;
    if (blockIdx.x >= sweeps) {
        attn_mod_rows<NW>(a, blockIdx.x - sweeps);
        return;
    }
    const int nqt = (a.nq + BQ - 1) / BQ;
    const uint32_t lid = xcd_contiguous_id(blockIdx.x, sweeps);
    const int hs = lid / nqt, qt = lid % nqt;
    const int h = FORM == PARTS ? hs / a.splits : hs, part = FORM == PARTS ? hs % a.splits : 0;       // head, and which part of the keys
    const int q0 = qt * BQ + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 32;
    const int NT = (a.nk + BKV - 1) / BKV;
    const int T0 = FORM == PARTS ? part * a.part_tiles : 0, T1 = FORM == PARTS ? min(NT, T0 + a.part_tiles) : NT;
    attn_sweep<HD, NW, FORM == ALL_PARTS>(a, h, q0, T0, T1, nullptr, [] { return true; }, [&](floatx16 (&o)[DT], float mc, float l_run) {
        const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0)), lj = lane & 31, lg = lane >> 5;
        const float l_tot = FORM == ALL_PARTS ? l_run : l_run + __shfl_xor(l_run, 32);
        if constexpr (FORM == PARTS) {
            // O^T, the reference it is taken against and the row sum as they lie in registers, 1 KiB per store
            if (q0 < a.nq) {
                const size_t tile32 = ((size_t)part * a.H + h) * ((a.nq + 31) / 32) + q0 / 32;
                float* const po = a.part_o + tile32 * (32 * HD);
#pragma unroll
                for (int d = 0; d < DT; ++d)
#pragma unroll
                    for (int vb = 0; vb < 4; ++vb) {
                        const floatx4 v = {o[d][vb * 4], o[d][vb * 4 + 1], o[d][vb * 4 + 2], o[d][vb * 4 + 3]};
                        *(floatx4*)(po + (d * 4 + vb) * 256 + lane * 4) = v;
                    }
                if (lg == 0) *(float2*)(a.part_ml + tile32 * 64 + lj * 2) = make_float2(mc, l_tot);
            }
        } else {
            store_rows<HD>(a, h, q0 + lj, lg, [&](int d, int v) { return o[d][v]; }, 1.0f / l_tot);
        }
    });
}

// The same work dealt out by the kernel itself: one workgroup per CU stays and takes one sweep after the other.  The unit is a
// group of 32 query tiles, one per CU of an XCD, swept in step (they share K and V tiles through the XCD's L2); "lane" j is the
// j-th tile of every group and the j-th CU of every XCD.  A sweep may be cut: the first tiles by one workgroup, which leaves
// the sweep's state in memory, the rest later by another, of another XCD, from there -- the same tiles in the same order, so
// the same bits as one sweep of an 8-wave workgroup.  Should the state not be there when it is needed (its workgroup has not been given a CU for
// kWaitTicks), the sweep starts over from the first tile.  Where a tile is out of the fast softmax's range no state is left,
// only word of it (kUnfit), and the workgroup with the last piece takes the whole sweep, which it then repeats as one
// workgroup would: the bits depend neither on the cut nor on what was waited for.
//
// Two plans.  Even shares (even_units = 0), for a few generations: XCD x takes the x-th eighth of the groups' key tiles laid end
// to end; where an eighth ends inside a group, XCD x sweeps the group's first tiles before anything else and XCD x + 1 goes on
// after its own groups, a generation or more later.  12 heads x 27280 x 128: 3.91 ms, against 4.38 in six generations of 7-wave
// workgroups for 5.72.
// Taken as they come (even_units > 0), for many generations of long sweeps: the XCDs' clocks differ by +-3 %, and dealt out
// alike the slowest decides (12 heads x 119056: XCDs done after 65.2 to 69.7 ms, now all after 66.6: 1306 TFLOP/s).  The
// workgroups of a lane draw groups from a counter; the last even_last groups go in even_cuts pieces each, all first pieces
// before all second ones, so that the end is ragged by a piece and not by a sweep.
constexpr unsigned long long kWaitTicks = 2000000;       // 20 ms of the 100 MHz counter
enum : uint32_t { kStateLeft = 1, kUnfit = 2 };          // flag of a cut sweep; 0 = not there yet
template <int HD>
__global__ __launch_bounds__(512, 2) void attn_even_kernel(AttnArgs a) {
    constexpr int NW = 8, BQ = 32 * NW, DT = HD / 32, STATE = NW * 64 * (HD / 2 + 2);
    __shared__ int shared_word;
    const int lane = threadIdx.x & 63, lj = lane & 31, lg = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int nqt = (a.nq + BQ - 1) / BQ, items = nqt * a.H, NT = (a.nk + BKV - 1) / BKV;
    const int groups = (items + 31) / 32;
    const long total = (long)groups * NT, u0 = total * x / 8, u1 = total * (x + 1) / 8;
    const int g0 = (int)(u0 / NT), t0 = (int)(u0 % NT), g1 = (int)(u1 / NT), t1 = (int)(u1 % NT);     // g1 > g0: at least 8 groups
    // even shares, in steps: the head of group g1 (left for XCD x + 1), the whole groups, the rest of group g0
    const int first_whole = t0 ? g0 + 1 : g0, n_steps = a.even_units ? a.even_units : 1 + (g1 - first_whole) + 1;
    for (int step = 0;; ++step) {
        int group, T0 = 0, T1 = NT, take = -1, leave = -1;      // take, leave: state slots, 32 lanes each
        if (a.even_units) {
            if (threadIdx.x == 0) shared_word = (int)__hip_atomic_fetch_add(a.even_flags + ATTN_FLAGS - 32 + j, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const int u = __builtin_amdgcn_readfirstlane(shared_word);
            __syncthreads();                   // the word is used again below
            if (u >= n_steps) break;
            const int whole = groups - a.even_last;
            group = u;
            if (u >= whole) {
                const int c = (u - whole) / a.even_last, r = (u - whole) % a.even_last;
                group = whole + r;
                T0 = (int)((long)NT * c / a.even_cuts);
                T1 = (int)((long)NT * (c + 1) / a.even_cuts);
                if (c > 0) take = (c - 1) * a.even_last + r;
                if (c + 1 < a.even_cuts) leave = c * a.even_last + r;
            }
        } else {
            if (step >= n_steps) break;
            group = first_whole + step - 1;
            if (step == 0) { if (!t1) continue; group = g1; T1 = t1; leave = x; }
            else if (step == n_steps - 1) { if (!t0) continue; group = g0; T0 = t0; take = x - 1; }
        }
        const int item = group * 32 + j;
        if (item >= items) continue;
        const float* from = nullptr;
        if (take >= 0) {
            if (threadIdx.x == 0) {
                uint32_t* const f = a.even_flags + take * 32 + j;
                const unsigned long long give_up = __builtin_amdgcn_s_memrealtime() + kWaitTicks;
                uint32_t r = 0;
                while (a.even_wait && !(r = __hip_atomic_load(f, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT)) && __builtin_amdgcn_s_memrealtime() < give_up)
                    __builtin_amdgcn_s_sleep(16);
                shared_word = (int)r;
            }
            __syncthreads();                   // orders every wave behind thread 0's acquire
            const uint32_t found = (uint32_t)__builtin_amdgcn_readfirstlane(shared_word);
            if (found == kUnfit && leave >= 0) {
                if (threadIdx.x == 0) __hip_atomic_store(a.even_flags + leave * 32 + j, (uint32_t)kUnfit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __syncthreads();               // the word is written again in the next step
                continue;
            }
            if (found == kStateLeft) from = a.even_state + ((size_t)take * 32 + j) * STATE;
            else T0 = 0;
        }
        const int h = item / nqt, q0 = item % nqt * BQ + wave * 32;
        bool unfit;                            // a tile was out of range, and this workgroup has not all of the sweep
        do {
            unfit = false;
            attn_sweep<HD, NW, false>(a, h, q0, T0, T1, from, [&] { unfit = leave >= 0 || from; return !unfit; }, [&](floatx16 (&o)[DT], float mc, float l_run) {
                if (leave >= 0) {
                    store_state<HD>(a.even_state + ((size_t)leave * 32 + j) * STATE, wave, lane, o, mc, l_run);
                    // One release per workgroup, by thread 0 behind the barrier: it writes back the XCD's whole L2.  By every wave
                    // it cost 57 us.  Its own wait covers its own wave's stores only, and the barrier waits for none: each wave
                    // waits for its stores to have reached the L2 that is written back.
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    __syncthreads();
                    if (threadIdx.x == 0) __hip_atomic_store(a.even_flags + leave * 32 + j, (uint32_t)kStateLeft, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    const float l_tot = l_run + __shfl_xor(l_run, 32);
                    store_rows<HD>(a, h, q0 + lj, lg, [&](int d, int v) { return o[d][v]; }, 1.0f / l_tot);
                }
            });
            T0 = 0;
            from = nullptr;
        } while (unfit && leave < 0);
        if (unfit && threadIdx.x == 0) __hip_atomic_store(a.even_flags + leave * 32 + j, (uint32_t)kUnfit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Keys in parts, a wave to each: the workgroup is 32 queries of a head and as many waves as there are parts, and joins them through
// LDS in the merge kernel's order and rounding (the same bits).  For launches with so few queries that their workgroups are a few
// dozen sweeps side by side.  Every wave copies the tiles of its part into LDS of its own and waits for nobody: the next tile's K
// goes where this one's was as soon as the scores are computed, V after the second contraction.  Bound by the latency of a tile
// and, from about one workgroup per CU on, by what a CU takes in (16 or 32 KB per tile that nobody shares).  (Fragments straight
// from memory, 32 rows x 32 bytes per load, took 0.43 us per tile of 64-wide heads, however many waves shared them.)
// 8 heads x 512 x 64: 7.6 us in two parts, whole 9.3; 3 x 2640 x 128 in three: 29.8, whole 44.8, in parts of their own 33.3 (attn_splits has the line).
constexpr int wave_parts_most(int hd) { return hd == 64 ? 8 : 4; }     // 16 or 32 KB of LDS each
template <int HD>
__global__ __launch_bounds__(64 * wave_parts_most(HD)) void attn_wave_parts_kernel(AttnArgs a) {
    constexpr int DT = HD / 32, KS = HD / 16, QUADS = DT * 4, KCH = HD / 8, KROW = HD * 2;
    constexpr int KL = BKV * KCH / 64, VL = HD * 8 / 64, K_RPL = 1024 / KROW;
    constexpr int K_TILE = BKV * KROW, V_TILE = HD * 128;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, lj = lane & 31, lg = lane >> 5;
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* const sK = smem + part * (K_TILE + V_TILE);
    char* const sV = sK + K_TILE;
    const int nqt = (a.nq + 31) / 32, NT = (a.nk + BKV - 1) / BKV;
    const uint32_t lid = xcd_contiguous_id(blockIdx.x, gridDim.x);
    const int h = lid / nqt, q0 = lid % nqt * 32;
    const int T0 = part * a.part_tiles, T1 = min(NT, T0 + a.part_tiles);       // every part has a tile (attn_check)
    const float c2 = a.scale * 1.4426950408889634f;
    const int krow = (lj & 0x13) | ((lj & 4) << 1) | ((lj & 8) >> 1);
    auto kswz = [](int key) { return HD == 128 ? (key & 15) : (((key >> 1) & 7) ^ ((key & 1) << 2)); };        // as attn_sweep
    auto vswz = [](int row) { return ((row >> 1) & 7) ^ ((row & 1) << 2); };
    const __amdgpu_buffer_rsrc_t k_rsrc = make_rsrc(a.K + (size_t)h * a.nk * HD, (uint64_t)a.nk * KROW);
    const __amdgpu_buffer_rsrc_t v_rsrc = make_rsrc(a.Vt + (size_t)h * HD * a.nk_pad, (uint64_t)HD * a.nk_pad * 2);
    auto issue_k = [&](int t) __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // this wave's reads of the tile before have returned
#pragma unroll
        for (int j = 0; j < KL; ++j) {
            const int key = j * K_RPL + lane / KCH;
            lds_bload16(k_rsrc, (uint32_t)key * KROW + (((lane % KCH) ^ kswz(key)) << 4), (uint32_t)t * K_TILE, sK + j * 1024);
        }
    };
    auto issue_v = [&](int t) __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int j = 0; j < VL; ++j) {
            const int row = j * 8 + (lane >> 3);
            lds_bload16(v_rsrc, (uint32_t)row * (uint32_t)a.nk_pad * 2 + (((lane & 7) ^ vswz(row)) << 4), (uint32_t)t * (BKV * 2), sV + j * 1024);
        }
    };
    auto landed = [](auto younger) __attribute__((always_inline)) {            // all but the `younger` last copies of this wave
        constexpr int N = decltype(younger)::value;
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
        asm volatile("" ::: "memory");
    };
    bf16x8 qf[KS];
    {
        const bf16* const qp = a.Q + ((size_t)h * a.nq + min(q0 + lj, a.nq - 1)) * HD + lg * 8;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) qf[kk] = *(const bf16x8*)(qp + kk * 16);
    }
    floatx16 o[DT];
    float mc, l_run;
    int out_of_range;
    // as attn_sweep's tiles: the same products in the same order.  (A repeated sweep is this wave's alone, and tracks.)
    auto tile = [&](int t, bool more, auto mode_c) __attribute__((always_inline)) {
        constexpr int mode = decltype(mode_c)::value;
        landed(std::integral_constant<int, VL>{});
        floatx16 s[2];
#pragma unroll
        for (int i = 0; i < 2 * KS; ++i) {
            const int key = (i & 1) * 32 + krow, c = (i >> 1) * 2 + lg;
            const bf16x8 kf = *(const bf16x8*)(sK + key * KROW + ((c ^ kswz(key)) << 4));
            if (i < 2) {
                floatx16 z;
#pragma unroll
                for (int v = 0; v < 16; ++v) z[v] = 0.f;
                s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[i >> 1], z, 0, 0, 0);
            } else {
                s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[i >> 1], s[i & 1], 0, 0, 0);
            }
        }
        if (more) issue_k(t + 1);
        if (t * BKV + BKV > a.nk) {
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (t * BKV + mt * 32 + 16 * (v >> 3) + 8 * lg + (v & 7) >= a.nk) s[mt][v] = -INFINITY;
        }
        float alpha = 1.f;
        if constexpr (mode != FAST) {
            float mx = s[0][0];
#pragma unroll
            for (int v = 1; v < 32; ++v) mx = fmaxf(mx, s[v >> 4][v & 15]);
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float mc_new = fmaxf(mc, mx * c2);
            if constexpr (mode == REPEATED) {
                alpha = __builtin_amdgcn_exp2f(mc - mc_new);
#pragma unroll
                for (int d = 0; d < DT; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[d][v] *= alpha;
            }
            mc = mc_new;
        }
        bf16x8 pf[4];
        float ps[4] = {0.f, 0.f, 0.f, 0.f};
        bf16x2 ones;
        ones[0] = (bf16)1.0f;
        ones[1] = (bf16)1.0f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                bf16x2 pp;
                pp[0] = (bf16)__builtin_amdgcn_exp2f(fmaf(s[ks >> 1][8 * (ks & 1) + e], c2, -mc));
                pp[1] = (bf16)__builtin_amdgcn_exp2f(fmaf(s[ks >> 1][8 * (ks & 1) + e + 1], c2, -mc));
                pf[ks][e] = pp[0];
                pf[ks][e + 1] = pp[1];
                ps[(e >> 1) & 3] = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, ps[(e >> 1) & 3], false);
            }
        const float psum = (ps[0] + ps[1]) + (ps[2] + ps[3]);
        l_run = mode == REPEATED ? fmaf(l_run, alpha, psum) : l_run + psum;
        if (more) landed(std::integral_constant<int, KL>{});
        else landed(std::integral_constant<int, 0>{});
#pragma unroll
        for (int i = 0; i < QUADS; ++i) {
            const int row = (i % DT) * 32 + lj, c = (i / DT) * 2 + lg;
            const bf16x8 vf = *(const bf16x8*)(sV + row * 128 + ((c ^ vswz(row)) << 4));
            o[i % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[i / DT], o[i % DT], 0, 0, 0);
        }
        if (more) issue_v(t + 1);
        if constexpr (mode == FAST) {
            const float row = psum + __shfl_xor(psum, 32);
            if (__any(!(row < 1048576.0f))) {
                if (__any(!(row < 18446744073709551616.0f))) {
                    out_of_range = 1;
                } else {
                    const int e = row < 1048576.0f ? 0 : (int)(__float_as_uint(row) >> 23) - 127;
                    const float alpha = __uint_as_float((uint32_t)(127 - e) << 23);
                    mc += (float)e;
                    l_run *= alpha;
#pragma unroll
                    for (int d = 0; d < DT; ++d)
#pragma unroll
                        for (int v = 0; v < 16; ++v) o[d][v] *= alpha;
                }
            }
        }
    };
    auto sweep = [&](auto mode_c) __attribute__((always_inline)) {
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[d][v] = 0.f;
        mc = kNoRef;
        l_run = 0.f;
        out_of_range = 0;
        issue_k(T0);
        issue_v(T0);
        tile(T0, T0 + 1 < T1, std::integral_constant<int, FIRST>{});
        for (int t = T0 + 1; t < T1; ++t) tile(t, t + 1 < T1, mode_c);
    };
    sweep(std::integral_constant<int, FAST>{});
    if (out_of_range) sweep(std::integral_constant<int, REPEATED>{});
    // joined in the order of the parts; of the row's QUADS pieces wave w puts together every parts-th
    auto po = [&](int p) { return (float*)(smem + p * (K_TILE + V_TILE)); };       // of part p, where its tiles were: [QUADS][64 * 4]
    auto ml = [&](int p) { return po(p) + QUADS * 256; };                          // [64 * 2]
    static_assert(QUADS * 1024 + 512 <= K_TILE + V_TILE, "a part's result in place of its tiles");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // this wave's last reads of them
#pragma unroll
    for (int i = 0; i < QUADS; ++i)
        *(floatx4*)(po(part) + i * 256 + lane * 4) = floatx4{o[i / 4][i % 4 * 4], o[i / 4][i % 4 * 4 + 1], o[i / 4][i % 4 * 4 + 2], o[i / 4][i % 4 * 4 + 3]};
    *(float2*)(ml(part) + lane * 2) = make_float2(mc, l_run + __shfl_xor(l_run, 32));
    __syncthreads();
    bf16* const op = out_row<HD>(a, h, q0 + lj);
    for (int i = part; i < QUADS; i += a.splits) {
        float m = kNoRef, l = 0.f;
        floatx4 sum = {0.f, 0.f, 0.f, 0.f};
        for (int p = 0; p < a.splits; ++p) {
            const float2 mp = *(const float2*)(ml(p) + lane * 2);
            const floatx4 v = *(const floatx4*)(po(p) + i * 256 + lane * 4);
            const Joint f = join_part(m, l, mp.x, mp.y);
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[c] = f.join(sum[c], v[c]);
        }
        const float inv = 1.0f / l;
        if (op) {
            bf16x4 w;
#pragma unroll
            for (int c = 0; c < 4; ++c) w[c] = (bf16)(sum[c] * inv);
            *(bf16x4*)(op + i / 4 * 32 + i % 4 * 8 + lg * 4) = w;
        }
    }
}

// Puts the parts of the keys together: a wave per 32 queries of a head, lanes as in attn_fwd_kernel, parts in order.
// Bound by the partial results it reads (3 heads x 4608 queries in four parts: 28 MB).
template <int HD>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a) {
    constexpr int DT = HD / 32;
    const int lane = threadIdx.x & 63, lj = lane & 31, lg = lane >> 5;
    const int n32 = (a.nq + 31) / 32;
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= a.H * n32) return;
    const int h = w / n32, q0 = (w % n32) * 32;
    const size_t part_stride = (size_t)a.H * n32, tile32 = (size_t)h * n32 + q0 / 32;
    float m = kNoRef, l = 0.f;
    floatx4 o[DT * 4];
#pragma unroll
    for (int i = 0; i < DT * 4; ++i) o[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int p = 0; p < a.splits; ++p) {
        const float2 ml = *(const float2*)(a.part_ml + (p * part_stride + tile32) * 64 + lj * 2);
        const float* const po = a.part_o + (p * part_stride + tile32) * (32 * HD);
        floatx4 v[DT * 4];
#pragma unroll
        for (int i = 0; i < DT * 4; ++i) v[i] = *(const floatx4*)(po + i * 256 + lane * 4);
        const Joint f = join_part(m, l, ml.x, ml.y);
#pragma unroll
        for (int i = 0; i < DT * 4; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) o[i][c] = f.join(o[i][c], v[i][c]);
    }
    store_rows<HD>(a, h, q0 + lj, lg, [&](int d, int v) { return o[d * 4 + v / 4][v % 4]; }, 1.0f / l);
}

template <int HD, int NW, int FORM>
hipError_t launch(const AttnArgs& a, hipStream_t s) {
    const size_t smem = 2 * (BKV * HD * 2 + HD * 128);
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)attn_fwd_kernel<HD, NW, FORM>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int nqt = (a.nq + 32 * NW - 1) / (32 * NW);
    AttnArgs b = a;
    b.mod_blocks = a.mod.n1 > a.mod.n0 ? (a.mod.n1 - a.mod.n0 + NW * MV_ROWS - 1) / (NW * MV_ROWS) * a.mod.mats * a.mod.batch : 0;
    hipLaunchKernelGGL((attn_fwd_kernel<HD, NW, FORM>), dim3(nqt * a.H * (FORM == PARTS ? a.splits : 1) + b.mod_blocks), dim3(64 * NW), smem, s, b);
    return hipGetLastError();
}

template <int HD, int FORM>
hipError_t launch_nw(int nw, const AttnArgs& a, hipStream_t s) {
    switch (nw) {
        case 7: return launch<HD, 7, FORM>(a, s);
        case 8: return launch<HD, 8, FORM>(a, s);
        default: return launch<HD, 4, FORM>(a, s);
    }
}
template <int HD>
hipError_t launch_nw(int nw, const AttnArgs& a, hipStream_t s) {
    if (a.splits <= 1) return launch_nw<HD, WHOLE>(nw, a, s);
    if (a.all_parts) {
        if constexpr (HD == 64) return launch<HD, 4, ALL_PARTS>(a, s);
        else return launch_nw<HD, ALL_PARTS>(nw, a, s);
    }
    return launch_nw<HD, PARTS>(nw, a, s);
}

}  // namespace

const char* attn_check(const AttnArgs& a) {
    if (a.hd != 64 && a.hd != 128) return "attention: head_dim must be 64 or 128";
    if (a.H <= 0 || a.nq <= 0 || a.nk <= 0) return "attention: empty shape";
    if (a.nk_pad % 64 || a.nk_pad < a.nk) return "attention: nk_pad must be a multiple of 64 covering nk";
    if ((uint64_t)a.nk_pad * a.hd * 2 >= (1ull << 32)) return "attention: a head's keys exceed the 4 GiB buffer range";
    if (!a.Q || !a.K || !a.Vt) return "attention: null operand";
    if (((uintptr_t)a.Q | (uintptr_t)a.K | (uintptr_t)a.Vt) % 16) return "attention: operands must be 16-byte aligned";
    if (a.scatter) {
        const TokenMap& m = a.map;
        if (!a.dst0 || (m.len1 > 0 && !a.dst1)) return "attention: scatter mode needs the projection operand";
        if (m.n_total != a.nq || m.len0 + m.len1 != m.n_local || m.pos0 < 0 || m.len0 < 0 || m.len1 < 0 ||
            m.pos0 + m.len0 > m.pos1 || m.pos1 + m.len1 > m.n_total)
            return "attention: scatter map must hold two ordered position ranges inside the query sequence";
        if ((((uintptr_t)a.dst0 | (uintptr_t)a.dst1 | (uintptr_t)a.send) % 8) || (a.ld % 4) || (a.bs0 % 4) || (a.bs1 % 4) || (a.send_bs % 4))
            return "attention: scatter targets must be 8-byte aligned";
        if (a.h0 < 0 || a.ld < (a.h0 + (a.hps ? a.hps : a.H)) * a.hd) return "attention: scatter columns exceed the operand's row";
    } else {
        if (!a.O) return "attention: null operand";
        if (((uintptr_t)a.O % 8) || (a.o_hs % 4) || (a.o_qs % 4) || (a.o_bs % 4)) return "attention: output must be 8-byte aligned";
    }
    if (a.hps < 0 || (a.hps && a.H % a.hps)) return "attention: H must be whole samples of hps heads";
    if ((long)((a.nq + 127) / 128) * a.H * std::max(1, a.splits) > 0x7fffffffL) return "attention: grid too large";
    if (a.splits > 1 && (a.part_tiles < 2 || (a.part_tiles & 1) || (long)(a.splits - 1) * a.part_tiles * BKV >= a.nk || (long)a.splits * a.part_tiles * BKV < a.nk))
        return "attention: bad split of the keys";
    if (a.splits > 1 && !a.all_parts && (!a.part_o || !a.part_ml || (((uintptr_t)a.part_o | (uintptr_t)a.part_ml) % 16)))
        return "attention: no scratch for the parts of the keys";
    if (a.all_parts == ALL_PARTS_WAVES && (a.splits > wave_parts_most(a.hd) || (long)((a.nq + 31) / 32) * a.H > 0x7fffffffL)) return "attention: too many parts for the waves of a workgroup";
    if (a.all_parts && a.splits < 2) return "attention: no parts for a workgroup to have all of";
    if (a.even_state && (a.splits > 1 || !a.even_flags || ((uintptr_t)a.even_state % 16) || a.hd != 128 || (long)((a.nq + 255) / 256) * a.H <= 7 * 32))
        return "attention: launch cannot be dealt out by the kernel";
    // a sweep works off its first tile whatever its end: an empty piece would count one twice
    if (a.even_state && a.even_units && (a.nk + BKV - 1) / BKV < a.even_cuts) return "attention: too few keys to cut a sweep in pieces";
    return nullptr;
}

// Waves per workgroup.  A CU holds 8 waves of this kernel, as one workgroup of 7 or 8 or as two of 4, and
// runs its workgroups generation after generation; a generation takes about as long whether the chip is
// full of workgroups or holds a handful.  Estimated time, in units of one K/V tile of an 8-wave workgroup
// (fitted to sweeps of 8 to 1861 tiles on 12 to 24 heads):
//   8 waves: generations x (tiles + 2.5)           the fixed part is the prologue and epilogue nothing overlaps
//   7 waves: generations x (0.96 tiles + 9)        a little faster per tile (one SIMD holds a single wave), its
//                                                  tile copies dealt unevenly; never fewer generations than 8
//   4 waves: generations x (1.08 tiles + 0.5)      twice the tile copies per query, but one workgroup's fixed
//                                                  part hides behind the other's tiles, and a last generation
//                                                  of at most one workgroup per CU takes 0.55 of a full one
// Short sweeps (cross-attention to a few hundred keys) and grids that end on a half-empty generation go to
// 4; very long sweeps whose 7- and 8-wave grids need the same number of generations to 7; the rest to 8.
// Heights 5 and 6 were built once and never won: three SIMDs share the work of four.
static int waves_and_cost(const AttnArgs& a, double* cost) {
    const int splits = a.all_parts ? 1 : std::max(1, a.splits);          // workgroups over one query tile
    const double tiles = splits > 1 ? a.part_tiles : (double)((a.nk + BKV - 1) / BKV);
    auto items = [&](int nw) { return (long)((a.nq + 32 * nw - 1) / (32 * nw)) * a.H * splits; };
    auto generations = [](long n, long slots) { return (double)((n + slots - 1) / slots); };
    const double c8 = generations(items(8), 256) * (tiles + 2.5);
    const double c7 = generations(items(7), 256) * (0.96 * tiles + 9.0);
    const long full4 = items(4) / 512, rest4 = items(4) % 512;
    const double c4 = ((double)full4 + (rest4 == 0 ? 0.0 : (rest4 <= 256 ? 0.55 : 1.0))) * (1.08 * tiles + 0.5);
    int best = 8;
    double best_cost = c8;
    if (c7 < best_cost - 1e-9) { best = 7; best_cost = c7; }
    if (c4 < best_cost - 1e-9) { best = 4; best_cost = c4; }
    // a grid that cannot even give every CU one 4-wave workgroup is spread as widely as possible
    if (items(4) <= 256) { best = 4; best_cost = c4; }
    *cost = best_cost;
    return best;
}

int attn_waves(const AttnArgs& a) {
    if (a.all_parts && a.hd == 64) return 4;       // see attn_fwd_kernel
    double cost;
    return waves_and_cost(a, &cost);
}

// Key tiles of a part: an even number, so that every part begins in the same one of the two tile buffers.
static int tiles_per_part(int tiles, int parts) { return parts > 1 ? ((tiles + parts - 1) / parts + 1) & ~1 : tiles; }

// Estimated times in us, past the launch itself.  Sweeps of `tiles` by `wgs` 4-wave workgroups, n to a CU: a tile takes each CU
// 0.97 + 0.25 n up to one of them and 0.25 + 0.97 n from there on with 128-wide heads, 0.68 and 0.45 + 0.48 n with 64-wide ones.
static double sweeps_us(double wgs, double tiles, int hd) {
    const double n = wgs / 256.0;
    return tiles * (hd == 64 ? (n <= 1.0 ? 0.68 : 0.45 + 0.48 * n) : n <= 1.0 ? 0.97 + 0.25 * n : 0.25 + 0.97 * n);
}
// The same, their parts merged by a kernel: 6 us and a pass over the partial results at 4 TB/s.
static double merged_us(int heads, int nq, int tiles, int hd, int parts) {
    return sweeps_us((double)((nq + 127) / 128) * heads * parts, tiles_per_part(tiles, parts), hd) + 6.0 + 4.0 * parts * (double)heads * nq * hd / 4e6;
}
// The same, a workgroup with all parts one after the other: joining one costs 0.4 of a tile (0.3 us, 64-wide, or 0.4).
static double in_turn_us(int heads, int nq, int tiles, int hd, int parts) {
    return sweeps_us((double)((nq + 127) / 128) * heads, tiles + 0.4 * (parts - 1), hd);
}
// A wave to each part, 32 queries to a workgroup, of which a CU holds 9 waves with 64-wide heads (8 in two parts) or 4 with 128-wide ones.
// Fitted to 286 launches of each width, 1 to 128 heads x 320 to 3584 in 2 to 4 parts: off by 6 and 4 % in the mean.
static double wave_parts_us(int heads, int nq, int tiles, int hd, int parts) {
    const long items = (long)((nq + 31) / 32) * heads;
    const long per_cu = hd == 64 ? (parts == 2 ? 4 : std::max(1, 9 / parts)) : std::max(1, 4 / parts), slots = 256 * per_cu;
    auto generation = [&](long n) {            // n workgroups to a CU
        return hd == 64 ? tiles_per_part(tiles, parts) * (0.6 + 0.085 * parts * n + (n > 1 ? 0.33 : 0.0)) + 2.0
                        : tiles_per_part(tiles, parts) * (1.03 + 0.16 * parts * n + (n > 1 ? 0.17 : 0.0)) + 3.7;
    };
    const long rest = items % slots;
    return (double)(items / slots) * generation(per_cu) + (rest ? generation((rest + 255) / 256) : 0.0) - (hd == 64 ? 1.3 : 2.5);
}

// Parts the keys of a launch are cut into.  Few heads over a short sequence (a Ulysses rank's share at degree 4 or 8, the toy model)
// are a few dozen workgroups that each sweep all keys; cut into parts they fill the chip, at the price of writing the
// partial results and merging them, or, where there are fewer queries still, the parts go to the waves of one workgroup, which costs
// neither.  A function of one sample's heads and lengths only, so that a sample's result does not depend on the batch it is part of;
// a batch that fills the chip, whose workgroups have all parts, pays for joining them and gains nothing, which sets a bound on
// their number.
// Parts that are workgroups: at least 6 tiles each (8 with 64-wide heads).  Estimated time in us for 128-wide heads: a tile takes a
// 4-wave workgroup 0.97 alone on its CU and 1.7 beside another, the merge 10 us and one pass over the partial results at 4 TB/s (3 heads
// x 4608: 72 us whole, 51 in two or four parts; 12 heads x 2640: 51 us whole, 58 in two).  Not where the planner would then give one
// sample's workgroups all parts.
// Parts that are waves: two to four (five to eight are no faster: 8 x 1000 x 64 in 2, 3, 4, 8 parts 11.3, 9.8, 8.3, 8.9 us), where they take
// at least 15 % off and a batch with a workgroup per CU joins them in a twenty-fifth of its time; or as many as were chosen for workgroups, where
// waves are the faster with those (1 x 2640 to 4680 x 64 in five to eight: merged 17.0 to 22.0, waves 14.3 to 20.2).  One sample whole or merged / so, and
// eight samples whole / all parts in turn: 8 x 512 x 64 9.3 / 7.6 and 10.2 / 10.4; 8 x 800 x 64 12.6 / 10.7 and 19.8 / 20.4; 8 x 1000 x 64 14.4 / 11.3 and
// 24.4 / 25.3; 3 x 2048 x 64 17.0 / 12.2 and 36.8 / 38.2; 8 x 512 x 128 13.1 / 11.5 and 15.8 / 16.7; 8 x 1000 x 128 20.9 / 15.4 and 40.9 / 41.6; 3 x 2048 x 128 28.7 / 20.5
// and 53.5 / 54.4.  (Four parts of 8 x 512 x 64: 6.1 us, and eight samples 11.2.)  Over 380 batches of 320 to 3584
// tokens whose samples are cut for their own sake, the median is even with whole sweeps, and the worst 7 % behind (one, 4 x 1280 x 128 of two samples,
// 24.4 against 27.2, merged where in turn would be better).
int attn_splits(int heads, int nq, int nk, int hd) {
    const long items = (long)((nq + 127) / 128) * heads;
    const int tiles = (nk + BKV - 1) / BKV, least = hd == 64 ? 8 : 6;
    auto cuts = [&](int s) { const int per = tiles_per_part(tiles, s); return (tiles + per - 1) / per == s; };
    int best = 1;
    double best_us = 0;
    for (int s = 1; s <= 8; ++s) {
        const int per = tiles_per_part(tiles, s);
        if (s > 1 && (per < least || !cuts(s))) continue;
        const long wgs = items * s;
        if (s > 1 && wgs > 512) break;
        double us = (wgs <= 256 ? 0.97 * per : 1.7 * per * (double)((wgs + 511) / 512)) * (hd == 64 ? 0.55 : 1.0) + 3.0;
        if (s > 1) us += 10.0 + 4.0 * s * (double)heads * nq * hd / 4e6;
        if (s == 1 || us < 0.95 * best_us) best = s, best_us = us;
    }
    if (best > 1 && attn_all_parts(heads, nq, nk, hd, best) == ALL_PARTS_IN_TURN) best = 1;
    best_us = best > 1 ? merged_us(heads, nq, tiles, hd, best) : sweeps_us(items, tiles, hd);
    const double join = hd == 64 ? 0.3 : 0.4, batch = sweeps_us(256, tiles, hd) + 4.0;
    bool waves = false;
    for (int s = 2; s <= 4 && (s - 1) * join <= 0.04 * batch; ++s) {
        const double us = wave_parts_us(heads, nq, tiles, hd, s);
        if (cuts(s) && attn_all_parts(heads, nq, nk, hd, s) == ALL_PARTS_WAVES && us < (waves ? 0.95 : 0.85) * best_us) best = s, best_us = us, waves = true;
    }
    return best;
}

// Whether a workgroup has all parts of its queries, for the heads of all samples together, and how: where the query tiles alone fill the
// chip, parts that are workgroups only cost (12 heads x 4608 x 128, four samples: 115 us in one sweep, 136 in two parts and their merge, 115 with
// both in one workgroup).  (3 heads x 4608 for 1, 2, 3, 4, 8 samples, in parts /
// in one workgroup: 55/74, 78/81, 126/108, 146/126, 286/248; 3 x 2640: 34/46, 44/47, -, 65/54, 119/95; 2 x 4696 x 64 for 1, 4, 16:
// 29/51, 64/75, 210/199.)
int attn_all_parts(int heads, int nq, int nk, int hd, int splits) {
    if (splits <= 1) return 0;
    const int tiles = (nk + BKV - 1) / BKV;
    const double parts = merged_us(heads, nq, tiles, hd, splits), in_turn = in_turn_us(heads, nq, tiles, hd, splits);
    if (splits <= wave_parts_most(hd) && wave_parts_us(heads, nq, tiles, hd, splits) < std::min(parts, in_turn)) return ALL_PARTS_WAVES;
    return in_turn < parts ? ALL_PARTS_IN_TURN : 0;
}

uint64_t attn_part_floats(int heads, int nq, int hd, int splits) {
    return splits > 1 ? (uint64_t)splits * heads * ((nq + 31) / 32) * 32 * (hd + 2) : 0;
}

void attn_set_split(AttnArgs* a, int splits, float* scratch) {
    const int tiles = (a->nk + BKV - 1) / BKV;
    a->splits = std::max(1, splits);
    a->part_tiles = tiles_per_part(tiles, a->splits);
    a->part_o = scratch;
    a->part_ml = scratch ? scratch + (uint64_t)a->splits * a->H * ((a->nq + 31) / 32) * 32 * a->hd : nullptr;
}

// How the launch is dealt out: 0 = by the grid, 1 = even shares, 2 = taken as they come.  Estimated in the units above for
// groups of 32 query tiles.  By the grid and in even shares the slowest XCD takes 3 % longer than the mean.  Even shares: an
// eighth of the groups per XCD, a fixed part per sweep (one more of them where an eighth ends inside a group) and about 15 for
// leaving (17 us, most of it the L2 write-back) and fetching the states.  As they come: 15 for each of the pieces an XCD takes
// of the last kEvenLast groups, and half a piece of ragged end.  At least eight groups: a workgroup's even share must cover a
// whole sweep, or three of them would queue up in one.
// 128-wide heads only: a CU holds two 8-wave workgroups of the 64-wide kernel, which one evenly dealt workgroup does not match
// (8 heads x 30950 x 64: 2.70 against 1.83 ms).
// Where the lines lie (us by the grid / even / drawn; the estimated even share of the grid's time in brackets): 48 heads x 4608
// 491 / 459 / 500 (0.97), 48 x 6000 806 / 756 / 805 (0.97), 96 x 4608 889 / 892 / 937 (1.00), 8 x 24000 1898 / 1926 / 1966
// (1.02), 24 x 13640 2114 / 1900 / 1927 (0.88), 24 x 20000 4072 / 3961 / 3999 (0.94), 4 x 60000 5952 / 5846 / 5889 (0.94: by the
// grid 8-wave sweeps, whose time is estimated too high by up to 4 %), 12 x 119056 69.2 / - / 66.65 ms.  The last sweeps in four
// pieces each; there, in two 66.96, in three 66.70.
constexpr int kEvenLast = 8, kEvenCuts = 4;
int attn_deal(int H, int nq, int nk, int hd, int splits) {
    const long groups = ((long)((nq + 255) / 256) * H + 31) / 32;
    if (splits > 1 || groups < 8 || hd != 128) return 0;
    AttnArgs a{};
    a.H = H; a.nq = nq; a.nk = nk; a.hd = hd; a.splits = 1;
    double plain;
    const int waves = waves_and_cost(a, &plain);
    const double tiles = (double)((nk + BKV - 1) / BKV), sweeps = groups / 8.0 * (tiles + 2.5);
    const double even = 1.03 * (sweeps + 2.5 + 15.0), drawn = sweeps + 15.0 * kEvenCuts + tiles / kEvenCuts / 2;
    if (groups >= 3 * kEvenLast && tiles >= kEvenCuts && drawn < 0.99 * even && drawn < 0.985 * 1.03 * plain) return 2;
    return even < (waves == 8 ? 0.96 : 0.98) * 1.03 * plain ? 1 : 0;
}

uint64_t attn_deal_floats(int deal) {
    return deal ? (uint64_t)(deal == 2 ? kEvenLast * (kEvenCuts - 1) : 7) * 32 * 512 * (128 / 2 + 2) : 0;
}

void attn_set_deal(AttnArgs* a, int deal, float* state, uint32_t* flags) {
    static_assert(kEvenLast * (kEvenCuts - 1) * 32 + 32 <= ATTN_FLAGS, "a flag per state and 32 counters");
    a->even_state = deal ? state : nullptr;
    a->even_flags = deal ? flags : nullptr;
    a->even_last = kEvenLast;
    a->even_cuts = kEvenCuts;
    a->even_wait = 1;
    const int groups = (int)(((long)((a->nq + 255) / 256) * a->H + 31) / 32);
    a->even_units = deal == 2 ? groups - kEvenLast + kEvenLast * kEvenCuts : 0;
}

static hipError_t launch_even(const AttnArgs& a, hipStream_t s) {
    const size_t smem = 2 * (BKV * 128 * 2 + 128 * 128);
    static const hipError_t allowed = hipFuncSetAttribute((const void*)attn_even_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (allowed != hipSuccess) return allowed;
    hipLaunchKernelGGL(attn_even_kernel<128>, dim3(256), dim3(512), smem, s, a);
    return hipGetLastError();
}

template <int HD>
static hipError_t launch_wave_parts(const AttnArgs& a, hipStream_t s) {
    const size_t smem = (size_t)a.splits * (BKV * HD * 2 + HD * 128);
    static const hipError_t allowed = hipFuncSetAttribute((const void*)attn_wave_parts_kernel<HD>, hipFuncAttributeMaxDynamicSharedMemorySize, wave_parts_most(HD) * (BKV * HD * 2 + HD * 128));
    if (allowed != hipSuccess) return allowed;
    hipLaunchKernelGGL(attn_wave_parts_kernel<HD>, dim3((a.nq + 31) / 32 * a.H), dim3(64 * a.splits), smem, s, a);
    return hipGetLastError();
}

// One generation of workgroups that leaves an eighth of the chip's places free, so that what streams there does not wait for a sweep to end;
// and sweeps that last (1.35 us a tile of 128-wide heads, half of that for 64-wide ones) as long as the rows take to be read at 5 TB/s,
// or the launch would end with a product that a launch of its own, with more of it in flight, does faster.  3 heads x 4608 x 128 in two parts, 50 us:
// 151 MB beside it, 27 us of a launch of their own, make it 61.
bool attn_takes_mod(const AttnArgs& a) {
    if (a.even_state || a.all_parts == ALL_PARTS_WAVES) return false;
    const int nw = attn_waves(a), own = a.splits > 1 && !a.all_parts ? a.splits : 1;
    const long groups = (long)((a.nq + 32 * nw - 1) / (32 * nw)) * a.H * own;
    const double sweep_us = (a.hd == 128 ? 1.35 : 0.68) * (own > 1 ? a.part_tiles : (a.nk + BKV - 1) / BKV);
    const double read_us = 2.0 * (a.mod.n1 - a.mod.n0) * a.mod.K * a.mod.mats * a.mod.batch / 5e6;
    return groups <= 7 * 32 * (nw == 4 ? 2 : 1) * (a.hd == 64 ? 2 : 1) && read_us <= sweep_us;
}

hipError_t attn_launch(const AttnArgs& a, hipStream_t s) {
    if (a.mod.n1 > a.mod.n0 && (!attn_takes_mod(a) || a.mod.K % 8 || a.mod.mats < 1 || a.mod.mats > 2 || a.mod.batch < 1)) return hipErrorInvalidValue;
    if (a.even_state) return launch_even(a, s);
    if (a.all_parts == ALL_PARTS_WAVES) return a.hd == 128 ? launch_wave_parts<128>(a, s) : launch_wave_parts<64>(a, s);
    const int nw = attn_waves(a);
    const hipError_t e = a.hd == 128 ? launch_nw<128>(nw, a, s) : launch_nw<64>(nw, a, s);
    if (e != hipSuccess || a.splits <= 1 || a.all_parts) return e;
    const dim3 grid((a.H * ((a.nq + 31) / 32) + 3) / 4);
    if (a.hd == 128) hipLaunchKernelGGL(attn_merge_kernel<128>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(attn_merge_kernel<64>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}
