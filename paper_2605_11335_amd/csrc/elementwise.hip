// HBM-bound kernels of the block: adaLN modulation vector, LayerNorm+modulate, q/k RMSNorm
// with the Ulysses head-major relayout, the receiving side of the two exchanges around attention
// (Sec. 2.1; the sending side of the second one is the attention kernel's own stores), and the
// streamed-bytes checksum.  All accesses are 8- or 16-byte per lane and
// consecutive lanes touch consecutive addresses.
#include "common.h"
#include "heads.h"
#include "kernels.h"
#include "modvec.h"

namespace {

// ---------------------------------------------------------------------------------------------
// modulation vectors (modvec.h): a workgroup per MV_ROWS rows of each of its waves, grid rows are samples, grid planes matrices
template <int U>
__global__ __launch_bounds__(256) void modvec_kernel(ModRows j, uint32x4* zero, uint32_t zeros) {
    for (uint32_t i = ((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * 256 + threadIdx.x; i < zeros; i += gridDim.x * gridDim.y * gridDim.z * 256)
        zero[i] = uint32x4{0u, 0u, 0u, 0u};
    modvec_rows<U>(j, blockIdx.z, blockIdx.y, j.n0 + (blockIdx.x * 4 + (threadIdx.x >> 6)) * MV_ROWS);
}

// ---------------------------------------------------------------------------------------------
// LayerNorm over d (no affine, biased variance, eps 1e-6) then modulate or affine; wave per row.  Workgroups from blocks0 on
// have the second of a launch's two parts.
struct LnPair { LnArgs part[2]; int blocks0; };
template <int NJ, bool AFFINE>
__global__ __launch_bounds__(256) void ln_kernel(LnPair p, WView W, uint64_t w_off, uint64_t b_off, int d) {
    const LnArgs& a = p.part[(int)blockIdx.x >= p.blocks0];
    const int lane = threadIdx.x & 63;
    const int row = ((int)blockIdx.x - ((int)blockIdx.x >= p.blocks0 ? p.blocks0 : 0)) * 4 + (threadIdx.x >> 6);
    if (row >= a.rows) return;
    // a batch stacks samples along the rows: each has its own modulation vectors and may sit at its own stride
    int smp = 0, ri = row;
    if (a.rows_per_sample) { smp = row / a.rows_per_sample; ri = row - smp * a.rows_per_sample; }
    const float* __restrict__ xr = a.x + (size_t)smp * a.x_bs + (size_t)ri * d;
    const float *__restrict__ shift = a.shift, *__restrict__ scale = a.scale;
    bf16* __restrict__ out = a.xn;
    if (!AFFINE) { shift += (size_t)smp * a.mod_bs; scale += (size_t)smp * a.mod_bs; }
    float4 v[NJ];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        v[j] = *(const float4*)(xr + (lane + 64 * j) * 4);
        s += v[j].x + v[j].y + v[j].z + v[j].w;
    }
    // the row-independent operands of the last step are requested now, so that they arrive while the
    // statistics are reduced instead of costing a round trip of their own afterwards
    floatx4 ma[NJ], mb[NJ];                      // modulate: scale, shift;  affine: weight | bias as bf16 pairs
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c = (lane + 64 * j) * 4;
        if (AFFINE) {
            const uint32x2 wa = *(const uint32x2*)wv_ptr(W, w_off + 2ull * c), wb = *(const uint32x2*)wv_ptr(W, b_off + 2ull * c);
            ma[j] = floatx4{__uint_as_float(wa.x << 16), __uint_as_float(wa.x & 0xffff0000u), __uint_as_float(wa.y << 16),
                            __uint_as_float(wa.y & 0xffff0000u)};
            mb[j] = floatx4{__uint_as_float(wb.x << 16), __uint_as_float(wb.x & 0xffff0000u), __uint_as_float(wb.y << 16),
                            __uint_as_float(wb.y & 0xffff0000u)};
        } else {
            ma[j] = *(const floatx4*)(scale + c);
            mb[j] = *(const floatx4*)(shift + c);
        }
    }
    const float mean = wave_sum(s) / d;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        v[j].x -= mean; v[j].y -= mean; v[j].z -= mean; v[j].w -= mean;
        q += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
    }
    const float rstd = rsqrtf(wave_sum(q) / d + 1e-6f);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c = (lane + 64 * j) * 4;
        float a[4], b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] = AFFINE ? ma[j][e] : 1.f + ma[j][e];
            b[e] = mb[j][e];
        }
        bf16x4 o;
        o[0] = (bf16)(v[j].x * rstd * a[0] + b[0]);
        o[1] = (bf16)(v[j].y * rstd * a[1] + b[1]);
        o[2] = (bf16)(v[j].z * rstd * a[2] + b[2]);
        o[3] = (bf16)(v[j].w * rstd * a[3] + b[3]);
        *(bf16x4*)(out + (size_t)row * d + c) = o;
    }
}

template <bool AFFINE>
hipError_t ln_dispatch(const LnArgs* parts, int n_parts, const WView& W, uint64_t w_off, uint64_t b_off, int d, hipStream_t s) {
    LnPair p{};
    int blocks = 0;
    for (int i = 0; i < n_parts; ++i) {
        const LnArgs& a = parts[i];
        if (a.rows_per_sample < 0 || (a.x_bs % 4) || (a.mod_bs % 4)) return hipErrorInvalidValue;
        p.part[i] = a;
        blocks += a.rows > 0 ? (a.rows + 3) / 4 : 0;
        if (i == 0) p.blocks0 = blocks;
    }
    if (blocks == 0) return hipSuccess;
    if (d % 256 || d > 4096) return hipErrorInvalidValue;
    const dim3 grid(blocks), blk(256);
#define CF_LN_CASE(NJ) case NJ: hipLaunchKernelGGL((ln_kernel<NJ, AFFINE>), grid, blk, 0, s, p, W, w_off, b_off, d); break;
    switch (d / 256) {
        CF_LN_CASE(1) CF_LN_CASE(2) CF_LN_CASE(3) CF_LN_CASE(4) CF_LN_CASE(6) CF_LN_CASE(8) CF_LN_CASE(12) CF_LN_CASE(16)
        default: return hipErrorInvalidValue;
    }
#undef CF_LN_CASE
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// q,k: optional per-head RMSNorm, then head-major placement (own heads) or send buffers (others).
// v of other heads: send buffer.  A wave takes one of q, k, v of one row; a group of hd/8 of its lanes owns a head's vector.
// Everything between HBM and HBM is index arithmetic here: with a flat item index taken apart by 64-bit divisions (three per
// 16 bytes) the kernel ran at 3.6-4.2 TB/s.
__device__ __forceinline__ void qk_relayout_part(const RelayoutArgs& r, int bid, int nblk) {
    const int lane = threadIdx.x & 63;
    const int lph = r.hd / 8, lsh = r.hd == 128 ? 4 : 3;        // lanes per head vector
    const int vpw = 64 >> lsh, grp = lane >> lsh, sub = lane & (lph - 1);
    uint32x4 w_raw[2] = {};            // (as they are in memory, for the registers' sake)
    if (r.has_norm) {
#pragma unroll
        for (int t = 0; t < 2; ++t) w_raw[t] = *(const uint32x4*)wv_ptr(r.W, (t ? r.kn_off : r.qn_off) + sub * 16);
    }
    const int n_other = r.n_heads - r.h_local;
    for (uint32_t item = (uint32_t)bid * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); item < (uint32_t)r.rows * 3u; item += (uint32_t)nblk * 4u) {
        const int row = item / 3u, tns = item % 3u;             // 0 q, 1 k, 2 v
        const int col = tns == 0 ? r.col_q : (tns == 1 ? r.col_k : r.col_v);
        bf16* const send = tns == 0 ? r.send_q : (tns == 1 ? r.send_k : r.send_v);
        if (col < 0 || (tns == 2 && (!send || n_other == 0))) continue;      // own v goes through the transposing part
        const int lrow = r.row0 + row;
        bf16* const own_dst = (tns == 0 ? r.Q : r.K) + (size_t)local_pos(r.map, lrow) * r.hd + sub * 8;
        const size_t own_hs = (size_t)r.map.n_total * r.hd, send_hs = (size_t)r.map.n_local * r.hd;
        bf16* const send_dst = send + (size_t)lrow * r.hd + sub * 8;
        const bf16* const src = r.src + (size_t)row * r.ld + col + sub * 8;
        const bool turn = r.rope_cos && tns < 2;
        floatx4 cs = {1.f, 1.f, 1.f, 1.f}, sn = {0.f, 0.f, 0.f, 0.f};
        if (turn) {          // this lane's 8 elements are pairs sub*4 .. sub*4+3 of the head vector, for every head
            const size_t ro = (size_t)lrow * (r.hd / 2) + sub * 4;
            cs = *(const floatx4*)(r.rope_cos + ro);
            sn = *(const floatx4*)(r.rope_sin + ro);
        }
        float w[8];
        unpack8(tns ? w_raw[1] : w_raw[0], w);
        for (int h4 = 0; h4 < r.n_heads; h4 += 4 * vpw) {        // four vectors of a lane group in flight
            uint32x4 u[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                u[q] = *(const uint32x4*)(src + min(h4 + q * vpw + grp, r.n_heads - 1) * r.hd);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int hh = h4 + q * vpw + grp;
                if (hh >= r.n_heads) continue;
                const bool own = hh >= r.h0 && hh < r.h0 + r.h_local;
                if (own ? tns == 2 : !send) continue;
                bf16* const dst = own ? own_dst + (hh - r.h0) * own_hs : send_dst + (hh < r.h0 ? hh : hh - r.h_local) * send_hs;
                if (tns == 2 || !(r.has_norm || turn)) {
                    *(uint32x4*)dst = u[q];
                    continue;
                }
                *(uint32x4*)dst = head_piece<false>(u[q], r.hd, r.has_norm, w, turn, cs, sn);
            }
        }
    }
}

// [token, hd] rows of one head -> Vt[head, d, position] (keys contiguous).  src element (h, i, d) at
// src + h*src_hs + i*src_rs + d; i counts local rows (remote=0) or remote rows (remote=1) and maps to its position in the
// joint sequence.  A lane turns 8 tokens x 8 elements round in its registers: it reads 16 bytes of eight tokens and writes
// 16 bytes (8 positions) of eight rows of Vt; the 64 lanes of a wave are 8 token groups x 8 element groups, so both sides
// touch whole 128-byte lines.  A workgroup takes V_TOKENS(hd) tokens of all hd elements.
__host__ __device__ __forceinline__ int v_tokens(int hd) { return hd == 128 ? 128 : 256; }
__device__ __forceinline__ void v_transpose_part(int bx, int h, const bf16* __restrict__ src, long src_hs, long src_rs, int n_rows,
                                                 int row0, bf16* __restrict__ Vt, int hd, int n_pad, const TokenMap& map, int remote) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = (lane & 7) + (hd == 128 ? (wave & 1) * 8 : 0);                             // 8-element group
    const int i0 = bx * v_tokens(hd) + (hd == 128 ? wave >> 1 : wave) * 64 + (lane >> 3) * 8;    // first token
    const int cnt = min(8, n_rows - i0);
    if (cnt > 0) {
        uint32x4 u[8];
        const bf16* const p = src + (size_t)h * src_hs + (size_t)i0 * src_rs + c * 8;
#pragma unroll
        for (int k = 0; k < 8; ++k) u[k] = *(const uint32x4*)(p + (size_t)min(k, cnt - 1) * src_rs);
        uint16_t* const vh = (uint16_t*)Vt + (size_t)h * hd * n_pad + (size_t)(c * 8) * n_pad;
        v_turned(u, cnt, n_pad, [&](int k) { const int i = row0 + i0 + k; return vh + (remote ? remote_pos(map, i) : local_pos(map, i)); });
    }
    // zero the pad columns once per (head, d) row
    if (bx == 0 && !remote) {
        for (int q = threadIdx.x; q < hd * (n_pad - map.n_total); q += 256) {
            const int dd = q / (n_pad - map.n_total), p = map.n_total + q % (n_pad - map.n_total);
            ((uint16_t*)Vt)[((size_t)h * hd + dd) * n_pad + p] = 0;
        }
    }
}

// peer q/k rows -> head-major operands at the remote positions: a workgroup copies PEER_PIECES 16-byte pieces of one head of
// one tensor
constexpr int PEER_PIECES = 256 * 8;
__device__ __forceinline__ void peer_qk_part(int bid, int blocks_per_head, const bf16* __restrict__ pq, const bf16* __restrict__ pk,
                                             bf16* __restrict__ Q, bf16* __restrict__ K, int h_local, int hd, const TokenMap& map) {
    const int lsh = hd == 128 ? 4 : 3, n_rem = map.n_total - map.n_local;
    const int th = bid / blocks_per_head, h = th % h_local;
    const bf16* const s = (th >= h_local ? pk : pq) + (size_t)h * n_rem * hd;
    bf16* const d = (th >= h_local ? K : Q) + (size_t)h * map.n_total * hd;
    const int first = (bid % blocks_per_head) * PEER_PIECES + threadIdx.x, total = n_rem << lsh;
    uint32x4 u[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
        u[q] = *(const uint32x4*)(s + (size_t)min(first + q * 256, total - 1) * 8);      // (loads behind branches each take registers of their own)
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int piece = first + q * 256;
        if (piece < total) *(uint32x4*)(d + (size_t)remote_pos(map, piece >> lsh) * hd + (piece & ((1 << lsh) - 1)) * 8) = u[q];
    }
}

// attention rows of the other ranks' heads for this rank's tokens -> their columns of the projection operand
__device__ __forceinline__ void peer_attn_part(int bid, const PeerAttnArgs& p) {
    const int lsh = p.hd == 128 ? 4 : 3;
    const uint32_t n_other = p.n_heads - p.h_local, total = ((uint32_t)p.map.n_local * n_other) << lsh;
    const uint32_t first = (uint32_t)bid * PEER_PIECES + threadIdx.x;
    uint32x4 u[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
        u[q] = *(const uint32x4*)(p.peer_attn + (size_t)min(first + q * 256, total - 1) * 8);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const uint32_t piece = first + q * 256;
        if (piece >= total) continue;
        const int i = (piece >> lsh) / n_other, ho = (piece >> lsh) % n_other;
        const int hh = ho < p.h0 ? ho : ho + p.h_local;
        bf16* const row = i < p.map.len0 ? p.dst + (size_t)i * p.ld : p.dst1 + (size_t)(i - p.map.len0) * p.ld;
        *(uint32x4*)(row + hh * p.hd + (piece & ((1u << lsh) - 1)) * 8) = u[q];
    }
}

// Everything between the QKV projection and attention in ONE launch: per part (one per stream; none where the projection has placed
// its heads itself)
// the q/k RMSNorm + head-major relayout and the transposition of the own heads' v, then the peer
// rows (q, k copied, v transposed).  Workgroups are dealt to the sub-tasks by index range.
struct PreAttnArgs {
    RelayoutArgs part[2];
    int n_parts;
    const bf16 *peer_q, *peer_k, *peer_v;      // may be NULL (sp_degree 1, or projection-only use)
    PeerAttnArgs pa;
    uint32_t* zero;                            // ATTN_FLAGS words to clear, or NULL
    int seg[7];                                // end of each segment: qk0, vt0, qk1, vt1, peer_qk, peer_vt, peer_attn
};

// Six workgroups on a CU at least: with five, which 81 registers leave, 1422 + 60 rows of 12 heads, two ranks, took 24 us instead of 17 (the
// double-stream block at batch 4 729 instead of 699), 1155 rows of 24 heads in blocks of two samples 529 to 532 instead of 521.
__global__ __launch_bounds__(256, 6) void pre_attention_kernel(PreAttnArgs a) {
    const int b = blockIdx.x;
    if (b == 0 && a.zero)
        for (int i = threadIdx.x; i < ATTN_FLAGS; i += 256) a.zero[i] = 0;
    int lo = 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        if (p >= a.n_parts) break;
        const RelayoutArgs& r = a.part[p];
        if (b < a.seg[2 * p]) { qk_relayout_part(r, b - lo, a.seg[2 * p] - lo); return; }
        lo = a.seg[2 * p];
        if (b < a.seg[2 * p + 1]) {
            const int nbx = (r.rows + v_tokens(r.hd) - 1) / v_tokens(r.hd), i = b - lo;
            v_transpose_part(i % nbx, i / nbx, r.src + r.col_v + (size_t)r.h0 * r.hd, (long)r.hd, (long)r.ld, r.rows,
                             r.row0, r.Vt, r.hd, r.n_pad, r.map, 0);
            return;
        }
        lo = a.seg[2 * p + 1];
    }
    const RelayoutArgs& r0 = a.part[0];
    const int n_rem = r0.map.n_total - r0.map.n_local;
    if (b < a.seg[4]) { peer_qk_part(b - lo, (a.seg[4] - lo) / (2 * r0.h_local), a.peer_q, a.peer_k, r0.Q, r0.K, r0.h_local, r0.hd, r0.map); return; }
    lo = a.seg[4];
    if (b < a.seg[5]) {
        const int nbx = (n_rem + v_tokens(r0.hd) - 1) / v_tokens(r0.hd), i = b - lo;
        v_transpose_part(i % nbx, i / nbx, a.peer_v, (long)n_rem * r0.hd, (long)r0.hd, n_rem, 0, r0.Vt, r0.hd, r0.n_pad,
                         r0.map, 1);
        return;
    }
    lo = a.seg[5];
    if (b < a.seg[6]) peer_attn_part(b - lo, a.pa);
}

// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void zero_u64_kernel(uint64_t* p) { if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0; }

// sum over 64-bit words of mix(word ^ (index+1)*GOLDEN), index counted from the blob start
__global__ __launch_bounds__(256) void checksum_kernel(const uint64_t* __restrict__ w, uint64_t n_words, uint64_t first_word,
                                                       unsigned long long* __restrict__ out) {
    uint64_t acc = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n_words; i += (uint64_t)gridDim.x * 256)
        acc += cf_mix64(w[i] ^ ((first_word + i + 1) * CF_GOLDEN64));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)acc, o), hi = __shfl_xor((uint32_t)(acc >> 32), o);
        acc += ((uint64_t)hi << 32) | lo;
    }
    if ((threadIdx.x & 63) == 0) atomicAdd(out, (unsigned long long)acc);
}

__global__ __launch_bounds__(256) void f32_to_bf16_kernel(const float* __restrict__ s, bf16* __restrict__ d, size_t n) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) d[i] = (bf16)s[i];
}

inline int grid_for(long items, int per_block, int cap = 256 * 16) {
    long b = (items + per_block - 1) / per_block;
    return (int)(b < 1 ? 1 : (b > cap ? cap : b));
}

}  // namespace

hipError_t modvec_launch(const ModRows& j, hipStream_t s, uint32_t* zero, uint32_t zero_words) {
    if (j.n1 <= j.n0) return hipSuccess;
    if (j.K % 8 || j.batch < 1 || j.batch > 65535 || j.mats < 1 || j.mats > 2) return hipErrorInvalidValue;
    const dim3 grid((j.n1 - j.n0 + 4 * MV_ROWS - 1) / (4 * MV_ROWS), j.batch, j.mats);
    const int steps = (j.K / 8 + 63) / 64;       // steps of a lane's walk over K; taken 3 or 4 at a time
#define CF_MV_CASE(U) hipLaunchKernelGGL(modvec_kernel<U>, grid, dim3(256), 0, s, j, (uint32x4*)zero, zero_words / 4)
    if (steps == 1) CF_MV_CASE(1);
    else if (steps == 2) CF_MV_CASE(2);
    else if (steps % 3 == 0) CF_MV_CASE(3);
    else CF_MV_CASE(4);
#undef CF_MV_CASE
    return hipGetLastError();
}

hipError_t ln_modulate_launch(const LnArgs* parts, int n_parts, int d, hipStream_t s) {
    if (n_parts < 1 || n_parts > 2) return hipErrorInvalidValue;
    return ln_dispatch<false>(parts, n_parts, WView{nullptr, nullptr, 0}, 0, 0, d, s);
}

hipError_t ln_affine_launch(const float* x, const WView& W, uint64_t w_off, uint64_t b_off, bf16* xn, int rows, int d,
                            hipStream_t s) {
    const LnArgs a{x, nullptr, nullptr, xn, rows, 0, 0, 0};
    return ln_dispatch<true>(&a, 1, W, w_off, b_off, d, s);
}

hipError_t pre_attention_launch(const RelayoutArgs* parts, int n_parts, const bf16* peer_q, const bf16* peer_k,
                                const bf16* peer_v, const PeerAttnArgs& pa, uint32_t* zero, hipStream_t s) {
    if (n_parts < 1 || n_parts > 2) return hipErrorInvalidValue;
    PreAttnArgs a{};
    a.n_parts = n_parts;
    a.peer_q = peer_q; a.peer_k = peer_k; a.peer_v = peer_v;
    a.pa = pa;
    a.zero = zero;
    int end = 0;
    for (int p = 0; p < 2; ++p) {
        if (p < n_parts) {
            const RelayoutArgs& r = parts[p];
            if (r.hd != 64 && r.hd != 128) return hipErrorInvalidValue;
            a.part[p] = r;
            if (r.rows > (1 << 29)) return hipErrorInvalidValue;             // 32-bit item indices
            if (r.rows > 0) end += grid_for((long)r.rows * 3, 4, 1 << 16);     // a wave per tensor of a row
            a.seg[2 * p] = end;
            if (r.rows > 0 && r.col_v >= 0 && r.Vt) end += ((r.rows + v_tokens(r.hd) - 1) / v_tokens(r.hd)) * r.h_local;
            a.seg[2 * p + 1] = end;
        } else {
            a.seg[2 * p] = a.seg[2 * p + 1] = end;
        }
    }
    const RelayoutArgs& r0 = parts[0];
    const int n_rem = r0.map.n_total - r0.map.n_local;
    if (peer_q && peer_k && peer_v && n_rem > 0) {
        if ((long)n_rem * (r0.hd / 8) > (1L << 30)) return hipErrorInvalidValue;
        end += 2 * r0.h_local * (int)(((long)n_rem * (r0.hd / 8) + PEER_PIECES - 1) / PEER_PIECES);
        a.seg[4] = end;
        end += ((n_rem + v_tokens(r0.hd) - 1) / v_tokens(r0.hd)) * r0.h_local;
        a.seg[5] = end;
    } else {
        a.seg[4] = a.seg[5] = end;
    }
    if (pa.peer_attn && pa.n_heads > pa.h_local && pa.map.n_local > 0) {
        if ((pa.hd != 64 && pa.hd != 128) || !pa.dst || (pa.ld % 8)) return hipErrorInvalidValue;
        if (!a.pa.dst1) a.pa.dst1 = pa.dst + (size_t)pa.map.len0 * pa.ld;
        const long pieces = (long)pa.map.n_local * (pa.n_heads - pa.h_local) * (pa.hd / 8);
        if (pieces > (1L << 31)) return hipErrorInvalidValue;
        end += (int)((pieces + PEER_PIECES - 1) / PEER_PIECES);
    }
    a.seg[6] = end;
    if (end == 0 && !zero) return hipSuccess;
    if (end == 0) end = 1;                      // (nothing but words to clear)
    hipLaunchKernelGGL(pre_attention_kernel, dim3(end), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t checksum_launch(const void* data, uint64_t bytes, uint64_t first_word, uint64_t* out, hipStream_t s) {
    if (bytes % 8 || ((uintptr_t)data % 8)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, s, out);
    if (bytes)
        hipLaunchKernelGGL(checksum_kernel, dim3(grid_for((long)(bytes / 8), 256 * 8, 2048)), dim3(256), 0, s,
                           (const uint64_t*)data, bytes / 8, first_word, (unsigned long long*)out);
    return hipGetLastError();
}

hipError_t f32_to_bf16_launch(const float* src, bf16* dst, size_t n, hipStream_t s) {
    if (!n) return hipSuccess;
    hipLaunchKernelGGL(f32_to_bf16_kernel, dim3(grid_for((long)n, 256 * 4)), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}
