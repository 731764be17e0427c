// Device code shared by the kernels that place heads as attention reads them: the pre-attention kernel, from projected rows in
// memory, and the GEMM's epilogue, from the tile it has just computed.  The arithmetic is written out (fmaf) so that both give
// the same bits.
#pragma once
#include "common.h"
#include "kernels.h"

namespace {

__device__ __forceinline__ void unpack8(const uint32x4& u, float* f) {
    f[0] = __uint_as_float(u.x << 16); f[1] = __uint_as_float(u.x & 0xffff0000u);
    f[2] = __uint_as_float(u.y << 16); f[3] = __uint_as_float(u.y & 0xffff0000u);
    f[4] = __uint_as_float(u.z << 16); f[5] = __uint_as_float(u.z & 0xffff0000u);
    f[6] = __uint_as_float(u.w << 16); f[7] = __uint_as_float(u.w & 0xffff0000u);
}

__device__ __forceinline__ int local_pos(const TokenMap& m, int i) {
    return i < m.len0 ? m.pos0 + i : m.pos1 + (i - m.len0);
}
// i-th position (ascending) that is NOT local
__device__ __forceinline__ int remote_pos(const TokenMap& m, int i) {
    if (i < m.pos0) return i;
    i += m.len0;
    if (m.len1 == 0 || i < m.pos1) return i;
    return i + m.len1;
}

// v of the lane whose number differs in bit O (of four): by a DPP move, where __shfl_xor goes through the LDS
template <int O>
__device__ __forceinline__ float lane_xor(float v) {
    const int x = __float_as_int(v);
    int t;
    if constexpr (O == 8) t = __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, true);            // rows of 16 turned by 8
    else if constexpr (O == 4) t = __builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, x, 0x104, 0xf, 0x5, true), x, 0x114, 0xf, 0xa, false);
    else if constexpr (O == 2) t = __builtin_amdgcn_update_dpp(0, x, 0x4e, 0xf, 0xf, true);        // within quads
    else t = __builtin_amdgcn_update_dpp(0, x, 0xb1, 0xf, 0xf, true);
    return __int_as_float(t);
}

// 8 elements of a q or k vector whose hd / 8 pieces lie in neighbouring lanes: RMSNorm over the vector with weights w, then the
// rotation of its pairs by (c, s).  DPP: where the registers that the moves take are there (the pre-attention kernel, bound by memory, has
// its waves instead: 19.1 us with shuffles, 22.6 without).
template <bool DPP>
__device__ __forceinline__ uint32x4 head_piece(const uint32x4& u, int hd, bool norm, const float (&w)[8], bool turn, const floatx4& c, const floatx4& s) {
    float f[8];
    unpack8(u, f);
    if (norm) {
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) ss = fmaf(f[e], f[e], ss);
        if constexpr (DPP) {
            const float far = lane_xor<8>(ss);
            ss = hd == 128 ? ss + far : ss;
            ss += lane_xor<4>(ss);
            ss += lane_xor<2>(ss);
            ss += lane_xor<1>(ss);
        } else {
            for (int o = hd >> 4; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
        }
        const float rs = rsqrtf(ss * (hd == 128 ? 1.f / 128 : 1.f / 64) + 1e-6f);
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = f[e] * rs * w[e];
    }
    if (turn) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = f[2 * e], b = f[2 * e + 1];
            f[2 * e] = fmaf(a, c[e], -(b * s[e]));
            f[2 * e + 1] = fmaf(a, s[e], b * c[e]);
        }
    }
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16)f[e];
    return __builtin_bit_cast(uint32x4, o);
}

// 16 bytes (8 elements) of each of eight tokens side by side, turned round in registers: element e of the tokens is 16 bytes at `off` + e rows
// of n_pad elements from `base` (on 16 bytes).
__device__ __forceinline__ void v_turned_line(const uint32x4 (&u)[8], char* base, uint32_t off, uint32_t n_pad) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        uint32x4 t;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            t[k] = __builtin_amdgcn_perm(u[2 * k + 1][e >> 1], u[2 * k][e >> 1], e & 1 ? 0x07060302u : 0x05040100u);
        *(uint32x4*)(base + (off + (uint32_t)e * n_pad * 2u)) = t;
    }
}
// The same of `cnt` <= 8 tokens wherever they are: element e of token k goes to to(k)[e * n_pad].
template <class To>
__device__ __forceinline__ void v_turned(const uint32x4 (&u)[8], int cnt, uint32_t n_pad, To to) {
    uint16_t* const dst = to(0);
    if (cnt == 8 && to(7) - dst == 7 && ((uintptr_t)dst & 15) == 0) {
        v_turned_line(u, (char*)dst, 0u, n_pad);
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (k >= cnt) break;
            uint16_t* const d = to(k);
#pragma unroll
            for (int e = 0; e < 8; ++e) d[(uint32_t)e * n_pad] = (uint16_t)(u[k][e >> 1] >> (16 * (e & 1)));
        }
    }
}

}  // namespace
