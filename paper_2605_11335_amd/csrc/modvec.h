// The modulation matrix-vector product, for a launch of its own (elementwise.hip) and for workgroups behind those of attention.
#pragma once
#include "common.h"
#include "heads.h"
#include "kernels.h"

namespace {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// m[n] = W[n,:] . t + b[n]; a wave owns MV_ROWS consecutive rows so that each slice of t is read
// once per MV_ROWS weight vectors and that many 16-byte loads are in flight per lane.  A row's sum
// is accumulated in the same lane order whatever rows share its wave.
constexpr int MV_ROWS = 4;
// U steps of the walk over K are fetched together (U * (MV_ROWS + 2) loads in flight per lane): with one
// step per round trip to memory the kernel ran at the latency of K / 512 + MV_ROWS dependent loads, not
// at the bandwidth of the weight matrix.  A lane whose step lies past the end re-reads the row's last
// chunk and adds nothing.  U changes no sum's order.
template <int U>
__device__ __forceinline__ void modvec_rows(const ModRows& j, int mat, int sample, int n) {
    const uint64_t w_off = mat ? j.w_off[1] : j.w_off[0], b_off = mat ? j.b_off[1] : j.b_off[0];
    const float* __restrict__ t = j.t + (size_t)sample * j.K;
    float* __restrict__ m = (mat ? j.m[1] : j.m[0]) + (size_t)sample * j.m_bs;
    const int lane = threadIdx.x & 63, K = j.K, n1 = j.n1;
    if (n >= n1) return;
    float acc[MV_ROWS];
#pragma unroll
    for (int r = 0; r < MV_ROWS; ++r) acc[r] = 0.f;
    const int nc = K / 8;                        // 16-byte chunks per row
    for (int c0 = lane; c0 < nc; c0 += 64 * U) {
        uint32x4 u[U][MV_ROWS];
        floatx4 t0[U], t1[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int c = min(c0 + 64 * q, nc - 1);
#pragma unroll
            for (int r = 0; r < MV_ROWS; ++r) {
                const int nr = min(n + r, n1 - 1);
                u[q][r] = *(const uint32x4*)wv_ptr(j.W, w_off + ((uint64_t)nr * K + (uint64_t)c * 8) * 2);
            }
            t0[q] = *(const floatx4*)(t + c * 8);
            t1[q] = *(const floatx4*)(t + c * 8 + 4);
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (c0 + 64 * q < nc) {
#pragma unroll
                for (int r = 0; r < MV_ROWS; ++r) {
                    float w[8];
                    unpack8(u[q][r], w);
                    acc[r] += w[0] * t0[q].x + w[1] * t0[q].y + w[2] * t0[q].z + w[3] * t0[q].w + w[4] * t1[q].x + w[5] * t1[q].y +
                              w[6] * t1[q].z + w[7] * t1[q].w;
                }
            }
        }
    }
    // lane r adds the bias of row r and writes it: the MV_ROWS bias loads go out side by side
    float mine = 0.f;
#pragma unroll
    for (int r = 0; r < MV_ROWS; ++r) {
        const float v = wave_sum(acc[r]);
        if (lane == r) mine = v;
    }
    if (lane < MV_ROWS && n + lane < n1) m[n + lane] = mine + wv_bf16(j.W, b_off, n + lane);
}

}  // namespace
