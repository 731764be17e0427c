/* chunkflow_diag.h -- diagnostic entry points of libchunkflow.so: single kernels exposed so that each
 * can be checked against the oracle in isolation, the host-only views of the launch planners, and a
 * matrix-core rate probe.  None of them is part of the block path's contract (chunkflow.h); tests and
 * microbenchmarks use them.  Same conventions: 0 or a negative cf_status, cf_last_error(NULL) for text,
 * every pointer is DEVICE memory unless named host_*, streams are hipStream_t passed as void*.
 */
#ifndef CHUNKFLOW_DIAG_H
#define CHUNKFLOW_DIAG_H

#include "chunkflow.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Host-only view of how an attention launch over H heads, nq queries and nk keys of width head_dim is
 * shaped (Sec. 2.1: each rank attends over the whole sequence for its heads; App. B: the 4*B*S^2*d
 * term): *waves_per_workgroup receives 4 (two workgroups per CU), 7 or 8 (one), each wave owning 32
 * queries.  The choice minimises an estimate of the launch's time: generations of workgroups times the
 * time of one generation, fitted to measurements.  No GPU is touched.  CF_ERR_ARG: non-positive
 * sizes, head_dim other than 64 or 128, NULL result.  cf_op_attention runs as this says, or, with few queries, with its keys in
 * parts that go to the waves of a workgroup; a block's attention may be cut or dealt out instead (cf_plan_block_attention). */
int cf_plan_attention(int32_t H, int32_t nq, int32_t nk, int32_t head_dim, int32_t* waves_per_workgroup);

/* Host-only view of how a block launches attention, `heads` heads for each of `batch` samples: with its keys in
 * `parts` parts (1 = whole).  all_parts: 0 = parts are computed by workgroups of their own and merged by a kernel afterwards, 1 = a
 * workgroup has all parts of its queries, one after the other (where the batch fills the chip), 2 = a wave to each (few queries), as in
 * cf_op_attention_form.  deal: sweeps dealt out by the grid (0), by the kernel in even shares (1) or as
 * workgroups come for the next sweep (2), whole sweeps of 8-wave workgroups in either case.  `waves`: of a workgroup.
 * The number of parts is a matter of one sample alone, and the bits of the result with it (whatever the scores: also
 * where those of 32 queries make their sweep start over, see attention.hip).  No GPU is touched. */
typedef struct cf_attention_plan {
    int32_t waves, parts, all_parts, deal;
} cf_attention_plan;
int cf_plan_block_attention(int32_t heads, int32_t batch, int32_t nq, int32_t nk, int32_t head_dim, cf_attention_plan* plan);

/* Host-only view of the tile a linear layer over m_rows tokens and n_features output features is
 * launched with (the GEMMs of App. B), for a layer of 3072 input features: *tile_rows receives 256 (256 or 192
 * tokens x 256 features, one workgroup per CU) or 128 (a smaller tile).  The big tile has the better arithmetic intensity; a
 * smaller one is taken where the big one would leave most CUs without a tile.  No GPU is touched.
 * CF_ERR_ARG: non-positive sizes, NULL result. */
int cf_plan_linear(int32_t m_rows, int32_t n_features, int32_t* tile_rows);

/* Host-only view of how a block launches a linear layer of k input features over `rows` tokens of each of `batch`
 * samples (rows2 > 0: with a second layer over rows2 tokens in the same launch, as the streams of a double-stream block): its
 * tile of tokens x features exactly (of a q, k, v projection: where it leaves rows; one that places its heads needs whole ones in a tile's half,
 * and may take another).  residual: with the gated fp32 residual, whose sum over k may be cut into `parts` parts
 * (a matter of one sample alone, and the bits with it); the tile is then that of the parts, and last_tile_* is not zero where
 * the last part has a launch of its own, which puts the sum together.  No GPU is touched. */
typedef struct cf_linear_plan {
    int32_t tile_tokens, tile_features, parts, last_tile_tokens, last_tile_features;
} cf_linear_plan;
int cf_plan_block_linear(int32_t rows, int32_t rows2, int32_t batch, int32_t n_features, int32_t k, int32_t residual, cf_linear_plan* plan);

/* Whether the workgroups of the parts of such a cut sum put it together themselves, within one launch: *meet 1 or 0 (a kernel of its
 * own does it, or the last part's launch; no cut sum).  Arguments and errors as above. */
int cf_plan_block_meet(int32_t rows, int32_t rows2, int32_t batch, int32_t n_features, int32_t k, int32_t* meet);

/* Host-only view of how that launch (of a cut sum: of its parts) lets CUs without a tile in the last round of workgroups fetch for the others:
 * `fetching` workgroups (0: none) behind `tiles` with a tile or as padding, which read every stride-th 512 bytes of the listed panels, one slab of 64
 * features per pace_ns, and stop deadline_ns after they began.  A panel is (XCD, first or second layer, 0 weights or 1 activations, first byte, bytes), of
 * weights at offset 0 in one buffer and activations of k per row; those of one XCD lie together, 64 at most. */
typedef struct cf_fetch_plan {
    int32_t tiles, fetching, with_activations, stride, pace_ns, deadline_ns, panels, pad;
    int64_t panel[8 * 64][5];
} cf_fetch_plan;
int cf_plan_block_fetch(int32_t rows, int32_t rows2, int32_t batch, int32_t n_features, int32_t k, int32_t residual, cf_fetch_plan* plan);

/* ---- single kernels.  `blob` holds W (and bias) at the given byte offsets. */
/* out[m,n] = A[m,:] . W[n,:] + bias[n]; features < n_split stored bf16 to out0[m*ld0+n], the rest
 * through GELU (tanh form, or erf form if gelu_erf) to out1[m*ld1 + n - n_split] (App. B linear layers). */
int cf_op_linear(const uint16_t* A, int32_t lda, const void* blob, uint64_t w_off, int64_t bias_off,
                 int32_t M, int32_t N, int32_t K, int32_t n0, int32_t n1, int32_t n_split,
                 uint16_t* out0, int32_t ld0, uint16_t* out1, int32_t ld1, int32_t gelu_erf, void* stream);
/* y = resid + gate * (A . W^T + bias), fp32 (gate NULL = 1). */
int cf_op_linear_residual(const uint16_t* A, int32_t lda, const void* blob, uint64_t w_off, int64_t bias_off,
                          int32_t M, int32_t N, int32_t K, const float* resid, const float* gate,
                          float* y, void* stream);
/* The same on tiles of the caller's choice (those of cf_plan_block_linear), with the sum over K in `parts` parts, put together by
 * a kernel of its own, (last_joins 1) by the launch of the last part or (2, up to three parts) by the workgroups of all parts in one
 * launch.  scratch, 16-byte aligned: parts * M * N floats; for 2, four words per tile that are ZERO and parts floats per output of whole tiles. */
int cf_op_linear_residual_form(const uint16_t* A, int32_t lda, const void* blob, uint64_t w_off, int64_t bias_off, int32_t M, int32_t N,
                               int32_t K, const float* resid, const float* gate, float* y, int32_t tile_tokens, int32_t tile_features,
                               int32_t parts, int32_t last_joins, void* scratch, uint64_t scratch_bytes, void* stream);
/* O[h,q,:] = softmax(Q K^T / sqrt(hd)) V; Q [H,nq,hd], K [H,nk,hd], Vt [H,hd,nk_pad] (pad zero),
 * O [H,nq,hd] (App. B attention term, no mask). */
int cf_op_attention(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O,
                    int32_t H, int32_t nq, int32_t nk, int32_t nk_pad, int32_t hd, void* stream);
/* The same in a form of the caller's choice, as a block may launch it: keys in `parts` parts, with all_parts those of
 * a query tile in one workgroup, one after the other (1) or a wave to each (2; up to 8 parts, 4 with 128-wide heads), or (parts = 1) dealt out as `deal` says; head width 128 and more than 7 * 32 query tiles of 256 for deal 1 and 2,
 * more than 192 keys for deal 2.  no_wait: a workgroup that would go on
 * with a sweep begun by another does not find it, as if that one had not run in time.  scratch: 16-byte aligned; none with
 * all_parts, parts * H * ceil(nq / 32) * 32 * (hd + 2) floats, or for a deal 4096 bytes that are ZERO followed by 24 * 32 * 512 * 66 floats. */
int cf_op_attention_form(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, int32_t H, int32_t nq, int32_t nk,
                         int32_t nk_pad, int32_t hd, int32_t parts, int32_t all_parts, int32_t deal, int32_t no_wait, void* scratch, uint64_t scratch_bytes,
                         void* stream);
/* xn = LayerNorm(x) * (1 + scale) + shift, bf16 out. */
int cf_op_ln_modulate(const float* x, const float* shift, const float* scale, uint16_t* xn,
                      int32_t rows, int32_t d, void* stream);
/* m = W t + b over a blob holding W [n,K] and b [n]. */
int cf_op_modvec(const void* blob, uint64_t w_off, uint64_t b_off, const float* t, float* m,
                 int32_t n, int32_t K, void* stream);
/* Diagnostic, not part of the block path: 256 workgroups of 4 waves issue `iters` x 16 bf16 MFMAs
 * (32x32x16) each on registers alone; a launch is 256 * 4 * iters * 16 * 32768 FLOPs.  Timed by the
 * caller, it gives the matrix-core rate the chip sustains under load (Sec. 3.1's eta_c * P_peak has
 * this as its ceiling, not the published peak).  The clock the chip settles to depends on the data:
 * random_operands = 0 repeats one pair of small-valued fragments, 1 cycles through sixteen pairs of
 * unit-variance pseudo-random fragments.  `out`: 65536 floats of device memory. */
int cf_op_mfma_rate(int32_t iters, int32_t random_operands, float* out, void* stream);
/* Diagnostic, not part of the block path: the same loop with the other work a kernel's waves have to issue
 * beside their MFMAs -- per 16 MFMAs a wave makes `reads_per_16` LDS fragment reads (16 bytes per lane, through a
 * ring of four fragments) and per MFMA `valu_per_mfma` fused multiply-adds and `exp_per_mfma` exp2's; `waves`
 * (4 or 8) waves per workgroup, one workgroup per CU, no global memory traffic, no barriers.  Timed by the
 * caller it gives the ceiling of an instruction mix: the attention kernel's is one read, about four VALU
 * operations and one exp2 per MFMA on 8 waves, the GEMM's one read per two MFMAs on 4 waves.  A launch is
 * 256 * waves * iters * 16 * 32768 FLOPs.  `out`: 256 * 64 * waves floats of device memory.  Built mixes:
 * reads_per_16 in {0, 8, 16} x (valu, exp) in {(0,0)}, and (2,0), (4,0) without reads, (2,1), (4,1) with any
 * reads; anything else is CF_ERR_ARG. */
int cf_op_mix_rate(int32_t iters, int32_t waves, int32_t reads_per_16, int32_t valu_per_mfma, int32_t exp_per_mfma,
                   float* out, void* stream);
#ifdef __cplusplus
}
#endif
#endif /* CHUNKFLOW_DIAG_H */
