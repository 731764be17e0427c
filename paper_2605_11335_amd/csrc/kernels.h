// Host-visible launchers of the block kernels.  Every launcher validates shapes against
// what its kernel assumes (`*_check` returns a message or nullptr) before anything runs.
#pragma once
#include "common.h"

enum { EPI_SPLIT_GELU = 0, EPI_GATE_RESID = 1 };

// Positions of this rank's tokens in the joint sequence: up to two contiguous segments
// (text rows, image rows).  Local row i < len0 sits at pos0 + i, else at pos1 + (i - len0).
struct TokenMap {
    int n_total, n_local;
    int pos0, len0, pos1, len1;
};

// Split a projection output into head-major attention operands, with optional per-head RMSNorm.
struct RelayoutArgs {
    const bf16* src;        // [rows, ld] ; head h of tensor t at column col0[t] + h*hd
    int ld, rows;
    int col_q, col_k, col_v;          // -1 = tensor absent
    int n_heads;                      // heads present in src (H)
    int h0, h_local;                  // heads kept for attention: [h0, h0 + h_local)
    int hd;
    WView W; uint64_t qn_off, kn_off; int has_norm;
    const float *rope_cos, *rope_sin; // [n_local, hd/2] by local row, or NULL: rotate q,k pairs (2i, 2i+1) after the norm
    TokenMap map; int row0;           // src row i is local row row0 + i
    bf16 *Q, *K, *Vt;                 // [h_local, n_total, hd] x2, [h_local, hd, n_pad]
    int n_pad;
    bf16 *send_q, *send_k, *send_v;   // [n_heads - h_local, n_local, hd] (may be NULL)
};

// A projection whose features are heads of q, k and v, placed as attention reads them by the launch that computes them (`on`),
// instead of going out as rows that a pass of their own relays: q, k normed and rotated, own v turned round, other heads to the send buffers.
struct HeadsOut {
    int on, first;                    // tensor of the first n_heads * hd features (0 q, 1 k, 2 v); the next ones follow
    int rps;                          // tokens of a sample of a batch (0 = one sample); sample strides:
    long op_bs, vt_bs, send_bs;       // of Q and K, of Vt, of the send buffers
    RelayoutArgs r;                   // (src, ld, rows and columns unused)
};

// What every linear-layer kernel is launched with: all of it is read by every one, but for `words`.
struct GemmCore {
    const bf16* A;      // [M, lda] activations
    int lda;
    WView W;            // weight blob view
    uint64_t w_off;     // blob offset of W[0][0]; W is [N, K] bf16 row-major
    uint64_t bias_off;  // blob offset of bias[N] (bf16)
    int has_bias;
    int M, N, K;
    int n0, n1;         // output-feature panel covered by this launch
    int epi;
    // EPI_SPLIT_GELU: features [0, n_split) -> out0[m*ld0 + n] (bf16);
    //                 features [n_split, N) -> GELU -> out1[m*ld1 + col1_off + n - n_split]
    bf16* out0; int ld0; int n_split;
    bf16* out1; int ld1; int col1_off;
    int act_erf;        // the activation of out1: 0 = tanh form of GELU, 1 = erf form
    // EPI_GATE_RESID: y[m*ldy + n] = resid[m*ldy + n] + gate[n] * (acc + bias)   (fp32; gate NULL = 1)
    const float* resid; const float* gate; float* y; int ldy;
    // A batch of samples stacked along M (rows_per_sample > 0): row m is row i = m % rows_per_sample of
    // sample b = m / rows_per_sample; it uses gate + b*gate_bs and sits at b*resid_bs + i*ldy in resid,
    // b*y_bs + i*ldy in y (strides in elements).  rows_per_sample = 0: one sample, strides unused.
    int rows_per_sample; long gate_bs, resid_bs, y_bs;
    // EPI_GATE_RESID with the sum over K cut into ksplits parts of part_slabs 64-wide slabs each (gemm_set_split), computed
    // by workgroups of their own into part[ksplits][M][N] and put together by a second launch; 0 or 1 = whole.
    int ksplits, part_slabs;
    float* part;
    uint32_t* words;    // where the parts' workgroups put the sum together themselves (GemmPlan::meet): gemm_meet_words words that are zero
};
// A layer as the host describes it.  Only launches that place heads take it all along: 264 bytes more cost a launch 0.2 us, whatever it
// does (307 x 1024 x 4224 24.9 us / 24.8 without, 300 x 1024 x 1024 11.5 / 11.3, 512 x 2048 x 512 9.24 / 9.08).
struct GemmArgs : GemmCore {
    int may_meet;       // the parts' workgroups may put the sum together: part holds gemm_meet_floats floats and words is set
    int col_step;       // > 1: feature-tiles are walked in steps of so many (set by the launch)
    HeadsOut heads;     // EPI_SPLIT_GELU: where features [0, n_split) go instead of out0
};
int gemm_splits(int rows, int rows2, int N, int K);      // parts to cut K into, for one sample's tokens (rows2: of a second layer in the launch)
void gemm_set_split(GemmArgs* g, int splits, float* part);
const char* gemm_check(const GemmArgs& g);
enum { GEMM_256x256 = 0, GEMM_128x128 = 1, GEMM_128x256 = 2, GEMM_128x64 = 3, GEMM_64x64 = 4, GEMM_192x256 = 5, GEMM_TILES = 6 };     // tokens x features
// How a layer, or two in one launch (`second` not NULL), is launched: its tile; of a cut sum the tile of the parts, and that of
// the last part where its launch puts the sum together (else -1).
// meet: the workgroups of the parts put the sum together.
struct GemmPlan { int tile, last, meet; };
uint32_t gemm_meet_words(const GemmPlan& plan, const GemmArgs& g, const GemmArgs* second);     // 0 unless plan.meet
uint64_t gemm_meet_floats(int parts, uint64_t rows, int problems, int N);      // scratch for any tile, N a multiple of 256
GemmPlan gemm_plan(const GemmArgs& g, const GemmArgs* second);
void gemm_tile_shape(int tile, int* tokens, int* features);
double gemm_fill(int M, int n);        // share of the launched rounds of workgroups that n features x M tokens fill
hipError_t gemm_launch(const GemmArgs& g, hipStream_t s);
hipError_t gemm_launch_as(const GemmPlan& plan, const GemmArgs& g, hipStream_t s);     // (diagnostic) as told
// Workgroups behind the tiles of a launch that fetch for its last round (gemm_kernel.h).
struct IdleFetch {
    uint32_t workgroups;                       // 0 = none
    uint32_t ticks_per_chunk, deadline;        // of 10 ns
    int stride, with_a;                        // every stride-th chunk; the activations too
};
// `tiles`: workgroups of the launch, with what pads the first problem's, tiles1 of them the second's; cut: the parts of a cut sum
IdleFetch gemm_idle_fetch_plan(int bm, int bn, bool cut, const GemmArgs& g, const GemmArgs* second, uint32_t tiles, uint32_t tiles1);
// (diagnostic) how the launch of a plan's tiles fetches; its panels by XCD, 64 of them at most, as (XCD, problem, 0 weights | 1 activations, first byte, bytes)
struct FetchPanel { int64_t xcd, problem, activations, begin, bytes; };
IdleFetch gemm_idle_fetch_view(const GemmPlan& plan, const GemmArgs& g, const GemmArgs* second, uint32_t* tiles, FetchPanel* panels, int* n_panels);
// per epilogue: one problem, or two in one launch (`second` not NULL), with the given tile
hipError_t gemm_launch_split_gelu(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s);
hipError_t gemm_launch_split_gelu_erf(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s);
hipError_t gemm_launch_heads(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s);           // features [0, n_split) are heads
hipError_t gemm_launch_heads_erf(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s);
hipError_t gemm_launch_gate_resid(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s);
hipError_t gemm_launch_partial(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s);     // the parts of a cut sum only
hipError_t gemm_launch_last_part(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s);   // its last part, added to the others
hipError_t gemm_launch_meet(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s);        // all parts, which put it together
hipError_t mfma_rate_launch(int iters, int random_operands, float* out, hipStream_t s);   // diagnostic: MFMAs on registers only
// diagnostic: MFMAs sharing the SIMD with LDS fragment reads and VALU work (see gemm.hip for the supported mixes)
hipError_t mix_rate_launch(int iters, int waves, int reads16, int valu, int exps, float* out, hipStream_t s);
// two independent problems in one launch
bool gemm_can_pair(const GemmArgs& g0, const GemmArgs& g1);
bool gemm_heads_pay(const GemmArgs& g, const GemmArgs* second, double separate_us);      // HeadsOut, or rows and a pass over them
hipError_t gemm_launch_pair(const GemmPlan& plan, const GemmArgs& g0, const GemmArgs& g1, hipStream_t s);

// m[b][n] = sum_k W[n,k] t[b][k] + bias[n]  (fp32 out), rows [n0, n1), for `batch` vectors t + b*K -> m + b*m_bs;
// mats = 2: a second matrix of the same shape (w_off[1], b_off[1]), its result at m[1].
struct ModRows {
    WView W;
    uint64_t w_off[2], b_off[2];
    const float* t;
    float* m[2];
    int n0, n1, K, batch, mats;
    long m_bs;
};
// zero: so many words to clear for the launches that follow (a multiple of 4, 16-byte aligned), or NULL.
hipError_t modvec_launch(const ModRows& j, hipStream_t s, uint32_t* zero = nullptr, uint32_t zero_words = 0);

struct AttnArgs {
    const bf16* Q;      // [H, nq, hd] head-major
    const bf16* K;      // [H, nk, hd]
    const bf16* Vt;     // [H, hd, nk_pad] keys contiguous, pad columns zero
    bf16* O;            // element (h, q, :) at O + (h / hps)*o_bs + (h % hps)*o_hs + q*o_qs
    long o_hs, o_qs, o_bs;
    int H, nq, nk, nk_pad, hd;
    int hps;            // heads per sample (a batch is H / hps samples of hps heads each); 0 = H
    float scale;        // 1/sqrt(hd)
    // Scatter mode (the second Ulysses exchange, Sec. 2.1, done by the attention kernel's own stores; O unused):
    // query position q of head h (sample b = h / hps, head hh = h % hps) is one of this rank's positions in `map`
    // -> columns (h0 + hh)*hd of the output projection's operand, row i of the map's first segment at
    // dst0 + b*bs0 + i*ld, of its second segment at dst1 + b*bs1 + i*ld; any other position -> row of the send
    // buffer, send + b*send_bs + (hh*(n_total - n_local) + index among the remote positions)*hd (send NULL: dropped).
    int scatter;
    TokenMap map;
    bf16 *dst0, *dst1, *send;
    int ld, h0;
    long bs0, bs1, send_bs;
    // The keys in `splits` parts of part_tiles 64-key tiles each (attn_set_split), merged by a second kernel; 1 = whole.
    // Scratch, float: part_o [splits][H][ceil(nq/32)][32 * hd] in register order, part_ml [..][32] (reference, row sum).
    // all_parts: a workgroup has all parts of its queries, one after the other or a wave to each, and merges them itself: same bits,
    // no scratch.
    int splits, part_tiles, all_parts;
    float *part_o, *part_ml;
    // Sweeps dealt out by the kernel (attn_set_deal) instead of one workgroup per query tile; state NULL = no.  Scratch: the
    // states of cut sweeps, and ATTN_FLAGS words that must be zero when the launch starts.  even_wait: 0 = no state is ever
    // waited for or taken, as when the wait runs out.
    float* even_state;
    uint32_t* even_flags;
    int even_units, even_last, even_cuts, even_wait;
    // Modulation rows that workgroups behind those of attention compute (attn_takes_mod); n1 = 0: none.
    ModRows mod;
    int mod_blocks;            // of them (set by the launch)
};
enum { ALL_PARTS_IN_TURN = 1, ALL_PARTS_WAVES = 2 };      // AttnArgs::all_parts
int attn_splits(int heads, int nq, int nk, int hd);      // parts to cut the keys into, for one sample's heads
int attn_all_parts(int heads, int nq, int nk, int hd, int splits);     // for all samples' heads: AttnArgs::all_parts
uint64_t attn_part_floats(int heads, int nq, int hd, int splits);      // scratch for all samples' heads, parts apart; 0 if splits is 1
void attn_set_split(AttnArgs* a, int splits, float* scratch);          // after H, nq, nk and hd are set
int attn_deal(int H, int nq, int nk, int hd, int splits);              // how the sweeps of all samples' heads are dealt out: 0 by the grid, 1 even, 2 drawn
uint64_t attn_deal_floats(int deal);                                   // scratch for the states of cut sweeps
void attn_set_deal(AttnArgs* a, int deal, float* state, uint32_t* flags);      // after attn_set_split
constexpr int ATTN_FLAGS = 1024;
bool attn_takes_mod(const AttnArgs& a);        // whether its launch has room for a.mod (host arithmetic only; after the set calls)
const char* attn_check(const AttnArgs& a);
hipError_t attn_launch(const AttnArgs& a, hipStream_t s);
int attn_waves(const AttnArgs& a);      // waves per workgroup attn_launch takes (host arithmetic only)

// xn = LN(x) * (1 + scale) + shift  (fp32 in, bf16 out); with ln_w/ln_b (blob offsets, has_affine)
// instead: xn = LN(x) * w + b.
// Row r of a batch is row r % rows_per_sample of sample b = r / rows_per_sample: read at x + b*x_bs, modulated
// with shift + b*mod_bs, scale + b*mod_bs; written densely to xn + r*d.  rows_per_sample = 0: one sample.
struct LnArgs {
    const float *x, *shift, *scale;
    bf16* xn;
    int rows, rows_per_sample;
    long x_bs, mod_bs;
};
// one or two (the streams of a double-stream block) in one launch, rows of width d
hipError_t ln_modulate_launch(const LnArgs* parts, int n_parts, int d, hipStream_t s);
hipError_t ln_affine_launch(const float* x, const WView& W, uint64_t w_off, uint64_t b_off, bf16* xn,
                            int rows, int d, hipStream_t s);

// What this rank receives from the second exchange (Sec. 2.1): the attention output of the other ranks' heads for
// its own tokens, peer_attn [n_local, n_heads - h_local, hd], copied into the columns of those heads in the
// output projection's operand (rows of the map's first segment at dst, of its second at dst1; leading dimension ld).
struct PeerAttnArgs {
    const bf16* peer_attn;            // NULL: nothing to copy
    bf16 *dst, *dst1;
    int ld, n_heads, h0, h_local, hd;
    TokenMap map;
};

// One launch for everything that does not depend on attention itself: the relayout of up to two parts (one per
// stream), when given the peer rows (what the first exchange delivers) placed at the remote positions of
// parts[0]'s operands (q, k copied; v transposed), and the peer attention rows of the second exchange.
// zero: ATTN_FLAGS words to clear for the attention launch that follows, or NULL.
hipError_t pre_attention_launch(const RelayoutArgs* parts, int n_parts, const bf16* peer_q, const bf16* peer_k,
                                const bf16* peer_v, const PeerAttnArgs& pa, uint32_t* zero, hipStream_t s);

hipError_t checksum_launch(const void* data, uint64_t bytes, uint64_t first_word, uint64_t* out, hipStream_t s);
hipError_t f32_to_bf16_launch(const float* src, bf16* dst, size_t n, hipStream_t s);
