// Host side of the linear layers: argument checks, the choice of the tile, dispatch; and the matrix-core rate
// diagnostics.  The kernels themselves are in gemm_kernel.h.
#include <algorithm>

#include "gemm_kernel.h"

const char* gemm_check(const GemmArgs& g) {
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return "gemm: empty shape";
    if (g.K % 64) return "gemm: K must be a multiple of 64";
    if (g.N % 8) return "gemm: N must be a multiple of 8";
    if (g.n0 < 0 || g.n1 > g.N || g.n0 >= g.n1 || (g.n0 % 8) || (g.n1 % 8)) return "gemm: bad feature panel";
    if (g.lda < g.K || (g.lda % 8)) return "gemm: lda must be >= K and a multiple of 8";
    if ((uint64_t)g.lda * 512 >= (1ull << 32)) return "gemm: lda too large for 32-bit offsets inside a tile";
    if ((uint64_t)g.M * g.lda * 2 >= (1ull << 32)) return "gemm: activations beyond 4 GiB (32-bit buffer range)";
    if ((g.w_off % 16) || (g.has_bias && (g.bias_off % 16))) return "gemm: weight/bias offsets must be 16-byte aligned";
    if (((uintptr_t)g.A) % 16) return "gemm: A must be 16-byte aligned";
    if (g.epi == EPI_SPLIT_GELU) {
        if (g.n_split % 8) return "gemm: n_split must be a multiple of 8";
        const HeadsOut& h = g.heads;
        const int section = h.r.n_heads * h.r.hd;
        if (h.on && ((h.r.hd != 64 && h.r.hd != 128) || section <= 0 || section % 256 || g.n_split % section || g.n_split / section > 3 - h.first || g.n0 % 256 ||
                     h.first < 0 || h.rps < 0 || (h.rps && (h.rps < 32 || g.M % h.rps))))
            return "gemm: heads must be whole tensors of 64 or 128 wide heads, of samples of 32 tokens and more";
        if (g.n_split > 0 && !h.on && (!g.out0 || (g.ld0 % 8) || ((uintptr_t)g.out0 % 16))) return "gemm: out0 must be 16-byte aligned with ld0 a multiple of 8";
        if (g.n_split < g.N && (!g.out1 || (g.ld1 % 8) || (g.col1_off % 8) || ((uintptr_t)g.out1 % 16)))
            return "gemm: out1 must be 16-byte aligned with ld1 and col1_off multiples of 8";
    } else if (g.epi == EPI_GATE_RESID) {
        if (!g.resid || !g.y || (g.ldy % 4) || ((uintptr_t)g.y % 16) || ((uintptr_t)g.resid % 16)) return "gemm: bad residual/output";
        if (g.gate && ((uintptr_t)g.gate % 16)) return "gemm: gate must be 16-byte aligned";
        if (g.rows_per_sample < 0 || (g.rows_per_sample && g.M % g.rows_per_sample)) return "gemm: M must be whole samples";
        if (g.ksplits > 1 && (!g.part || ((uintptr_t)g.part % 16) || g.part_slabs < 1 || (g.ksplits - 1) * g.part_slabs >= g.K / 64 ||
                              g.ksplits * g.part_slabs < g.K / 64))
            return "gemm: bad split of K";
        if (g.may_meet && g.ksplits > 1 && (!g.words || g.ksplits > 3)) return "gemm: two or three parts can meet, with words to meet by";
        if (g.rows_per_sample && ((g.gate_bs % 4) || (g.resid_bs % 4) || (g.y_bs % 4) || g.gate_bs < 0 || g.resid_bs < 0 || g.y_bs < 0))
            return "gemm: sample strides must be non-negative multiples of 4 elements";
    } else {
        return "gemm: unknown epilogue";
    }
    return nullptr;
}

// How a launch over n features fills the chip, for cutting a streamed layer into panels: estimated with the two
// square tiles only (cost = rounds x tile area / relative efficiency of the shape).
namespace {
// cost of a launch over n output features in units of one round of 256x256 tiles on all CUs
void tile_costs(int M, long n, double* c256, double* c128) {
    const long m256 = (M + 255) / 256, m128 = (M + 127) / 128;
    const long n256 = (n + 255) / 256, n128 = (n + 127) / 128;
    auto rounds = [](long tiles, long slots) { return (double)((tiles + slots - 1) / slots); };
    *c256 = rounds(m256 * n256, 256) * 1.0;
    *c128 = rounds(m128 * n128, 512) * 2.0 * 0.25 / 0.65;
}
}  // namespace

// Tile shape for a launch.  The larger a tile, the fewer bytes a CU has to take in per FLOP, but the fewer
// workgroups there are and the longer the last round of them.  Estimated time in us = rounds x (slabs x time
// per slab + fixed part), fitted to layers of 64 to 13640 tokens and K = 512 to 15360 with weights read cold
// (one MI355X): a slab takes a lone 256x256 workgroup per CU 1.05 us on a nearly empty chip and 1.35 on a full
// one, a 128x256 one 0.76 to 0.88, 128x128 0.55 alone and 1.07 for the two a CU holds,
// 128x64 0.43 and 0.92, 64x64 0.30 and 0.51; 192x256, for grids that end a little past whole rounds of the big tile,
// 0.85 to 1.05 (1531 x 12288 x 3072: 118 us in 384 tiles, 131 in 288 of 256x256 or 576 of 128x256).
namespace {
struct TileCost { int bm, bn, per_cu; double lone, full, fixed; };      // us per slab of a CU's workgroups: few CUs busy | chip full
constexpr TileCost kTileCost[GEMM_TILES] = {
    {256, 256, 1, 1.05, 1.35, 9.0},
    {128, 128, 2, 0.55, 1.07, 4.5},
    {128, 256, 1, 0.76, 0.88, 6.0},
    {128, 64, 2, 0.43, 0.92, 3.5},
    {64, 64, 2, 0.30, 0.51, 3.0},
    {192, 256, 1, 0.85, 1.05, 7.5},
};
double tile_time(const TileCost& t, long tiles, int K) {
    const double slabs = (K + 63) / 64;
    const long slots = 256L * t.per_cu, rest = tiles % slots;
    double us = (double)(tiles / slots) * (slabs * t.full + t.fixed);
    if (rest) {
        // The last round.  A CU with one workgroup where it could hold two works off its slab alone; where some CUs hold
        // two, those decide, at 0.7 of a full chip's time per slab if they are few (1320 x 3072 x 14336, 264 workgroups of
        // 128x128: 0.76 us) and all of it from 70 % on.
        double slab;
        if (rest > 256) slab = t.full * (0.7 + 0.3 * std::min(1.0, (double)(rest - 256) / 179.0));
        else if (t.per_cu > 1) slab = t.lone;
        else slab = t.lone + (t.full - t.lone) * (double)rest / 256.0;
        us += slabs * slab + t.fixed;
    }
    return us;
}
// Whether a tile's epilogue has whole heads where they are normed: a quadrant's half of the features, or on small tiles all of them
// (gemm_epilogue).
bool heads_fit(const TileCost& t, const GemmArgs& g) {
    return !g.heads.on || !g.heads.r.has_norm || (t.bn < 256 ? t.bn : t.bn / 2) >= g.heads.r.hd;
}
// What a launch covers of a cut sum: all its parts, all but the last, the last
enum Share { ALL_OF_IT, BEFORE_LAST, LAST };
int best_tile(const GemmArgs* const (&g)[2], Share share = ALL_OF_IT, double* time = nullptr) {
    int best = -1;
    double best_us = 0;
    for (int i = 0; i < GEMM_TILES; ++i) {
        if (i == GEMM_256x256 && g[1] && g[1]->ksplits > 1 && share != LAST) continue;        // not built: registers
        if (!heads_fit(kTileCost[i], *g[0]) || (g[1] && !heads_fit(kTileCost[i], *g[1]))) continue;
        const TileCost& t = kTileCost[i];
        long tiles = 0;
        int K = 0;                       // the longest walk
        for (const GemmArgs* p : g)
            if (p) {
                const int parts = p->ksplits <= 1 || share == LAST ? 1 : share == BEFORE_LAST ? p->ksplits - 1 : p->ksplits;
                tiles += (long)((p->M + t.bm - 1) / t.bm) * ((p->n1 - p->n0 + t.bn - 1) / t.bn) * parts;
                K = std::max(K, p->ksplits > 1 ? p->part_slabs * 64 : p->K);
            }
        const double us = tile_time(t, tiles, K);
        if (best < 0 || us < best_us) best = i, best_us = us;
    }
    if (time) *time = best_us;
    return best;
}
// Parts meet where every one of their workgroups has a CU (of two layers with the padding between them, behind which the last ones would wait for
// a whole round on CUs of their XCD: 1653 + 16 x 1536 x 7232 in three, 258, 92 us instead of 67 and 12) and it costs less than a kernel that reads them all: meeting is some 3 us
// (two parts) or 7 (three) and a third of a microsecond per MB of sums, on tiles of 64 features 10 and more; the kernel 5.5 and 0.5 or 0.6 per MB.
// Apart / meeting, with weights from HBM: 576 x 3072 x 12288 in two 64.2 / 62.4 us, 1600 x 3072 x 12288 in two 120.7 / 114.0, 1000 x 2048 x 10240 in three
// 51.4 / 52.6, 1152 x 3072 x 12288 in three 97.5 / 95.5, 1320 x 3072 x 14336 in three 111.0 / 108.6; 64x64 tiles: 150 x 3072 x 13376 in three 43.9 / 51.7.
bool can_meet(int tile, uint32_t workgroups, int parts, double sums) {
    return workgroups <= 256 && kTileCost[tile].bn >= 128 && (parts == 2 || sums >= 2.5e6);
}
}  // namespace

// How a cut sum is put together: by a kernel of its own that reads all parts, or by the launch of its last part, which
// follows that of the others and reads those alone: a pass over a partial result written and read less, a launch of workgroups
// that may fill the chip badly more.  The passes run at 3.5 TB/s.  It pays where a batch fills the chip (9216 tokens x 3072 x 15360
// in two parts: 778 us put together by the kernel, 700 by the last part; 4608 tokens: 373 and 350; 576 tokens: 78 and 106).
GemmPlan gemm_plan(const GemmArgs& g, const GemmArgs* second) {
    const GemmArgs* const both[2] = {&g, second};
    double all, before, last, bytes = 0;
    GemmPlan one = {best_tile(both, ALL_OF_IT, &all), -1, 0};
    if (g.ksplits <= 1) return one;
    const TileCost& t = kTileCost[one.tile];
    const uint32_t tiles = tile_count(g, t.bm, t.bn, true), workgroups = second ? pad_tiles(tiles) + tile_count(*second, t.bm, t.bn, true) : tiles;
    const GemmPlan two = {best_tile(both, BEFORE_LAST, &before), best_tile(both, LAST, &last), 0};
    for (const GemmArgs* p : both)
        if (p) bytes += 4.0 * p->M * (p->n1 - p->n0);
    if (g.may_meet && can_meet(one.tile, workgroups, g.ksplits, bytes / 4)) {
        one.meet = 1;
        return one;
    }
    return before + last + 3.0 + (g.ksplits + 1) * bytes / 3.5e6 < all + 6.0 + (g.ksplits + 2) * bytes / 3.5e6 ? two : one;
}

void gemm_tile_shape(int tile, int* tokens, int* features) {
    *tokens = kTileCost[tile].bm;
    *features = kTileCost[tile].bn;
}

// Which launches fetch ahead for their last round, and how (gemm_kernel.h).  A fetching workgroup gets about 50 GB/s of data that misses
// L2.  Where those of an XCD cannot keep up with its tiles they leave the activations out, and then chunks.  Up to two rounds of
// workgroups: behind more of them the last one is too little of a launch, and its CUs begin it too far apart, to gain anything (4608 x 9216 x
// 3072, 2.5 rounds, none / fetching: 232.0 / 233.5 us; 13640 x 3072 x 14336, 2.5: 959 / 966; 13640 x 9216 x 3072, 7.6: 628 / 633).  The pace is that of
// a tile whose operands lie in L2.  A workgroup stops at the latest when a round at that pace is over since it began itself: one
// that gets its CU late, because another stream's work was there, can make the launch longer by as much as it was late, and at most by that.
IdleFetch gemm_idle_fetch_plan(int bm, int bn, bool cut, const GemmArgs& g, const GemmArgs* second, uint32_t tiles, uint32_t tiles1) {
    IdleFetch f{};
    const uint32_t rest = tiles % 256;
    const int slabs = cut ? g.part_slabs : g.K / BK;
    if (tiles > 512 || rest == 0 || rest > IDLE_MOST || slabs < 4 * FETCH_SLABS) return f;
    if (second && (g.K != second->K || g.part_slabs != second->part_slabs)) return f;
    const double slab_us = bm * bn <= 128 * 256 ? 0.45 : bm * bn <= 192 * 256 ? 0.7 : 1.0;
    double w_bytes = 0, a_bytes = 0;                           // per slab, of an XCD's tiles in the last round
    for (int i = 0; i < (second ? 2 : 1); ++i) {
        const double of = (i ? std::min(rest, tiles1) : rest - std::min(rest, tiles1)) / 8.0;
        const double sharers = std::min(((i ? second->M : g.M) + bm - 1) / bm, 9);       // row-tiles that walk a weight panel together
        w_bytes += std::ceil(of / sharers) * bn * ROWB;
        a_bytes += std::min(std::ceil(of), sharers) * bm * ROWB;
    }
    const double can = (256 - rest) / 8 * 50e3 * slab_us;
    f.workgroups = 256 - rest;
    f.with_a = w_bytes + a_bytes <= can;
    f.stride = (int)std::ceil(w_bytes / can);
    f.ticks_per_chunk = (uint32_t)(slab_us * FETCH_SLABS * 100.0);
    f.deadline = (uint32_t)(slabs * slab_us * 100.0);
    return f;
}

namespace {
// The panels that list_panels lists on each XCD, by the same arithmetic.
template <int BM, int BN>
int panels_of(const GemmArgs& g, const GemmArgs* second, bool cut, uint32_t tiles0, uint32_t tiles0_pad, uint32_t tiles, bool with_a, FetchPanel* out) {
    int n = 0;
    for (uint32_t x = 0; x < 8; ++x)
        for (int i = 0; i < (second ? 2 : 1); ++i) {
            const GemmArgs& p = i ? *second : g;
            const uint32_t first = i ? tiles0_pad : 0, count = i ? tiles - tiles0_pad : tiles0;
            int lane0 = -1;
            for (int lane = 0; lane < 64; ++lane) {
                const uint32_t b = (tiles & ~255u) + x + 8u * lane;
                if (b < first || b >= first + count) continue;
                if (lane0 < 0) lane0 = lane;
                const TilePanels<BM, BN> t(p, cut, xcd_contiguous_id(b - first, count));
                if (t.lists_w(lane, lane0)) out[n++] = FetchPanel{x, i, 0, (int64_t)(t.w_begin + t.k0), (int64_t)t.w_bytes};
                if (with_a && t.lists_a(lane, lane0)) out[n++] = FetchPanel{x, i, 1, (int64_t)t.a_begin, (int64_t)t.a_bytes};
            }
        }
    return n;
}
}  // namespace

IdleFetch gemm_idle_fetch_view(const GemmPlan& plan, const GemmArgs& g, const GemmArgs* second, uint32_t* tiles, FetchPanel* panels, int* n_panels) {
    const int bm = kTileCost[plan.tile].bm, bn = kTileCost[plan.tile].bn;
    const bool cut = g.epi == EPI_GATE_RESID && g.ksplits > 1;
    GemmArgs a[2] = {g, second ? *second : g};
    if (cut && plan.last >= 0)
        for (GemmArgs& p : a) --p.ksplits;
    const uint32_t tiles0 = tile_count(a[0], bm, bn, cut), pad = second ? pad_tiles(tiles0) : tiles0;
    *tiles = second ? pad + tile_count(a[1], bm, bn, cut) : tiles0;
    *n_panels = 0;
    if (!can_idle_fetch(bm, bn, cut ? EPI_PARTIAL : g.epi, second != nullptr)) return IdleFetch{};
    const IdleFetch f = gemm_idle_fetch_plan(bm, bn, cut, a[0], second ? &a[1] : nullptr, *tiles, *tiles - pad);
    if (f.workgroups) {
        auto list = [&](auto panels_of_tile) { *n_panels = panels_of_tile(a[0], second ? &a[1] : nullptr, cut, tiles0, pad, *tiles, f.with_a != 0, panels); };
        if (plan.tile == GEMM_256x256) list(panels_of<256, 256>);
        else if (plan.tile == GEMM_192x256) list(panels_of<192, 256>);
        else list(panels_of<128, 256>);
    }
    return f;
}

// Parts K is cut into.  A layer with few outputs and a long sum (the MLP-out layers of a short sequence or of a rank at
// degree 4 or 8) has few tiles whatever their shape: cut, its workgroups multiply, each with a share of the walk.  The price
// is writing the partial sums and a second kernel that adds them, in the order of the parts, and applies the epilogue: 6 us and two
// passes over them at 4 TB/s.  Taken where the estimate promises a twentieth (2304 x 3072 x 15360 in two parts: a Flux-like
// single-stream block 660 -> 645 us).  A function of one sample's tokens and
// the whole layer only, so that results depend neither on the batch nor on the panels a streamed layer is cut into.
// Priced so also where one sample's parts meet within the launch for less: a batch does not fit the chip at once, and of the layers that
// the lower price would cut besides, it pays for the sums in memory.  30 such, blocks of one / two / four samples, whole and cut: cut 2.2 % faster / 1.4 %
// slower / 1.8 % slower in the mean (2760 x 1536 x 7232 in two: 292 -> 259, 484 -> 509, 882 -> 889 us; 1671 x 2048 x 10176 in three: 357 -> 360,
// 586 -> 590, 1009 -> 1080).
// At most three parts, because a batch that fills the chip pays for each and gains nothing (576 tokens x 3072 x 15360 per sample,
// one sample / eight of them in 1, 2, 3, 4, 5 parts: 103/347, 79/363, 83/395, 69/442, 72/485 us).
int gemm_splits(int rows, int rows2, int N, int K) {
    GemmArgs g{}, g2{};
    g.M = rows; g.N = g.n1 = N; g.K = K;
    g2 = g;
    g2.M = rows2;
    const int slabs = K / 64;
    int best = 1;
    double best_us = 0;
    for (int parts = 1; parts <= 3 && slabs >= 8 * parts; ++parts) {
        gemm_set_split(&g, parts, nullptr);
        if (g.ksplits != parts) continue;
        gemm_set_split(&g2, parts, nullptr);
        double us;
        best_tile({&g, rows2 > 0 ? &g2 : nullptr}, ALL_OF_IT, &us);
        if (parts > 1) us += 6.0 + 2.0 * 4.0 * parts * (double)(rows + rows2) * N / 4e6;
        if (parts == 1 || us < (best == 1 ? 0.95 : 1.0) * best_us) best = parts, best_us = us;
    }
    return best;
}

uint32_t gemm_meet_words(const GemmPlan& plan, const GemmArgs& g, const GemmArgs* second) {
    const TileCost& t = kTileCost[plan.tile];
    return plan.meet ? 4 * (tile_count(g, t.bm, t.bn, false) + (second ? tile_count(*second, t.bm, t.bn, false) : 0)) : 0;
}
uint64_t gemm_meet_floats(int parts, uint64_t rows, int problems, int N) { return parts * (rows + 255ull * problems) * N; }

void gemm_set_split(GemmArgs* g, int splits, float* part) {
    const int slabs = g->K / 64;
    g->part_slabs = splits > 1 ? (slabs + splits - 1) / splits : slabs;
    g->ksplits = splits > 1 ? (slabs + g->part_slabs - 1) / g->part_slabs : 1;
    g->part = part;
}

// How well a launch over n output features uses the chip: work in rounds of 256x256 tiles divided
// by the estimated cost of the better square tile (1 = whole rounds of the big tile).
double gemm_fill(int M, int n) {
    double c256, c128;
    tile_costs(M, n, &c256, &c128);
    const double work = (double)((M + 255) / 256) * (double)((n + 255) / 256) / 256.0;
    return work / std::min(c256, c128);
}

// Diagnostic: nothing but 32x32x16 bf16 MFMAs on registers, one wave per SIMD on every CU, four
// independent accumulators per wave.  Its rate is what the matrix cores sustain at the clock the
// chip settles to under this load (the published peak assumes the maximum clock).  The clock depends
// on what the operands look like: `random_operands` = 0 feeds the same small values to every MFMA,
// 1 feeds sixteen different pairs of pseudo-random fragments spread like N(0,1) data, as a GEMM does.
namespace {
__global__ __launch_bounds__(256) void mfma_rate_kernel(int iters, int random_operands, float* out) {
    bf16x8 a[4], b[4];
    uint32_t h = (blockIdx.x * 256u + threadIdx.x) * 2654435761u + 12345u;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            h = h * 1664525u + 1013904223u;
            const float u = (float)(h >> 8) * (1.0f / 16777216.0f);          // [0, 1)
            h = h * 1664525u + 1013904223u;
            const float w = (float)(h >> 8) * (1.0f / 16777216.0f);
            a[i][e] = random_operands ? (bf16)(3.46f * (u - 0.5f)) : (bf16)(0.001f * (threadIdx.x + e));   // unit variance
            b[i][e] = random_operands ? (bf16)(3.46f * (w - 0.5f)) : (bf16)(0.002f * (e + 1));
        }
    floatx16 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    for (int it = 0; it < iters; ++it)
#pragma unroll
        for (int q = 0; q < 16; ++q)
            acc[q & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[random_operands ? (q & 3) : 0], b[random_operands ? (q >> 2) : 0],
                                                                 acc[q & 3], 0, 0, 0);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) s += acc[i][v];
    out[blockIdx.x * 256 + threadIdx.x] = s;
}
}  // namespace

// `out` holds 256 * 256 floats; FLOPs of a launch = 256 workgroups x 4 waves x iters x 16 MFMAs x 32768
hipError_t mfma_rate_launch(int iters, int random_operands, float* out, hipStream_t s) {
    hipLaunchKernelGGL(mfma_rate_kernel, dim3(256), dim3(256), 0, s, iters, random_operands, out);
    return hipGetLastError();
}

// Diagnostic: what the matrix cores deliver when a wave's MFMAs share the SIMD with the other work a kernel
// has to issue -- LDS fragment reads (ds_read_b128 through a ring of four fragments) and ordinary / transcendental
// VALU instructions.  Per 16 MFMAs (four independent accumulators) a wave issues READS16 fragment reads,
// 16 * VALU fused multiply-adds and 16 * EXPS exp2's; `waves` waves per workgroup, one workgroup per CU.
// No global memory traffic, no barriers: the rate is the ceiling of an instruction mix, whatever the schedule.
namespace {
template <int READS16, int VALU, int EXPS>
__global__ void mix_rate_kernel(int iters, float* out) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    typedef __attribute__((address_space(3))) const volatile bf16x8 lds_frag;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nthr = blockDim.x;
    for (int i = threadIdx.x; i < 65536 / 4; i += nthr) {           // pairs of small bf16 values
        const bf16 lo = (bf16)(0.01f * (i % 37 - 18)), hi = (bf16)(0.01f * (i % 41 - 20));
        ((uint32_t*)smem)[i] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
    }
    __syncthreads();
    bf16x8 a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            a[i][e] = (bf16)(0.01f * ((lane * 7 + e * 3 + i) % 97 - 48));
            b[i][e] = (bf16)(0.02f * ((lane * 5 + e + i * 11) % 89 - 44));
        }
    floatx16 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    float vv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) vv[i] = 0.5f + 0.01f * (lane + i);
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + ((wave * 4096) & 0xffff) + lane * 16;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            acc[q & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[q & 3], b[q >> 2], acc[q & 3], 0, 0, 0);
            if (READS16 > 0 && (q % (16 / (READS16 > 0 ? READS16 : 1))) == 0)
                a[q & 3] = *(lds_frag*)(uintptr_t)(base + ((q * 1024 + it * 64) & 0x3fff));     // the fragment four slots ahead
#pragma unroll
            for (int u = 0; u < VALU; ++u) vv[(q * VALU + u) & 7] = __builtin_fmaf(vv[(q * VALU + u) & 7], 0.9999f, 0.0001f);   // -> 1
#pragma unroll
            for (int u = 0; u < EXPS; ++u) vv[(q + 3) & 7] = __builtin_amdgcn_exp2f(-vv[(q + 3) & 7]);                       // stays in (0, 1]
        }
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) s += acc[i][v];
#pragma unroll
    for (int i = 0; i < 8; ++i) s += vv[i];
    out[blockIdx.x * nthr + threadIdx.x] = s;
}

template <int READS16, int VALU, int EXPS>
hipError_t mix_rate_go(int iters, int waves, float* out, hipStream_t s) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)mix_rate_kernel<READS16, VALU, EXPS>, hipFuncAttributeMaxDynamicSharedMemorySize, 65536);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((mix_rate_kernel<READS16, VALU, EXPS>), dim3(256), dim3(64 * waves), 65536, s, iters, out);
    return hipGetLastError();
}
}  // namespace

// `out`: 256 * 64 * waves floats.  FLOPs of a launch = 256 * waves * iters * 16 * 32768.  Supported mixes:
// reads16 in {0, 8, 16}, valu in {0, 2, 4}, exps in {0, 1}, waves in {4, 8}.
hipError_t mix_rate_launch(int iters, int waves, int reads16, int valu, int exps, float* out, hipStream_t s) {
    if (waves != 4 && waves != 8) return hipErrorInvalidValue;
#define CF_MIX(R, V, E) if (reads16 == R && valu == V && exps == E) return mix_rate_go<R, V, E>(iters, waves, out, s);
    CF_MIX(0, 0, 0) CF_MIX(8, 0, 0) CF_MIX(16, 0, 0)
    CF_MIX(0, 2, 0) CF_MIX(0, 4, 0) CF_MIX(0, 2, 1) CF_MIX(0, 4, 1)
    CF_MIX(8, 2, 1) CF_MIX(8, 4, 1) CF_MIX(16, 2, 1) CF_MIX(16, 4, 1)
#undef CF_MIX
    return hipErrorInvalidValue;
}

// The parts of one or two cut layers added up in order, and the epilogue of gemm_kernel.h: y = resid + gate * (sum + bias).
// A thread per 4 features of a token.  Bound by the partial sums it reads (1320 x 3072 in three parts: 49 MB).
namespace {
struct ReduceArgs { GemmCore g[2]; uint32_t blocks0; };
__global__ __launch_bounds__(256) void gemm_reduce_kernel(ReduceArgs a) {
    const bool second = blockIdx.x >= a.blocks0;
    const GemmCore& g = a.g[second];
    const int quads = (g.n1 - g.n0) / 4;
    const long q = (long)(blockIdx.x - (second ? a.blocks0 : 0)) * 256 + threadIdx.x;
    if (q >= (long)g.M * quads) return;
    const int m = q / quads, n = g.n0 + (q % quads) * 4;
    const float* p = g.part + (size_t)m * g.N + n;
    floatx4 v = *(const floatx4*)p;
    for (int s = 1; s < g.ksplits; ++s) {
        const floatx4 t = *(const floatx4*)(p + (size_t)s * g.M * g.N);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += t[e];
    }
    if (g.has_bias) {
        const uint32x2 b = *(const uint32x2*)wv_ptr(g.W, g.bias_off + 2ull * n);
        v[0] += __uint_as_float(b.x << 16); v[1] += __uint_as_float(b.x & 0xffff0000u);
        v[2] += __uint_as_float(b.y << 16); v[3] += __uint_as_float(b.y & 0xffff0000u);
    }
    int smp = 0, i = m;
    if (g.rows_per_sample) { smp = m / g.rows_per_sample; i = m - smp * g.rows_per_sample; }
    const floatx4 r = *(const floatx4*)(g.resid + (size_t)smp * g.resid_bs + (size_t)i * g.ldy + n);
    floatx4 gt = {1.f, 1.f, 1.f, 1.f};
    if (g.gate) gt = *(const floatx4*)(g.gate + (size_t)smp * g.gate_bs + n);
    floatx4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = __fadd_rn(r[e], __fmul_rn(gt[e], v[e]));
    *(floatx4*)(g.y + (size_t)smp * g.y_bs + (size_t)i * g.ldy + n) = o;
}

// one or two layers; those with a cut sum go through their parts
hipError_t dispatch(const GemmPlan& plan, const GemmArgs& g, const GemmArgs* second, hipStream_t s) {
    // the erf form of the activation is some seventeen VALU operations per element against the tanh form's four: it gets kernels
    // of its own rather than a run-time choice inside the tanh one
    if (g.epi != EPI_GATE_RESID && g.heads.on) return g.act_erf ? gemm_launch_heads_erf(plan.tile, g, second, s) : gemm_launch_heads(plan.tile, g, second, s);
    if (g.epi != EPI_GATE_RESID) return g.act_erf ? gemm_launch_split_gelu_erf(plan.tile, g, second, s) : gemm_launch_split_gelu(plan.tile, g, second, s);
    if (g.ksplits <= 1) return gemm_launch_gate_resid(plan.tile, g, second, s);
    if (plan.meet) {
        if (!second) return gemm_launch_meet(plan.tile, g, nullptr, s);
        GemmArgs g2 = *second;                 // its words and sums follow the first's
        const TileCost& t = kTileCost[plan.tile];
        const uint32_t tiles = tile_count(g, t.bm, t.bn, false);
        g2.words = g.words + 4 * tiles;
        g2.part = g.part + (size_t)tiles * g.ksplits * t.bm * t.bn;
        return gemm_launch_meet(plan.tile, g, &g2, s);
    }
    GemmArgs parts[2] = {g, second ? *second : g};
    if (plan.last >= 0)
        for (GemmArgs& p : parts) --p.ksplits;
    const hipError_t e = gemm_launch_partial(plan.tile, parts[0], second ? &parts[1] : nullptr, s);
    if (e != hipSuccess) return e;
    if (plan.last >= 0) return gemm_launch_last_part(plan.last, g, second, s);
    auto blocks = [](const GemmArgs& p) { return (uint32_t)(((long)p.M * ((p.n1 - p.n0) / 4) + 255) / 256); };
    ReduceArgs a{};
    a.g[0] = g;
    a.blocks0 = blocks(g);
    if (second) a.g[1] = *second;
    hipLaunchKernelGGL(gemm_reduce_kernel, dim3(a.blocks0 + (second ? blocks(*second) : 0)), dim3(256), 0, s, a);
    return hipGetLastError();
}
}  // namespace

hipError_t gemm_launch_as(const GemmPlan& plan, const GemmArgs& g, hipStream_t s) { return dispatch(plan, g, nullptr, s); }
hipError_t gemm_launch(const GemmArgs& g, hipStream_t s) { return gemm_launch_as(gemm_plan(g, nullptr), g, s); }

// Whether a launch had better place its heads itself (`second`: two layers at once) than leave them to a pass that takes separate_us.
// What it costs there: the tile may have to be another (heads_fit), and a quadrant's slices of 32 tokens take 1.2 us each longer than
// plain rows, 2 where they are normed and 3 where they are rotated, in every round, or in as many as there are tiles of heads if there are
// several (even_step).  1320 x 9216 x 3072, normed, one round of 192x256 tiles: 67.6 us and 9.1 of the pass, or 73; 2304 x 21504 x 3072,
// three rounds: 265.4 and 17, or 266.  Rotated, 512 + 64 rows: 51 and 6, or 58.
// On tiles of up to 128 features (one slice a wave, nothing to hide the first loads of tables and weights behind) that is 1.5 us and more, a
// 128x128 tile a whole slice: 32 + 604 x 3072 x 1024, rotated, 15.0 us and 9.9 of the pass that moves the peers' rows besides, or 20.1 and 8.4;
// 180 x 3968 x 512 6.7 and 6.3, or 8.6 and 6.2.  Beside 128-feature tiles that apply the activation half a slice's time is left of it (blocks of 128 to
// 1600 rows and 512 to 3072 features -0.8 to +2.6 us of 50 to 160).
bool gemm_heads_pay(const GemmArgs& g, const GemmArgs* second, double separate_us) {
    const GemmArgs* const with[2] = {&g, second};
    GemmArgs plain[2] = {g, second ? *second : g};
    for (GemmArgs& p : plain) p.heads.on = 0;
    double placed, apart;
    best_tile({&plain[0], second ? &plain[1] : nullptr}, ALL_OF_IT, &apart);
    const TileCost& t = kTileCost[best_tile(with, ALL_OF_IT, &placed)];
    long tiles = 0;
    for (const GemmArgs* p : with)
        if (p) tiles += (long)((p->M + t.bm - 1) / t.bm) * ((p->N + t.bn - 1) / t.bn);
    const double slice_us = g.heads.r.rope_cos ? 3.0 : g.heads.r.has_norm ? 2.0 : 1.2;
    const double rounds = std::ceil((double)tiles / (256 * t.per_cu));
    double extra = (t.bn < 256 ? 0.5 : t.bm / 64) * slice_us * std::max(1.0, rounds * std::min(g.n_split, g.N) / g.N);
    if (t.bn < 128 || (t.bn < 256 && g.n_split >= g.N)) extra = 1.5 + t.bm * t.bn / 16384.0 * (0.5 + slice_us);
    return placed + extra <= apart + separate_us;
}

// two layers share a launch if they have one epilogue, both or neither have their sum in parts and both or neither place heads
bool gemm_can_pair(const GemmArgs& g0, const GemmArgs& g1) {
    return g0.epi == g1.epi && g0.act_erf == g1.act_erf && g0.heads.on == g1.heads.on && (g0.ksplits > 1) == (g1.ksplits > 1);
}

hipError_t gemm_launch_pair(const GemmPlan& plan, const GemmArgs& g0, const GemmArgs& g1, hipStream_t s) {
    return gemm_can_pair(g0, g1) ? dispatch(plan, g0, &g1, s) : hipErrorInvalidValue;
}
