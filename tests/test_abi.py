"""CPU-side checks of the C ABI: the library loads, exports what the header declares, and the
planning calls (which touch no GPU) behave: layout, chunking, argument errors."""
import ctypes as C
import os
import re

import numpy as np

import itertools

import pytest

import workload as wl
from oracle import chunks as och
from oracle import overlap_model as om
from paper_2605_11335_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions(name=None):
    """Functions declared by include/<name> (every header of include/ when no name is given)."""
    inc = os.path.join(ROOT, "include")
    names = []
    for h in sorted(os.listdir(inc)) if name is None else [name]:
        text = open(os.path.join(inc, h)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names += re.findall(r"^\s*(?:int|const char\*)\s+(\w+)\s*\(", text, flags=re.M)
    return names


def test_library_exports_every_declared_symbol():
    names = header_functions()
    assert len(names) >= 25 and "dit_block_fwd" in names and "set_resident_fraction" in names
    lib = B.lib()
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(names) == sorted(B.EXPORTS)
    # the block path's contract and the diagnostics are separate headers
    core, diag = header_functions("chunkflow.h"), header_functions("chunkflow_diag.h")
    assert sorted(core) == sorted(B.CORE_EXPORTS) and sorted(diag) == sorted(B.DIAG_EXPORTS)
    assert not any(n.startswith("cf_op_") or n in ("cf_plan_attention", "cf_plan_linear") for n in core
                   if not n.startswith("cf_op_checksum"))


def ctx_for(cfg, chunk):
    return B.Context(B.desc_from_config(cfg, chunk))


def test_blob_bytes_follow_app_b_formulas():
    flux = wl.CONFIGS["flux"]
    c = ctx_for(flux, 16 << 20)
    extra = c.cf_blob_bytes() - om.bytes_single(flux.d, flux.f)       # biases + norm weights + padding
    assert 0 < extra < 100_000
    hy = wl.CONFIGS["hunyuan"]
    c2 = ctx_for(hy, 16 << 20)
    extra = c2.cf_blob_bytes() - om.bytes_double(hy.d, hy.f)
    assert 0 < extra < 300_000
    wan = wl.CONFIGS["wan"]
    c3 = ctx_for(wan, 16 << 20)
    d, f = wan.d, wan.f
    assert 0 < c3.cf_blob_bytes() - 2 * (6 * d * d + 4 * d * d + 4 * d * d + 2 * d * f) < 300_000


@pytest.mark.parametrize("name", ["toy", "flux", "wan", "hunyuan"])
def test_layout_is_aligned_ordered_and_complete(name):
    cfg = wl.CONFIGS[name]
    c = ctx_for(cfg, 1 << 20)
    lay = c.cf_blob_layout()
    specs = {n: shape for n, shape, _, _ in wl.param_specs(cfg)}
    assert {t["name"] for t in lay} == set(specs)
    end = 0
    for t in lay:
        assert t["offset"] % 256 == 0 and t["offset"] >= end
        shape = specs[t["name"]]
        assert t["rows"] * t["cols"] == int(__import__("numpy").prod(shape))
        if len(shape) == 2:
            assert (t["rows"], t["cols"]) == shape
        end = t["offset"] + 2 * t["rows"] * t["cols"]
    assert end <= c.cf_blob_bytes() < end + 256
    assert c.cf_workspace_bytes() > 0


def test_chunk_count_matches_oracle_arithmetic():
    cfg = wl.CONFIGS["flux"]
    for chunk in (16 << 20, 64 << 20, 256 << 20, 1 << 20):
        c = ctx_for(cfg, chunk)
        assert c.cf_n_chunks() == len(och.chunk_bounds(c.cf_blob_bytes(), chunk))


def test_toy_config_is_four_chunks():
    from paper_2605_11335_amd.runner import chunk_bytes_for
    cfg = wl.CONFIGS["toy"]
    cb = chunk_bytes_for(cfg)
    assert cb % 256 == 0
    assert ctx_for(cfg, cb).cf_n_chunks() == 4
    assert ctx_for(wl.CONFIGS["flux"], chunk_bytes_for(wl.CONFIGS["flux"])).cf_n_chunks() == 8


@pytest.mark.parametrize("field,value", [("chunk_bytes", 0), ("chunk_bytes", 1000), ("head_dim", 96), ("sp_degree", 5),
                                         ("n_total", 4607), ("d", 3000), ("kind", 7), ("n_blocks", 0), ("f", 100),
                                         ("sp_rank", 2)])
def test_create_rejects_bad_descriptions(field, value):
    d = B.desc_from_config(wl.CONFIGS["flux"], 16 << 20)
    setattr(d, field, value)
    with pytest.raises(B.ChunkflowError) as e:
        B.Context(d)
    assert e.value.code == B.CF_ERR_ARG and str(e.value)


def test_block_range_is_checked_without_a_gpu():
    c = ctx_for(wl.CONFIGS["toy"], 1 << 20)
    with pytest.raises(B.ChunkflowError) as e:
        c.chunked_prefetch_begin(5, None)
    assert e.value.code == B.CF_ERR_ARG


@pytest.mark.parametrize("name,chunk_mib", [("flux", 16), ("flux", 35.4), ("wan", 64), ("toy", 0.5), ("hunyuan", 256)])
def test_panel_plans_cover_every_row_once_behind_the_right_chunk(name, chunk_mib):
    """Host logic of the per-chunk consumer waits: for every weight matrix and every resident
    prefix, panels tile the rows exactly, are tile-aligned, and every byte of a panel lies in a
    chunk that is resident or not later than the chunk the panel waits for; for several token
    counts of the layer, since the panel ends depend on how the launch fills the chip."""
    cfg = wl.CONFIGS[name]
    cb = int(chunk_mib * (1 << 20)) // 256 * 256
    c = ctx_for(cfg, cb)
    n_chunks = c.cf_n_chunks()
    bounds = och.chunk_bounds(c.cf_blob_bytes(), cb)
    for t in c.cf_blob_layout():
        if t["rows"] == 1:
            continue
        row_bytes = 2 * t["cols"]
        for n_res, m_rows in itertools.product(sorted({0, 1, n_chunks // 3, n_chunks // 2, n_chunks - 1, n_chunks}),
                                               (0, 1, cfg.n_local, 5 * cfg.n_local)):
            plan = c.cf_plan_panels(t["name"], m_rows, n_res)
            assert plan[0][0] == 0 and plan[-1][1] == t["rows"]
            for (a0, a1, w), nxt in zip(plan, plan[1:] + [None]):
                assert a0 < a1
                if nxt is not None:
                    assert a1 == nxt[0] and a1 % (256 if m_rows else 8) == 0 and w < nxt[2]
                last_byte = t["offset"] + a1 * row_bytes - 1
                need = next(k for k, (s, e) in enumerate(bounds) if s <= last_byte < e)
                assert need < n_res or need <= w, (t["name"], n_res, a0, a1, w, need)
                if w >= 0:
                    assert w >= n_res        # never waits for a resident chunk
            if n_res == n_chunks:
                assert plan == [(0, t["rows"], -1)]     # fully resident: one launch, no wait


def test_panels_fill_their_rounds_of_workgroups():
    """Every launch ends with a partly filled round of workgroups, so a layer is not cut wherever a
    chunk ends.  Flux-like lin1 (84 feature tiles of 256) on 2304 tokens (9 token tiles): 28
    feature tiles make 252 of the 256 workgroups of one round; although a 16 MiB chunk ends every
    10.7 tiles, the first panel leaves at most 7 % of its rounds empty and no panel but the last
    more than a quarter (such a remainder would have stayed with the next panel)."""
    cfg = wl.CONFIGS["flux"]
    c = ctx_for(cfg, 16 << 20)
    plan = c.cf_plan_panels("w1", cfg.n_local, 0)
    assert len(plan) >= 3
    for i, (a0, a1, w) in enumerate(plan[:-1]):
        tiles = (a1 - a0) // 256 * 9
        launched = -(-tiles // 256) * 256
        assert (a1 - a0) % 256 == 0 and launched - tiles <= (0.07 if i == 0 else 0.25) * launched, plan
    # lin2 (12 feature tiles x 9 token tiles): no cut fills a round; one launch behind its last chunk
    plan2 = c.cf_plan_panels("w2", cfg.n_local, 0)
    assert len(plan2) == 1 and plan2[0][:2] == (0, cfg.d)
    # the modulation product is cut at every chunk end
    assert len(c.cf_plan_panels("w_mod", 0, 0)) >= 2 or c.cf_n_chunks() == 1


def test_mixed_block_kinds_are_planned_per_block():
    """App. B composition: double-stream blocks then single-stream ones; each kind has its own
    layout and chunk count, the workspace covers both."""
    cfg = wl.CONFIGS["toy_mm"]
    chunk = 1 << 20
    ctx = B.Context(B.desc_from_config(cfg, chunk))
    try:
        single_bytes, single_ws = ctx.cf_blob_bytes(), ctx.cf_workspace_bytes()
        ctx.cf_set_block_kinds(cfg.kinds)
        assert [ctx.cf_block_kind_of(b) for b in range(cfg.n_blocks)] == [wl.KIND_DOUBLE, wl.KIND_SINGLE, wl.KIND_SINGLE]
        assert ctx.cf_blob_bytes(1) == ctx.cf_blob_bytes(2) == single_bytes
        assert ctx.cf_workspace_bytes() >= single_ws
        for b in range(cfg.n_blocks):
            specs = wl.param_specs(cfg.block_cfg(b))
            lay = ctx.cf_blob_layout(b)
            assert sorted(t["name"] for t in lay) == sorted(s[0] for s in specs)
            want = sum(-(-2 * int(np.prod(s[1])) // 256) * 256 for s in specs)
            assert ctx.cf_blob_bytes(b) == want
            assert ctx.cf_n_chunks(b) == -(-want // chunk)
        with pytest.raises(B.ChunkflowError):
            ctx.cf_set_block_kinds([0, 0])                      # one kind per block
        with pytest.raises(B.ChunkflowError):
            ctx.cf_set_block_kinds([wl.KIND_DIT, 0, 0])         # no cross-attention context in this model
    finally:
        ctx.close()
    no_txt = B.Context(B.desc_from_config(wl.CONFIGS["toy"], chunk))
    try:
        with pytest.raises(B.ChunkflowError):
            no_txt.cf_set_block_kinds([wl.KIND_DOUBLE, 0])      # double-stream needs text rows
    finally:
        no_txt.close()


def test_attention_launch_shapes():
    """The launch planner's choices by the grid for the shapes they were measured on (one MI355X; a block may deal
    the sweeps out otherwise, test_block_attention_plans): 8 waves per
    workgroup for the Flux-like and the Hunyuan-like self-attention, 7 for the Wan-like one (7- and 8-wave
    grids take six generations either way, and a 7-wave generation of such a long sweep is shorter), 4 for
    the cross-attention to 512 context tokens (short sweeps: one workgroup's fixed part hides behind the
    other's tiles) and for grids that end on a half-empty generation; tiny grids are spread over 4-wave
    workgroups.  Growing the key count alone never moves a choice from 8 towards 4."""
    assert B.cf_plan_attention(12, 4608, 4608, 128) == 8
    assert B.cf_plan_attention(12, 119056, 119056, 128) == 8
    assert B.cf_plan_attention(12, 59528, 59528, 128) == 8
    assert B.cf_plan_attention(12, 27280, 27280, 128) == 7
    assert B.cf_plan_attention(24, 13640, 512, 128) == 4
    assert B.cf_plan_attention(12, 8192, 8192, 128) == 4
    assert B.cf_plan_attention(24, 4096, 4096, 128) == 4
    assert B.cf_plan_attention(8, 512, 512, 64) == 4
    for nq, H in ((4608, 12), (13640, 24), (5120, 8)):
        picks = [B.cf_plan_attention(H, nq, nk, 128) for nk in (128, 512, 2048, 8192, 32768)]
        assert all(p in (4, 7, 8) for p in picks)
        first_tall = next((i for i, p in enumerate(picks) if p != 4), len(picks))
        assert all(p != 4 for p in picks[first_tall:]), picks
    for bad in ((0, 10, 10, 128), (1, 0, 10, 128), (1, 10, 0, 128), (1, 10, 10, 96)):
        with pytest.raises(B.ChunkflowError):
            B.cf_plan_attention(*bad)


def test_linear_tile_shapes():
    """The tile choice for layer shapes on which both tiles were timed (one MI355X, operands read cold): the
    listed choice was the faster one by 5-45 % (the Flux-like and Wan-like shares' layers, the context
    projection of the Wan-like cross-attention, the image stream of the mixed stack's double-stream blocks)."""
    for m, n, want in ((2304, 21504, 256), (2304, 3072, 128), (13640, 3072, 256), (13640, 9216, 256), (2048, 3072, 128),
                       (512, 6144, 128), (4608, 3072, 256), (4608, 9216, 256), (1024, 21504, 256)):
        assert B.cf_plan_linear(m, n) == want, (m, n)
    assert B.cf_plan_linear(64, 64) == 128                       # one tile either way: the small one
    with pytest.raises(B.ChunkflowError):
        B.cf_plan_linear(0, 64)


def test_no_alloc_checksum_rejects_oversize_and_misaligned_requests_before_touching_a_gpu():
    """The argument checks of cf_op_checksum_noalloc come before any HIP call: a request beyond what
    its fixed partial-sum array covers (1 GiB) is an argument error with a message that says so."""
    lib = B.lib()
    fake = C.c_void_p(4096)             # never dereferenced: the call must fail on its arguments
    assert lib.cf_op_checksum_noalloc(fake, (1 << 30) + 8, 0, fake, None) == B.CF_ERR_ARG
    assert b"exceed" in lib.cf_last_error(None)
    assert lib.cf_op_checksum_noalloc(fake, 12, 0, fake, None) == B.CF_ERR_ARG
    assert lib.cf_op_checksum_noalloc(fake, 8, 0, None, None) == B.CF_ERR_ARG
    assert lib.cf_op_checksum_noalloc(C.c_void_p(4097), 8, 0, fake, None) == B.CF_ERR_ARG


def test_block_attention_plans():
    """How a block launches attention: the Flux-like share whole, by the grid; its share on eight GPUs with its keys in parts,
    at any batch; the video shares dealt out by the kernel, evenly or drawn from a counter.  Bad requests for a form fail on
    their arguments."""
    def plan(*shape):
        p = B.cf_plan_block_attention(*shape)
        return p.waves, p.parts, p.deal
    assert plan(12, 1, 4608, 4608, 128) == (8, 1, 0)
    assert plan(12, 1, 27280, 27280, 128) == (8, 1, 1)
    assert plan(12, 1, 119056, 119056, 128) == (8, 1, 2)
    # merged by a kernel (0) or a wave to each part (2) where one sample runs; a batch that fills the chip has as many parts (the bits
    # depend on them), but pays for neither: its workgroups have all parts, one after the other (1)
    for shape, form in (((3, 4608, 128), 0), ((3, 2640, 128), 2), ((1, 4696, 128), 0), ((2, 4696, 64), 0), ((1, 2264, 64), 2), ((8, 512, 64), 2)):
        one = B.cf_plan_block_attention(shape[0], 1, shape[1], shape[1], shape[2])
        many = B.cf_plan_block_attention(shape[0], 64, shape[1], shape[1], shape[2])
        assert many.parts == one.parts > 1 and (one.all_parts, many.all_parts) == (form, 1), shape
        assert form != 2 or one.waves == one.parts, shape
    # One sample's keys are cut where that gives it workgroups or waves, not where its workgroups would have all parts in turn; and for waves
    # in few parts only, which a batch joins at little cost: no more than one to five tiles of a sweep.
    for hd in (64, 128):
        for heads in (1, 2, 3, 4, 6, 8, 12, 14, 16, 24, 25, 33, 64):
            for n in (64, 200, 320, 512, 640, 800, 1000, 1280, 1536, 1955, 2048, 2565, 2640, 3584, 4639, 9000):
                p = B.cf_plan_block_attention(heads, 1, n, n, hd)
                assert p.all_parts != 1, (heads, n, hd)
                assert p.all_parts != 2 or -(-n // 64) >= 5 * (p.parts - 1), (heads, n, hd, p.parts)
    for bad in ((0, 1, 10, 10, 128), (1, 0, 10, 10, 128), (1, 1, 0, 10, 128), (1, 1, 10, 0, 128), (1, 1, 10, 10, 96), (1 << 20, 1 << 20, 10, 10, 64)):
        with pytest.raises(B.ChunkflowError):
            B.cf_plan_block_attention(*bad)
    lib, p = B.lib(), C.c_void_p(4096)             # never dereferenced
    for H, nq, nk, hd, parts, deal, nbytes in ((1, 64, 512, 128, 0, 0, 1 << 30), (1, 64, 512, 128, 65, 0, 1 << 30), (1, 64, 512, 128, 9, 0, 1 << 30),
                                               (1, 64, 512, 128, 2, 1, 1 << 30), (1, 64, 512, 128, 1, 3, 1 << 30), (1, 64, 512, 128, 2, 0, 1000),
                                               (12, 64, 512, 128, 1, 1, 1 << 30), (12, 4800, 512, 64, 1, 1, 1 << 30), (12, 4800, 512, 128, 1, 1, 4096), (12, 4800, 192, 128, 1, 2, 1 << 30)):
        assert lib.cf_op_attention_form(p, p, p, p, H, nq, nk, nk, hd, parts, 0, deal, 0, p, nbytes, None) == B.CF_ERR_ARG
    # a drawn sweep is cut in four pieces of at least a tile, however many there are
    assert all(plan(48, b, nq, nk, 128)[2] != 2 for b in (1, 16, 256) for nq in (4608, 119056) for nk in (1, 64, 128, 192))


def test_block_linear_plans():
    """How a block launches its linear layers: the number of parts of a sum follows from one sample, is at most three (a batch that
    fills the chip pays for each), and where such a batch puts it together the last part does."""
    def plan(*shape, **kw):
        p = B.cf_plan_block_linear(*shape, **kw)
        return (p.tile_tokens, p.tile_features), p.parts, (p.last_tile_tokens, p.last_tile_features)
    assert plan(2304, 21504, 3072, False) == ((256, 256), 1, (0, 0))
    for shape in ((576, 3072, 15360), (1320, 3072, 14336), (2304, 3072, 15360)):
        alone = plan(*shape, True)
        assert 1 < alone[1] <= 3 and alone[2] == (0, 0)
        assert all(plan(*shape, True, batch=b)[1] == alone[1] for b in (2, 4, 8, 64))
    assert plan(576, 3072, 15360, True, batch=8)[2] == (256, 256) and plan(1320, 3072, 14336, True, batch=4)[2] == (256, 256)
    for bad in ((0, 64, 64), (64, 0, 64), (64, 64, 0)):
        with pytest.raises(B.ChunkflowError):
            B.cf_plan_block_linear(*bad, True)
    lib, p = B.lib(), C.c_void_p(4096)             # never dereferenced
    for tile, parts, nbytes in (((256, 64), 1, 0), ((128, 64), 0, 0), ((128, 64), 9, 1 << 30), ((128, 64), 2, 4096)):
        assert lib.cf_op_linear_residual_form(p, 512, p, 0, -1, 64, 64, 512, p, None, p, tile[0], tile[1], parts, 0, p, nbytes, None) == B.CF_ERR_ARG


def test_sums_that_a_batch_would_pay_for_stay_whole():
    """A layer whose sum only one sample gains from cutting, because its parts meet within a launch that holds no more of them, is not cut:
    the parts are those of every batch, which would put them together through memory."""
    for rows, rows2, n, k in ((2760, 0, 1536, 7232), (2444, 400, 1536, 5952), (5485, 0, 1024, 4608), (1865, 0, 2048, 9408), (1591, 80, 2048, 10176), (2783, 64, 2048, 6336),
                              (1131, 26, 3072, 11264), (2472, 0, 3072, 10560), (2000, 0, 3072, 9216), (4000, 0, 1536, 4608), (996, 0, 4096, 18176)):
        assert B.cf_plan_block_linear(rows, n, k, True, rows2=rows2).parts == 1, (rows, rows2, n, k)
    assert [B.cf_plan_block_linear(*shape, True).parts for shape in ((2304, 3072, 15360), (1320, 3072, 14336), (576, 3072, 15360))] == [2, 3, 2]


def test_parts_meet_where_all_their_workgroups_have_a_cu():
    """Of two layers in one launch with the padding to eight workgroups between them: 18 + 6 + 234 do not."""
    assert B.cf_plan_block_meet(2304, 3072, 15360) and B.cf_plan_block_meet(1320, 3072, 14336) and B.cf_plan_block_meet(512, 3072, 12288, rows2=64)
    for rows, rows2 in ((1653, 16), (1659, 32)):
        p = B.cf_plan_block_linear(rows, 1536, 7232, True, rows2=rows2)
        assert (p.parts, p.tile_tokens, p.tile_features) == (3, 128, 256) and not B.cf_plan_block_meet(rows, 1536, 7232, rows2=rows2)
    assert B.cf_plan_block_meet(1653 - 128, 1536, 7232, rows2=128)                        # 18 + 6 + 216
    assert not B.cf_plan_block_meet(2304, 3072, 15360, batch=4) and not B.cf_plan_block_meet(40000, 512, 512)
    for bad in ((0, 64, 64), (64, 0, 64), (64, 64, 0)):
        with pytest.raises(B.ChunkflowError):
            B.cf_plan_block_meet(*bad)


def _tiles_of_the_last_round(problems, tile, parts):
    """(XCD, problem, first token, first feature, part) of the tiles past whole rounds of 256 workgroups, in the order in which the kernel
    walks them: an XCD's ids together, groups of row-tiles of one size, feature-tile-major."""
    bm, bn = tile
    first, out = 0, []
    counts = [-(-m // bm) * -(-n // bn) * parts for m, n in problems]
    begins = [0, -(-counts[0] // 8) * 8]
    tiles = begins[len(problems) - 1] + counts[-1]
    for i, (m, n) in enumerate(problems):
        tm, tn = -(-m // bm), -(-n // bn)
        gm = -(-tm // max(1, (tm + 4) // 8))
        order = [(r, c) for g0 in range(0, tm, gm) for c in range(tn) for r in range(g0, min(tm, g0 + gm))] * parts
        for b in range(max(0, tiles // 256 * 256 - begins[i]), counts[i]):
            q, r = divmod(counts[i], 8)
            lid = b % 8 * q + min(b % 8, r) + b // 8
            out.append((b % 8, i, order[lid][0] * bm, order[lid][1] * bn, lid // (tm * tn)))
    return tiles, out


def test_idle_fetch_plans():
    """Which launches let idle CUs fetch, for how long, and what: up to two rounds of workgroups, no longer than a round takes at their
    pace, and on every XCD the weights (and activations) of its own tiles, whole, once, and nothing past the operands' ends."""
    seen = set()
    for rows, rows2, n, k, residual in ((2304, 0, 3072, 12288, True), (1531, 0, 12288, 3072, False), (1320, 0, 14336, 3072, False), (1320, 0, 3072, 14336, True),
                                        (512, 64, 9216, 3072, False), (1500, 70, 4104, 1088, False), (300, 0, 25000, 1024, False), (2304, 0, 3080, 15360, True),
                                        (4608, 0, 3072, 12288, True), (2304, 0, 3072, 15360, True), (1500, 0, 3072, 12288, True),
                                        (900, 512, 2048, 10240, True), (1320, 70, 1536, 6144, True), (6000, 256, 1024, 4096, True), (6000, 256, 1536, 6144, True),
                                        (2640, 256, 3072, 1024, False), (4608, 0, 9216, 3072, False), (13640, 0, 9216, 3072, False), (5, 0, 8, 4096, False)):
        p = B.cf_plan_block_linear(rows, n, k, residual, rows2=rows2)
        f = B.cf_plan_block_fetch(rows, n, k, residual, rows2=rows2)
        tile, slabs = (p.tile_tokens, p.tile_features), -(-(k // 64) // p.parts)
        problems = [(m, n) for m in (rows, rows2) if m]
        tiles, last = _tiles_of_the_last_round(problems, tile, p.parts)
        assert f.tiles == tiles
        if not f.fetching:
            assert f.panels == 0
            continue
        seen.add((tile, p.parts > 1, rows2 > 0))
        assert tile in ((256, 256), (192, 256), (128, 256)) and tiles <= 512 and f.fetching == 256 - tiles % 256
        assert f.stride >= 1 and f.deadline_ns <= slabs * f.pace_ns
        for x in range(8):
            mine = [q for q in f.panel[:f.panels] if q[0] == x]
            assert len(mine) <= 64
            for i, (m, _) in enumerate(problems):
                at = [t for t in last if t[0] == x and t[1] == i]
                got = [(q[3], q[3] + q[4]) for q in mine if q[1] == i and not q[2]]
                want = [(2 * (n0 * k + part * slabs * 64), 2 * min(n, n0 + tile[1]) * k) for _, _, _, n0, part in at]
                assert set(got) == set(want) and len(set(got)) == len(got) and all(0 <= a < b <= 2 * n * k for a, b in got)
                got = [(q[3], q[3] + q[4]) for q in mine if q[1] == i and q[2]]
                want = {(2 * (m0 * k + part * slabs * 64), 2 * min(m, m0 + tile[0]) * k) for _, _, m0, _, part in at}
                # of a second part of the sum on the same XCD the activations are left out
                assert not f.with_activations or (set(got) <= want and len(set(got)) == len(got) and (p.parts > 1 or set(got) == want))
                assert f.with_activations or not got
                assert all(0 <= a < b <= 2 * m * k for a, b in got)
    assert {t for t, _, _ in seen} == {(256, 256), (192, 256), (128, 256)} and {c for _, c, _ in seen} == {True, False} == {t for _, _, t in seen}, seen
    for bad in ((0, 64, 64), (64, 0, 64), (64, 64, 32)):
        with pytest.raises(B.ChunkflowError):
            B.cf_plan_block_fetch(*bad, False)


def test_the_tile_tests_take_every_tile():
    """The sizes of tests/test_gpu_gemm_tiles.py still reach all tiles: on the longest sum, with few slabs all but 128 x 256, and with
    two layers in one launch."""
    from tests import test_gpu_gemm_tiles as t

    def tile(m, k, n=t.N, m2=0):
        p = B.cf_plan_block_linear(m, n, k, False, rows2=m2)
        return p.tile_tokens, p.tile_features
    assert {tile(m, t.KS[-1]) for m in t.FEWER + (t.M,)} == t.TILES
    assert all({tile(m, k) for m in t.FEWER + (t.M,)} >= t.TILES - {(128, 256)} for k in t.KS)
    assert {tile(m, 512, 2048, t.TXT) for m in t.IMAGES} == t.TILES
