"""The persistent kernel that spreads the heads of a tile over compute units (circuits with few gates per level):
every hidden size and type, rows of every width class, every tile size, against the oracle and, bit for bit,
against itself under other schedules and cuts. The level-by-level path (other kernels) is the second opinion."""
import numpy as np
import pytest
import torch

import dg4_synth as synth
import oracle
import paper_2502_01681_amd as dg4
from gpu_utils import TOL, cfg_of, device_weights, row_rel_err, tdtype, to_dev, to_np

pytestmark = pytest.mark.gpu


def make(n_and, window, hidden, dtype, hops, layers, n_pi=40):
    return synth.make(synth.Config("heads", 77, n_pi, n_and, window, 1.0, 0, hidden, hidden // 32, hops, layers, dtype))


def run(w, cfg, g, ffn=None, level_begin=0, level_end=None, H0=None):
    X, W = to_dev(w.x, cfg.dtype), device_weights(w, cfg.dtype)
    if ffn is not None:
        W = [lw + (to_dev(ffn[0][l], cfg.dtype), to_dev(ffn[1][l], cfg.dtype)) for l, lw in enumerate(W)]
    H = torch.full((w.cfg.n_nodes, cfg.hidden), float("nan"), dtype=tdtype(cfg.dtype), device="cuda") if H0 is None else H0
    ws = torch.empty(dg4.dg4_layer_workspace_bytes(cfg, g), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)                          # NaN patterns: nothing may be read before it is written
    dg4.dg4_layer_fwd(cfg, g, X, W, H, level_begin, level_end, workspace=ws)
    torch.cuda.synchronize()
    dg4.dg4_layer_status(cfg, g, ws)
    return H


@pytest.mark.parametrize("hidden,dtype", [(128, "f32"), (128, "bf16"), (256, "f32"), (256, "bf16")])
@pytest.mark.parametrize("n_and,window,hops,layers,ffn", [
    (3, 2, 1, 2, False),                    # fewer gates than a tile, fewer tiles than groups
    (700, 60, 2, 2, False), (700, 60, 3, 1, False),
    (2_500, 2_400, 2, 2, False),            # a hundred gates per level: tiles of two (hidden 128) and four
    (600, 60, 2, 2, True), (700, 60, 2, 1, True), (700, 60, 3, 1, True),
    (500, 20, 5, 2, False),                 # wide rows, tiles of two gates (16 lane groups and more per gate)
    (1_500, 900, 5, 1, False),              # ... of two
    (4_000, 3_900, 4, 2, False),            # ... of four (hidden 128) and eight
    (900, 300, 6, 2, True), (900, 300, 6, 1, True),
])
def test_heads_kernel_against_oracle(hidden, dtype, n_and, window, hops, layers, ffn):
    print(f"heads kernel {dtype} {hidden} n_and={n_and} window={window} hops={hops} layers={layers} ffn={ffn}", flush=True)
    w = make(n_and, window, hidden, dtype, hops, layers)
    c = w.cfg
    fw = synth.ffn_weights(c) if ffn else None
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    cfg = cfg_of(c, ffn=ffn)
    H = run(w, cfg, g, fw)
    assert not torch.isnan(H.float()).any()
    og = oracle.build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    kw = dict(w1=fw[0], w2=fw[1]) if ffn else {}
    ref = oracle.layer_fwd(og, w.x, w.wqkv, w.wo, w.rel_bias, c.heads, store=dtype, **kw)
    err = row_rel_err(to_np(H), ref).max()
    print(f"  {g.n_levels} levels, max rel err {err:.3e}", flush=True)
    assert err <= TOL[dtype]
    # other kernels, another summation order: each within TOL of the oracle
    assert row_rel_err(to_np(H), to_np(run(w, cfg_of(c, ffn=ffn, per_level=True), g, fw)).astype(np.float64)).max() <= 2 * TOL[dtype]
    assert torch.equal(H, run(w, cfg_of(c, ffn=ffn, level_order=True), g, fw))
    mid = g.n_levels // 2
    assert torch.equal(H, run(w, cfg, g, fw, mid, None, H0=run(w, cfg, g, fw, 0, mid)))


@pytest.mark.parametrize("hidden,dtype", [(128, "bf16"), (256, "f32")])
def test_heads_kernel_without_epilogue_and_with_masking_biases(hidden, dtype):
    # relation biases of -inf and of the type's lowest value take entries out of the softmax; the gate itself stays
    w = make(600, 50, hidden, dtype, 3, 1)
    c = w.cfg
    for code, value in ((3, -np.inf), (1, np.finfo(np.float32).min)):
        w.rel_bias[0][:, code] = value
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, 3)
    og = oracle.build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, 3)
    for epilogue in (True, False):
        H = run(w, cfg_of(c, epilogue=epilogue), g)
        ref = oracle.layer_fwd(og, w.x, w.wqkv, w.wo, w.rel_bias, c.heads, store=dtype, epilogue=epilogue)
        assert row_rel_err(to_np(H), ref).max() <= TOL[dtype], epilogue


def test_heads_kernel_bounded_wait_two_streams_and_packed_weights():
    # A spin limit of one may end the sweep early: it returns, says so, and the same workspace then serves a
    # normal sweep. Two sweeps at once on two streams (more workgroups than compute units): the same bits.
    w = make(2_000, 200, 128, "f32", 2, 3)
    c = w.cfg
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, 2)
    cfg = cfg_of(c)
    H = run(w, cfg, g)
    X, W = to_dev(w.x, c.dtype), device_weights(w, c.dtype)
    out = torch.full_like(H, float("nan"))
    ws = torch.empty(dg4.dg4_layer_workspace_bytes(cfg, g), dtype=torch.uint8, device="cuda")
    print("heads kernel: spin limit 1", flush=True)
    dg4.dg4_layer_fwd(cfg_of(c, spin_limit=1), g, X, W, out, workspace=ws)
    torch.cuda.synchronize()
    assert dg4.dg4_layer_status(cfg, g, ws, check=False) in (0, -10)
    for again in (cfg, cfg_of(c, weights_packed=True)):
        out.fill_(float("nan"))
        dg4.dg4_layer_fwd(again, g, X, W, out, workspace=ws)
        torch.cuda.synchronize()
        dg4.dg4_layer_status(cfg, g, ws)
        assert torch.equal(out, H)
    print("heads kernel: two streams", flush=True)
    streams = [torch.cuda.Stream() for _ in range(2)]
    both = [(torch.full_like(H, float("nan")), torch.empty_like(ws)) for _ in streams]
    torch.cuda.synchronize()
    for s, (o, k) in zip(streams, both):
        with torch.cuda.stream(s):
            dg4.dg4_layer_fwd(cfg, g, X, W, o, workspace=k)
    torch.cuda.synchronize()
    for o, k in both:
        dg4.dg4_layer_status(cfg, g, k)
        assert torch.equal(o, H)


@pytest.mark.parametrize("hidden,dtype,hops,ffn", [(128, "f32", 2, False), (256, "bf16", 3, False), (128, "bf16", 5, True)])
def test_heads_kernel_under_graph_capture(hidden, dtype, hops, ffn):
    # captured right after dg4_graph_upload (no sweep before it: nothing may be allocated), replayed with eager work
    # and new inputs in between
    w = make(900, 90, hidden, dtype, hops, 2)
    c = w.cfg
    fw = synth.ffn_weights(c) if ffn else None
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    captured_sweeps(w, g, fw)


@pytest.mark.parametrize("hidden,dtype,hops,ffn", [(256, "f32", 2, False), (128, "bf16", 3, True)])
def test_heads_kernel_under_graph_capture_on_a_deeper_levelling(hidden, dtype, hops, ffn):
    # ... of a graph built on the GPU under a caller's levelling: nothing to allocate there either
    w = make(900, 90, hidden, dtype, hops, 2)
    c = w.cfg
    level = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops).array("level")
    hint = np.where(level > 0, 2 * level + np.arange(c.n_nodes) % 2, 0).astype(np.int32)
    edges = [torch.from_numpy(a).cuda() for a in (w.edge_src, w.edge_dst, w.edge_inv, hint)]
    captured_sweeps(w, dg4.dg4_build_levels_device(c.n_nodes, *edges[:3], hops, edges[3]), synth.ffn_weights(c) if ffn else None)


def captured_sweeps(w, g, fw):
    c = w.cfg
    hidden, dtype, hops, ffn = c.hidden, c.dtype, c.hops, fw is not None
    g.upload()
    cfg = cfg_of(c, ffn=ffn)
    X, W = to_dev(w.x, dtype), device_weights(w, dtype)
    if ffn:
        W = [lw + (to_dev(fw[0][l], dtype), to_dev(fw[1][l], dtype)) for l, lw in enumerate(W)]
    out = torch.full_like(X, float("nan"))
    ws = torch.empty(dg4.dg4_layer_workspace_bytes(cfg, g), dtype=torch.uint8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    print(f"heads kernel captured: {dtype} {hidden} hops={hops} ffn={ffn}", flush=True)
    with torch.cuda.graph(graph):
        dg4.dg4_layer_fwd(cfg, g, X, W, out, workspace=ws)
    for replay in range(3):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        dg4.dg4_layer_status(cfg, g, ws)
        eager = torch.full_like(X, float("nan"))
        dg4.dg4_layer_fwd(cfg, g, X, W, eager)
        torch.cuda.synchronize()
        assert torch.equal(out, eager), replay
        X.mul_(-1)


@pytest.mark.parametrize("hidden,dtype,n_and,window,hops,ffn", [
    (128, "f32", 900, 90, 2, False),        # a handful of gates per level: the list schedule's tiles one by one
    (256, "bf16", 4_000, 3_000, 3, True),   # a round of its tiles of 8
    (128, "bf16", 700, 60, 5, False),       # wide rows: tiles cut from the caller's levels
])
def test_heads_kernel_on_a_deeper_levelling(hidden, dtype, n_and, window, hops, ffn):
    # a caller's levelling deeper than Eq. 1 changes the schedule, not a bit of the result; host- and device-built
    w = make(n_and, window, hidden, dtype, hops, 2)
    c = w.cfg
    fw = synth.ffn_weights(c) if ffn else None
    cfg = cfg_of(c, ffn=ffn)
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    level = g.array("level")
    hint = np.where(level > 0, 2 * level + np.arange(c.n_nodes) % 2, 0).astype(np.int32)
    print(f"deeper levelling {dtype} {hidden} hops={hops}: {g.n_levels} levels of {c.n_nodes // g.n_levels}", flush=True)
    H = run(w, cfg, g, fw)
    deeper = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops, hint)
    assert torch.equal(H, run(w, cfg, deeper, fw))
    edges = [torch.from_numpy(a).cuda() for a in (w.edge_src, w.edge_dst, w.edge_inv)]
    on_gpu = dg4.dg4_build_levels_device(c.n_nodes, *edges, hops, torch.from_numpy(hint).cuda())
    assert torch.equal(H, run(w, cfg, on_gpu, fw))
    assert torch.equal(H, run(w, cfg_of(c, ffn=ffn, level_order=True), deeper, fw))
    mid = deeper.n_levels // 2
    assert torch.equal(H, run(w, cfg, deeper, fw, mid, None, H0=run(w, cfg, deeper, fw, 0, mid)))


def test_path_goes_by_the_circuits_own_depth():
    # Eq. 1 depth 4 under a levelling of hundreds of levels: the path (and so every bit) is that of the wide circuit,
    # whoever built the graph
    w = synth.make(synth.Config("flat", 78, 500, 9_000, 4_000, 0.5, 3, 128, 4, 2, 2, "f32"))
    c = w.cfg
    cfg = cfg_of(c)
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, 2)
    level = g.array("level")
    hint = np.where(level > 0, 200 * level + np.arange(c.n_nodes) % 150, 0).astype(np.int32)
    H = run(w, cfg, g)
    edges = [torch.from_numpy(a).cuda() for a in (w.edge_src, w.edge_dst, w.edge_inv)]
    assert torch.equal(H, run(w, cfg, dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, 2, hint)))
    assert torch.equal(H, run(w, cfg, dg4.dg4_build_levels_device(c.n_nodes, *edges, 2, torch.from_numpy(hint).cuda())))


def test_path_goes_by_the_circuits_own_depth_with_one_fanin_gates():
    # ... where some gates have one fanin, and where a device-built graph's levelling is the circuit's own one
    w = synth.make(synth.Config("flat", 78, 500, 9_000, 4_000, 0.5, 3, 128, 4, 2, 2, "f32"))
    c = w.cfg
    cfg = cfg_of(c)
    keep = np.ones(len(w.edge_src), dtype=bool)
    keep[1::6] = False                      # every third gate keeps one of its two fanins
    host = [np.ascontiguousarray(a[keep]) for a in (w.edge_src, w.edge_dst, w.edge_inv)]
    g = dg4.dg4_build_levels(c.n_nodes, *host, 2)
    level = g.array("level")
    H = run(w, cfg, g)
    edges = [torch.from_numpy(a).cuda() for a in host]
    for hint in (level, np.where(level > 0, 200 * level + np.arange(c.n_nodes) % 150, 0)):
        hint = np.ascontiguousarray(hint.astype(np.int32))
        on_gpu = dg4.dg4_build_levels_device(c.n_nodes, *edges, 2, torch.from_numpy(hint).cuda())
        assert np.array_equal(on_gpu.array("level"), hint)
        assert torch.equal(H, run(w, cfg, on_gpu))
        assert torch.equal(H, run(w, cfg, dg4.dg4_build_levels(c.n_nodes, *host, 2, hint)))


@pytest.mark.parametrize("hidden,dtype,hops,ffn", [(256, "bf16", 2, False), (128, "f32", 3, False), (256, "f32", 2, True), (128, "bf16", 5, False)])
def test_heads_kernel_in_groups_by_order_of_arrival(hidden, dtype, hops, ffn):
    # A spin limit below 4096 makes a workgroup close a group that is not complete the moment it sits down, so most
    # groups consist of whichever workgroups come next: the same bits, cut in two as well (the finished gates' rows then
    # come from workgroups of other slices).
    w = make(1_500, 200, hidden, dtype, hops, 2)
    c = w.cfg
    fw = synth.ffn_weights(c) if ffn else None
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    print(f"heads kernel, groups by arrival: {dtype} {hidden} hops={hops} ffn={ffn}", flush=True)
    H = run(w, cfg_of(c, ffn=ffn), g, fw)
    at_once = cfg_of(c, ffn=ffn, spin_limit=4095)
    assert torch.equal(H, run(w, at_once, g, fw))
    mid = g.n_levels // 2
    assert torch.equal(H, run(w, at_once, g, fw, mid, None, H0=run(w, at_once, g, fw, 0, mid)))


@pytest.mark.parametrize("hidden,dtype,n_streams", [(256, "bf16", 2), (256, "f32", 3)])
def test_heads_kernel_on_streams_that_share_the_compute_units(hidden, dtype, n_streams):
    # hidden 256: one workgroup fills a compute unit, and every sweep asks for all of them
    w = make(6_000, 600, hidden, dtype, 2, 3)
    c = w.cfg
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, 2)
    cfg = cfg_of(c)
    H = run(w, cfg, g)
    X, W = to_dev(w.x, c.dtype), device_weights(w, c.dtype)
    streams = [torch.cuda.Stream() for _ in range(n_streams)]
    outs = [(torch.full_like(H, float("nan")), torch.empty(dg4.dg4_layer_workspace_bytes(cfg, g), dtype=torch.uint8, device="cuda"))
            for _ in streams]
    torch.cuda.synchronize()
    print(f"heads kernel: {n_streams} streams, {dtype} {hidden}", flush=True)
    for _ in range(3):
        for s, (o, k) in zip(streams, outs):
            with torch.cuda.stream(s):
                dg4.dg4_layer_fwd(cfg, g, X, W, o, workspace=k)
    torch.cuda.synchronize()
    for o, k in outs:
        dg4.dg4_layer_status(cfg, g, k)
        assert torch.equal(o, H)


def shape_of(w, levels, ffn):
    """What the rules make of a circuit with this many (Eq. 1) levels: whether it takes the heads kernel, gates per tile."""
    c = w.cfg
    groups, width = 256 // c.heads, c.n_nodes // levels
    streamed = (c.dtype, c.hidden) in (("f32", 128), ("bf16", 256)) and (not ffn or c.hops <= 3)
    rows = 2
    while rows < 16 and 4 * width > 5 * groups * rows:
        rows *= 2
    return width <= groups * 16 * (4 if not streamed else 2 if c.hops >= 6 else 1), rows


def make_flat(n_pi, n_and, cap, hidden, dtype, hops, layers):
    return synth.make(synth.Config("heads", 79, n_pi, n_and, 2_000, 0.5, cap, hidden, hidden // 32, hops, layers, dtype))


@pytest.mark.parametrize("hidden,dtype,n_pi,n_and,cap,hops,layers,ffn,rows", [
    (256, "bf16", 400, 2_000, 14, 2, 2, False, 16), (128, "f32", 400, 6_000, 8, 3, 2, False, 16),
    (256, "bf16", 400, 2_000, 14, 4, 2, False, 16), (256, "f32", 400, 2_000, 14, 4, 1, False, 16),
    (128, "f32", 400, 6_000, 8, 4, 2, False, 16), (128, "bf16", 400, 6_000, 8, 5, 1, False, 16),
    (256, "bf16", 400, 2_000, 14, 5, 2, True, 16), (256, "f32", 400, 2_000, 14, 4, 2, True, 16),
    (128, "f32", 400, 6_000, 8, 4, 1, True, 16), (128, "bf16", 400, 6_000, 8, 4, 2, True, 16),
    (128, "f32", 400, 3_500, 8, 5, 2, False, 8), (256, "bf16", 150, 1_400, 9, 5, 2, False, 8), (256, "f32", 150, 1_400, 9, 6, 1, True, 8),
    (128, "bf16", 150, 1_400, 9, 4, 2, True, 4), (256, "f32", 60, 700, 9, 6, 2, False, 4),
])
def test_heads_kernel_with_every_tile_size_on_wide_rows(hidden, dtype, n_pi, n_and, cap, hops, layers, ffn, rows):
    w = make_flat(n_pi, n_and, cap, hidden, dtype, hops, layers)
    c = w.cfg
    fw = synth.ffn_weights(c) if ffn else None
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    assert shape_of(w, g.n_levels, ffn) == (True, rows)
    print(f"heads kernel, tiles of {rows}: {dtype} {hidden} {c.n_nodes // g.n_levels} gates per level hops={hops} ffn={ffn}", flush=True)
    cfg = cfg_of(c, ffn=ffn)
    H = run(w, cfg, g, fw)
    og = oracle.build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    assert (int(np.diff(og.nbr_ptr).max()) > 16) == (hops > 3)
    kw = dict(w1=fw[0], w2=fw[1]) if ffn else {}
    ref = oracle.layer_fwd(og, w.x, w.wqkv, w.wo, w.rel_bias, c.heads, store=dtype, **kw)
    assert row_rel_err(to_np(H), ref).max() <= TOL[dtype]
    mid = g.n_levels // 2
    assert torch.equal(H, run(w, cfg, g, fw, mid, None, H0=run(w, cfg, g, fw, 0, mid)))


@pytest.mark.parametrize("hidden,dtype,n_pi,n_and,cap,hops,ffn", [
    (256, "bf16", 400, 2_000, 14, 2, False), (256, "bf16", 400, 2_000, 14, 3, True),
    (128, "f32", 400, 6_000, 8, 3, False), (128, "f32", 400, 6_000, 8, 2, True),
])
def test_heads_kernel_takes_two_tiles_of_the_pair_table_at_a_time(hidden, dtype, n_pi, n_and, cap, hops, ffn):
    # a deeper levelling of a circuit whose levels hold more than one round of the table's tiles of 8
    w = make_flat(n_pi, n_and, cap, hidden, dtype, hops, 2)
    c = w.cfg
    fw = synth.ffn_weights(c) if ffn else None
    cfg = cfg_of(c, ffn=ffn)
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    level = g.array("level")
    hint = np.where(level > 0, 2 * level + np.arange(c.n_nodes) % 2, 0).astype(np.int32)
    deeper = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops, hint)
    assert deeper.n_levels > g.n_levels and shape_of(w, g.n_levels, ffn) == (True, 16)
    tiles = np.diff(deeper.array("pair_tile_ptr"))
    assert tiles.max() == 8 and tiles.min() >= 0
    print(f"heads kernel, two tiles of 8: {dtype} {hidden} {c.n_nodes // g.n_levels} gates per level hops={hops} ffn={ffn}", flush=True)
    H = run(w, cfg, g, fw)
    og = oracle.build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    kw = dict(w1=fw[0], w2=fw[1]) if ffn else {}
    ref = oracle.layer_fwd(og, w.x, w.wqkv, w.wo, w.rel_bias, c.heads, store=dtype, **kw)
    assert row_rel_err(to_np(H), ref).max() <= TOL[dtype]
    assert torch.equal(H, run(w, cfg, deeper, fw))
    edges = [torch.from_numpy(a).cuda() for a in (w.edge_src, w.edge_dst, w.edge_inv, hint)]
    assert torch.equal(H, run(w, cfg, dg4.dg4_build_levels_device(c.n_nodes, *edges[:3], hops, edges[3]), fw))


@pytest.mark.parametrize("hidden,dtype,layers", [(128, "f32", 1), (128, "bf16", 2), (256, "f32", 2), (256, "bf16", 1)])
@pytest.mark.parametrize("hops,trees", [(4, 3), (5, 3), (6, 20), (7, 20), (8, 3)])
def test_heads_kernel_on_rows_that_end_a_round(hidden, dtype, layers, hops, trees):
    # complete trees: rows of 2^(h+1) - 1 entries, so that whole rounds of a lane group's eight entries, one entry
    # short (the gate itself included), come in every tile size and lane split
    leaves = 2 ** hops
    n_pi, n_and = trees * leaves, trees * (leaves - 1)
    w = make(n_and, 2, hidden, dtype, hops, layers, n_pi=n_pi)
    src, dst, below, nxt = [], [], np.arange(n_pi), n_pi
    while len(below) > trees:
        above = np.arange(nxt, nxt + len(below) // 2)
        src.append(below)
        dst.append(np.repeat(above, 2))
        below, nxt = above, nxt + len(above)
    src, dst = np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)
    inv = (np.arange(len(src)) % 3 == 0).astype(np.uint8)
    g = dg4.dg4_build_levels(w.cfg.n_nodes, src, dst, inv, hops)
    assert max(np.diff(g.array("nbr_ptr"))) == 2 ** (hops + 1) - 1
    print(f"tree rows {dtype} {hidden} hops={hops} trees={trees} layers={layers}", flush=True)
    H = run(w, cfg_of(w.cfg), g)
    og = oracle.build_levels(w.cfg.n_nodes, src, dst, inv, hops)
    assert row_rel_err(to_np(H), oracle.layer_fwd(og, w.x, w.wqkv, w.wo, w.rel_bias, w.cfg.heads, store=dtype)).max() <= TOL[dtype]
