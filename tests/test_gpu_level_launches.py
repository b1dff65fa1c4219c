"""Level-by-level launches in every shape, levels around the 32 rows of a tile (64 for the feed-forward sub-block in bf16)
and above the 4096 gates up to which the attention runs in the output projection's launch: against the oracle, and the
same bits when the sweep is cut in two."""
import numpy as np
import pytest
import torch

import dg4_synth as synth
import oracle
import paper_2502_01681_amd as dg4
from gpu_utils import TOL, cfg_of, device_weights, row_rel_err, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden", [128, 256])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_pi,n_and,cap,hops,layers,ffn", [
    (2, 2, 1, 1, 1, False), (31, 63, 2, 2, 1, True), (33, 65, 1, 2, 1, False), (64, 1_301, 20, 2, 2, True),
    (100, 400, 6, 3, 1, False), (100, 400, 6, 4, 2, True), (200, 8_500, 2, 2, 1, False), (4_200, 4_300, 1, 1, 2, True),
])
def test_level_by_level(hidden, dtype, n_pi, n_and, cap, hops, layers, ffn):
    w = synth.make(synth.Config("launches", 17, n_pi, n_and, 500, 0.5, cap, hidden, hidden // 32, hops, layers, dtype))
    c = w.cfg
    fw = synth.ffn_weights(c) if ffn else None
    X, W = to_dev(w.x, dtype), device_weights(w, dtype)
    if ffn:
        W = [lw + (to_dev(fw[0][l], dtype), to_dev(fw[1][l], dtype)) for l, lw in enumerate(W)]
    cfg = cfg_of(c, ffn=ffn, per_level=True)
    g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    print(f"level by level {dtype} {hidden}: {c.n_nodes} gates, {g.n_levels} levels, hops {hops}, layers {layers}, ffn {ffn}", flush=True)
    ws = torch.full((dg4.dg4_layer_workspace_bytes(cfg, g),), 0xFF, dtype=torch.uint8, device="cuda")
    H = torch.full_like(X, float("nan"))
    dg4.dg4_layer_fwd(cfg, g, X, W, H, workspace=ws)
    og = oracle.build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    kw = dict(w1=fw[0], w2=fw[1]) if ffn else {}
    ref = oracle.layer_fwd(og, w.x, w.wqkv, w.wo, w.rel_bias, c.heads, store=dtype, **kw)
    assert row_rel_err(to_np(H), ref).max() <= TOL[dtype]
    cut = torch.full_like(X, float("nan"))
    mid = g.n_levels // 2
    ws.fill_(0xFF)
    for begin, end in ((0, mid), (mid, None)):
        dg4.dg4_layer_fwd(cfg, g, X, W, cut, begin, end, workspace=ws)
    assert torch.equal(H, cut)


@pytest.mark.parametrize("n_pi,n_and,ffn", [(2_000, 4_000, False), (2_000, 4_000, True), (2_300, 4_700, False), (2_300, 4_700, True)])
@pytest.mark.parametrize("hops", [2, 3])
def test_one_layer_bf16_128_on_both_sides_of_2048_gates_per_level(n_pi, n_and, ffn, hops):
    """Below: the heads of a tile over compute units; above: level-by-level launches, unless a caller's levelling is deeper than
    the circuit. Each against the oracle, and cut in two to the same bits."""
    w = synth.make(synth.Config("sides", 23, n_pi, n_and, 3_000, 0.5, 2, 128, 4, hops, 1, "bf16"))
    c = w.cfg
    fw = synth.ffn_weights(c) if ffn else None
    X, W = to_dev(w.x, c.dtype), device_weights(w, c.dtype)
    if ffn:
        W = [lw + (to_dev(fw[0][l], c.dtype), to_dev(fw[1][l], c.dtype)) for l, lw in enumerate(W)]
    cfg = cfg_of(c, ffn=ffn)
    og = oracle.build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    kw = dict(w1=fw[0], w2=fw[1]) if ffn else {}
    ref = oracle.layer_fwd(og, w.x, w.wqkv, w.wo, w.rel_bias, c.heads, store=c.dtype, **kw)
    hint = (3 * og.level).astype(np.int32)
    for deeper in (None, hint):
        g = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops, deeper)
        print(f"one layer bf16 128: {c.n_nodes // og.n_levels} gates per level, hops {hops}, ffn {ffn}, deeper {deeper is not None}", flush=True)
        ws = torch.full((dg4.dg4_layer_workspace_bytes(cfg, g),), 0xFF, dtype=torch.uint8, device="cuda")
        H, cut = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
        dg4.dg4_layer_fwd(cfg, g, X, W, H, workspace=ws)
        assert row_rel_err(to_np(H), ref).max() <= TOL[c.dtype]
        ws.fill_(0xFF)
        for begin, end in ((0, 1), (1, None)):
            dg4.dg4_layer_fwd(cfg, g, X, W, cut, begin, end, workspace=ws)
        assert torch.equal(H, cut)
