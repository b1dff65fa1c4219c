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


@pytest.mark.parametrize("n_pi,n_and,launches", [(2_300, 4_700, False), (4_000, 8_200, False), (4_200, 8_200, True)])
@pytest.mark.parametrize("hops,ffn", [(2, False), (2, True), (3, False), (3, True)])
def test_one_layer_bf16_128_is_the_same_bits_under_every_levelling(n_pi, n_and, launches, hops, ffn):
    """Up to 4096 gates per level the heads of a tile over compute units, above level-by-level launches: by the circuit, not by
    the levelling, so that a caller's deeper one, host- or device-built, whole or cut in two, changes no bit."""
    w = synth.make(synth.Config("sides", 23, n_pi, n_and, 3_000, 0.5, 2, 128, 4, hops, 1, "bf16"))
    c = w.cfg
    fw = synth.ffn_weights(c) if ffn else None
    X, W = to_dev(w.x, c.dtype), device_weights(w, c.dtype)
    if ffn:
        W = [lw + (to_dev(fw[0][l], c.dtype), to_dev(fw[1][l], c.dtype)) for l, lw in enumerate(W)]
    cfg = cfg_of(c, ffn=ffn, time_sweep=True)
    edges = [torch.from_numpy(a).cuda() for a in (w.edge_src, w.edge_dst, w.edge_inv)]

    def run(g, cuts=((0, None),), cfg=cfg):
        ws = torch.full((dg4.dg4_layer_workspace_bytes(cfg, g),), 0xFF, dtype=torch.uint8, device="cuda")
        H = torch.full_like(X, float("nan"))
        for begin, end in cuts:
            dg4.dg4_layer_fwd(cfg, g, X, W, H, begin, end, workspace=ws)
        torch.cuda.synchronize()
        dg4.dg4_layer_status(cfg, g, ws)
        return H

    own = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    width = c.n_nodes // own.n_levels
    assert (width > 4096) == launches
    print(f"one layer bf16 128: {width} gates per level, hops {hops}, ffn {ffn}", flush=True)
    H = run(own)
    if launches:            # (no persistent kernel ran: nothing was timed)
        with pytest.raises(dg4.DG4Error):
            dg4.dg4_sweep_elapsed_ms()
        assert torch.equal(H, run(own, cfg=cfg_of(c, ffn=ffn, per_level=True)))
    else:
        assert dg4.dg4_sweep_elapsed_ms() > 0
    og = oracle.build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)
    kw = dict(w1=fw[0], w2=fw[1]) if ffn else {}
    ref = oracle.layer_fwd(og, w.x, w.wqkv, w.wo, w.rel_bias, c.heads, store=c.dtype, **kw)
    assert row_rel_err(to_np(H), ref).max() <= TOL[c.dtype]
    level = og.level
    for hint in (3 * level, np.where(level > 0, 5 * level + np.arange(c.n_nodes) % 5, 0)):
        hint = np.ascontiguousarray(hint.astype(np.int32))
        on_host = dg4.dg4_build_levels(c.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops, hint)
        on_gpu = dg4.dg4_build_levels_device(c.n_nodes, *edges, hops, torch.from_numpy(hint).cuda())
        mid = on_host.n_levels // 2
        assert torch.equal(H, run(on_host)) and torch.equal(H, run(on_gpu))
        assert torch.equal(H, run(on_host, ((0, mid), (mid, None)))) and torch.equal(H, run(on_gpu, ((0, 1), (1, None))))
    assert torch.equal(H, run(dg4.dg4_build_levels_device(c.n_nodes, *edges, hops)))
    assert torch.equal(H, run(own, ((0, 1), (1, None))))
