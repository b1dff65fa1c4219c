"""Sizes of dg4_layer_fwd's workspace (host calls): they depend on the configuration, the number of gates and the
largest level, not on the path a sweep takes."""
import numpy as np
import pytest

import dg4_synth as synth
import paper_2502_01681_amd as dg4


def build(n_pi, n_and, window, cap, hops):
    w = synth.make(synth.Config("ws", 31, n_pi, n_and, window, 0.9, cap, 128, 4, hops, 1, "f32"))
    return dg4.dg4_build_levels(w.cfg.n_nodes, w.edge_src, w.edge_dst, w.edge_inv, hops)


def largest_level(g):
    return int(np.diff(g.array("level_ptr")).max())


@pytest.mark.parametrize("hops", [2, 3, 5])
@pytest.mark.parametrize("hidden,dtype", [(128, "f32"), (128, "bf16"), (256, "f32"), (256, "bf16")])
def test_a_size_covers_every_path_and_every_smaller_circuit(hidden, dtype, hops):
    narrow = build(40, 300, 40, 0, hops)            # a few gates per level
    middle = build(90, 5_000, 100, 0, hops)         # ... and more gates than the wide one next to it in size
    wide = build(2_600, 2_700, 2_000, 1, hops)      # two levels
    assert narrow.n < middle.n < wide.n
    assert largest_level(narrow) < largest_level(middle) < largest_level(wide)
    for layers in (1, 4):
        for ffn in (False, True):
            def size(g, **kw):
                return dg4.dg4_layer_workspace_bytes(dg4.LayerConfig(hidden, hidden // 32, hops, layers, dtype, ffn=ffn, **kw), g)

            for g in (narrow, middle, wide):
                assert size(g, per_level=True) == size(g) == size(g, level_order=True)
            assert size(narrow) <= size(middle) <= size(wide)
