"""dg4_ffn_fwd at the edges of its row tiles (32 rows in fp32, 64 in bf16), every shape: against 64 bits, and the
same bits for a row whatever the range of rows it was asked for in."""
import pytest
import torch

import paper_2502_01681_amd as dg4
from gpu_utils import TOL, tdtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden", [128, 256])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_ffn_fwd_at_tile_edges(hidden, dtype):
    td = tdtype(dtype)
    gen = torch.Generator(device="cuda").manual_seed(5)
    n = 161
    S = torch.randn(n, hidden, generator=gen, device="cuda").to(td)
    W1 = (torch.randn(hidden, 4 * hidden, generator=gen, device="cuda") * hidden ** -0.5).to(td)
    W2 = (torch.randn(4 * hidden, hidden, generator=gen, device="cuda") * (4 * hidden) ** -0.5).to(td)
    s = S.double()
    ref = torch.nn.functional.layer_norm(s + torch.relu(s @ W1.double()) @ W2.double(), (hidden,), eps=1e-5)
    cfg = dg4.LayerConfig(hidden, hidden // 32, 2, 1, dtype)
    whole = torch.full_like(S, float("nan"))
    dg4.dg4_ffn_fwd(cfg, S, W1, W2, whole)
    err = ((whole.double() - ref).norm(dim=1) / ref.norm(dim=1)).max()
    print(f"{dtype} {hidden}: max row error {err:.2e}", flush=True)
    assert err <= TOL[dtype]
    for begin, end in ((0, 1), (0, 31), (0, 32), (0, 33), (5, 68), (5, 69), (5, 70), (32, 161), (160, 161), (7, 7)):
        part = torch.full_like(S, float("nan"))
        dg4.dg4_ffn_fwd(cfg, S, W1, W2, part, row_begin=begin, row_end=end)
        assert torch.equal(part[begin:end], whole[begin:end]), (begin, end)
        assert torch.isnan(part[:begin].float()).all() and torch.isnan(part[end:].float()).all(), (begin, end)
