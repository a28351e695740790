"""moe_combine_residual alone, on expert outputs, weights and slots given
directly, against float64: every number of experts per round of loads (top_k 1,
2, 3 to 4, 5 to 8 and more), rows over one and two blocks with a short last
one, few tokens and the many-token form. Slots outside the expert rows (as
experts past a group's end leave them) add nothing, also where the row they
would clamp to holds NaN. Bound per element: one rounding to bf16 (2^-8) and
fp32 sums of k products and the residual ((k + 2) 2^-24 of their sizes)."""
import sys

import pytest
import torch

import workloads as W
from harness import Setup

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("hidden,batch", [(520, 3), (2056, 40), (2048, 1100), (4096, 1427), (520, 1100)])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 11])
def test_combine_against_float64(hidden, batch, k):
    print(f"[case] combine hidden {hidden} batch {batch} k {k}", file=sys.stderr, flush=True)
    cfg = W.LayerCfg(hidden=hidden, n_q=2, n_kv=1, head_dim=64, n_experts=12, top_k=k, moe_ffn=64)
    s = Setup(W.Workload("combine", (cfg,), batch=batch, ctx_lo=1, ctx_hi=8), seed=k)
    g = torch.Generator(device="cuda").manual_seed(hidden + k)
    n = batch * k
    yp = s.buf("yp", n, hidden).normal_(0, 1, generator=g)
    w = s.buf("topk_w", batch, k).copy_(torch.rand(batch, k, device="cuda", generator=g))
    pos = torch.randperm(n, device="cuda", generator=g).int().view(batch, k)
    yp[0] = float("nan")
    yp[n - 1] = float("nan")
    pos[pos == 0] = -1
    pos[pos == n - 1] = n
    pos[batch // 2, k - 1] = 2 ** 31 - 1
    s.buf("slot_pos", batch, k).copy_(pos)
    s.reset_resid()
    s.run(13, 14)
    torch.cuda.synchronize()
    live = (pos >= 0) & (pos < n)
    rows = yp[pos.clamp(0, n - 1).long()].double() * w.double()[..., None]
    rows = torch.where(live[..., None], rows, torch.zeros_like(rows))
    x = s.x.double()
    ref = x + rows.sum(1)
    bound = 2.0 ** -8 * ref.abs() + (k + 2) * 2.0 ** -24 * (x.abs() + rows.abs().sum(1)) + 1e-30
    worst = ((s.buf("resid", batch, hidden).double() - ref).abs() / bound).max().item()
    assert worst <= 1.0, f"{worst:.2f} times the bound"
