"""Split-K sum + residual + RMSNorm as one kernel, against the two kernels.

When the norm that reads a residual GEMM's result is next in the range
(ffn_norm after o_proj, the next layer's attn_norm after down), a split-K GEMM
hands its partials to a kernel that does both. It adds and rounds in the order
of the separate kernels, so the whole block in one call and the block cut
before every norm leave the same bits in resid, hn and xn. Widths: not a
multiple of 64, one pass of the kernel's 1024 threads, and more than one."""
import sys

import pytest
import torch

import workloads as W
from harness import Setup

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("hidden,tiled,batch", [(520, False, 40), (520, False, 100), (1024, True, 33),
                                                (1024, True, 300), (4608, True, 64)])
def test_one_call_equals_cuts_at_the_norms(hidden, tiled, batch):
    print(f"[case] reduce + norm, hidden {hidden} batch {batch}", file=sys.stderr, flush=True)
    cfg = W.LayerCfg(hidden=hidden, n_q=16, n_kv=4, head_dim=64, ffn=2048)
    w = W.Workload("reduce_norm", (cfg, cfg), batch=batch, ctx_lo=1, ctx_hi=60)
    s = Setup(w, seed=7, tiled=tiled)
    got = []
    for cuts in ([0, 20], [0, 6, 10, 16, 20]):
        s.reset_resid()
        for a, b in zip(cuts[:-1], cuts[1:]):
            s.run(a, b)
        torch.cuda.synchronize()
        got.append([s.buf(name, batch, hidden).clone() for name in ("resid", "xn", "hn")])
    for name, one, cut in zip(("resid", "xn", "hn"), *got):
        assert torch.isfinite(one.float()).all()
        assert torch.equal(one, cut), f"{name}: {int((one != cut).sum())} values differ"
