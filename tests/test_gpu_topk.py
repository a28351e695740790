"""Top-k routing on special logits, through the C ABI."""
import sys

import numpy as np
import pytest
import torch

import workloads as W
from harness import Setup

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


@pytest.mark.parametrize("E,k", [(5, 5), (64, 1), (64, 8), (64, 64), (65, 8), (256, 64)])
def test_topk_special_logits(E, k):
    """Top-k of logits given directly: ties (equal values, -0 and +0), infinities, NaN and rows with fewer numbers than
    k, for the one-expert-per-lane kernel (E <= 64) and the general one alike. Choice: larger value first, ties to the
    lower id, NaN never; a slot with no number left gets id 0x7fffffff and the weight of -inf."""
    say("top-k special logits", E, k)
    cfg = W.LayerCfg(hidden=64, n_q=1, n_kv=1, head_dim=64, n_experts=E, top_k=k, moe_ffn=64)
    n = 9
    w = W.Workload("topk", (cfg,), batch=n, ctx_lo=1, ctx_hi=4)
    s = Setup(w, seed=3)
    z = np.random.default_rng(E * 100 + k).standard_normal((n, E)).astype(np.float32)
    z[1] = 0.5                                     # all equal
    z[2, ::2], z[2, 1::2] = 0.0, -0.0              # equal zeros
    z[3] = np.round(z[3])                          # many ties
    z[4, E // 2] = np.inf
    z[4, 0] = -np.inf
    z[5, 1:] = -np.inf                             # -inf is chosen, by id
    z[6, ::3] = np.nan
    z[7, : E - 1] = np.nan                         # one number left
    z[8] = np.finfo(np.float32).min                # the type's lowest value
    s.buf("logits", n, E).copy_(torch.from_numpy(z))
    s.run(8, 9)
    torch.cuda.synchronize()
    ids, wts = s.buf("topk_ids", n, k).cpu().numpy(), s.buf("topk_w", n, k).cpu().numpy()
    for b in range(n):
        order = sorted((e for e in range(E) if not np.isnan(z[b, e])), key=lambda e: (-z[b, e], e))[:k]
        want = order + [0x7FFFFFFF] * (k - len(order))
        assert ids[b].tolist() == want, (b, ids[b], want)
        zz = np.array([z[b, e] for e in order] + [-np.inf] * (k - len(order)), dtype=np.float64)
        with np.errstate(invalid="ignore"):
            p = np.exp(zz - zz[0])
            p = p / p.sum()
        np.testing.assert_allclose(wts[b], p, rtol=1e-5, atol=1e-6, equal_nan=True, err_msg=str(b))


@pytest.mark.parametrize("E,k", [(64, 1), (64, 2), (48, 1), (100, 1)])
def test_topk_joined_to_the_router_equals_the_cut(E, k):
    """Router and top-k in one call (split-K partials summed by the top-k kernel) and as two calls: the same logits and
    ids, weights to fp32 exp rounding. Top-1 of up to 64 experts takes another kernel in either form."""
    say("top-k joined to the router", E, k)
    cfg = W.LayerCfg(hidden=2048, n_q=2, n_kv=1, head_dim=64, n_experts=E, top_k=k, moe_ffn=64)
    n = 40
    s = Setup(W.Workload("topk_join", (cfg,), batch=n, ctx_lo=1, ctx_hi=4), seed=E + k)
    s.reset_resid()
    s.run(6, 7)
    got = []
    for cuts in ([7, 9], [7, 8, 9]):
        for a, b in zip(cuts[:-1], cuts[1:]):
            s.run(a, b)
        torch.cuda.synchronize()
        got.append([s.buf(x, n, m).clone() for x, m in (("logits", E), ("topk_ids", k), ("topk_w", k))])
    (z0, i0, w0), (z1, i1, w1) = got
    assert torch.equal(z0, z1) and torch.equal(i0, i1)
    assert (w0 - w1).abs().max() <= 1e-6
