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
