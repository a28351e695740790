"""The whole-K GEMM kernel of the smallest batches (up to 32 rows), operator by
operator through the C ABI, against float64 products of the operator's own
bf16 inputs as the GPU left them.

Sizes sit where it can go wrong: 1, 8 / 9 and 16 / 17 rows (one, two and four
8-row groups of activations), 32 / 33 rows (its last batch and the first of
the kernels after it); K that ends inside a 64-wide step, K of one step or
less than one step per wave, N that ends inside a 16- or 32-column block, and
outputs wide enough for each of its block shapes, on both weight layouts.

Bound per element: one rounding to bf16 (2^-8 of the value), and fp32 sums
over K products in any order (K 2^-24 of sum |a||b|); SiLU(gate) * up carries
the two sums' errors through (their sensitivities are at most 1.1 |up| and
|silu|) and its fp32 exp (1e-6 of the value)."""
import sys

import pytest
import torch

import workloads as W
from harness import Setup

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

SHAPES = {
    # hidden and FFN widths that are not multiples of 64 (nor, for hidden, of 16)
    "ragged": W.LayerCfg(hidden=520, n_q=3, n_kv=3, head_dim=64, ffn=696),
    # one K step for o_proj, K shorter than the waves of a block
    "short_k": W.LayerCfg(hidden=192, n_q=1, n_kv=1, head_dim=64, ffn=320),
    # 257 to 512 fragments (two per block), and a SiLU output past 256 blocks
    "wide": W.LayerCfg(hidden=256, n_q=40, n_kv=4, head_dim=128, ffn=4224),
    # hidden wide enough that o_proj and down take two fragments; a long K
    "tall": W.LayerCfg(hidden=4608, n_q=2, n_kv=1, head_dim=64, ffn=1088),
}
# past 512 fragments on row-major weights: gate_up on its own (2 * 4224 columns of "wide")


def gemm64(a, w):
    a, w = a.double(), w.double()
    return a @ w.T, a.shape[1] * 2.0 ** -24 * (a.abs() @ w.abs().T)


def check(name, got, ref, slack):
    bound = 2.0 ** -8 * ref.abs() + slack + 1e-30
    worst = ((got.double() - ref).abs() / bound).max().item()
    assert worst <= 1.0, f"{name}: {worst:.2f} times the bound"


@pytest.mark.parametrize("batch", [1, 8, 9, 16, 17, 32, 33])
@pytest.mark.parametrize("shape,tiled", [("ragged", False), ("short_k", False), ("short_k", True), ("wide", False),
                                         ("wide", True), ("tall", False), ("tall", True)])
def test_operators_against_float64(shape, tiled, batch):
    cfg = SHAPES[shape]
    print(f"[case] whole-K GEMMs {shape} batch {batch} {'tiled' if tiled else 'rows'}", file=sys.stderr, flush=True)
    w = W.Workload(f"skinny_{shape}", (cfg,), batch=batch, ctx_lo=1, ctx_hi=40)
    s = Setup(w, seed=batch, tiled=tiled)
    wt, H, F = s.weights[0], cfg.hidden, cfg.ffn
    s.reset_resid()
    s.run(0, 2)
    ref, slack = gemm64(s.buf("xn", batch, H), wt["w_qkv"])
    check("qkv", s.buf("qkv", batch, cfg.qkv_dim), ref, slack)
    s.run(2, 5)
    before = s.buf("resid", batch, H).double()
    s.run(5, 6)
    ref, slack = gemm64(s.buf("o", batch, cfg.n_q * cfg.head_dim), wt["w_o"])
    check("o_proj", s.buf("resid", batch, H), before + ref, slack)
    s.run(6, 8)
    ref, slack = gemm64(s.buf("hn", batch, H), wt["w_gate_up"])
    check("gate_up", s.buf("gu", batch, 2 * F), ref, slack)
    s.run(7, 9)  # gate_up and SiLU in one call: the fused epilogue
    gate, up = ref[:, :F], ref[:, F:]
    act = torch.nn.functional.silu(gate)
    check("gate_up+silu", s.buf("act", batch, F), act * up,
          1.1 * up.abs() * slack[:, :F] + act.abs() * slack[:, F:] + 1e-6 * (act * up).abs())
    before = s.buf("resid", batch, H).double()
    s.run(9, 10)
    ref, slack = gemm64(s.buf("act", batch, F), wt["w_down"])
    check("down", s.buf("resid", batch, H), before + ref, slack)


@pytest.mark.parametrize("batch", [1, 16, 17])
@pytest.mark.parametrize("hidden,experts", [(256, 8), (520, 100), (4096, 256)])
def test_router_against_float64(hidden, experts, batch):
    cfg = W.LayerCfg(hidden=hidden, n_q=2, n_kv=1, head_dim=64, n_experts=experts, top_k=2, moe_ffn=64)
    print(f"[case] router {hidden} -> {experts} batch {batch}", file=sys.stderr, flush=True)
    s = Setup(W.Workload("skinny_router", (cfg,), batch=batch, ctx_lo=1, ctx_hi=20), seed=batch)
    s.reset_resid()
    s.run(6, 8)
    ref, slack = gemm64(s.buf("hn", batch, hidden), s.weights[0]["w_router"])
    err = ((s.buf("logits", batch, experts).double() - ref).abs() / (slack + 1e-30)).max().item()
    assert err <= 1.0, f"logits: {err:.2f} times the bound"  # fp32 output: no bf16 rounding
