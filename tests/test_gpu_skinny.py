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


@pytest.mark.parametrize("batch", [1, 8, 9, 16])
@pytest.mark.parametrize("hidden,ffn,tiled", [
    (2056, 64, False), (520, 16, False), (4104, 128, False),
    # one gate and one up fragment per block, two and two (past 4096 columns), four and four (past 8192)
    (704, 1088, False), (704, 1088, True), (1000, 4232, False), (1024, 4224, True), (1000, 8264, False),
    (1024, 8320, True), (7680, 8320, False), (7680, 8320, True)])
def test_norm_joins_gate_up(hidden, ffn, tiled, batch):
    """ffn_norm, gate_up and SiLU in one call: hn is the norm of the residual to one bf16 rounding (2^-8), act the gated
    products of the float64 normalised rows. Bound: each factor of a product is rounded to bf16 once (2^-9, here the row
    before or after its 1 / rms), so a sum is off by at most 2^-8 of sum |hn||w| with the fp32 order; SiLU(gate) * up
    carries both through (sensitivities at most 1.1 |up| and |silu|) and is rounded once. Few blocks against rows whose
    last 64-wide slice is short: every thread writes several slices of hn, with short ones among them. Wide outputs on
    tiled weights run this launch only with their norm; hidden 7680 is the widest gain it holds, at 16 rows and four
    fragments the most LDS it asks for."""
    print(f"[case] norm + gate_up + SiLU hidden {hidden} ffn {ffn} {'tiled' if tiled else 'rows'} batch {batch}",
          file=sys.stderr, flush=True)
    cfg = W.LayerCfg(hidden=hidden, n_q=2, n_kv=1, head_dim=64, ffn=ffn)
    s = Setup(W.Workload("skinny_norm", (cfg,), batch=batch, ctx_lo=1, ctx_hi=20), seed=batch + hidden, tiled=tiled)
    s.reset_resid()
    s.run(6, 9)
    torch.cuda.synchronize()
    x, g = s.x.double(), s.weights[0]["g_ffn"].double()
    hn = x * torch.rsqrt((x * x).mean(-1, keepdim=True) + cfg.rms_eps) * g
    check("hn", s.buf("hn", batch, hidden), hn, 1e-6 * hn.abs())
    w = s.weights[0]["w_gate_up"].double()
    gu, mag = hn @ w.T, 2.0 ** -8 * (hn.abs() @ w.abs().T)
    gate, up = gu[:, :ffn], gu[:, ffn:]
    act = torch.nn.functional.silu(gate)
    check("act", s.buf("act", batch, ffn), act * up,
          1.1 * up.abs() * mag[:, :ffn] + act.abs() * mag[:, ffn:] + 1.1 * mag[:, :ffn] * mag[:, ffn:]
          + 1e-6 * (act * up).abs())


@pytest.mark.parametrize("batch", [1, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("D,n_q,n_kv,hidden,tiled", [(64, 4, 2, 520, False), (128, 4, 1, 256, True),
                                                     (128, 6, 3, 1000, False), (64, 8, 8, 7680, True),
                                                     (64, 1, 1, 2056, False),
                                                     (128, 2, 1, 8192, False)])
def test_norm_rope_and_append_join_qkv(D, n_q, n_kv, hidden, tiled, batch):
    """attn_norm .. kv_append in one call: xn is the norm of the residual to one bf16 rounding (2^-8), qkv the rotated
    products of the float64 normalised rows. Bound: each factor of a product is rounded to bf16 once (2^-9, here the
    row before or after its 1 / rms), so a pair's two sums are off by at most 2^-8 of sum |xn||w| each with the fp32
    sums' order, rotation adds the two, and each value is rounded to bf16 before and after it (2^-8 of their sizes).
    The pool holds the very bits of the k and v columns in the new slots and is untouched elsewhere; hidden sizes end
    inside a K step and reach the widest gain the launch holds and past it. Row 0 has no context: it is projected,
    not rotated, and appends nothing."""
    print(f"[case] norm + qkv + rope + append D {D} hidden {hidden} batch {batch}", file=sys.stderr, flush=True)
    cfg = W.LayerCfg(hidden=hidden, n_q=n_q, n_kv=n_kv, head_dim=D, ffn=64)
    w = W.Workload("skinny_rope", (cfg,), batch=batch, ctx_lo=1, ctx_hi=70)
    s = Setup(w, seed=batch + D, tiled=tiled)
    if batch > 1:
        s.batch.ctx_lens[0] = 0
    ctx = s.batch.ctx_lens.long()
    s.reset_resid()
    before = s.pools[0].clone()
    s.run(0, 4)
    torch.cuda.synchronize()
    x, g = s.x.double(), s.weights[0]["g_attn"].double()
    xn = x * torch.rsqrt((x * x).mean(-1, keepdim=True) + cfg.rms_eps) * g
    check("xn", s.buf("xn", batch, hidden), xn, 1e-6 * xn.abs())
    wq = s.weights[0]["w_qkv"].double()
    heads = lambda t: t.view(batch, n_q + 2 * n_kv, D)  # noqa: E731
    v64, mag = heads(xn @ wq.T), heads(2.0 ** -8 * (xn.abs() @ wq.abs().T))
    half = D // 2
    inv = cfg.rope_theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / D)
    ang = ((ctx - 1).clamp(min=0).double()[:, None] * inv)[:, None, :]
    live = ((ctx > 0)[:, None, None] & (torch.arange(n_q + 2 * n_kv, device=x.device) < n_q + n_kv)[None, :, None])
    c, sn = torch.where(live, ang.cos(), 1.0), torch.where(live, ang.sin(), 0.0)
    a, b = v64[..., :half], v64[..., half:]
    ref = torch.cat([a * c - b * sn, b * c + a * sn], -1)
    both = mag[..., :half] + mag[..., half:] + (2.0 ** -8 + 1e-6) * (a.abs() + b.abs())
    got = heads(s.buf("qkv", batch, cfg.qkv_dim))
    check("qkv", got, ref, torch.cat([both, both], -1))
    after = before.clone()
    pages = s.batch.page_table.long()
    for r in range(batch):
        p = int(ctx[r]) - 1
        if p < 0:
            continue
        page, slot = int(pages[r, p // 16]), p % 16
        after[page, 0].view(n_kv, 16, D)[:, slot] = got[r, n_q:n_q + n_kv]
        after[page, 1].view(n_kv, D, 16)[:, :, slot] = got[r, n_q + n_kv:]
    assert torch.equal(s.pools[0], after)
