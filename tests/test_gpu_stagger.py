"""Unsplit streaming GEMMs that start each weight tile at a K step of its own.

gate_up + SiLU against float64 products of the GPU's own hn, either side of the
rule: 64-row tiles (33, 64 rows) with K a multiple of 2048 and not, the 256-row
tile (65 and 256 rows, the last wrap of a K range of one step more than the
tiles), on both weight layouts, and tiled weights of more tiles than compute
units, which stay in step. Bound per element as in test_gpu_skinny: one rounding
to bf16 (2^-8) plus fp32 sums over K products in any order (K 2^-24 of
sum |a||b|) through SiLU(gate) * up (sensitivities at most 1.1 |up| and |silu|)
and its fp32 exp (1e-6 of the value)."""
import sys

import pytest
import torch

import workloads as W
from harness import Setup

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("hidden,ffn,tiled,batch", [
    (2048, 8320, True, 33), (2048, 8320, True, 64), (2048, 8320, False, 64), (1984, 8320, False, 64),
    (1984, 8320, True, 65), (1984, 8320, False, 256), (704, 16448, True, 65), (704, 16448, False, 65),
    (64, 8320, True, 100)])
def test_gate_up_against_float64(hidden, ffn, tiled, batch):
    print(f"[case] staggered gate_up hidden {hidden} ffn {ffn} batch {batch} {'tiled' if tiled else 'rows'}",
          file=sys.stderr, flush=True)
    cfg = W.LayerCfg(hidden=hidden, n_q=2, n_kv=1, head_dim=64, ffn=ffn)
    s = Setup(W.Workload("stagger", (cfg,), batch=batch, ctx_lo=1, ctx_hi=16), seed=batch, tiled=tiled)
    s.reset_resid()
    s.run(6, 9)
    torch.cuda.synchronize()
    hn, w = s.buf("hn", batch, hidden).double(), s.weights[0]["w_gate_up"].double()
    gu, slack = hn @ w.T, hidden * 2.0 ** -24 * (hn.abs() @ w.abs().T)
    act = torch.nn.functional.silu(gu[:, :ffn])
    ref = act * gu[:, ffn:]
    bound = ((2.0 ** -8 + 1e-6) * ref.abs() + 1.1 * gu[:, ffn:].abs() * slack[:, :ffn] + act.abs() * slack[:, ffn:] + 1e-30)
    worst = ((s.buf("act", batch, ffn).double() - ref).abs() / bound).max().item()
    assert worst <= 1.0, f"act: {worst:.2f} times the bound"
