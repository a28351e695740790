"""Attention split over waves and the merge of its records, through the C ABI.

Ranges of one page (split_pages = 1) leave a record per page, so the number of
records of a row is its page count: rows with 1, 2, 5, 31 to 33 and 63 to 65
pages and more meet every loop of the merge (the first four loads of a group,
the loop past them, the weights past the 64th record), with rows few enough
for four waves each and too many for that. The library's own split covers
ranges from its shortest to several sequences long. From 6144 (sequence, KV head)
pairs it takes fewer waves than the grid has, spread over all workgroups."""
import sys

import numpy as np
import pytest
import torch

import workloads as W
from harness import Setup, assert_close, f64, oracle_run

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

CTX = [1, 16, 17, 80, 31 * 16, 33 * 16 - 3, 63 * 16, 64 * 16 + 1, 70 * 16 + 5]


@pytest.mark.parametrize("split", [0, 1, 3])
@pytest.mark.parametrize("D,n_q,n_kv,repeat", [(64, 4, 2, 1), (64, 16, 1, 8), (128, 8, 2, 1), (128, 16, 2, 8)])
def test_attention_records(D, n_q, n_kv, repeat, split):
    cfg = W.LayerCfg(hidden=256, n_q=n_q, n_kv=n_kv, head_dim=D, ffn=256)
    ctx = np.array(CTX * repeat, dtype=np.int32)
    B = len(ctx)
    print(f"[case] attention records D {D} rows {B * n_q} split {split}", file=sys.stderr, flush=True)
    w = W.Workload("attn_split", (cfg,), batch=B, ctx_lo=1, ctx_hi=int(ctx.max()))
    s = Setup(w, seed=D + split, split_pages=split, ctx=ctx)
    inp = s.oracle_inputs()
    ref = oracle_run(inp, w.layers, 0, 5)
    s.reset_resid()
    s.run(0, 5)
    torch.cuda.synchronize()
    got = f64(s.buf("o", B, n_q * D))
    for b in range(B):
        assert_close(f"row {b} (context {ctx[b]})", got[b], ref["o"][b])


@pytest.mark.parametrize("D,n_q,n_kv,batch", [(64, 4, 2, 3071), (64, 4, 2, 3072), (64, 4, 2, 3500), (64, 4, 2, 4096),
                                              (64, 16, 1, 4096), (128, 8, 4, 1536), (128, 8, 4, 1700)])
def test_attention_many_pairs(D, n_q, n_kv, batch):
    cfg = W.LayerCfg(hidden=256, n_q=n_q, n_kv=n_kv, head_dim=D, ffn=256)
    print(f"[case] attention D {D} {n_q}/{n_kv} heads batch {batch}", file=sys.stderr, flush=True)
    ctx = np.random.default_rng(batch).integers(1, 113, batch).astype(np.int32)
    ctx[:3] = 1, 2000, 16
    w = W.Workload("attn_pairs", (cfg,), batch=batch, ctx_lo=1, ctx_hi=2000)
    s = Setup(w, seed=D, ctx=ctx)
    rows = np.concatenate([np.arange(8), np.arange(8, batch - 8, 97), np.arange(batch - 8, batch)])
    ref = oracle_run(s.oracle_inputs(rows), w.layers, 0, 5)
    s.reset_resid()
    s.run(0, 5)
    torch.cuda.synchronize()
    got = f64(s.buf("o", batch, n_q * D))[rows]
    for i, b in enumerate(rows):
        assert_close(f"row {b} (context {ctx[b]})", got[i], ref["o"][i])
