"""bf16 dispatch edges, against the fp64 oracle: shapes on both sides of the line between statistics taken on chip from
a row's proxies and from the pooled keys' moments (query blocks x key blocks of a head), and causal launches on both
sides of the line between the two queue orders (query blocks of all heads)."""
import math

import numpy as np
import pytest
import torch

from oracle import sol_attn_oracle as ora
from paper_2607_24027_amd import binding as sb
from paper_2607_24027_amd import synth
from tests.parity import assert_mask_matches, assert_output_close, small_workload, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sb.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("N,d,bq,text,mode", [
    (387 * 64, 64, 64, 0, "sparse"),                         # 149,769 pairs: on chip
    (387 * 64 + 1, 64, 64, 0, "sparse"),                     # 150,544: moments and order, a last block of one row
    (24640 + 192, 64, 64, 192, "sparse_no_correction"),      # 388 x 385 with a forced tail: on chip
    (548 * 64 - 5, 128, 128, 0, "sparse"),                   # 274 x 548 = 150,152: moments
    (130, 128, 64, 64, "sparse"),                            # two routable blocks, a forced one
])
def test_statistics_on_chip_or_from_moments(dev, N, d, bq, text, mode):
    w = small_workload("line", (N - text,), d, bq, text_tokens=text, H=1, seed=N)
    q, k, v = synth.make_qkv(w)
    nkr = w.NK - text // 64
    print(f"[dispatch] N={N} d={d} bq={bq} NQ={w.NQ} NKr={nkr} {mode}", flush=True)
    mask = torch.zeros((1, 1, w.NQ, sb.mask_words(nkr)), dtype=torch.int32, device=dev)
    counts = torch.full((1, 1), -1, dtype=torch.int32, device=dev)
    out = torch.full(q.shape, math.nan, dtype=torch.bfloat16, device=dev)
    sb.forward(q.to(dev), k.to(dev), v.to(dev), bq, 64, 0.7, mode, keep_tail_tokens=text, out=out, counts=counts,
               mask_out=mask)
    gmask = sb.unpack_mask(mask.cpu().numpy().view(np.uint32), nkr)
    assert bool(torch.isfinite(out).all())
    qn, kn, vn = to_np(q), to_np(k), to_np(v)
    r = ora.routing(qn, kn, bq, 64, 0.7, keep_tail_tokens=text)
    assert_mask_matches(gmask, r["mask"], r["s_hat"], r["tau"])
    assert np.array_equal(counts.cpu().numpy(), gmask.sum(axis=(2, 3)))
    blocks = sorted({0, w.NQ // 2, w.NQ - 1})
    ref = ora.forward(qn, kn, vn, bq, 64, 0.7, mode, keep_tail_tokens=text, query_blocks=blocks, mask=gmask)["out"]
    assert_output_close(to_np(out), ref, "bf16", mode)


@pytest.mark.parametrize("H,N,d,bq,g,mode", [
    (1, 70, 64, 64, 1, "sparse"),                 # 2 blocks: most queues are empty
    (3, 9 * 64 + 1, 128, 64, 1, "sparse"),        # 10 blocks a head, not a multiple of 8
    (96, 1024, 64, 64, 130, "sparse"),            # 1,536 blocks: dealt block by block
    (97, 1023, 64, 64, 130, "sparse"),            # 1,552 blocks: head by head
    (5, 2049, 64, 128, 1, "dense"),               # 128-row blocks at d = 64, two workgroups a CU
    (121, 1089, 64, 128, 64, "sparse_no_correction"),   # 1,089 of them: three
])
def test_causal_queue_orders(dev, H, N, d, bq, g, mode):
    w = small_workload("queue", (N,), d, bq, H=H, seed=N + H)
    q, k, v = synth.make_qkv(w)
    print(f"[dispatch] causal H={H} N={N} d={d} bq={bq} G={g} {mode}", flush=True)
    mask = torch.zeros((1, H, w.NQ, sb.mask_words(w.NK)), dtype=torch.int32, device=dev)
    counts = torch.full((1, H), -1, dtype=torch.int32, device=dev)
    out = torch.full(q.shape, math.nan, dtype=torch.bfloat16, device=dev)
    sb.forward(q.to(dev), k.to(dev), v.to(dev), bq, 64, 0.5, mode, out=out, counts=counts, mask_out=mask, causal_granule=g)
    assert bool(torch.isfinite(out).all()), "rows left unwritten"
    heads = sorted({0, H // 2, H - 1})
    qn, kn, vn = (to_np(x[:, heads]) for x in (q, k, v))
    ref = ora.forward(qn, kn, vn, bq, 64, 0.5, mode, causal_granule=g)
    if mode != "dense":
        gmask = sb.unpack_mask(mask.cpu().numpy().view(np.uint32), w.NK)
        assert np.array_equal(counts.cpu().numpy(), gmask.sum(axis=(2, 3)))
        if assert_mask_matches(gmask[:, heads], ref["mask"], ref["s_hat"], ref["tau"]):
            ref = ora.forward(qn, kn, vn, bq, 64, 0.5, mode, causal_granule=g, mask=gmask[:, heads])
    assert_output_close(to_np(out)[:, heads], ref["out"], "bf16", mode)
