"""bf16 dispatch edges, against the fp64 oracle: heads of few and many (query block, key block) pairs, whose thresholds
all come from the pooled keys' moments, and causal launches on both sides of the line between the two queue orders
(query blocks of all heads)."""
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
    (387 * 64, 64, 64, 0, "sparse"),                         # 149,769 pairs
    (387 * 64 + 1, 64, 64, 0, "sparse"),                     # a last block of one row
    (24640 + 192, 64, 64, 192, "sparse_no_correction"),      # 388 x 385 with a forced tail
    (548 * 64 - 5, 128, 128, 0, "sparse"),                   # 274 x 548 = 150,152
    (130, 128, 64, 64, "sparse"),                            # two routable blocks, a forced one
])
def test_statistics_from_moments(dev, N, d, bq, text, mode):
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


def kernel_proxies(qbar, kbar, tpk):
    """The forward's f32 proxies, operation by operation: a key's row in 16-byte chunks over tpk threads, four fused
    sums per thread (in 64 bits the products of two f32 are exact, so one rounding per step), then the threads'."""
    nq, d = qbar.shape
    nk = kbar.shape[0]
    qc = qbar.reshape(nq, 1, d // (4 * tpk), tpk, 4).astype(np.float64)
    kc = kbar.reshape(1, nk, d // (4 * tpk), tpk, 4).astype(np.float64)
    a = np.zeros((nq, nk, tpk, 4), np.float32)
    for i in range(d // (4 * tpk)):
        a = (a.astype(np.float64) + qc[:, :, i] * kc[:, :, i]).astype(np.float32)
    dot = (a[..., 0] + a[..., 1]) + (a[..., 2] + a[..., 3])
    while dot.shape[-1] > 1:
        dot = dot[..., 0::2] + dot[..., 1::2]
    return np.float32(1.0 / math.sqrt(d)) * dot[..., 0]


@pytest.mark.parametrize("dtype,d,bq", [("bf16", 64, 64), ("bf16", 64, 128), ("bf16", 128, 64), ("bf16", 128, 128),
                                        ("f32", 64, 64), ("f32", 128, 128)])
def test_forward_selects_by_the_threshold_entry_points_tau(dev, dtype, d, bq):
    # Two kinds of key block, half of each: at beta = 1 the larger proxy of every row equals tau_i in exact
    # arithmetic, so rounding alone decides, and only a forward that takes its tau from the same moments
    # agrees with sol_attn_thresholds on every row.  Tokens of a block are equal: their means are exact.
    H, nk, tpk = 2, 66, 2 if dtype == "bf16" and d == 64 and bq == 64 else 4
    g = torch.Generator().manual_seed(d + bq)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    kinds = torch.randn(H, 2, d, generator=g).bfloat16()
    k = kinds[:, torch.arange(nk) % 2].repeat_interleave(64, dim=1)[None].to(dt)
    q = torch.randn(1, H, nk * 64 // bq, d, generator=g).bfloat16().repeat_interleave(bq, dim=2).to(dt)
    q, k, v = (x.contiguous().to(dev) for x in (q, k, torch.randn(k.shape, generator=g).to(dt)))
    mask = torch.zeros((1, H, q.shape[2] // bq, sb.mask_words(nk)), dtype=torch.int32, device=dev)
    sb.forward(q, k, v, bq, 64, 1.0, "sparse", mask_out=mask)
    got = sb.unpack_mask(mask.cpu().numpy().view(np.uint32), nk)
    qbar, kbar, _ = sb.pool_blocks(q, k, v, bq, 64)
    tau = sb.thresholds(qbar, kbar, 1.0)[0].cpu().numpy()
    for h in range(H):
        s_hat = kernel_proxies(qbar[0, h].cpu().numpy(), kbar[0, h].cpu().numpy(), tpk)
        assert np.array_equal(got[0, h], s_hat > tau[0, h][:, None])


@pytest.mark.parametrize("H,N,d,bq,g,mode", [
    (1, 70, 64, 64, 1, "sparse"),                 # 2 blocks: most queues are empty
    (3, 9 * 64 + 1, 128, 64, 1, "sparse"),        # 10 blocks a head, not a multiple of 8
    (96, 1024, 64, 64, 130, "sparse"),            # many heads: head by head
    (97, 1023, 64, 64, 130, "sparse"),
    (5, 2049, 64, 128, 1, "dense"),               # 128-row blocks at d = 64, two waves a SIMD
    (121, 1089, 64, 128, 64, "sparse_no_correction"),   # 1,089 of them: two
    (160, 1023, 64, 128, 1, "sparse"),            # 1,280: two
    (183, 895, 64, 128, 1, "sparse"),             # 1,281: three
    (16, 6144, 64, 64, 130, "sparse"),            # 16 heads, 1,536 blocks: block by block
    (16, 6145, 64, 64, 130, "sparse_no_correction"),    # 1,552: head by head
    (15, 9 * 128, 128, 128, 1, "sparse"),         # 135 blocks, 9 a head: block by block, the last round is one block
    (14, 9 * 128, 128, 128, 1, "dense"),          # 126: head by head
    (17, 8 * 128, 64, 128, 1, "sparse"),          # 17 heads: head by head
    (2, 66 * 128 - 1, 128, 128, 64, "sparse"),    # 132 blocks of 2 heads, key blocks on the granule
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


@pytest.mark.parametrize("dtype,N,bq", [("bf16", 2048, 128), ("bf16", 1024, 64), ("f32", 1024, 64)])
def test_counts_shared_by_overlapping_calls_hold_one_calls_sums(dev, dtype, N, bq):
    # Two forwards with other selections overlap on two streams, each with its own workspace, and write the same
    # counts buffer (the caller's, then the library's): every head's count is the sum of one of the two calls.
    w = small_workload("counts", (N,), 128, bq, dtype=dtype, H=24, B=2, seed=13)
    q, k, v = (t.to(dev) for t in synth.make_qkv(w))
    code = sb.SOL_BF16 if dtype == "bf16" else sb.SOL_F32
    ws = [torch.empty(sb.workspace_bytes(w.B, w.H, N, 128, bq, 64, "sparse", code), dtype=torch.uint8, device=dev)
          for _ in range(2)]
    outs = [torch.empty_like(q) for _ in range(2)]
    betas = (0.2, 1.1)
    want = []
    for beta, o, s in zip(betas, outs, ws):
        c = torch.empty((w.B, w.H), dtype=torch.int32, device=dev)
        sb.forward(q, k, v, bq, 64, beta, "sparse", out=o, workspace=s, counts=c)
        want.append(c.cpu().numpy().ravel())
    assert (want[0] != want[1]).all()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]   # default priority
    shared = torch.empty((w.B, w.H), dtype=torch.int32, device=dev)
    for counts in (shared, None):
        for _ in range(5):
            torch.cuda.synchronize()
            for i in range(2):
                with torch.cuda.stream(streams[i]):
                    sb.forward(q, k, v, bq, 64, betas[i], "sparse", out=outs[i], workspace=ws[i], counts=counts)
            torch.cuda.synchronize()
            got = np.array(sb.stats(w.B, w.H, counts=counts)) * (w.NQ * w.NK)
            assert all(round(g) in (a, b) for g, a, b in zip(got, *want)), (got, want)


@pytest.mark.parametrize("dtype,d,bq", [("bf16", 128, 64), ("f32", 64, 128)])
def test_counts_of_one_query_block(dev, dtype, d, bq):
    w = small_workload("oneblock", (bq - 3,), d, bq, dtype=dtype, H=3, seed=2)
    q, k, v = (t.to(dev) for t in synth.make_qkv(w))
    mask = torch.zeros((1, 3, 1, 1), dtype=torch.int32, device=dev)
    counts = torch.full((1, 3), -1, dtype=torch.int32, device=dev)
    sb.forward(q, k, v, bq, 64, 0.0, "sparse", counts=counts, mask_out=mask)
    assert np.array_equal(counts.cpu().numpy(), sb.unpack_mask(mask.cpu().numpy().view(np.uint32), w.NK).sum(axis=(2, 3)))


@pytest.mark.parametrize("mode,g,d,bq,off", [("dense", 0, 64, 64, 1), ("sparse", 0, 128, 128, 1), ("sparse", 0, 128, 64, 2),
                                             ("sparse", 1, 64, 128, 1), ("sparse_no_correction", 100, 128, 64, 4)])
def test_bf16_tensors_off_16_bytes(dev, mode, g, d, bq, off):
    # views that start 2 bytes or more into an allocation: the same results as aligned tensors, bit for bit
    w = small_workload("off", (601,), d, bq, H=2, seed=4)
    aligned = [t.to(dev) for t in synth.make_qkv(w)]
    moved = []
    for t in aligned + [torch.empty_like(aligned[0])]:
        moved.append(torch.empty(t.numel() + off, device=dev, dtype=t.dtype)[off:].view(t.shape))
        moved[-1].copy_(t)
        assert moved[-1].data_ptr() % 16 == 2 * off
    out = moved.pop()
    ref = sb.forward(*aligned, bq, 64, 0.5, mode, causal_granule=g)
    sb.forward(*moved, bq, 64, 0.5, mode, causal_granule=g, out=out)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("dtype,off", [("bf16", 2), ("bf16", 8), ("f32", 4)])
def test_workspace_off_16_bytes(dev, dtype, off):
    w = small_workload("wsoff", (601,), 128, 64, dtype=dtype, H=2, seed=4)
    q, k, v = (t.to(dev) for t in synth.make_qkv(w))
    ref = sb.forward(q, k, v, 64, 64, 0.5, "sparse")
    n = sb.workspace_bytes(1, 2, 601, 128, 64, 64, "sparse", sb.SOL_BF16 if dtype == "bf16" else sb.SOL_F32)
    buf = torch.full((n + off + 4096,), 0x5A, dtype=torch.uint8, device=dev)
    out = sb.forward(q, k, v, 64, 64, 0.5, "sparse", workspace=buf[off:off + n])
    assert torch.equal(out, ref)
    assert bool((buf[:off] == 0x5A).all()) and bool((buf[off + n:] == 0x5A).all()), "written outside the workspace"


def test_pooling_of_inputs_past_one_launch(dev):
    # 1.1 GB of inputs: a launch per tensor; the same means as of a slice small enough for one launch, bit for bit
    g = torch.Generator(device=dev).manual_seed(3)
    q, k, v = (torch.randn(1, 24, 60001, 128, generator=g, device=dev).bfloat16() for _ in range(3))
    assert 3 * q.numel() * 2 > 1 << 30
    got = sb.pool_blocks(q, k, v, 128, 64)
    for h in (0, 23):
        part = sb.pool_blocks(*(x[:, h:h + 1].contiguous() for x in (q, k, v)), 128, 64)
        for a, b in zip(got, part):
            assert torch.equal(a[:, h:h + 1], b)


@pytest.mark.parametrize("dtype,d,bq", [("bf16", 64, 64), ("bf16", 128, 128), ("f32", 64, 128), ("f32", 128, 64)])
def test_a_single_routable_block_ties_with_its_mean(dev, dtype, d, bq):
    # sigma = 0: the proxy equals mu, and selection is strict, whichever way their rounding falls; 64 heads so that
    # rounding would select some.  Without a tail, with one forced block, and under a mask.
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(d + bq)
    for n, keep, granule in ((1, 0, 0), (33, 0, 0), (64, 0, 0), (100, 64, 0), (50, 0, 50)):
        q, k, v = (torch.randn(4, 16, n, d, generator=g).to(dt).to(dev) for _ in range(3))
        for beta, want in ((0.0, 0), (0.7, 0), (-0.7, 0), (math.inf, 0), (-math.inf, 1)):
            counts = torch.full((4, 16), -1, dtype=torch.int32, device=dev)
            sb.forward(q, k, v, bq, 64, beta, "sparse", keep_tail_tokens=keep, counts=counts, causal_granule=granule)
            assert bool((counts == want * -(-n // bq)).all()), (n, keep, granule, beta)
