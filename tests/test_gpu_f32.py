"""f32 inputs: the sharing of query blocks between workgroups, tile edges, masked values and long rows, against the
fp64 oracle with the f32 tolerances of the other parity tests."""
import math

import numpy as np
import pytest
import torch

from oracle import sol_attn_oracle as ora
from paper_2607_24027_amd import binding as sb
from paper_2607_24027_amd import synth
from tests.parity import assert_mask_matches, assert_output_close, small_workload, to_np

pytestmark = pytest.mark.gpu

# (H, N, d, block_q, granule, mode): every rule of the sharing (fewer than 128 query blocks, fewer than 512, more), both
# block heights and head sizes, last blocks of 1 and 63 rows, none, and of a full block.
CASES = [
    (1, 63, 64, 64, 0, "dense"),
    (2, 1024, 128, 64, 0, "sparse"),
    (3, 1025, 128, 128, 0, "sparse"),
    (2, 1087, 64, 128, 0, "sparse_no_correction"),
    (7, 2497, 64, 128, 0, "sparse"),            # 140 query blocks, not a multiple of 8
    (17, 1984, 64, 64, 0, "sparse"),            # 527 query blocks
    (17, 1985, 64, 64, 0, "dense"),
    (2, 1025, 128, 128, 1, "dense"),
    (2, 1025, 128, 64, 100, "sparse"),
    (5, 1903, 64, 64, 1, "sparse"),             # 150 query blocks
    (18, 1921, 64, 64, 130, "sparse_no_correction"),   # 558 query blocks
]


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sb.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("H,N,d,bq,g,mode", CASES)
def test_f32_shared_blocks_parity(dev, H, N, d, bq, g, mode):
    w = small_workload("f32", (N,), d, bq, dtype="f32", H=H, seed=5 + N)
    q, k, v = synth.make_qkv(w)
    print(f"[f32] H={H} N={N} d={d} bq={bq} G={g} {mode}", flush=True)
    mask = torch.zeros((1, H, w.NQ, sb.mask_words(w.NK)), dtype=torch.int32, device=dev)
    counts = torch.full((1, H), -1, dtype=torch.int32, device=dev)
    out = torch.full(q.shape, math.nan, device=dev)
    sb.forward(q.to(dev), k.to(dev), v.to(dev), bq, 64, 0.5, mode, out=out, counts=counts, mask_out=mask, causal_granule=g)
    torch.cuda.synchronize()
    qn, kn, vn = to_np(q), to_np(k), to_np(v)
    ref = ora.forward(qn, kn, vn, bq, 64, 0.5, mode, causal_granule=g)
    if mode != "dense":
        gmask = sb.unpack_mask(mask.cpu().numpy().view(np.uint32), w.NK)
        if assert_mask_matches(gmask, ref["mask"], ref["s_hat"], ref["tau"]):
            ref = ora.forward(qn, kn, vn, bq, 64, 0.5, mode, causal_granule=g, mask=gmask)
        assert np.array_equal(counts.cpu().numpy(), gmask.sum(axis=(2, 3)))
    assert_output_close(to_np(out), ref["out"], "f32", mode)


@pytest.mark.parametrize("d,bq", [(64, 64), (128, 128)])
def test_f32_causal_masked_values_do_not_enter(dev, d, bq):
    # the last token's value is infinite: only the last row may see it
    w = small_workload("f32inf", (700,), d, bq, dtype="f32", H=2, seed=3)
    q, k, v = synth.make_qkv(w)
    ref = sb.forward(q.to(dev), k.to(dev), v.to(dev), bq, 64, 0.0, "dense", causal_granule=1)
    v[:, :, -1] = math.inf
    out = sb.forward(q.to(dev), k.to(dev), v.to(dev), bq, 64, 0.0, "dense", causal_granule=1)
    assert torch.equal(out[:, :, :-1], ref[:, :, :-1])
    assert bool((out[:, :, -1] == math.inf).all())


def test_f32_long_rows_take_the_moment_thresholds(dev):
    # 4,099 key blocks: past the rows whose statistics are taken on chip
    w = small_workload("f32long", (2, 262, 501), 64, 128, dtype="f32", H=1, seed=9)
    assert w.NK > 4096
    q, k, v = synth.make_qkv(w)
    mask = torch.zeros((1, 1, w.NQ, sb.mask_words(w.NK)), dtype=torch.int32, device=dev)
    out = sb.forward(q.to(dev), k.to(dev), v.to(dev), 128, 64, 1.5, "sparse", mask_out=mask)
    gmask = sb.unpack_mask(mask.cpu().numpy().view(np.uint32), w.NK)
    qn, kn, vn = to_np(q), to_np(k), to_np(v)
    rows = [0, w.NQ // 2, w.NQ - 1]
    ref = ora.forward(qn, kn, vn, 128, 64, 1.5, "sparse", query_blocks=rows, mask=gmask)
    s_hat = (ora.pool_means(qn, 128)[0] @ ora.pool_means(kn, 64)[0].transpose(0, 1, 3, 2)) / 8.0
    tau = s_hat.mean(-1) + 1.5 * s_hat.std(-1)
    assert_mask_matches(gmask, s_hat > tau[..., None], s_hat, tau)
    assert_output_close(to_np(out), ref["out"], "f32", "long")


@pytest.mark.parametrize("mode,g,d,bq", [("dense", 0, 64, 64), ("sparse", 0, 128, 128), ("sparse", 1, 64, 128)])
def test_f32_tensors_off_16_bytes(dev, mode, g, d, bq):
    # views that start 4 bytes into an allocation: the same results as aligned tensors, bit for bit
    w = small_workload("f32off", (601,), d, bq, dtype="f32", H=2, seed=4)
    aligned = [t.to(dev) for t in synth.make_qkv(w)]
    off = []
    for t in aligned:
        buf = torch.empty(t.numel() + 1, device=dev)
        off.append(buf[1:].view(t.shape))
        off[-1].copy_(t)
        assert off[-1].data_ptr() % 16 == 4
    out = torch.empty(aligned[0].numel() + 1, device=dev)[1:].view(aligned[0].shape)
    ref = sb.forward(*aligned, bq, 64, 0.5, mode, causal_granule=g)
    sb.forward(*off, bq, 64, 0.5, mode, causal_granule=g, out=out)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("mode", ["dense", "sparse"])
def test_f32_workspace_of_a_longer_sequence_serves_a_shorter_one(dev, mode):
    # 512 query blocks want less room for partial outputs than 504: the longer call's workspace holds all that the
    # shorter one needs but that room, and its blocks are computed whole
    H, d, bq = 8, 128, 64
    size = {n: sb.workspace_bytes(1, H, n, d, bq, 64, mode, sb.SOL_F32) for n in (4032, 4096)}
    assert size[4032] > size[4096]
    w = small_workload("f32ws", (4032,), d, bq, dtype="f32", H=H, seed=6)
    q, k, v = (t.to(dev) for t in synth.make_qkv(w))
    ref = sb.forward(q, k, v, bq, 64, 0.5, mode)
    guard = 1 << 16
    buf = torch.full((size[4096] + guard,), 0x5A, dtype=torch.uint8, device=dev)
    out = sb.forward(q, k, v, bq, 64, 0.5, mode, workspace=buf[:size[4096]])
    assert bool((buf[size[4096]:] == 0x5A).all()), "written past the workspace"
    assert_output_close(to_np(out), to_np(ref), "f32", mode)
    with pytest.raises(sb.SolAttnError) as ei:
        sb.forward(q, k, v, bq, 64, 0.5, "sparse", workspace=buf[:1 << 20])
    assert ei.value.code == sb.SOL_ERR_WORKSPACE


@pytest.mark.parametrize("H,N,d,bq,text", [(8, 7680, 128, 128, 0), (17, 1985, 64, 64, 64), (2, 1087, 64, 128, 0)])
def test_f32_every_block_selected_is_dense_bit_for_bit(dev, H, N, d, bq, text):
    # the sharing of query blocks must not depend on the mode, whichever workspace the calls have: 480 blocks whose
    # partial outputs and routing buffers exceed 64 MiB together, launches of more and of fewer blocks
    w = small_workload("f32dense", (N - text,), d, bq, dtype="f32", text_tokens=text, H=H, seed=8)
    q, k, v = (t.to(dev) for t in synth.make_qkv(w))
    dense = sb.forward(q, k, v, bq, 64, 0.0, "dense")
    assert torch.equal(sb.forward(q, k, v, bq, 64, -math.inf, "sparse", keep_tail_tokens=text), dense)
    outs = [torch.empty_like(q) for _ in range(2)]
    counts = torch.empty((1, H), dtype=torch.int32, device=dev)
    sb.forward_noalloc(q, k, v, outs[0], counts, bq, 64, 0.0, "dense")
    sb.forward_noalloc(q, k, v, outs[1], counts, bq, 64, -math.inf, "sparse")
    assert torch.equal(outs[0], outs[1])
    size = [sb.workspace_bytes(1, H, N, d, bq, 64, m, sb.SOL_F32) for m in ("dense", "sparse")]
    assert size[0] == size[1]   # one room for partial outputs
    ws = torch.empty(size[0] - 1024, dtype=torch.uint8, device=dev)   # just short of it
    for o, (beta, m) in zip(outs, ((0.0, "dense"), (-math.inf, "sparse"))):
        sb.forward(q, k, v, bq, 64, beta, m, out=o, workspace=ws)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("H,N,d,bq", [(2, 1024, 128, 64), (2, 1087, 64, 128), (20, 1984, 64, 64)])
def test_f32_infinite_scores_reach_the_output(dev, H, N, d, bq):
    # One key component is infinite.  Rows that score it +inf have no finite softmax and must not come out finite,
    # whichever share of the block held the key; rows that score it -inf give it no weight, as for a huge finite
    # component of the same sign.
    w = small_workload("f32score", (N,), d, bq, dtype="f32", H=H, seed=12)
    q, k, v = synth.make_qkv(w)
    low = q[..., 0] < 0
    for key in (5, N // 2, N - 1):
        res = []
        for x in (math.inf, 1e30):
            kk = k.clone()
            kk[:, :, key, 0] = x
            res.append(sb.forward(q.to(dev), kk.to(dev), v.to(dev), bq, 64, 0.0, "dense").cpu())
        assert not torch.isfinite(res[0][~low]).any()
        assert torch.equal(res[0][low], res[1][low])
