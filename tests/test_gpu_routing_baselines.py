"""Top-k and top-p maps at the edges of their dispatch (keys per lane, mask words, tied and negative proxies, all or
one block kept) against the oracle's rules on the proxies the library returned."""
import numpy as np
import pytest
import torch

from oracle import sol_attn_oracle as ora
from paper_2607_24027_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sb.lib()
    return torch.device("cuda:0")


def pooled(nq, nk, d, tied, dev):
    g = torch.Generator().manual_seed(nk * 7 + nq)
    q = torch.randn(1, 2, nq, d, generator=g)
    k = torch.randn(1, 2, nk, d, generator=g)
    if tied:   # every key block three times: runs of equal proxies cross the cut
        k = k[:, :, torch.arange(nk) // 3]
    return q.to(dev), k.to(dev)


@pytest.mark.parametrize("tied", [False, True])
@pytest.mark.parametrize("nq,nk,nkr,d", [(1, 1, 1, 64), (3, 33, 33, 128), (65, 256, 256, 64), (5, 257, 250, 128),
                                         (7, 513, 513, 128), (4, 1500, 1500, 64), (3, 4096, 4096, 64)])
def test_route_baseline_masks(dev, nq, nk, nkr, d, tied):
    q, k = pooled(nq, nk, d, tied, dev)
    want = (q[..., :, :].double() @ k[:, :, :nkr].double().transpose(2, 3)) / d ** 0.5
    for rule, params in (("topk", sorted({1, max(1, nkr // 7), nkr - 1 or 1, nkr})), ("topp", (1e-3, 0.3, 0.9))):
        for param in params:
            prox, mask = sb.route_materialized(q, k, rule, param, nk_routable=nkr)
            # f32 products and sums of d terms: d ulp of the largest term sum at most
            assert float((prox.double() - want).abs().max()) <= d * 2.0 ** -24 * float(want.abs().max() + 8)
            s = prox.cpu().numpy().astype(np.float64)
            got = sb.unpack_mask(mask.cpu().numpy().view(np.uint32), nkr)
            ref = ora.route_topk(s, param) if rule == "topk" else ora.route_topp(s, param)
            if rule == "topk":
                assert np.array_equal(got, ref)
                continue
            # the mass before a block, in 64 bits, may only disagree where it meets the cut within f32 rounding
            order = np.argsort(-s, axis=-1, kind="stable")
            w = np.exp(s - s.max(-1, keepdims=True))
            ws = np.take_along_axis(w, order, -1)
            before = np.empty_like(s)
            np.put_along_axis(before, order, np.cumsum(ws, -1) - ws, -1)
            near = np.abs(before / w.sum(-1, keepdims=True) - param) < 1e-5
            assert not ((got != ref) & ~near).any()


def test_topk_longest_row(dev):
    q, k = pooled(2, 8192, 64, False, dev)
    prox, mask = sb.route_materialized(q, k, "topk", 1000)
    got = sb.unpack_mask(mask.cpu().numpy().view(np.uint32), 8192)
    assert np.array_equal(got, ora.route_topk(prox.cpu().numpy().astype(np.float64), 1000))


@pytest.mark.parametrize("nkr,d", [(100, 64), (300, 128)])
def test_rows_without_a_softmax(dev, nkr, d):
    # One key component is infinite: rows whose query component is positive have a proxy of +inf, zero gives not a
    # number, and both have no softmax, so top-p keeps nothing; a negative one gives -inf, a block without weight.
    q, k = pooled(9, nkr, d, False, dev)
    q[..., 0] = torch.tensor([1.0, 0.0, -1.0], device=dev).repeat(3)
    k[:, 1, nkr // 2, 0] = float("inf")   # the second head; the first stays finite
    prox, mask = sb.route_materialized(q, k, "topp", 0.5)
    s = prox.cpu().numpy().astype(np.float64)
    got = sb.unpack_mask(mask.cpu().numpy().view(np.uint32), nkr)
    for h in range(2):
        for i in range(9):
            if h == 1 and i % 3 < 2:
                assert not got[0, h, i].any()
                continue
            assert not got[0, h, i][np.isneginf(s[0, h, i])].any()
            w = np.exp(s[0, h, i] - s[0, h, i].max())
            mass = w[got[0, h, i]].sum() / w.sum()
            assert 0.5 - 1e-5 <= mass <= 0.5 + w[got[0, h, i]].min() / w.sum() + 1e-5
    _, mask = sb.route_materialized(q, k, "topk", 7)
    assert (sb.unpack_mask(mask.cpu().numpy().view(np.uint32), nkr).sum(-1) == 7).all()
