"""The moment scratch of the thresholds entry point: growth, calls too large to keep it, release, and calls on two
threads and streams, against the statistics of the proxies in 64 bits."""
import threading

import numpy as np
import pytest
import torch

from paper_2607_24027_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sb.lib()
    return torch.device("cuda:0")


def pooled(H, nq, nk, d, seed, dev):
    g = torch.Generator().manual_seed(seed)
    return tuple(torch.randn(1, H, n, d, generator=g).to(dev) for n in (nq, nk))


def check(q, k, got):
    s = (q.cpu().double() @ k.cpu().double().transpose(2, 3)) / q.shape[-1] ** 0.5
    mu, sigma = s.mean(-1), s.std(-1, correction=0)
    for x, y in zip(got, (mu + 0.7 * sigma, mu, sigma)):
        # f32 moments and sums of d = 128 terms: relative errors of at most 128 * 2^-24 = 8e-6 of values of a few units;
        # sigma, from its square, has half of that (40 keys or more: sigma is near 1, never near 0)
        assert float((x.cpu().double() - y).abs().max()) < 2e-5


def test_scratch_grows_is_given_back_and_comes_again(dev):
    # 4 and 64 heads keep the scratch, 800 heads of d = 128 need 112 MB, above what is kept
    for H in (4, 64, 800, 4, None, 4, 64):
        if H is None:
            sb.release()
            continue
        q, k = pooled(H, 3, 40, 128, H, dev)
        check(q, k, sb.thresholds(q, k, 0.7))


def test_calls_on_two_streams_do_not_wait_for_each_other(dev):
    q, k = pooled(4, 9, 70, 64, 1, dev)
    x = torch.randn(8192, 8192, device=dev, dtype=torch.bfloat16)
    y = torch.empty_like(x)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]   # default priority
    sb.release()
    sb.thresholds(q, k, 0.7)
    torch.mm(x, x, out=y)
    torch.cuda.synchronize()
    first, started = [], threading.Event()
    busy = torch.cuda.Event()

    def blocked():
        torch.cuda.set_device(dev)
        with torch.cuda.stream(streams[0]):
            for _ in range(400):   # about half a second of work ahead of the call
                torch.mm(x, x, out=y)
            busy.record(streams[0])
            started.set()
            first.append(sb.thresholds(q, k, 0.7))

    t = threading.Thread(target=blocked)
    t.start()
    assert started.wait(60)
    with torch.cuda.stream(streams[1]):
        second = sb.thresholds(q, k, 0.7)
        done_early = not busy.query()
    t.join(60)
    torch.cuda.synchronize()
    assert done_early, "the second call waited for the first one's stream"
    check(q, k, first[0])
    check(q, k, second)
