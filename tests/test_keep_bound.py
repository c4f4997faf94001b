"""The bound on packed fields that autograd graphs keep (CPU: the accounting
alone, without a field)."""

import gc
import threading

import torch

from paper_2001_07557_amd import autograd as A


def test_shares_stay_within_the_bound_and_come_back():
    dev, part = "test-device", A.KEEP_BYTES // 8
    shares = [A._take_share(dev, part) for _ in range(8)]
    assert all(s is not None for s in shares)
    assert A._take_share(dev, 1) is None
    assert A._take_share("another-device", part) is not None
    shares.pop()
    assert A._take_share(dev, part + 1) is None
    s = A._take_share(dev, part)
    assert s is not None
    del shares, s
    gc.collect()
    assert A._take_share(dev, A.KEEP_BYTES) is not None


def test_shares_from_many_threads():
    dev, part, limit = "threads", A.KEEP_BYTES // 5, 5
    live, most, lock = [0], [0], threading.Lock()

    def work():
        for _ in range(2000):
            s = A._take_share(dev, part)
            if s is None:
                continue
            with lock:
                live[0] += 1
                most[0] = max(most[0], live[0])
            with lock:
                live[0] -= 1
            del s

    threads = [threading.Thread(target=work) for _ in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert 0 < most[0] <= limit
    assert A._take_share(dev, A.KEEP_BYTES) is not None


def test_a_share_goes_with_the_saved_buffer():
    """What the bound counts is freed when the graph's saved tensors are, not
    when a result that the caller still holds is."""
    dev = "saved"

    class Doubled(torch.autograd.Function):
        @staticmethod
        def forward(ctx, x):
            b = torch.zeros(8, dtype=torch.uint8)
            b.share = A._take_share(dev, A.KEEP_BYTES)
            assert b.share is not None
            ctx.save_for_backward(x, b)
            return 2 * x

        @staticmethod
        def backward(ctx, g):
            assert len(ctx.saved_tensors) == 2
            return 2 * g

    x = torch.ones(3, requires_grad=True)
    y = Doubled.apply(x)
    assert A._take_share(dev, 1) is None
    y.sum().backward(retain_graph=True)
    assert A._take_share(dev, 1) is None
    y.sum().backward()
    assert A._take_share(dev, A.KEEP_BYTES) is not None  # y is alive
    y = Doubled.apply(x)
    del y
    assert A._take_share(dev, A.KEEP_BYTES) is not None
