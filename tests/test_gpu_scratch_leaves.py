"""Scratch calls on networks with much leaf data: what they upload is right on both
sides of the size from which it goes by a copy of its own, and takes about as long as
copying it."""
import time

import numpy as np
import pytest

from tests.gpu_util import banner, rel_l2
from tests.test_gpu_parts import torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _case(rank):
    """A leaf of 2^rank elements times a vector, and another vector: two steps."""
    import paper_2205_00393_amd as P
    rng = np.random.default_rng(rank)
    cplx = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)
    a, b, c = cplx(1 << rank), cplx(2), cplx(4)
    net = P.Network.from_arrays([list(range(rank)), [0], [1, 2]], [a, b, c], list(range(3, rank)), rank)
    want = np.einsum("ijkr,i,jk->r", a.astype(complex).reshape(2, 2, 2, -1), b, c.reshape(2, 2))
    return P.Plan(net, [(0, 1), (2, 3)], []), want


# 2^17 elements with the other leaves are just above 1 MiB
@pytest.mark.parametrize("rank", [4, 12, 16, 17, 18, 20])
def test_scratch_leaf_data(torch, rank):  # noqa: F811
    plan, want = _case(rank)
    banner(f"scratch call with 2^{rank} leaf elements")
    for _ in range(2):
        assert rel_l2(plan.execute_scratch([0]).cpu().numpy(), want) < 1e-6


def test_scratch_leaf_data_time(torch):  # noqa: F811
    """8 MiB: at most 1.5 times a small scratch call and a copy of as many bytes from
    pageable memory."""
    def best(f):
        t = []
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t) * 1e6
    large, small = _case(20)[0], _case(4)[0]
    out, out4 = large.new_output(), small.new_output()
    host = torch.randn(2 << 20, dtype=torch.float32)
    dev = torch.empty_like(host, device="cuda")
    us = best(lambda: large.execute_scratch([0], out))
    copy, call = best(lambda: dev.copy_(host)), best(lambda: small.execute_scratch([0], out4))
    banner(f"scratch call with 8 MiB of leaf data {us:.0f} us; copy {copy:.0f} us, small call {call:.0f} us")
    assert us < 1.5 * (copy + call)
