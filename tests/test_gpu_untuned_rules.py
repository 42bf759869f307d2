"""Untuned choices at the edges of their rules: the kernel that a plan takes for a
step by itself is not clearly slower than the one on the other side of the edge, and
gives the same result."""
import numpy as np
import pytest

from tests.gpu_util import banner, rel_l2
from tests.test_gpu_parts import torch  # noqa: F401

pytestmark = pytest.mark.gpu


# (m, k, n), slices, mode, the other kernel's kind and tile: split fp16 tiles of
# several slices, sums of 2^4 and 2^6, and of one slice; 64 columns and one tile a CU on
# three parts; narrow steps whose rows hold the output's lowest bit; rows of one element
# with and without maxima
@pytest.mark.parametrize("m,k,n,sl,mode,kind,cfg", [
    (10, 4, 8, 5, "split_f16", 2, 0), (11, 4, 7, 4, "split_f16", 2, 0), (9, 4, 8, 8, "split_f16", 2, 0),
    (8, 6, 7, 5, "split_f16", 2, 0), (15, 5, 8, 0, "split_f16", 2, 0), (18, 4, 6, 0, "c64", 1, 13),
    (15, 4, 7, 0, "c64", 1, 10), (17, 1, 6, 2, "c64", 3, 0), (11, 1, 6, 8, "split_bf16", 3, 0),
    (17, 2, 6, 2, "c64", 3, 0), (19, 0, 0, 0, "c64", 3, 0), (16, 0, 0, 2, "split_f16", 3, 0),
    (13, 1, 1, 5, "split_f16", 3, 0)])
def test_untuned_choice_is_not_slow(torch, m, k, n, sl, mode, kind, cfg):  # noqa: F811
    import paper_2205_00393_amd as P
    rng = np.random.default_rng(m + k + n)
    mi, ki, ni = list(range(m)), list(range(m, m + k)), list(range(m + k, m + k + n))
    si = list(range(m + k + n, m + k + n + sl))
    cplx = lambda s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)
    a, b = cplx(1 << (m + k + sl)), cplx(1 << (n + k + sl))
    # columns and rows in turn from the lowest bit, which is a row
    low = [x for p in zip(mi[::-1], ni[::-1]) for x in p]
    out = ([x for x in mi + ni if x not in low] + low[::-1])
    net = P.Network.from_arrays([si + mi + ki, si + ni + ki], [a, b], out, m + k + n + sl)
    plan = P.Plan(net, [(0, 1)], si)
    plan.bind(batch=1 << sl)
    step = plan.step(0)
    own = plan.step_kernel(0, mode)

    def best():
        return min(plan.profile_steps(0, mode)[0] for _ in range(20)) * 1e3

    mine, got = best(), plan.execute_range(0, 1 << sl, mode=mode)
    name, other = plan.step_kernel_name(0, mode), None
    for swap in (0, 1):
        try:
            plan.set_step_kernel(0, mode, kind, cfg, swap, 1)
        except P.LtnError:
            continue
        us = best()
        if other is None or us < other:
            other, want = us, plan.execute_range(0, 1 << sl, mode=mode)
    plan.set_step_kernel(0, mode, *own)
    mine = min(mine, best())  # before and after: the first launches may run at low clocks
    banner(f"({step['m']},{k},{step['n']}) x {1 << sl} {mode}: {name} (swap {own[2]}) {mine:.1f} us, "
           f"{P.kernel_name(kind, cfg, mode)} {other:.1f} us")
    assert rel_l2(got.cpu().numpy(), want.cpu().numpy()) < 1e-5
    assert mine < 1.1 * other + 1
