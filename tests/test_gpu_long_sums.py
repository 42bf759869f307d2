"""Sums of 2^14 and more on tiles of parts: the untuned choice and the tuner's are the
split-K form where it fits, whose error is below the full tile's at the same time."""
import pytest

from tests.gpu_util import banner
from tests.test_gpu_parts import torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,full", [("c64", 0), ("split_f16", 4)])
def test_long_sums_are_split(torch, mode, full):  # noqa: F811
    import paper_2205_00393_amd as P
    m, k, n = 11, 14, 11  # with two slices, two full tiles per CU
    g = torch.Generator().manual_seed(4)
    a = torch.randn(2, 1 << m, 1 << k, dtype=torch.complex64, generator=g)
    b = torch.randn(2, 1 << n, 1 << k, dtype=torch.complex64, generator=g)
    mi, ki, ni, si = list(range(m)), list(range(m, m + k)), list(range(m + k, m + k + n)), [m + k + n]
    net = P.Network.from_arrays([si + mi + ki, si + ni + ki], [a.numpy(), b.numpy()], mi + ni, m + k + n + 1)
    plan = P.Plan(net, [(0, 1)], si)
    plan.bind(batch=2)
    exact = torch.zeros(1 << m, 1 << n, dtype=torch.complex128, device="cuda")
    for x, y in zip(a, b):
        exact += x.cuda().to(torch.complex128) @ y.cuda().to(torch.complex128).T.contiguous()

    def error():
        return float((plan.execute_range(0, 2, mode=mode).reshape(exact.shape) - exact).norm() / exact.norm())

    errs = {}
    for what in ("untuned", "tuned"):
        if what == "tuned":
            plan.autotune(mode)
        name = plan.step_kernel_name(0, mode)
        errs[what] = error()
        banner(f"({m},{k},{n}) x 2 {mode} {what}: {name}, error {errs[what]:.2e}")
        assert name.startswith("splitk_")
    plan.set_step_kernel(0, mode, 6, full, 0, 1)
    banner(f"full tile: error {error():.2e}")
    assert max(errs.values()) < error()
