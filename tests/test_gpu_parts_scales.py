"""Two-part fp16 tiles over the whole range of operand scales: results that FP32
holds come out whatever the operands' largest numbers are, as on the split tiles.

The bound is that of the two-part tiles at ordinary scales (it goes by |x y| and by
max|x| max|y|, so it moves with the scales), plus FP32's smallest number, 2^-149,
once for every rounding below 2^-126: one per output, and one per chunk on the
split-K form. Where no output lies down there, the norm-wise error is the split
tile's too (1.05 for the spread of one draw)."""
import numpy as np
import pytest

from tests.gpu_util import banner, rel_l2
from tests.test_gpu_parts import U, _operands, _plan, _tiles, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# log2 of the operands' scales (their largest numbers are four times that): products
# of 2^-122 (normal) and 2^-134 (below 2^-126),
# numbers whose own scale factor FP32 does not hold, and large times small
@pytest.mark.parametrize("ea,eb", [(-64, -64), (-70, -70), (-122, 40), (40, -124), (-100, 90), (110, -120), (40, 60)])
@pytest.mark.parametrize("m,k,n,order", [(7, 10, 7, "rows"), (8, 11, 7, "mixed")])
def test_two_parts_at_any_scale(torch, m, k, n, order, ea, eb):  # noqa: F811
    import paper_2205_00393_amd as P
    a, b = _operands(m, k, n, "normal")
    a *= np.float32(2.0 ** ea)
    b *= np.float32(2.0 ** eb)
    plan, rows_cols = _plan(P, a, b, m, k, n, order)
    A, B = a.astype(np.complex128), b.astype(np.complex128)
    exact = A @ B.T
    S1, S2 = np.abs(A.real) @ np.abs(B.real).T, np.abs(A.imag) @ np.abs(B.imag).T
    S3 = (np.abs(A.real) + np.abs(A.imag)) @ (np.abs(B.real) + np.abs(B.imag)).T
    K = 1 << k
    floor = K * 2.0 ** -36 * np.abs(A).max() * np.abs(B).max()
    small = 2.0 ** -149 * (1 + K // 256)
    plan.set_step_kernel(0, "split_f16", 2, 3, 0, 1)
    base = rel_l2(rows_cols(plan.execute([0], mode="split_f16").cpu().numpy()), exact)
    ran = 0
    for name, cfg, swap in _tiles(P, plan, "split_f16", (4, 5)):
        L = 3 * K + 256
        got = rows_cols(plan.execute([0], mode="split_f16").cpu().numpy())
        d = got - exact
        r_re = float((np.abs(d.real) / (1.5 * (L + 4) * U * (S1 + S2) + 2 * floor + small)).max())
        r_im = float((np.abs(d.imag) / (1.5 * (L + 8) * U * (S1 + S2 + S3) + 6 * floor + small)).max())
        err = rel_l2(got, exact)
        banner(f"two parts ({m},{k},{n}) {order} 2^{ea} x 2^{eb} {name} swap {swap}: max err/bound re {r_re:.3f} "
               f"im {r_im:.3f}, rel {err:.2e} (split tile {base:.2e})")
        assert r_re <= 1.0 and r_im <= 1.0
        if ea + eb > -130:
            assert err <= 1.05 * base
        ran += 1
    assert ran == 4
