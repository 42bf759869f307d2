"""Infinities, NaN and very large numbers on the kernels with a way of their own:
three-part tiles (row-major, split-K and in place), runs of small steps, products
with few columns."""
import numpy as np
import pytest

from tests.gpu_util import banner, rel_l2
from tests.test_gpu_parts import _operands, _plan, _tiles, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", ["one", "rows", "all"])
@pytest.mark.parametrize("m,k,n,order", [(8, 5, 8, "cols"), (7, 12, 8, "mixed"), (8, 4, 8, "rows")])
def test_parts_large_and_non_finite(torch, m, k, n, order, what):  # noqa: F811
    """The three-part tiles give what the FP32 three-product tile gives, in the same
    places: results above 2^79 and operands above 2^104 (finite in FP32, not in the
    scaled parts) to rounding, infinities and NaN as such."""
    import paper_2205_00393_amd as P
    a, b = _operands(m, k, n, "normal")
    if what == "one":
        a[5, 3] = complex(2.0 ** 110, 2.0 ** 108)
        b[:, 3] *= np.float32(2.0 ** -40)
        a[9, 1] = complex(1, np.nan)
    elif what == "rows":
        a[::16] *= np.float32(2.0 ** 60)
        b[::32] *= np.float32(2.0 ** 50)
        a[1, 0], b[1, 0] = complex(np.inf, 1), complex(0.5, -np.inf)
    else:
        a *= np.float32(2.0 ** 60)
        b *= np.float32(2.0 ** 30)
        a[::2, 0] = np.nan
    plan, rows_cols = _plan(P, a, b, m, k, n, order)
    plan.set_step_kernel(0, "c64", 1, 10 if n >= 6 and m >= 7 else 13, 0, 1)
    want = rows_cols(plan.execute([0]).cpu().numpy())
    scale = np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64).T
    ran = 0
    for name, cfg, swap in _tiles(P, plan):
        banner(f"parts, {what} large or not finite, ({m},{k},{n}) {order} {name} swap {swap}")
        got = rows_cols(plan.execute([0]).cpu().numpy())
        for part in (np.real, np.imag):
            g, w = part(got), part(want)
            assert np.array_equal(np.isnan(g), np.isnan(w)), name
            inf = np.isinf(w)
            assert np.array_equal(g[inf], w[inf]) and np.array_equal(np.isinf(g), inf), name
            fin = np.isfinite(w)
            # both within K 2^-23 of the absolute sums, thrice for the three products
            assert (np.abs(g[fin] - w[fin]) <= 6 * (1 << k) * 2.0 ** -23 * scale[fin]).all()
        ran += 1
    assert ran >= 2


def test_parts_time_with_non_finite_operands(torch):  # noqa: F811
    """A step whose operands are all NaN takes its time once more on the FP32 matrix
    cores (1/16 of the rate of the six products of parts: 2.7 times as much), not the
    time of serial sums: below eight times the finite step's."""
    import paper_2205_00393_amd as P
    m, k, n = 12, 10, 10
    ms = {}
    for what in ("finite", "nan"):
        a, b = _operands(m, k, n, "normal")
        if what == "nan":
            a[:] = np.nan
        plan, _ = _plan(P, a, b, m, k, n, "cols")
        plan.set_step_kernel(0, "c64", 6, 0, 0, 1)
        plan.profile_steps(0, "c64")
        ms[what] = min(plan.profile_steps(0, "c64")[0] for _ in range(3))
    banner(f"(12,10,10) on three parts: {ms['finite']:.3f} ms finite, {ms['nan']:.3f} ms all NaN")
    assert ms["nan"] < 8 * ms["finite"]


# sums and rows at random address bits, either operand role; the last on the kernel
# for few columns
@pytest.mark.parametrize("m,k,n,sl", [(8, 7, 8, 7), (7, 8, 9, 7), (9, 6, 8, 8), (8, 2, 7, 6)])
def test_adjoint_of_large_rows(torch, m, k, n, sl):  # noqa: F811
    """Adjoint products of operands that lie in the forward step's order, a quarter of
    whose numbers are of 2^90: the gradient against the oracle's contraction. With an
    infinity among them nothing of it is finite."""
    import paper_2205_00393_amd as P
    from oracle import gradients as gr, network as onw
    banner(f"adjoint of large rows ({m},{k},{n}) x {1 << sl}")
    rng = np.random.default_rng(m + 10 * k + 100 * n)
    M, K, N = list(range(m)), list(range(m, m + k)), list(range(m + k, m + k + n))
    S = list(range(m + k + n, m + k + n + sl))
    ta = m + k + n + sl
    shuffled = lambda x: [x[i] for i in rng.permutation(len(x))]
    T = shuffled([ta if i == M[0] else i for i in M] + K + S)
    V = N[:2] + shuffled(N[2:] + K + S)
    rand = lambda ix: (rng.standard_normal([2] * len(ix)) + 1j * rng.standard_normal([2] * len(ix))).astype(np.complex64)
    data = [rand(T), np.eye(2, dtype=np.complex64), rand(V)]
    data[2][1, 0] *= np.float32(2.0 ** 90)
    indices, opens, path = [T, [M[0], ta], V], shuffled(M + N), [(0, 1), (2, 3)]
    angles = rng.uniform(0, 3, 3)
    cot = rng.standard_normal(1 << (m + n)) + 1j * rng.standard_normal(1 << (m + n))
    u, du = gr._u3_parts(*angles)

    def gradient(v):
        net = P.Network.from_arrays(indices, data[:2] + [v], opens, ta + 1, param=[-1, 0, -1])
        plan = P.Plan(net, path, S)
        plan.bind(batch=1 << sl, grad=True)
        plan.set_params(torch.tensor(angles, dtype=torch.float64, device="cuda"))
        return plan.execute_grad(range(1 << sl), torch.tensor(cot, device="cuda")).cpu().numpy()

    def psi(x):
        net = onw.Network(indices, [data[0].astype(complex), x, data[2].astype(complex)], [-1] * 3, opens, ta + 1)
        return onw.contract_path(net, path)

    ref = [np.real(np.vdot(cot, psi(d))) for d in du]
    g = gradient(data[2])
    assert rel_l2(g, ref) < 5e-5
    v = data[2].copy()
    v[(0,) * v.ndim] = complex(np.inf, 0)
    assert not np.isfinite(gradient(v)).any()


@pytest.mark.parametrize("value", [complex(np.inf, 0.5), complex(0.25, np.nan)])
def test_run_of_small_steps(torch, value):  # noqa: F811
    """A chain of small steps in one launch: an infinity or NaN reaches the
    outputs it has a path to and no others."""
    import paper_2205_00393_amd as P
    from oracle import network as onw
    rng = np.random.default_rng(17)
    # A[o, i, s] B[i, j, p] C[j, q, s]: o is A's own, so A[1, 0, 1] reaches o = 1 only
    o, p, q = [0, 1], [2, 3], [4, 5]
    i, j, s = [6, 7, 8], [9, 10], [11]
    indices, opens, path = [o + i + s, i + j + p, j + q + s], o + p + q, [(0, 1), (2, 3)]
    rand = lambda ix: (rng.standard_normal([2] * len(ix)) + 1j * rng.standard_normal([2] * len(ix))).astype(np.complex64)
    data = [rand(ix) for ix in indices]
    clean = onw.contract_path(onw.Network(indices, [x.astype(complex) for x in data], [-1] * 3, opens, 12), path)
    data[0][0, 1, 0, 0, 0, 1] = value
    net = P.Network.from_arrays(indices, data, opens, 12)
    banner(f"run of small steps with {value}")
    for mode in ("c64", "split_f16"):
        plan = P.Plan(net, path, s)
        plan.bind(batch=2)
        got = plan.execute([0, 1], mode=mode).cpu().numpy().reshape(4, -1)
        want = clean.reshape(4, -1)
        assert not np.isfinite(got[1]).any()
        rest = [0, 2, 3]
        assert np.isfinite(got[rest]).all() and rel_l2(got[rest], want[rest]) < 1e-5
