"""Complex64 GEMM tiles on three bf16 parts (kernel kind 6) against their
rounding bound, element by element.

A one-step network C = A B runs on every tile that fits, in both operand
roles, with the output's low bits from rows, columns or both. With three real
products P1 = Ar Br, P2 = Ai Bi, P3 = (Ar + Ai)(Br + Bi) of FP32 operands:

* the parts of an operand sum to it exactly; the products of parts that are
  left out are below 2^-26 of |x y| and those taken add up to at most
  1 + 2^-7 times it;
* each real product of K terms is a sum of 6 K products of parts in FP32: at
  most 6 K u of the absolute sum, u = 2^-23 (as in the bound of the FP32
  tiles, so as not to assume round-to-nearest inside the matrix core); split-K
  adds one term per chunk (at most 2^8);
* the rest is as on the three-product FP32 tiles: rounded operand sums (2 u
  S3) and subtractions.

With S1 = |Ar||Br|, S2 = |Ai||Bi|, S3 = (|Ar| + |Ai|)(|Br| + |Bi|) and L =
6 K (+ 256), a factor 1.5 for second-order terms:

    |Re| <= 1.5 (L + 2) u (S1 + S2),   |Im| <= 1.5 (L + 6) u (S1 + S2 + S3).

Operands: normal; "tiny" (rows of A scaled by 2^-100 and 2^-118, columns of B
by 2^100: unscaled, their last parts are below bf16's smallest number);
"sparse" (whole k-tiles of zeros). The norm-wise error must also stay below the FP32
three-product tile's on normal operands."""
import numpy as np
import pytest

from tests.gpu_util import banner, rel_l2

pytestmark = pytest.mark.gpu

U = 2.0 ** -23


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def _operands(m, k, n, kind):
    rng = np.random.default_rng(700 + 10 * k + m)
    M, K, N = 1 << m, 1 << k, 1 << n
    a = rng.standard_normal((M, K)) + 1j * rng.standard_normal((M, K))
    b = rng.standard_normal((N, K)) + 1j * rng.standard_normal((N, K))
    if kind == "tiny":
        a[::3] *= 2.0 ** -100
        a[1::3] *= 2.0 ** -118
        b *= 2.0 ** 100
    if kind == "sparse":
        a[:, : K // 2] = 0
        b[::2, K // 4:] = 0
    return a.astype(np.complex64), b.astype(np.complex64)


def _plan(P, a, b, m, k, n, order):
    """One-step plan; order of the output's indices, lowest bits last: rows
    lowest, columns lowest, or interleaved."""
    mi, ki, ni = list(range(m)), list(range(m, m + k)), list(range(m + k, m + k + n))
    out = {"rows": ni + mi, "cols": mi + ni,
           "mixed": [x for p in zip(mi, ni) for x in p] + mi[min(m, n):] + ni[min(m, n):]}[order]
    net = P.Network.from_arrays([mi + ki, ni + ki], [a, b], out, m + k + n)
    plan = P.Plan(net, [(0, 1)], [])
    plan.bind(batch=1)
    pos = {x: j for j, x in enumerate(out)}
    axes = [pos[x] for x in mi + ni]  # output axes in (rows, columns) order

    def rows_cols(v):
        return v.reshape([2] * (m + n)).transpose(axes).reshape(1 << m, 1 << n)
    return plan, rows_cols


def _tiles(P, plan, mode="c64", cfgs=range(4)):
    for cfg in cfgs:
        for swap in (0, 1):
            try:
                plan.set_step_kernel(0, mode, 6, cfg, swap, 1)
            except P.LtnError:
                continue
            yield P.kernel_name(6, cfg, mode), cfg, swap


@pytest.mark.parametrize("operands", ["normal", "tiny", "sparse"])
@pytest.mark.parametrize("m,k,n,order", [(7, 4, 7, "rows"), (8, 5, 6, "cols"), (7, 6, 8, "mixed"), (7, 10, 7, "rows"),
                                         (6, 11, 8, "mixed")])
def test_parts_within_analytic_bound(torch, m, k, n, order, operands):
    import paper_2205_00393_amd as P
    a, b = _operands(m, k, n, operands)
    plan, rows_cols = _plan(P, a, b, m, k, n, order)
    A, B = a.astype(np.complex128), b.astype(np.complex128)
    exact = A @ B.T
    S1, S2 = np.abs(A.real) @ np.abs(B.real).T, np.abs(A.imag) @ np.abs(B.imag).T
    S3 = (np.abs(A.real) + np.abs(A.imag)) @ (np.abs(B.real) + np.abs(B.imag)).T
    ran = 0
    for name, cfg, swap in _tiles(P, plan):
        L = 6 * (1 << k) + (256 if name.startswith("splitk") else 0)
        got = rows_cols(plan.execute([0]).cpu().numpy())
        d = got - exact
        tiny = 2.0 ** -149
        r_re = float((np.abs(d.real) / (1.5 * (L + 2) * U * (S1 + S2) + tiny)).max())
        r_im = float((np.abs(d.imag) / (1.5 * (L + 6) * U * (S1 + S2 + S3) + tiny)).max())
        err = rel_l2(got, exact)
        banner(f"parts ({m},{k},{n}) {order} {operands} {name} swap {swap}: max err/bound re {r_re:.3f} im {r_im:.3f}, "
               f"rel {err:.2e}")
        assert r_re <= 1.0 and r_im <= 1.0
        if operands == "normal" and not name.startswith("splitk") and min(m, n) >= 6:
            for c in (10, 13):  # the FP32 three-product tiles 128 x 64 and 64 x 64
                try:
                    plan.set_step_kernel(0, "c64", 1, c, swap, 1)
                except P.LtnError:
                    continue
                assert err <= rel_l2(rows_cols(plan.execute([0]).cpu().numpy()), exact)
                break
        ran += 1
    assert ran >= 1


def test_parts_non_finite_operands(torch):
    """Infinities, NaN and numbers that overflow in the scaled parts give what
    the FP32 three-product tile gives, in the same places."""
    import paper_2205_00393_amd as P
    m, k, n = 7, 5, 7
    a, b = _operands(m, k, n, "normal")
    a[3, 7] = complex(np.inf, 1)
    a[77, 31] = complex(0.5, np.nan)
    a[20, 0] = complex(3.4e38, 0)
    a[20, 1:] = 0
    b[:, 0] *= 2.0 ** -10
    plan, rows_cols = _plan(P, a, b, m, k, n, "cols")
    plan.set_step_kernel(0, "c64", 1, 10, 0, 1)
    want = rows_cols(plan.execute([0]).cpu().numpy())
    assert np.isfinite(want[20]).all() and not np.isfinite(want[3]).all()
    for name, cfg, swap in _tiles(P, plan):
        got = rows_cols(plan.execute([0]).cpu().numpy())
        for part in (np.real, np.imag):
            g, w = part(got), part(want)
            assert np.array_equal(np.isnan(g), np.isnan(w)), name
            inf = np.isinf(w)
            assert np.array_equal(g[inf], w[inf]) and np.array_equal(np.isinf(g), inf), name
            fin = np.isfinite(w)
            assert np.abs(g[fin] - w[fin]).max() <= 1e-5 * np.abs(w[fin]).max()


@pytest.mark.parametrize("mode", ["split_f16", "split_bf16"])
def test_parts_write_split_layout(torch, mode):
    """In the split modes a full three-part tile writes its output in the
    split layout for a split consumer: T = A B, then C = T^T D on a split
    tile, with T's low bits from either operand."""
    import paper_2205_00393_amd as P
    J, K, M, N = 8, 6, 7, 6
    rng = np.random.default_rng(41)
    cplx = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)
    a, b, d = cplx(1 << J, 1 << K), cplx(1 << K, 1 << M), cplx(1 << J, 1 << N)
    ji, ki = list(range(J)), list(range(J, J + K))
    mi, ni = list(range(J + K, J + K + M)), list(range(J + K + M, J + K + M + N))
    net = P.Network.from_arrays([ji + ki, ki + mi, ji + ni], [a, b, d], mi + ni, J + K + M + N)
    plan = P.Plan(net, [(0, 1), (2, 3)], [])
    plan.bind(batch=1)
    exact = ((a.astype(np.complex128) @ b).T @ d).reshape(-1)
    plan.set_step_kernel(1, mode, 2, 3, 0 if plan.step(1)["m"] >= 6 else 1, 1)
    ran = 0
    for name, cfg, swap in _tiles(P, plan, mode):
        err = rel_l2(plan.execute([0], mode=mode).cpu().numpy(), exact)
        banner(f"parts -> split {mode} {name} swap {swap}: rel err {err:.2e}")
        # bf16 hi + lo keeps 2^-17 of each operand, fp16 2^-22
        assert err < (3e-6 if mode == "split_f16" else 3e-5)
        ran += 1
    assert ran >= 2


@pytest.mark.parametrize("operands", ["normal", "wide", "sparse"])
@pytest.mark.parametrize("m,k,n,order", [(7, 10, 7, "rows"), (8, 10, 7, "cols"), (7, 12, 8, "mixed")])
def test_two_parts_within_analytic_bound(torch, m, k, n, order, operands):
    """Split fp16 mode: tiles on two scaled fp16 parts, three real products.
    x = h + l + e with |e| <= 2^-24 |x| + 2^-38 max|x| (l's own rounding; fp16's
    smallest number under the scale that takes the maximum to [2^13, 2^14)), and
    l l' <= 2^-24 |x y| left out: 3.1 2^-24 |x y| + 2^-36 max|x| max|y| per
    product; 3 K products of parts in FP32 per real product. The norm-wise error
    on normal operands is the split tiles' (1.05 for the spread of one draw).
    "wide": magnitudes over 2^16 by row, 2^8 by column."""
    import paper_2205_00393_amd as P
    a, b = _operands(m, k, n, operands)
    if operands == "wide":
        rng = np.random.default_rng(5)
        a *= (2.0 ** -rng.integers(0, 17, size=(1 << m, 1)) * 2.0 ** -20).astype(np.float32)
        b *= (2.0 ** -rng.integers(0, 9, size=(1 << n, 1))).astype(np.float32)
    plan, rows_cols = _plan(P, a, b, m, k, n, order)
    A, B = a.astype(np.complex128), b.astype(np.complex128)
    exact = A @ B.T
    S1, S2 = np.abs(A.real) @ np.abs(B.real).T, np.abs(A.imag) @ np.abs(B.imag).T
    S3 = (np.abs(A.real) + np.abs(A.imag)) @ (np.abs(B.real) + np.abs(B.imag)).T
    K = 1 << k
    floor = K * 2.0 ** -36 * np.abs(A).max() * np.abs(B).max()
    plan.set_step_kernel(0, "split_f16", 2, 3, 0, 1)
    base = rel_l2(rows_cols(plan.execute([0], mode="split_f16").cpu().numpy()), exact)
    ran = 0
    for name, cfg, swap in _tiles(P, plan, "split_f16", (4, 5)):
        L = 3 * K + 256
        d = rows_cols(plan.execute([0], mode="split_f16").cpu().numpy()) - exact
        r_re = float((np.abs(d.real) / (1.5 * (L + 4) * U * (S1 + S2) + 2 * floor)).max())
        r_im = float((np.abs(d.imag) / (1.5 * (L + 8) * U * (S1 + S2 + S3) + 6 * floor)).max())
        err = float(np.linalg.norm(d) / np.linalg.norm(exact))
        banner(f"two parts ({m},{k},{n}) {order} {operands} {name} swap {swap}: max err/bound re {r_re:.3f} "
               f"im {r_im:.3f}, rel {err:.2e} (split tile {base:.2e})")
        assert r_re <= 1.0 and r_im <= 1.0
        if operands == "normal":
            assert err <= 1.05 * base
        ran += 1
    assert ran == 4


def test_two_parts_only_where_they_are_as_exact(torch):
    """Sums below 2^10 and the other modes refuse the two-part tiles."""
    import paper_2205_00393_amd as P
    for k, mode in ((9, "split_f16"), (10, "split_bf16"), (10, "c64")):
        a, b = _operands(7, k, 7, "normal")
        plan, _ = _plan(P, a, b, 7, k, 7, "rows")
        assert not list(_tiles(P, plan, mode, (4, 5)))
        assert plan.execute([0], mode=mode).isfinite().all()
