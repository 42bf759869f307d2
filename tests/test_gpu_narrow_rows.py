"""The narrow kernel's rows form with several rows per thread, element by element.

An output sums K = 2^k complex products in FP32: it errs by at most sqrt(2)
(2 K + 2) u of the sum over absolute values, u = 2^-24 (2 K real terms and a
rounded product each, in any order; 1 % for second-order terms).

Sizes: 256 blocks of 256 U rows (where U = 16 / max(K, N) rows per thread are
taken from) and half of that, slices of exactly one block and of half a block,
and slices whose blocks move on to the next slice. The output's lowest bits
belong to rows, to columns (pairs of columns are written together) or to both."""
import numpy as np
import pytest

from tests.gpu_util import banner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.mark.parametrize("m,k,n,sl", [(20, 0, 0, 0), (19, 0, 0, 0), (19, 1, 0, 0), (18, 2, 2, 0), (17, 2, 2, 0),
                                      (17, 3, 1, 0), (17, 1, 3, 0), (12, 0, 0, 8), (11, 0, 1, 8), (10, 0, 2, 8),
                                      (9, 3, 3, 3), (18, 0, 4, 0), (21, 0, 0, 3)])
@pytest.mark.parametrize("order", ["rows", "cols", "mixed"])
def test_rows_per_thread(torch, m, k, n, sl, order):
    import paper_2205_00393_amd as P
    if n == 0 and order != "rows":
        pytest.skip("no columns")
    banner(f"narrow rows ({m},{k},{n}) x {1 << sl} {order}")
    rng = np.random.default_rng(100 * m + 10 * k + n)
    S, M, K, N = 1 << sl, 1 << m, 1 << k, 1 << n
    a = (rng.standard_normal((S, M, K)) + 1j * rng.standard_normal((S, M, K))).astype(np.complex64)
    b = (rng.standard_normal((S, N, K)) + 1j * rng.standard_normal((S, N, K))).astype(np.complex64)
    mi, ki, ni = list(range(m)), list(range(m, m + k)), list(range(m + k, m + k + n))
    si = list(range(m + k + n, m + k + n + sl))
    out_ix = {"rows": ni + mi, "cols": mi + ni, "mixed": mi[:-2] + ni + mi[-2:]}[order]
    # slice ids take the sliced indices lowest bit first, leaves store them highest first
    net = P.Network.from_arrays([si[::-1] + mi + ki, si[::-1] + ni + ki], [a, b], out_ix, m + k + n + sl)
    plan = P.Plan(net, [(0, 1)], si)
    plan.bind(batch=S)
    swap = 0 if plan.step(0)["m"] == m and plan.step(0)["n"] == n else 1

    def placed(x):
        x = x.reshape([2] * (m + n))
        return np.transpose(x, [(mi + ni).index(i) for i in out_ix]).reshape(-1)

    ids = sorted({0, S // 2, S - 1})
    a64, b64 = a.astype(np.complex128), b.astype(np.complex128)
    for mode in ("c64", "split_f16"):
        plan.set_step_kernel(0, mode, 3, 1, swap, 1)
        # every slice runs in one launch; three are looked at one at a time
        total = plan.execute(list(range(S)), mode=mode).cpu().numpy()
        bound = np.sqrt(2) * 1.01 * (2 * K + 2) * 2.0 ** -24
        ref = placed(sum(a64[s] @ b64[s].T for s in range(S)))
        top = placed(sum(np.abs(a64[s]) @ np.abs(b64[s]).T for s in range(S)))
        assert np.all(np.abs(total - ref) <= bound * top)
        for s in ids:
            one = plan.execute([s], mode=mode).cpu().numpy()
            top = placed(np.abs(a64[s]) @ np.abs(b64[s]).T)
            assert np.all(np.abs(one - placed(a64[s] @ b64[s].T)) <= bound * top), s


@pytest.mark.parametrize("m,k,n,order,cfg", [(12, 2, 2, "cols", 1), (12, 2, 3, "rows", 1), (12, 2, 3, "cols", 0),
                                             (12, 2, 4, "cols", 1), (12, 5, 2, "rows", 0), (6, 2, 6, "rows", 0)])
def test_form_taken(torch, m, k, n, order, cfg):
    import paper_2205_00393_amd as P
    mi, ki, ni = list(range(m)), list(range(m, m + k)), list(range(m + k, m + k + n))
    net = P.Network.from_arrays([mi + ki, ni + ki], [np.ones(1 << (m + k)), np.ones(1 << (n + k))],
                                ni + mi if order == "rows" else mi + ni, m + k + n)
    plan = P.Plan(net, [(0, 1)], [])
    plan.bind(batch=1)
    assert plan.step_kernel(0, "c64")[:2] == (3, cfg)
