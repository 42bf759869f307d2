"""Large adjoint products on both sides of the line between operands read in place
and operands permuted first, with the output's rows as its upper bits (nothing of the
cotangent to permute) and at random bits, against the oracle's contraction.

The amplitudes are linear in the leaf, so the gradient of Re <cotangent, psi> is that
of psi with dU in place of U. Bound: as for the products with few columns, sums of at
most 2^13 products of random sign, 2^6.5 2^-24 a step, three steps each way: 5e-5."""
import numpy as np
import pytest

from tests.gpu_util import banner, rel_l2
from tests.test_gpu_parts import torch  # noqa: F401

pytestmark = pytest.mark.gpu


# (rows, sum, columns): 8 rows; 9 and 9; 9 rows, 8 columns; 10 and 10; 64 columns
@pytest.mark.parametrize("in_order", [True, False])
@pytest.mark.parametrize("m,n,k,sl", [(8, 6, 8, 6), (9, 5, 9, 4), (9, 6, 8, 5), (10, 5, 10, 2), (10, 7, 6, 7)])
def test_adjoint_routes(torch, m, n, k, sl, in_order):  # noqa: F811
    import paper_2205_00393_amd as P
    from oracle import gradients as gr, network as onw
    banner(f"adjoint: {m} row, {n} sum, {k} column bits x {1 << sl}, {'in order' if in_order else 'any order'}")
    rng = np.random.default_rng(100 * m + 10 * n + k)
    M, K, N = list(range(m)), list(range(m, m + k)), list(range(m + k, m + k + n))
    S = list(range(m + k + n, m + k + n + sl))
    ta = m + k + n + sl
    shuffled = lambda x: [x[i] for i in rng.permutation(len(x))]
    opens = M + N if in_order else shuffled(M + N)
    T, V = shuffled([ta if i == M[0] else i for i in M] + K + S), shuffled(N + K + S)
    rand = lambda ix: (rng.standard_normal([2] * len(ix)) + 1j * rng.standard_normal([2] * len(ix))).astype(np.complex64)
    data = [rand(T), np.eye(2, dtype=np.complex64), rand(V)]
    indices, path = [T, [M[0], ta], V], [(0, 1), (2, 3)]
    angles = rng.uniform(0, 3, 3)
    net = P.Network.from_arrays(indices, data, opens, ta + 1, param=[-1, 0, -1])
    plan = P.Plan(net, path, S)
    plan.bind(batch=1 << sl, grad=True)
    plan.set_params(torch.tensor(angles, dtype=torch.float64, device="cuda"))
    cot = rng.standard_normal(1 << (m + n)) + 1j * rng.standard_normal(1 << (m + n))
    g = plan.execute_grad(range(1 << sl), torch.tensor(cot, device="cuda")).cpu().numpy()

    def psi(x):
        net = onw.Network(indices, [data[0].astype(complex), x, data[2].astype(complex)], [-1] * 3, opens, ta + 1)
        return onw.contract_path(net, path)

    ref = [np.real(np.vdot(cot, psi(d))) for d in gr._u3_parts(*angles)[1]]
    assert rel_l2(g, ref) < 5e-5
