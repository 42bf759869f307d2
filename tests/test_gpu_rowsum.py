"""Adjoint products with few columns, read in place (both operands in the forward
step's order), against the oracle's contraction with the derivative of a leaf.

T and V, each behind a u3 leaf, are contracted over k indices into m + n open
indices in random order, for slices that differ in every element of T and V; the
adjoint of that step has sums of 2^n and 2^m, columns 2^k (or 2^m, 2^n where k is
above 4), and rows and sums at random address bits. The amplitudes are linear in
each u3, so the gradient of Re <cotangent, psi> is that of psi with dU in place of
U. Bound: sums of at most 2^13 products of random sign gather rounding errors
like a random walk, 2^6.5 2^-24 a step, three steps each way: below 5e-5."""
import numpy as np
import pytest

from tests.gpu_util import banner, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


# sums shorter than a tile, of one tile, of many; 16 to 2^11 rows a tile; 1 to 16
# columns; rows from the other operand (k > 4); batches too small for the kernel
@pytest.mark.parametrize("m,k,n,sl", [(8, 2, 7, 6), (6, 4, 6, 8), (9, 1, 4, 8), (12, 3, 1, 4), (1, 3, 12, 4),
                                      (3, 9, 4, 6), (4, 11, 1, 5), (13, 0, 3, 5), (2, 2, 11, 6), (7, 2, 7, 1),
                                      (5, 4, 9, 5), (10, 0, 10, 3)])
def test_adjoint_products_in_place(torch, m, k, n, sl):
    import paper_2205_00393_amd as P
    from oracle import gradients as gr, network as onw
    banner(f"adjoint in place ({m},{k},{n}) x {1 << sl}")
    rng = np.random.default_rng(1000 * m + 100 * k + n)
    M, K, N = list(range(m)), list(range(m, m + k)), list(range(m + k, m + k + n))
    S = list(range(m + k + n, m + k + n + sl))
    ta, tb = m + k + n + sl, m + k + n + sl + 1
    shuffled = lambda x: [x[i] for i in rng.permutation(len(x))]
    T = shuffled([ta if i == M[0] else i for i in M] + K + S)
    V = shuffled([tb if i == N[0] else i for i in N] + K + S)
    indices = [T, [M[0], ta], V, [N[0], tb]]
    opens = shuffled(M + N)
    rand = lambda ix: (rng.standard_normal([2] * len(ix)) + 1j * rng.standard_normal([2] * len(ix))).astype(np.complex64)
    data = [rand(T), np.eye(2, dtype=np.complex64), rand(V), np.eye(2, dtype=np.complex64)]
    angles = rng.uniform(0, 3, 6)
    net = P.Network.from_arrays(indices, data, opens, tb + 1, param=[-1, 0, -1, 1])
    path = [(0, 1), (2, 3), (4, 5)]
    plan = P.Plan(net, path, S)
    plan.bind(batch=1 << sl, grad=True)
    plan.set_params(torch.tensor(angles, dtype=torch.float64, device="cuda"))
    cot = rng.standard_normal(1 << (m + n)) + 1j * rng.standard_normal(1 << (m + n))
    out = plan.new_output()
    g = plan.execute_grad(range(1 << sl), torch.tensor(cot, device="cuda"), out)
    torch.cuda.synchronize()

    (ua, da), (ub, db) = gr._u3_parts(*angles[:3]), gr._u3_parts(*angles[3:])

    def psi(x, y):
        # all slices at once: the sum over them is a contraction over S
        net = onw.Network(indices, [data[0].astype(complex), x, data[2].astype(complex), y], [-1] * 4, opens, tb + 1)
        return onw.contract_path(net, path)

    assert rel_l2(out.cpu().numpy(), psi(ua, ub)) < 5e-5
    ref = [np.real(np.vdot(cot, psi(d, ub))) for d in da] + [np.real(np.vdot(cot, psi(ua, d))) for d in db]
    assert rel_l2(g.cpu().numpy(), ref) < 5e-5
