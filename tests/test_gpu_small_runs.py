"""Runs of small contraction steps (one block per slice) against the oracle,
element by element, on random networks with random leaves.

A step that sums K = 2^k complex products in FP32 errs by at most
sqrt(2) (2 K + 2) u of the same sum over absolute values, u = 2^-24, in any
order (2 K real terms and a rounded product each). The FP32 tiles, which wide steps with sums of 2 and 4 take, may use three
real products: 1.5 (2 K + 6) 2^-23 (S1 + S2 + S3) a part, and S1 + S2 + S3 is at most 3
times the sum over absolute values. Errors of the operands enter each product
once, so a tree's outputs err by at most the sum of its steps'
factors (1 % more for second-order terms) times the contraction of the
absolute values; the leaves are FP32 numbers and slices are summed in FP64.

Gradients are linear in the cotangent and compared with the state vector's; the
bound 1e-5 is a hundred roundings of 2^-23 in a row, of a relative error that
grows with the square root of the number of steps (about 100) if they are
random."""
import numpy as np
import pytest

from tests.gpu_util import banner, rel_l2
from tests.netgen import random_network

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def _greedy_path(indices):
    """Pairwise path that joins neighbours with the smallest result first."""
    tens = {i: set(ix) for i, ix in enumerate(indices)}
    path = []
    while len(tens) > 1:
        ids = sorted(tens)
        pairs = [(len(tens[a] ^ tens[b]), a, b) for i, a in enumerate(ids) for b in ids[i + 1:]
                 if tens[a] & tens[b]]
        pairs = pairs or [(len(tens[a] ^ tens[b]), a, b) for i, a in enumerate(ids) for b in ids[i + 1:]]
        _, a, b = min(pairs)
        tens[len(indices) + len(path)] = tens.pop(a) ^ tens.pop(b)
        path.append((a, b))
    return path


def _step_sums(indices, path, S):
    """k of every step."""
    tens = {i: set(ix) - set(S) for i, ix in enumerate(indices)}
    ks = []
    for a, b in path:
        ks.append(len(tens[a] & tens[b]))
        tens[len(indices) + len(ks) - 1] = tens.pop(a) ^ tens.pop(b)
    return ks


def _bound(ks, tiles=()):
    return 1.01 * np.sqrt(2) * (sum(2 * 2 ** k + 2 for k in ks) * 2.0 ** -24 +
                                sum(4.5 * (2 * 2 ** k + 6) for k in tiles) * 2.0 ** -23)


def _check(torch, indices, data, opens, n_indices, path, S, batch, mode, force=None, tiles=()):
    import paper_2205_00393_amd as P
    from oracle import network as onw
    onet = onw.Network(indices, [d.astype(np.complex128) for d in data], [-1] * len(indices), opens, n_indices)
    anet = onw.Network(indices, [np.abs(d) + 0j for d in onet.data], onet.param, opens, n_indices)
    plan = P.Plan(P.Network.from_arrays(indices, data, opens, n_indices), path, S)
    plan.bind(batch=batch)
    plan.set_fusion(False)
    if force is not None:
        for s in range(plan.info()["n_steps"]):
            plan.set_step_kernel(s, mode, 0, 0, 0, force)
    ids = list(range(1 << len(S)))[::-1]  # the last batch is ragged
    ref, top = onw.sliced_sum(onet, path, S, ids), onw.sliced_sum(anet, path, S, ids).real
    for _ in range(3):  # graph replays
        out = plan.execute(ids, mode=mode)
        torch.cuda.synchronize()
        err = np.abs(out.cpu().numpy() - ref)
        bound = _bound(_step_sums(indices, path, S), tiles) * top
        assert np.all(err <= bound), float((err / bound).max())
    return plan


# leaves, closed indices, open indices: many tiny steps; tensors past 64 elements
# as inputs and between steps; sums of 2^6 and more
@pytest.mark.parametrize("L,E,n_open", [(3, 2, 2), (40, 60, 4), (12, 40, 3), (8, 44, 2), (130, 140, 5)])
@pytest.mark.parametrize("batch,mode", [(1, "c64"), (3, "c64"), (8, "split_f16")])
def test_runs_of_small_steps(torch, L, E, n_open, batch, mode):
    banner(f"runs L={L} E={E} batch={batch} {mode}")
    indices, n, opens = random_network(L + E, L, E, n_open)
    rng = np.random.default_rng(L)
    data = [(rng.standard_normal([2] * len(ix)) + 1j * rng.standard_normal([2] * len(ix))).astype(np.complex64)
            for ix in indices]
    S = [opens[0], 0, 1]
    if L == 3:
        S = [0, opens[1]]
    _check(torch, indices, data, opens, n, _greedy_path(indices), S, batch, mode,
           force=8 if E > 3 * L else None)


@pytest.mark.parametrize("tk", [1, 8, 64])
def test_runs_with_forced_generic_steps(torch, tk):
    """Every step generic, also those too large for a run, which then ends."""
    banner(f"forced generic tk={tk}")
    indices, n, opens = random_network(5, 14, 52, 6)
    rng = np.random.default_rng(6)
    data = [(rng.standard_normal([2] * len(ix)) + 1j * rng.standard_normal([2] * len(ix))).astype(np.complex64)
            for ix in indices]
    path = _greedy_path(indices)
    _check(torch, indices, data, opens, n, path, [opens[2], 3, 4], 3, "c64", force=tk)


@pytest.mark.parametrize("k", [1, 2])
@pytest.mark.parametrize("mode", ["c64", "split_f16", "split_bf16"])
def test_wide_short_sums(torch, k, mode):
    """Sums of 2 and 4 with many outputs take FP32 tiles by themselves, and the
    generic kernel on plans bound for a complex64 gradient."""
    import paper_2205_00393_amd as P
    m = n = 8
    S, opens = [m + n + k, m + n + k + 1], list(range(m + n))
    indices = [list(range(m)) + [m + n + j for j in range(k)] + [S[0]],
               list(range(m, m + n)) + [m + n + j for j in range(k)] + [S[1]], [S[0]], [S[1]]]
    rng = np.random.default_rng(k)
    data = [(rng.standard_normal([2] * len(ix)) + 1j * rng.standard_normal([2] * len(ix))).astype(np.complex64)
            for ix in indices]
    banner(f"wide short sums k={k} {mode}")
    plan = _check(torch, indices, data, opens, m + n + k + 2, [(0, 1), (2, 4), (3, 5)], S, 4, mode, tiles=[k])
    assert plan.step_kernel(0, mode)[0] == 1
    if mode == "c64":
        plan.bind(batch=4, grad=True)
        assert plan.step_kernel(0, mode)[0] == 0


@pytest.mark.parametrize("batch", [1, 3, 32])
def test_adjoint_runs(torch, batch):
    import paper_2205_00393_amd as P
    from oracle import gradients as gr, statevector as sv
    from workload import make_rqc, Workload
    c = make_rqc(3, 3, 5, u3_seed=9)
    w = Workload("u3_9", c, tuple(range(7)), {7: 1, 8: 0}, None, True, None)
    net = P.Network.from_circuit(c, w.open_qubits, w.closed_bits)
    indices = net.indices
    S = [indices[0][0], indices[3][0], net.open_ids[1]]
    S = list(dict.fromkeys(S))
    plan = P.Plan(net, _greedy_path(indices), S)
    plan.bind(batch=batch, grad=True)
    plan.set_params(torch.tensor(c.angles(), dtype=torch.float64, device="cuda"))
    rng = np.random.default_rng(10)
    cot = rng.standard_normal(128) + 1j * rng.standard_normal(128)
    banner(f"adjoint runs batch={batch}")
    pick = lambda phi: np.asarray(phi).reshape([2] * 9)[..., 1, 0].reshape(-1)
    which = range(len(c.angles()))
    ref = [float(np.real(np.vdot(cot, 0.5 * pick(sv.final_state(c, gr._with_angle(c, i, np.pi))))))
           for i in which]
    for _ in range(3):
        out = plan.new_output()
        g = plan.execute_grad(range(1 << len(S)), torch.tensor(cot, device="cuda"), out)
        torch.cuda.synchronize()
        assert rel_l2(out.cpu().numpy(), pick(sv.final_state(c))) < 1e-5
        assert rel_l2(g.cpu().numpy(), ref) < 1e-5
