"""One tuning file for plans of different bindings, and files whose entries do not
fit. The complex64 forward of a plan bound for gradients keeps the FP32 tiles (its
loss may magnify a change of rounding); other plans take the three-part tiles where
they are faster, which on (10,10,10) x 16 they are by half."""
import json

import numpy as np
import pytest

from tests.gpu_util import banner, rel_l2

pytestmark = pytest.mark.gpu
M = K = N = 10
BATCH = 16


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def _network(P):
    """T behind a leaf of angles, then T V over K indices, in 2^4 slices."""
    rng = np.random.default_rng(8)
    mi, ki = list(range(M)), list(range(M, M + K))
    ni, si, t = list(range(M + K, M + K + N)), list(range(M + K + N, M + K + N + 4)), M + K + N + 4
    cplx = lambda n: ((rng.standard_normal([2] * n) + 1j * rng.standard_normal([2] * n)) / 8).astype(np.complex64)
    data = [cplx(M + K + 4), np.eye(2, dtype=np.complex64), cplx(K + N + 4)]
    indices = [si + [t] + mi[1:] + ki, [mi[0], t], ni + ki + si]
    net = P.Network.from_arrays(indices, data, mi + ni, t + 1, param=[-1, 0, -1])
    return net, [(0, 1), (2, 3)], si


def _plan(P, torch, grad, cache):
    net, path, si = _network(P)
    plan = P.Plan(net, path, si)
    assert plan.bind(batch=BATCH, grad=grad) == BATCH
    plan.set_params(torch.tensor([0.3, 0.7, -0.4], dtype=torch.float64, device="cuda"))
    plan.autotune("c64", cache)
    step = next(i for i, s in enumerate(plan.steps()) if (s["m"], s["k"], s["n"]) == (M, K, N))
    return plan, step


@pytest.mark.parametrize("first", ["amplitudes", "gradient"])
def test_bindings_share_a_file(torch, tmp_path, first):
    import paper_2205_00393_amd as P
    cache = str(tmp_path / "tune.json")
    kinds = {}
    for grad in ((False, True) if first == "amplitudes" else (True, False)):
        plan, step = _plan(P, torch, grad, cache)
        kinds[grad] = plan.step_kernel(step)[0]
        banner(f"{first} first: {'gradient' if grad else 'amplitude'} plan takes {plan.step_kernel_name(step)}")
    assert kinds[False] == 6
    assert kinds[True] in (1, 5)
    # both read it again
    written = json.load(open(cache))
    for grad in (False, True):
        plan, step = _plan(P, torch, grad, cache)
        assert plan.step_kernel(step)[0] == kinds[grad]
    assert json.load(open(cache)) == written


# a tile of another mode, none, a tile larger than the step, no lane count
@pytest.mark.parametrize("entry", [[6004, 0], [1999, 0], [2000, 0], [9000, 1], [-5, 0], [4000, 0], [6002, 7]])
def test_entries_that_do_not_fit(torch, tmp_path, entry):
    """Each is passed over and its step tuned anew."""
    import paper_2205_00393_amd as P
    cache = str(tmp_path / "tune.json")
    rng = np.random.default_rng(3)
    a = (rng.standard_normal((128, 32)) + 1j * rng.standard_normal((128, 32))).astype(np.complex64)
    b = (rng.standard_normal((32, 32)) + 1j * rng.standard_normal((32, 32))).astype(np.complex64)
    mi, ki, ni = list(range(7)), list(range(7, 12)), list(range(12, 17))
    net = P.Network.from_arrays([mi + ki, ni + ki], [a, b], mi + ni, 17)

    def tuned():
        plan = P.Plan(net, [(0, 1)], [])
        plan.bind(batch=1)
        plan.autotune("c64", cache)
        return plan
    tuned()
    keys = list(json.load(open(cache)))
    json.dump({k: entry for k in keys}, open(cache, "w"))
    banner(f"tuning file with {entry} for {keys}")
    plan = tuned()
    kind, cfg, swap, tk = plan.step_kernel(0)
    plan.set_step_kernel(0, "c64", kind, cfg, swap, tk)  # refuses what does not fit
    got = plan.execute([0]).cpu().numpy().reshape(128, 32)
    assert rel_l2(got, a.astype(complex) @ b.T.astype(complex)) < 1e-5
    assert all(v != entry for v in json.load(open(cache)).values())
