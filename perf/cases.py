"""What a program does with this framework, as cases that can be timed.

Four kinds of call, each over the range in which it is used:

* ``amps``: amplitudes of a random circuit, contracted slice by slice on a
  bound plan (``Plan.execute`` / ``Plan.execute_range``), in the three
  precision modes, on greedy and on reconfigured paths, with and without the
  autotuner. The program keeps the amplitudes as complex64, the accuracy
  that they have.
* ``scratch``: the same without a workspace (``Plan.execute_scratch``).
* ``grad``: forward and backward of a loss over bitstring amplitudes with
  respect to float32 rotation angles (``Amplitudes``).
* ``permute``: bit permutations of batches of complex64 tensors.

A seed draws the circuit's gates, the closed bits, the bitstrings, the angles
and the tensors. It does not change the network's structure, so a program
plans (and tunes) a circuit shape once and keeps the path.
"""
import functools
import math
import os
import tempfile

import numpy as np
import torch

import paper_2205_00393_amd as P
from paper_2205_00393_amd.autograd import Amplitudes
from workload import make_workload

_TUNING = tempfile.mkdtemp(prefix="ltn_tuning_")  # autotuner cache of this process

_AMPS = dict(kind="amps", rows=4, cols=5, cycles=10, n_open=6, max_rank=12, mode="c64", reconf_k=0,
             trials=16, slices=0, batch=0, tune=False)
_GRAD = dict(kind="grad", rows=4, cols=5, cycles=12, bitstrings=256, tune=False)


def listed():
    return [
        # one closed amplitude of a small circuit: nothing but launches and latency
        dict(_AMPS, name="amplitude 12q c64", rows=3, cols=4, cycles=8, n_open=0, max_rank=-1, batch=1),
        # the same in a serving loop that may not allocate or bind anything
        dict(_AMPS, name="amplitude 12q scratch", kind="scratch", rows=3, cols=4, cycles=8, n_open=0, max_rank=-1),
        # 64 correlated amplitudes of 20 qubits, cut into many small slices
        dict(_AMPS, name="slices 20q c64", max_rank=12),
        # a deeper circuit with wider tensors, the mixed-precision mode, a ragged last batch
        dict(_AMPS, name="slices 20q split_f16", cycles=12, max_rank=14, mode="split_f16", batch=96),
        # the 30-qubit workload on its greedy path, all slices: large complex GEMMs
        dict(_AMPS, name="slices 30q c64", rows=5, cols=6, cycles=14, max_rank=26, batch=16),
        # the same in the fastest mode, tuned as a long run is
        dict(_AMPS, name="slices 30q split_bf16 tuned", rows=5, cols=6, cycles=14, max_rank=26, batch=16,
             mode="split_bf16", tune=True),
        # the 30-qubit workload on a reconfigured path that needs no slicing: narrow steps
        dict(_AMPS, name="one pass 30q c64 tuned", rows=5, cols=6, cycles=14, max_rank=26, reconf_k=10, batch=1,
             tune=True),
        # the same untuned in split fp16
        dict(_AMPS, name="one pass 30q split_f16", rows=5, cols=6, cycles=14, max_rank=26, reconf_k=10, batch=1,
             mode="split_f16"),
        # one slice of the 53-qubit workload, 2^20 amplitudes: the largest work on one GPU
        dict(_AMPS, name="slice 53q split_f16", rows=6, cols=9, cycles=20, n_open=20, max_rank=30, batch=1,
             slices=1, mode="split_f16"),
        # training of rotation angles: loss over 256 bitstrings, forward and backward
        dict(_GRAD, name="gradient 20q tuned", tune=True),
        # reordering the indices of two large tensors
        dict(kind="permute", name="permute 2 x 2^26", rank=26, batch=2, perm_seed=1),
        # many small tensors, a batch that fills no round number of blocks
        dict(kind="permute", name="permute 37 x 2^13", rank=13, batch=37, perm_seed=2),
    ]


def draw(rng):
    kind = rng.choice(["amps", "amps", "amps", "scratch", "grad", "permute"])
    if kind == "permute":
        rank = rng.randint(4, 27)
        most = min(2000, (1 << 27) >> rank)
        return dict(kind="permute", rank=rank, batch=int(round(math.exp(rng.uniform(0, math.log(most))))),
                    perm_seed=rng.randint(3, 999))
    # work spread evenly over its logarithm: the circuit of a few that comes nearest to a drawn amount
    aim = rng.uniform(15, 22 if kind == "scratch" else 36 if kind == "grad" else 42)
    best, left = None, 12
    while left or best is None:
        left = max(0, left - 1)
        if kind == "grad":
            c = dict(_GRAD, rows=rng.randint(3, 4), cols=rng.randint(3, 5), cycles=rng.randint(4, 12),
                     bitstrings=int(round(math.exp(rng.uniform(0, math.log(256))))), tune=rng.random() < 0.25)
        else:
            c = dict(_AMPS, kind=kind, rows=rng.randint(3, 5), cols=rng.randint(4, 6), cycles=rng.randint(6, 14),
                     n_open=rng.randint(0, 10), max_rank=rng.choice([-1, 12, 16, 20, 24, 26]),
                     mode=rng.choice(["c64", "split_f16", "split_bf16"]), reconf_k=rng.choice([0, 0, 8]),
                     trials=rng.randint(1, 8), tune=kind == "amps" and rng.random() < 0.25)
        path, sliced = _planned(*_shape(c))
        if len(sliced) > 10 and kind != "grad":
            continue
        info = P.Plan(_network(c, 0)[1], path, sliced).info()
        n = c["bitstrings"] if kind == "grad" else 1 << len(sliced)
        work = math.log2(info["macs_per_slice"] * n)
        if work <= 42 and info["arena_bytes_per_slice"] <= (8 << 20 if kind == "scratch" else 4 << 30):
            if best is None or abs(work - aim) < best[0]:
                best = abs(work - aim), c
    return best[1]


# ------------------------------------------------------------------ circuits
def _workload(case, seed):
    grad = case["kind"] == "grad"
    rank = None if grad or case["max_rank"] < 0 else case["max_rank"]
    over = dict(rows=case["rows"], cols=case["cols"], cycles=case["cycles"], max_rank=rank, bit_seed=seed + 1)
    if grad:
        return make_workload("rqc20_grad", n_open=case["rows"] * case["cols"], u3_seed=seed + 2,
                             n_bitstrings=case["bitstrings"], **over)
    return make_workload("rqc53" if case["rows"] * case["cols"] == 54 else "rqc30", n_open=case["n_open"], seed=seed,
                         **over)


def _shape(case):
    """What the path and the slicing set depend on."""
    grad = case["kind"] == "grad"
    return (case["kind"], case["rows"], case["cols"], case["cycles"], case.get("n_open", 0), case.get("max_rank", -1),
            0 if grad else case["reconf_k"], 16 if grad else case["trials"])


@functools.lru_cache(maxsize=None)
def _planned(kind, rows, cols, cycles, n_open, max_rank, reconf_k, trials):
    w = _workload(dict(kind=kind, rows=rows, cols=cols, cycles=cycles, n_open=n_open, max_rank=max_rank,
                       bitstrings=1), 0)
    pr = P.prepare(w, n_seeds=trials, reconf_k=reconf_k)
    return pr.path, pr.sliced


def _network(case, seed):
    w = _workload(case, seed)
    return w, P.Network.from_circuit(w.circuit, w.open_qubits, w.closed_bits)


def _slice_ids(case, sliced, seed):
    if case["slices"] == 0:
        return np.arange(1 << len(sliced), dtype=np.uint64)
    rng = np.random.default_rng(seed + 3)
    return np.sort(rng.integers(0, 1 << min(62, len(sliced)), size=case["slices"], dtype=np.int64)).astype(np.uint64)


def _bits(perm_seed, rank):
    return [int(j) for j in np.random.default_rng(perm_seed).permutation(rank)]


# -------------------------------------------------------------------- passes
def prepare(case, seed):
    if case["kind"] == "permute":
        g = torch.Generator(device="cuda").manual_seed(seed)
        x = torch.randn(case["batch"], 1 << case["rank"], dtype=torch.complex64, device="cuda", generator=g)
        return dict(case=case, x=x, perm=_bits(case["perm_seed"], case["rank"]))
    w, net = _network(case, seed)
    path, sliced = _planned(*_shape(case))
    plan = P.Plan(net, path, sliced, max_rank=w.max_rank if w.max_rank is not None else -1)
    state = dict(case=case, plan=plan)
    if case["kind"] == "grad":
        # one batch holds every bitstring of the loss
        plan.bind(batch=case["bitstrings"], grad=True)
        if case["tune"]:
            plan.autotune("c64", _cache(case))
        state["bits"] = torch.as_tensor(w.bitstrings, device="cuda")
        state["ids"] = [int(x) for x in w.bitstrings]  # slice id == bitstring
        state["angles"] = torch.tensor(w.circuit.angles(), dtype=torch.float32, device="cuda", requires_grad=True)
        return state
    state["ids"] = _slice_ids(case, sliced, seed)
    if case["kind"] == "amps":
        if case["batch"]:
            plan.bind(batch=case["batch"])
        else:
            plan.bind(budget_bytes=8 << 30)
        if case["tune"]:
            plan.autotune(case["mode"], _cache(case))
    return state


def _cache(case):
    return os.path.join(_TUNING, "_".join(str(v) for v in _shape(case)) + "_" + case.get("mode", "c64") + ".json")


def run(state):
    case = state["case"]
    if case["kind"] == "permute":
        return P.permute(state["x"], state["perm"])
    plan = state["plan"]
    if case["kind"] == "grad":
        angles = state["angles"]
        angles.grad = None
        psi = Amplitudes.apply(angles, plan, state["ids"])[state["bits"]]
        torch.sum(torch.log(torch.abs(psi) ** 2)).backward()
        return dict(amplitudes=psi.detach().to(torch.complex64), grad=angles.grad)
    if case["kind"] == "scratch":
        out = plan.execute_scratch(state["ids"], mode=case["mode"])
    elif case["slices"] == 0:
        out = plan.execute_range(0, len(state["ids"]), mode=case["mode"])
    else:
        out = plan.execute(state["ids"], mode=case["mode"])
    return out.to(torch.complex64)


def work(case):
    """8 flops per complex multiply-add of the plan's steps; leaves read once, outputs written once."""
    if case["kind"] == "permute":
        return dict(bytes=16.0 * case["batch"] * (1 << case["rank"]), flops=0)
    net = _network(case, 0)[1]
    path, sliced = _planned(*_shape(case))
    info = P.Plan(net, path, sliced).info()
    leaves = sum(1 << len(ix) for ix in net.indices)
    if case["kind"] == "grad":
        # forward, and two adjoint products for each step
        n = case["bitstrings"]
        return dict(bytes=8.0 * leaves + 8.0 * n + 8.0 * info["n_params"], flops=24.0 * info["macs_per_slice"] * n)
    n = case["slices"] or 1 << len(sliced)
    return dict(bytes=8.0 * leaves + 8.0 * (1 << info["n_open"]), flops=8.0 * info["macs_per_slice"] * n)


# --------------------------------------------------- the same in 64 bits
def _gate(name, params):
    if name == "fsim":
        t, phi = params
        c, s = math.cos(t), -1j * math.sin(t)
        return np.array([[1, 0, 0, 0], [0, c, s, 0], [0, s, c, 0], [0, 0, 0, np.exp(-1j * phi)]])
    x, y = np.array([[0, 1], [1, 0]], dtype=complex), np.array([[0, -1j], [1j, 0]])
    p = {"sqrt_x": x, "sqrt_y": y, "sqrt_w": (x + y) / math.sqrt(2)}[name]
    return 0.5 * (1 + 1j) * np.eye(2) + 0.5 * (1 - 1j) * p


def _state_vector(circuit, n, dev):
    """The circuit's output state, gate after gate, in place."""
    psi = torch.zeros(1 << n, dtype=torch.complex128, device=dev)
    psi[0] = 1
    for g in circuit.gates:
        u = _gate(g.name, g.params)
        if len(g.qubits) == 1:
            v = psi.view(1 << g.qubits[0], 2, -1)
            a = v[:, 0].clone()
            v[:, 0].mul_(u[0, 0]).add_(v[:, 1], alpha=u[0, 1])
            v[:, 1].mul_(u[1, 1]).add_(a, alpha=u[1, 0])
        else:
            p, q = g.qubits
            v = psi.view(1 << p, 2, 1 << (q - p - 1), 2, -1)
            a, b = v[:, 0, :, 1], v[:, 1, :, 0]
            keep = a.clone()
            a.mul_(u[1, 1]).add_(b, alpha=u[1, 2])
            b.mul_(u[2, 2]).add_(keep, alpha=u[2, 1])
            v[:, 1, :, 1].mul_(u[3, 3])
    return psi


def _u3(a, b, c):
    def e(t):
        return torch.polar(torch.ones_like(t), t)
    co, si = torch.cos(b / 2), torch.sin(b / 2)
    return e(-(a + c) / 2) * co, -e(-(a - c) / 2) * si, e((a - c) / 2) * si, e((a + c) / 2) * co


def _u3_state(circuit, n, angles):
    """The output state as a differentiable function of the angles."""
    psi = torch.zeros(1 << n, dtype=torch.complex128, device=angles.device)
    psi[0] = 1
    for g in circuit.gates:
        if g.name == "u3":
            u = _u3(*angles[3 * g.param_id:3 * g.param_id + 3])
            v = psi.view(1 << g.qubits[0], 2, -1)
            psi = torch.stack([u[0] * v[:, 0] + u[1] * v[:, 1], u[2] * v[:, 0] + u[3] * v[:, 1]], 1).reshape(-1)
        else:
            u = [[complex(z) for z in r] for r in _gate(g.name, g.params)]
            p, q = g.qubits
            v = psi.view(1 << p, 2, 1 << (q - p - 1), 2, -1)
            psi = torch.stack([torch.stack([v[:, 0, :, 0], u[1][1] * v[:, 0, :, 1] + u[1][2] * v[:, 1, :, 0]], 2),
                               torch.stack([u[2][1] * v[:, 0, :, 1] + u[2][2] * v[:, 1, :, 0],
                                            u[3][3] * v[:, 1, :, 1]], 2)], 1).reshape(-1)
    return psi


def exact(case, seed):
    if case["kind"] == "permute":
        x = prepare(case, seed)["x"]
        y = torch.arange(x.shape[1], device=x.device)
        at = torch.zeros_like(y)
        for j, to in enumerate(_bits(case["perm_seed"], case["rank"])):
            at |= ((y >> to) & 1) << j
        return x[:, at].to(torch.complex128)
    n = case["rows"] * case["cols"]
    if n > 30 or case.get("slices"):
        return None  # no state vector of this size; a slice alone has none
    w = _workload(case, seed)
    if case["kind"] == "grad":
        a = torch.tensor(w.circuit.angles(), dtype=torch.float32, device="cuda").double().requires_grad_()
        psi = _u3_state(w.circuit, n, a)[torch.as_tensor(w.bitstrings, device="cuda")]
        torch.sum(torch.log(torch.abs(psi) ** 2)).backward()
        return dict(amplitudes=psi.detach(), grad=a.grad)
    # qubit 0 is the most significant bit; the open qubits are the last ones
    at = 0
    for q, b in w.closed_bits.items():
        at |= b << (n - 1 - q)
    return _state_vector(w.circuit, n, "cuda")[at:at + (1 << case["n_open"])]
