"""Tuning of the adjoint products: what is timed, and on what."""
import json

import pytest

from tests.gpu_util import banner
from tests.test_gpu_tuning_file import BATCH, _network, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def test_adjoint_tuning_on_a_dirty_workspace(torch, tmp_path):  # noqa: F811
    """The adjoint candidates are timed on numbers, whatever the workspace held:
    after NaN in all of it, three-part tiles (kind 6, or -1 for the fixed rule, which
    takes them) still come out for the product they are fastest on."""
    import paper_2205_00393_amd as P
    net, path, si = _network(P)
    plan = P.Plan(net, path, si)
    nbytes = plan.workspace_size(BATCH, True)
    dirty = torch.full(((nbytes + 3) // 4,), float("nan"), dtype=torch.float32, device="cuda")
    where = dirty.data_ptr()
    del dirty
    plan.bind(batch=BATCH, grad=True)
    assert plan._ws.data_ptr() == where, "the allocator gave other memory"
    plan.set_params(torch.tensor([0.3, 0.7, -0.4], dtype=torch.float64, device="cuda"))
    cache = str(tmp_path / "tune.json")
    plan.autotune("c64", cache)
    adj = {k: v for k, v in json.load(open(cache)).items() if k.startswith("g0_")}
    banner(f"adjoint choices {adj}")
    large = [v[0] for k, v in adj.items() if k.startswith("g0_10_10_10_")]
    assert len(large) == 1 and (large[0] == -1 or large[0] // 1000 == 6)
