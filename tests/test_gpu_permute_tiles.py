"""Permutations around the sizes at which the tile is filled to 2^10, 2^11 or 2^12
elements (256 tiles), bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import banner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.mark.parametrize("rank,batch", [(1, 3), (9, 300), (10, 255), (11, 127), (11, 128), (12, 127), (12, 128),
                                        (12, 255), (12, 256), (13, 1), (18, 3), (18, 4), (19, 1), (20, 1), (21, 1)])
@pytest.mark.parametrize("kind", ["random", "reverse", "identity"])
def test_tile_sizes(torch, rank, batch, kind):
    import paper_2205_00393_amd as P
    banner(f"permute {batch} x 2^{rank} {kind}")
    rng = np.random.default_rng(100 * rank + batch)
    perm = {"random": rng.permutation(rank), "reverse": np.arange(rank)[::-1], "identity": np.arange(rank)}[kind]
    words = rng.integers(0, 2 ** 32, size=(batch << rank, 2), dtype=np.uint32).view(np.float32)
    x = torch.tensor(words, device="cuda").view(torch.complex64).reshape(batch, 1 << rank)
    got = P.permute(x, [int(p) for p in perm]).view(torch.int64)
    y = torch.arange(1 << rank, device="cuda")
    at = torch.zeros_like(y)
    for j, to in enumerate(perm):
        at |= ((y >> int(to)) & 1) << j
    assert torch.equal(got, x.view(torch.int64)[:, at])
