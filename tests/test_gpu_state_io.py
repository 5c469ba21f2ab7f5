"""State in and out of a handle, bit for bit: the tiles of 64 rows at their
edges, buffers off the 16-byte grid, and masked loads."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2306_09537_amd import workloads as W  # noqa: E402
from paper_2306_09537_amd.quadswarm import QuadSwarm  # noqa: E402

pytestmark = pytest.mark.gpu


def shifted(shape, by):
    """A contiguous tensor that starts `by` floats into its allocation."""
    n = int(np.prod(shape))
    return torch.empty(n + 8, device="cuda")[by:by + n].view(shape)


@pytest.mark.parametrize("by", [0, 1])
@pytest.mark.parametrize("n_envs", [1, 21, 22, 43, 300])
def test_state_round_trip(n_envs, by):
    w = W.custom([3] * n_envs, seed=n_envs, k=0, name="io")
    sim = QuadSwarm.from_workload(w)
    rng = np.random.default_rng(n_envs)
    new = torch.from_numpy(rng.standard_normal((w.n_quads, 27)).astype(np.float32)).cuda()
    src, dst = shifted(new.shape, by), shifted(new.shape, by)
    src.copy_(new)
    sim.get_state(dst)
    assert np.array_equal(dst.cpu().numpy(), w.state0)
    mask = torch.from_numpy((rng.random(n_envs) < 0.4).astype(np.uint8)).cuda()
    sim.set_state(src, 5, mask)
    want = torch.where(torch.repeat_interleave(mask, 3)[:, None] != 0, new,
                       torch.from_numpy(w.state0).cuda())
    assert torch.equal(sim.get_state(dst)[0], want)
    sim.set_state(src, 5)
    assert torch.equal(sim.get_state(dst)[0], new)
