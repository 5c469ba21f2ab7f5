"""Uneven swarm sizes: calls of few substeps by packed blocks, calls of many by
work items ordered over the XCDs.  Which lanes serve a quad, and when, changes no
result, so every route equals the packed blocks bit for bit (tolerance zero)."""
import numpy as np
import pytest
import torch

from paper_2306_09537_amd import workloads as W
from paper_2306_09537_amd.quadswarm import QuadSwarm

pytestmark = pytest.mark.gpu

# full slots; sorted, so that a run of items has one slot size, in more than one
# group of runs with a ragged last one; padded slots; one size, no power of two
SIZES = {
    "powers": [1, 2, 4, 8, 16, 32, 64] * 9,
    "sorted": [64] * 700 + [16] * 900 + [3] * 1500 + [1] * 2000,
    "padded": [17, 33, 5, 9, 2, 40] * 30,
    "twelves": [12] * 37,
}


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("sizes", sorted(SIZES))
def test_routes_are_bitwise_equal(sizes, monkeypatch):
    w = W.custom(SIZES[sizes], seed=11, k=6, name="routes")
    monkeypatch.setenv("QS_BUCKETED", "0")
    ref = QuadSwarm.from_workload(w)
    monkeypatch.setenv("QS_BUCKETED", "1")
    items = QuadSwarm.from_workload(w)
    monkeypatch.delenv("QS_BUCKETED")
    auto = QuadSwarm.from_workload(w)
    g = dev(w.goals)
    for c, nsub in enumerate((1, 7, 8, 3, 12)):
        a = dev(w.actions(c))
        want = ref.step_observe(a, nsub, g).clone()
        for sim in (items, auto):
            assert torch.equal(sim.step_observe(a, nsub, g), want)
        if c == 2:  # whatever the tuner picks, from here on
            auto.autotune(a, 3, g, torch.empty_like(want))
    state = ref.get_state()[0]
    assert torch.equal(items.get_state()[0], state)
    assert torch.equal(auto.get_state()[0], state)


def test_explicit_launch_after_the_tuner(monkeypatch):
    w = W.custom(SIZES["powers"], seed=12, k=6, name="routes")
    monkeypatch.setenv("QS_BUCKETED", "0")
    ref = QuadSwarm.from_workload(w)
    monkeypatch.delenv("QS_BUCKETED")
    sim = QuadSwarm.from_workload(w)
    g = dev(w.goals)
    for c, (block, grid) in enumerate(((128, 0), (64, 5), (128, 3))):
        sim.set_launch(block, grid)
        a = dev(w.actions(c))
        assert torch.equal(sim.step_observe(a, 2, g), ref.step_observe(a, 2, g))


def kernels_of(call):
    """Names of the kernels that a call launches."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA, ProfilerActivity.CPU]) as prof:
        call()
        torch.cuda.synchronize()
    return [e.key for e in prof.key_averages() if "qs::" in e.key]


def test_the_tuner_leaves_a_forced_launch(monkeypatch):
    """A batch of three workgroups, which the table serves faster than any grid of
    items does: QS_BUCKETED=1 keeps the items all the same."""
    monkeypatch.setenv("QS_BUCKETED", "1")
    w = W.custom([12] * 15, seed=13, k=6, name="routes")
    sim = QuadSwarm.from_workload(w)
    g, a = dev(w.goals), dev(w.actions(0))
    o = torch.empty((w.n_quads, w.obs_dim), device="cuda")
    sim.autotune(a, 4, g, o)
    names = kernels_of(lambda: sim.step_observe(a, 4, g, o))
    assert len(names) == 1 and "bucket_kernel" in names[0], names
