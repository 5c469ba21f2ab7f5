"""Calls of several substeps on two wavefronts per workgroup, for every swarm
size with a kernel of its own and for the table of sizes: the same arithmetic in
the same order as on one, so bit for bit the same (tolerance zero)."""
import numpy as np
import pytest
import torch

from paper_2306_09537_amd import workloads as W
from paper_2306_09537_amd.quadswarm import QuadSwarm

pytestmark = pytest.mark.gpu

# the last workgroup is not full; the table's hold 60, 51 or fewer of 64
SIZES = {"1": [1] * 131, "2": [2] * 67, "4": [4] * 37, "16": [16] * 9, "32": [32] * 5,
         "64": [64] * 3, "12": [12] * 11, "17": [17] * 7, "mixed": [1, 40, 7, 16, 3, 64, 2, 33]}


@pytest.mark.parametrize("k", [6, 0, 3])
@pytest.mark.parametrize("sizes", sorted(SIZES))
def test_two_wavefronts_equal_one(sizes, k, monkeypatch):
    w = W.custom(SIZES[sizes], seed=21, k=k, name="pipe")
    monkeypatch.setenv("QS_BUCKETED", "0")
    sims = []
    for on in ("0", "1"):
        monkeypatch.setenv("QS_STEP_PIPE", on)
        sim = QuadSwarm.from_workload(w)
        sim.record_contacts(True)
        g = torch.from_numpy(np.ascontiguousarray(w.goals)).cuda()
        got = []
        for c, nsub in enumerate((2, 5, 1, 9)):
            a = torch.from_numpy(np.ascontiguousarray(w.actions(c))).cuda()
            if c == 1:
                got += [x.clone() for x in sim.step_observe_reward(a, nsub, g)]
            elif c == 3:
                sim.step(a, nsub)
            else:
                got.append(sim.step_observe(a, nsub, g).clone())
        got += [sim.get_state()[0], sim.debug_contacts()]
        sims.append(got)
    for one, two in zip(*sims):
        assert torch.equal(one, two)
