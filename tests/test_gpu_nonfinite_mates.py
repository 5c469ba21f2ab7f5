"""A quad whose position is not a number is in contact with nobody: its mates
move as they do without it, in every form of the in-swarm pass."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2306_09537_amd import workloads as W  # noqa: E402
from paper_2306_09537_amd.quadswarm import QuadSwarm, QuadSwarmError  # noqa: E402

pytestmark = pytest.mark.gpu
# responses to every contact, approaching or not: a false one would be seen
FLAGS = W.QS_COLLIDE | W.QS_MOTOR_NOISE


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def lost(w, value):
    """The state with the third quad of every swarm at `value`, and the mates."""
    state, out = w.state0.copy(), w.env_offsets[:-1] + 2
    state[:, 2] += 2.0
    state[out, :3] = value
    rest = np.ones(w.n_quads, bool)
    rest[out] = False
    return state, rest


@pytest.mark.parametrize("downwash", [False, True])
@pytest.mark.parametrize("value", [np.nan, -np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("n", [4, 8, 13, 16, 32, 64])
def test_mates_of_a_lost_quad(n, value, downwash, monkeypatch):
    # no downwash reaches anybody: the flag only takes the pass over every partner
    w = W.custom([n] * (160 // n), seed=n, k=0, name="lost", dw_radius=0.0,
                 flags=FLAGS | (W.QS_DOWNWASH if downwash else 0))
    state, rest = lost(w, value)
    away, _ = lost(w, 3.0e9)
    Q, acts = w.n_quads, dev(np.random.default_rng(n).random((3, w.n_quads, 4)))
    for pipe in ("0", "1"):
        for k in ("STEP", "ROLLOUT"):
            monkeypatch.setenv(f"QS_{k}_PIPE", pipe)
        sim = QuadSwarm.from_workload(w)
        sim.record_contacts(True)
        got = []
        for s in (state, away):
            sim.set_state(dev(s), 0)
            sim.step(acts[0], 3)
            contacts = sim.debug_contacts()[rest]
            stepped = sim.get_state()[0][rest]
            sim.set_state(dev(s), 0)
            sim.rollout(acts, 1, 0, None, torch.zeros(Q, device="cuda"), 100.0)
            got.append((contacts, stepped, sim.get_state()[0][rest]))
            try:
                sim.sync()
            except QuadSwarmError as e:
                assert e.code == -5
        for a, b in zip(*got):
            assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("lost_quad,weight", [(True, 1.0), (False, np.inf), (False, np.nan)])
@pytest.mark.parametrize("sizes", [[13] * 9, [40] * 3, [50, 50, 17, 9]])
def test_a_lost_mate_in_the_other_wavefront(sizes, lost_quad, weight, monkeypatch):
    """Workgroups of 128 may hold a swarm in two wavefronts: its penalty and its
    adjoint are those of workgroups of 64, where it lies in one."""
    w = W.custom(sizes, seed=1, k=0, name="lost", flags=W.QS_MOTOR_NOISE)
    Q, state = w.n_quads, w.state0.copy()
    env = int(np.searchsorted(w.env_offsets, 64, side="right")) - 1
    first, end = w.env_offsets[env], w.env_offsets[env + 1]
    assert first < 64 < end <= 128
    rng = np.random.default_rng(2)
    state[:, :3] = 6.0 * rng.uniform(-1, 1, size=(Q, 3))  # few within 1.2 m
    if lost_quad:
        state[first, 1] = np.nan
    acts, g = dev(rng.random((2, Q, 4))), dev(rng.standard_normal((Q, 27)))
    gpen = np.ones(Q)
    gpen[first] = weight
    outs = []
    for block in ("64", "128"):
        monkeypatch.setenv("QS_BLOCK_SIZE", block)
        sim = QuadSwarm.from_workload(w)
        sim.set_state(dev(state), 0)
        pen, ckpt = torch.zeros(Q, device="cuda"), torch.empty((1, 27, Q), device="cuda")
        sim.rollout(acts, 2, 2, ckpt, pen, 100.0)
        gs, ga = g.clone(), torch.empty((2, Q, 4), device="cuda")
        sim.rollout_backward(acts, 2, 2, ckpt, 0, gs, dev(gpen), 100.0, ga,
                             torch.zeros((Q, 6), device="cuda"))
        outs.append((pen, gs, ga))
    if lost_quad:  # a swarm with a lost quad has no penalty that is a number
        assert outs[0][0][first:end].isnan().all()
    for a, b in zip(*outs):
        assert torch.equal(a.isnan(), b.isnan())
        assert torch.equal(a.nan_to_num(), b.nan_to_num())
