"""The ways the kernels pass over a swarm's partners give the same bits.

The same swarms run in a handle of their own (sizes known at compile time) and
in one with an environment more (table of sizes), with the multi-wavefront
kernels and without, at spreads where the penalty is summed over the near
partners only, over all of them, and from a far origin, where the expanded
screen does not hold.  Sums leave out exact zeros only, so every result is
compared bit for bit; the penalty of loose swarms also against the oracle.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2306_09537_amd import workloads as W  # noqa: E402
from paper_2306_09537_amd.quadswarm import QuadSwarm  # noqa: E402

pytestmark = pytest.mark.gpu
FLAGS = W.QS_COLLIDE | W.QS_MOTOR_NOISE | W.QS_APPROACH_ONLY
CALLS, NSUB, CE = 6, 2, 4


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def differentiate(w, acts, g_state, g_pen, beta):
    sim = QuadSwarm.from_workload(w)
    Q = w.n_quads
    ckpt = torch.empty(((CALLS + CE - 1) // CE, 27, Q), device="cuda")
    pen = torch.zeros(Q, device="cuda")
    sim.rollout(acts, NSUB, CE, ckpt, pen, beta)
    end, _ = sim.get_state()
    gs, gact = g_state.clone(), torch.empty_like(acts)
    gpar = torch.zeros(Q, 6, device="cuda")
    sim.rollout_backward(acts, NSUB, CE, ckpt, 0, gs, g_pen, beta, gact, gpar)
    sim.sync()
    return end, pen, gs, gact, gpar


@pytest.mark.parametrize("beta", [100.0, 20.0])
@pytest.mark.parametrize("origin,spread", [(0.0, 0.15), (0.0, 2.0), (9.5, 2.0), (60.0, 2.0)])
@pytest.mark.parametrize("n", [2, 8, 13, 16, 32, 40])
def test_paths_agree(monkeypatch, n, origin, spread, beta):
    n_envs = max(2, 160 // n)
    rng = np.random.default_rng(n * 7 + int(origin))
    w = W.custom([n] * n_envs, seed=n, k=0, flags=FLAGS, name="paths")
    w1 = W.custom([n] * n_envs + [3], seed=n, k=0, flags=FLAGS, name="paths+")
    Q = w.n_quads
    state, params = w1.state0.copy(), w1.params.copy()
    state[:, :3] = origin + spread * rng.uniform(-1, 1, size=(w1.n_quads, 3))
    w = w.with_(state0=state[:Q], params=params[:Q])
    w1 = w1.with_(state0=state, params=params)
    acts = dev(rng.random((CALLS, w1.n_quads, 4)))
    g_state, g_pen = dev(rng.standard_normal((w1.n_quads, 27))), dev(rng.random(w1.n_quads))
    runs = []
    for pipe in ("1", "0"):
        for k in ("ROLLOUT", "RECOMPUTE", "REVERSE"):
            monkeypatch.setenv(f"QS_{k}_PIPE", pipe)
        runs.append(differentiate(w, acts[:, :Q].contiguous(), g_state[:Q], g_pen[:Q], beta))
        more = differentiate(w1, acts, g_state, g_pen, beta)
        runs.append(tuple(v[:, :Q] if v.dim() == 3 else v[:Q] for v in more))
    for other in runs[1:]:
        for k, (a, b) in enumerate(zip(runs[0], other)):
            assert torch.equal(a, b), (k, float((a - b).abs().max()))
    if spread < 1.0:  # packed swarms: contacts amplify float32's rounding
        return
    _, pen = O.Oracle.from_workload(w).rollout(w.state0, acts[:, :Q].cpu().numpy(), NSUB, 0, beta)
    # a term changes by beta times the error of its distance: two positions
    # rounded once per substep (half an ulp, 2^-24 relative)
    rtol = 2e-4 + beta * 2 * CALLS * NSUB * (origin + spread) * 2.0 ** -24
    np.testing.assert_allclose(runs[0][1].cpu().numpy(), pen, rtol=rtol, atol=1e-7)
