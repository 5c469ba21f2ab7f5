"""A tape that does not hold every segment is filled and swept chunk by chunk:
the state adjoint and the action gradients have the bits of one chunk, and the
parameter gradient is a sum of its own, added to the caller's array once."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2306_09537_amd import workloads as W  # noqa: E402
from paper_2306_09537_amd.quadswarm import QuadSwarm  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("pipe", ["0", "1"])
@pytest.mark.parametrize("beta", [0.0, 100.0])
@pytest.mark.parametrize("sizes", [[1] * 70, [8] * 21, [32] * 3, [13] * 11, [40, 3, 64, 17, 1]])
def test_chunks_equal_one_pass(sizes, beta, pipe, monkeypatch):
    for k in ("RECOMPUTE", "REVERSE"):
        monkeypatch.setenv(f"QS_{k}_PIPE", pipe)
    w = W.custom(sizes, seed=len(sizes), k=0, name="chunks")
    Q, calls, nsub, ce = w.n_quads, 9, 2, 2
    rng = np.random.default_rng(1)
    acts, g, gpen = dev(rng.random((calls, Q, 4))), dev(rng.standard_normal((Q, 27))), dev(rng.random(Q))
    start = dev(100.0 * rng.standard_normal((Q, 6)))
    sim = QuadSwarm.from_workload(w)
    ckpt = torch.empty(((calls + ce - 1) // ce, 27, Q), device="cuda")
    sim.rollout(acts, nsub, ce, ckpt, torch.zeros(Q, device="cuda") if beta else None, beta)

    def backward(gp):
        gs, ga, gp = g.clone(), torch.empty_like(acts), gp.clone()
        sim.rollout_backward(acts, nsub, ce, ckpt, 0, gs, gpen if beta else None, beta, ga, gp)
        return gs, ga, gp

    whole = backward(torch.zeros_like(start))
    words = 34 if beta else 31
    for segments in (1, 2, 3):  # of five: the last chunk holds one, one and two
        monkeypatch.setenv("QS_TAPE_BYTES", str(segments * ce * nsub * words * Q * 4))
        alone, added = backward(torch.zeros_like(start)), backward(start)
        for a, b in zip(whole[:2], alone[:2]):
            assert torch.equal(a, b)
        # two sums of the same 18 terms of a quad, in two orders
        size = whole[2].abs().amax(0)
        assert ((whole[2] - alone[2]).abs() <= 2 * 18 * 2.0 ** -23 * size).all()
        assert torch.equal(added[0], alone[0]) and torch.equal(added[1], alone[1])
        assert torch.equal(added[2], start + alone[2])
    sim.sync()
