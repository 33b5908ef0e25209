"""Knot-gradient samples inside run_switching when a chunk is replayed after its
rows overflowed: every sampled step counts once, from whole rows, as in a run
that had room from the start, with a caller's workspace and without."""
import numpy as np
import pytest

from gpu_common import say
from paper_2201_04622_amd import inputs as I

pytestmark = pytest.mark.gpu
FP64, FP32 = 0, 1


# a replay of the first chunk follows the run that had room bit for bit; one of a later chunk builds its lists at
# another step, which changes the sums' order: round-off (1e-15 a step), grown over 400 steps
@pytest.mark.parametrize("prec,chunk,tol", [(FP64, 1000, 0.0), (FP32, 1000, 0.0), (FP64, 150, 1e-6)])
@pytest.mark.parametrize("reduce", [False, True])
@pytest.mark.parametrize("workspace", [True, False])
def test_samples_of_a_replayed_chunk_count_once(workspace, reduce, prec, chunk, tol):
    import torch

    import paper_2201_04622_amd.eamfe as E
    # verbatim crystals densify under this potential: rows of 64 slots overflow within the equilibration
    reps = [I.Replica("bcc", 6, I.A_BCC_VERBATIM, 1200.0, 5.0, 3), I.Replica("fcc", 5, I.A_FCC_VERBATIM, 900.0, 5.0, 4)]
    p = E.protocol("fl", 400, 600, 0, 0)
    out = []
    for cap in (64, 0):
        ctx = E.Context(0, prec, workspace=workspace)
        ctx.set_launch(4, 256)
        ctx.eam_setup(I.synthetic_eam_knots())
        x = E.to_soa(I.batch_arrays(reps)["x0"])
        ctx.system_setup(reps, x)
        v = torch.zeros_like(x)
        ctx.init_velocities(v, True)
        ctx.neigh_build(x, 0.3, cap)
        ctx.set_chunk(chunk)
        shape = (3, I.N_KNOTS) if reduce else (2, 3, I.N_KNOTS)
        d = torch.ones(shape, dtype=torch.float64, device="cuda")   # the caller's own start value stays in
        ctx.set_adjoint_sampling(20, d, weights=[1.0, -0.5], reduce=reduce)
        ctx.run_switching(p, x, v, 0, 400)
        say(f"cap {cap}: samples {ctx.adjoint_samples()}, replays {ctx.replays()}")
        out.append((x.cpu().numpy(), d.cpu().numpy(), ctx.adjoint_samples()))
        if cap:
            assert ctx.replays() >= 1
        ctx.close()
    assert out[0][2] == out[1][2] == 20
    for a, b in zip(out[0][:2], out[1][:2]):
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b)


def test_tuner_takes_no_samples():
    import torch

    import paper_2201_04622_amd.eamfe as E
    reps = [I.Replica("bcc", 6, I.A_BCC_STABLE, 300.0, 5.0, 3)]
    ctx = E.Context(0, FP32)
    ctx.eam_setup(I.synthetic_eam_knots())
    x = E.to_soa(I.batch_arrays(reps)["x0"])
    ctx.system_setup(reps, x)
    v = torch.zeros_like(x)
    ctx.init_velocities(v, True)
    ctx.neigh_build(x, 0.3, 0)
    d = torch.zeros(1, 3, I.N_KNOTS, dtype=torch.float64, device="cuda")
    ctx.set_adjoint_sampling(2, d)
    p = E.protocol("fl", 200, 10, 0, 0)
    ctx.autotune(p, 0, x, v, trial_steps=2)
    assert ctx.adjoint_samples() == 0 and float(d.abs().max()) == 0.0
    ctx.run_switching(p, x, v, 0, 10)
    assert ctx.adjoint_samples() == 5 and float(d.abs().max()) > 0.0
    ctx.close()
