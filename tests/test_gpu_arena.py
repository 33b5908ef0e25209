"""A context whose device memory the library owns (no caller's workspace) and
whose arena moves in the middle of a call: the first list plan inside
run_switching, an overflow replay whose larger rows outgrow the arena, and
the tuner's trials.  Each run is bitwise the run of a context that had room
from the start."""
import numpy as np
import pytest

from gpu_common import say
from paper_2201_04622_amd import inputs as I

pytestmark = pytest.mark.gpu
FP64, FP32 = 0, 1


def _ctx(reps, prec, workspace, shape=(2, 256)):
    import torch

    import paper_2201_04622_amd.eamfe as E
    ctx = E.Context(0, prec, workspace=workspace)
    if shape:
        ctx.set_launch(*shape)
    ctx.eam_setup(I.synthetic_eam_knots())
    x = E.to_soa(I.batch_arrays(reps)["x0"])
    ctx.system_setup(reps, x)
    v = torch.zeros_like(x)
    ctx.init_velocities(v, True)
    return ctx, x, v


def _run(ctx, x, v, n_rep, S, p, steps=None):
    import torch
    W = torch.zeros(n_rep, S, dtype=torch.float64, device="cuda")
    before = ctx.device_allocations()
    ctx.run_switching(p, x, v, 0, steps or S, W_out=W)
    return (x.cpu().numpy(), v.cpu().numpy(), W.cpu().numpy()), ctx.device_allocations() - before


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_first_plan_inside_a_run(prec):
    import paper_2201_04622_amd.eamfe as E
    reps = [I.Replica("bcc", 8, I.A_BCC_VERBATIM, 300.0, 5.0, 3), I.Replica("fcc", 7, I.A_FCC_VERBATIM, 300.0, 5.0, 4)]
    p = E.protocol("fl", 10, 25, 0, 0)
    out = []
    for workspace in (True, False):
        ctx, x, v = _ctx(reps, prec, workspace)
        if workspace:
            ctx.neigh_build(x, 0.3, 0)
        got, allocs = _run(ctx, x, v, 2, 60, p)
        say(f"workspace {workspace}: allocations in the run {allocs}")
        if not workspace:
            assert allocs >= 1   # the arena moved inside the call
        out.append(got)
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("chunk", [1000, 10, 11])   # replay of the first chunk; of a later one, in either buffer
@pytest.mark.parametrize("prec", [FP64, FP32])
def test_replay_that_outgrows_the_arena(prec, chunk):
    import paper_2201_04622_amd.eamfe as E
    # verbatim crystals densify under this potential: rows of 64 slots overflow and grow until they hold
    reps = [I.Replica("bcc", 10, I.A_BCC_VERBATIM, 1200.0, 5.0, 3), I.Replica("fcc", 8, I.A_FCC_VERBATIM, 900.0, 5.0, 4)]
    p = E.protocol("fl", 200, 600, 100, 100)
    out = []
    if chunk < 1000:   # the first chunk's rows fit
        ctx, x, v = _ctx(reps, prec, True)
        ctx.neigh_build(x, 0.3, 64)
        ctx.run_switching(p, x, v, 0, chunk)
        assert ctx.replays() == 0
        ctx.close()
    for workspace in (True, False):
        ctx, x, v = _ctx(reps, prec, workspace)
        ctx.neigh_build(x, 0.3, 64)
        ctx.set_chunk(chunk)
        got, allocs = _run(ctx, x, v, 2, 1600, p, 800)
        say(f"workspace {workspace}: allocations in the run {allocs}, replays {ctx.replays()}, rows {ctx.list_stats()}")
        assert ctx.replays() >= 1
        if not workspace:
            assert allocs >= 1
        out.append(got)
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_tuner_without_lists():
    import torch

    import paper_2201_04622_amd.eamfe as E
    reps = [I.Replica("bcc", 14, I.A_BCC_VERBATIM, 300.0, 5.0, 3), I.Replica("fcc", 7, I.A_FCC_VERBATIM, 300.0, 5.0, 4)]
    p = E.protocol("fl", 10, 25, 0, 0)
    out = []
    for tune in (False, True):
        ctx, x, v = _ctx(reps, FP32, not tune)
        if tune:   # plans the lists inside its first trial, and again for the other builder
            x0, v0, before = x.clone(), v.clone(), ctx.device_allocations()
            ctx.autotune(p, 0, x, v, trial_steps=2)
            assert ctx.device_allocations() > before
            assert torch.equal(x, x0) and torch.equal(v, v0)
        else:
            ctx.neigh_build(x, 0.3, 0)
        got, _ = _run(ctx, x, v, 2, 60, p)   # FP32 bits do not depend on the shape or the builder
        out.append(got)
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
