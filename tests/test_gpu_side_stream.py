"""Contexts on a stream that the null stream does not wait for: calls whose
rows overflow and which clear the latched status and try again give bitwise
what they give on the default stream, a latched condition is reported once,
and buffers moved to a larger workspace or copied out are complete when the
call returns.  Graph replays that a call leaves in flight end before the next
call drops their graph."""
import numpy as np
import pytest

from gpu_common import say
from paper_2201_04622_amd import inputs as I

pytestmark = pytest.mark.gpu
FP64, FP32 = 0, 1


def _calls(prec):
    import torch

    import paper_2201_04622_amd.eamfe as E
    reps = [I.Replica("fcc", 5, I.A_FCC_VERBATIM, 300.0, 5.0, 1), I.Replica("fcc", 11, I.A_FCC_VERBATIM, 300.0, 5.0, 2)]
    ctx = E.Context(0, prec, workspace=False)   # the calls enlarge the lists themselves
    ctx.eam_setup(I.synthetic_eam_knots())
    arrs = I.batch_arrays(reps)
    x0 = E.to_soa(arrs["x0"])
    ctx.system_setup(reps, x0)
    x = E.to_soa(I.displaced(arrs["x0"], 0.2, seed=5))
    out = []
    f, U = torch.zeros_like(x), torch.zeros(2, dtype=torch.float64, device="cuda")
    try:
        ctx.neigh_build(x, 0.3, 32)
        raise AssertionError("rows of 32 slots cannot hold")
    except E.EamfeError as e:
        assert e.code == 6
    ctx.check()                      # the condition was reported and is gone
    for call in ("forces", "pressure", "run"):
        ctx.neigh_build(x0, 0.3, 64)   # holds the crystal's 54 neighbours, not all of the displaced atoms'
        n = ctx.replays()
        if call == "forces":
            ctx.eam_forces(x, f, U)
            out += [f.cpu().numpy().copy(), U.cpu().numpy().copy()]
        elif call == "pressure":
            out.append(ctx.pressure(x).copy())
        else:
            xx, v = x.clone(), torch.zeros_like(x)
            ctx.init_velocities(v, True)
            W = torch.zeros(2, 12, dtype=torch.float64, device="cuda")
            ctx.run_switching(E.protocol("fl", 2, 5, 0, 0), xx, v, 0, 12, W_out=W)
            out += [xx.cpu().numpy(), v.cpu().numpy(), W.cpu().numpy(), ctx.get_state()[1].cpu().numpy()]
        ctx.check()
        assert ctx.replays() > n
        say(f"{call}: replays {ctx.replays() - n}, rows {ctx.list_stats()}")
    ctx.close()
    ctx = E.Context(0, prec)                    # a workspace that grows in the call
    ctx.eam_setup(I.synthetic_eam_knots())
    ctx.system_setup(reps, x0)
    ctx.neigh_build(x0, 0.3, 64)
    ctx.eam_forces(x, f, U)
    out += [f.cpu().numpy().copy(), U.cpu().numpy().copy()]
    ctx.close()
    return out


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_retries_on_a_side_stream(prec):
    import torch
    ref = _calls(prec)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        got = _calls(prec)
    s.synchronize()
    for a, b in zip(ref, got):
        assert np.array_equal(a, b)


def test_graph_replays_left_in_flight():
    # harmonic runs that are not waited for, one after another: each drops the graphs of the one before
    import torch

    import paper_2201_04622_amd.eamfe as E
    reps = [I.Replica("bcc", 10, I.A_BCC_STABLE, 300.0, 5.0, 1 + q, k2=4.0) for q in range(4)]
    x0 = E.to_soa(I.batch_arrays(reps)["x0"])
    p = E.protocol("hh", 20, 200, 20, 0)
    out = []
    for graph in (0, 8):
        ctx = E.Context(0, FP64)
        ctx.set_launch(4, 256)
        ctx.system_setup(reps, x0)
        ctx.set_graph(graph)
        x, v = x0.clone(), torch.zeros_like(x0)
        ctx.init_velocities(v, True)
        W = torch.zeros(4, 440, dtype=torch.float64, device="cuda")
        for s in range(0, 440, 55):
            ctx.run_switching(p, x, v, s, s + 55, W_out=W, sync=False)
        ctx.check()
        out.append([t.cpu().numpy() for t in (x, v, W)])
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
