"""The launch shape that the library chooses in EAMFE_FP64 where the caller
sets none, at the edges of its rule (sixteen lanes or eight, units counted
per replica, tables that fit a block's LDS or not, and tables that change
after the system is set up): the forces are those of an explicit shape.  The
harmonic modes have a shape of their own, which leaves no trace in the runs
with pair sums around them."""
import numpy as np
import pytest

from paper_2201_04622_amd import inputs as I

pytestmark = pytest.mark.gpu
FP64, FP32 = 0, 1


def _reps(kind, n, n_rep, vac):
    a = I.A_FCC_VERBATIM if kind == "fcc" else I.A_BCC_VERBATIM
    return [I.Replica(kind, n, a, 300.0, 5.0, 3 + k, vacancies=tuple(range(vac))) for k in range(n_rep)]


@pytest.mark.parametrize("kind,n,n_rep,vac,knots,want", [
    ("fcc", 8, 1, 5, 2000, (16, 64)),        # 2,043 atoms: 511 units, two per CU are not reached
    ("fcc", 8, 1, 1, 2000, (16, 1024)),      # 2,047: 512 units, the last one partly filled
    ("bcc", 8, 2, 1, 2000, (16, 1024)),      # 2 x 1,023: 512 units, two of them partly filled
    ("fcc", 8, 1, 1, 2562, (16, 128)),       # tables one knot beyond a block's LDS
    ("bcc", 15, 1, 606, 2000, (16, 1024)),   # 6,144 atoms: six wavefronts per CU at sixteen lanes
    ("bcc", 15, 1, 602, 2000, (8, 256)),     # 6,148
    ("fcc", 14, 1, 0, 2000, (8, 384)),       # 10,976: 5.4 units per CU
    ("bcc", 10, 8, 0, 2000, (8, 512)),       # 8 x 2,000: 7.8
    ("bcc", 10, 8, 0, 2562, (8, 128)),
])
def test_shape_and_forces(kind, n, n_rep, vac, knots, want):
    import torch

    import paper_2201_04622_amd.eamfe as E
    reps = _reps(kind, n, n_rep, vac)
    arrs = I.batch_arrays(reps)
    x = E.to_soa(I.displaced(arrs["x0"], 0.05, seed=5))
    out = []
    for shape in (None, (4, 256)):
        ctx = E.Context(0, FP64)
        if shape:
            ctx.set_launch(*shape)
        ctx.eam_setup(I.synthetic_eam_knots(knots))
        ctx.system_setup(reps, E.to_soa(arrs["x0"]))
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert ctx.get_launch() == (shape or want)
        f, U = torch.zeros_like(x), torch.zeros(n_rep, dtype=torch.float64, device="cuda")
        ctx.eam_forces(x, f, U)
        out.append((f.cpu().numpy(), U.cpu().numpy()))
        ctx.close()
    for a, b in zip(*out):   # sums of under 1e3 terms in another order
        assert np.linalg.norm(a - b) <= 1e-12 * np.linalg.norm(b)


def test_shape_follows_the_tables():
    import torch

    import paper_2201_04622_amd.eamfe as E
    reps = _reps("bcc", 10, 8, 0)
    ctx = E.Context(0, FP64)
    ctx.eam_setup(I.synthetic_eam_knots(2562))
    ctx.system_setup(reps, E.to_soa(I.batch_arrays(reps)["x0"]))
    got = [ctx.get_launch()]
    for knots in (2000, 2562):
        ctx.eam_setup(I.synthetic_eam_knots(knots))
        got.append(ctx.get_launch())
    ctx.set_launch(8, 256)
    ctx.eam_setup(I.synthetic_eam_knots(2000))   # the caller's shape stands
    assert ctx.get_launch() == (8, 256)
    ctx.close()
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert got == [(8, 128), (8, 512), (8, 128)]


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("kind,n,n_rep,harmonic", [
    ("bcc", 4, 1, (4, 256)), ("fcc", 16, 1, (4, 256)),   # 128 and 16,384 atoms
    ("bcc", 21, 1, (1, 256)),                            # 18,522
])
def test_harmonic_modes_between_runs_with_pairs(prec, kind, n, n_rep, harmonic):
    import torch

    import paper_2201_04622_amd.eamfe as E
    reps = _reps(kind, n, n_rep, 0)
    x0 = E.to_soa(I.batch_arrays(reps)["x0"])
    fl, hh = E.protocol("fl", 2, 4, 0, 0), E.protocol("hh", 2, 4, 0, 0)
    out = {}
    for name in ("with", "without", "harmonic alone", "harmonic fixed"):
        ctx = E.Context(0, prec)
        if name == "harmonic fixed":
            ctx.set_launch(*harmonic)
        if not name.startswith("harmonic"):
            ctx.eam_setup(I.synthetic_eam_knots())
        ctx.system_setup(reps, x0)
        shape = ctx.get_launch()

        def run(p):
            x, v = x0.clone(), torch.zeros_like(x0)
            ctx.init_velocities(v, True)
            W = torch.zeros(n_rep, 10, dtype=torch.float64, device="cuda")
            ctx.run_switching(p, x, v, 0, 10, W_out=W)
            return [t.cpu().numpy() for t in (x, v, W)]

        if name == "with":
            ctx.set_launch(0, 0)   # keeps the automatic shape
            run(hh)
            assert ctx.get_launch() == harmonic
            out[name] = run(fl)
            assert ctx.get_launch() == shape
        elif name == "without":
            out[name] = run(fl)
        else:
            assert shape == harmonic
            out[name] = run(hh)
        ctx.close()
    for a, b in (("with", "without"), ("harmonic alone", "harmonic fixed")):
        for u, w in zip(out[a], out[b]):
            assert np.array_equal(u, w)
