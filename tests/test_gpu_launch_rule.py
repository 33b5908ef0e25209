"""The launch shape that the library chooses in EAMFE_FP64 where the caller
sets none, at the edges of its rule (sixteen lanes or eight, units counted
per replica, tables that fit a block's LDS or not, and tables that change
after the system is set up): the forces are those of an explicit shape."""
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
