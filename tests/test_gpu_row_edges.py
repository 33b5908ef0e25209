"""Both row builders at the sizes where their work is cut: a stencil's
candidates exactly filling one register chunk (1024), the chunks of larger
stencils, all-pairs boxes up to and beyond a chunk with a partial last group,
cells of more members than one round of a wavefront takes, and rows so wide
that fewer wavefronts (and shorter chunks) fit a block.  Rows of both builders
are equal slot for slot and hold exactly the brute-force pairs.  The launch
shape chosen for a system where the caller sets none gives the bits of an
explicit one."""
import numpy as np
import pytest

from gpu_common import make_ctx, say
from paper_2201_04622_amd import inputs as I

pytestmark = pytest.mark.gpu
FP64, FP32 = 0, 1

B = I.A_BCC_STABLE
CASES = {   # replicas, skin, max_neighbors, cells per edge of the first replica
    "1024 of one chunk": ([("bcc", 8, B), ("bcc", 5, I.A_BCC_VERBATIM)], 0.3, 0, 5),
    "1458 in two chunks": ([("bcc", 9, B)], 0.65, 0, 5),
    "all pairs of 1024": ([("bcc", 8, B)], 1.1, 0, 4),
    "all pairs of 1458": ([("bcc", 9, B)], 1.9, 0, 4),
    "all pairs, partial group": ([("bcc", 5, I.A_BCC_VERBATIM)], 0.5, 0, 4),
    "16 members per cell": ([("bcc", 12, B), ("bcc", 9, B)], 1.7, 0, 6),
    "16 members, beyond LDS": ([("bcc", 14, B)], 1.7, 0, 7),
    "wide rows, four wavefronts": ([("bcc", 12, B), ("bcc", 8, B)], 0.3, 3584, 8),
    "wide rows, two wavefronts": ([("bcc", 12, B), ("bcc", 8, B)], 0.3, 6144, 8),
}


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("case", list(CASES))
def test_rows_at_the_cuts(case, prec):
    import paper_2201_04622_amd.eamfe as E
    spec, skin, cap, ncell = CASES[case]
    reps = [I.Replica(lat, n, a, 300.0, 5.0, 3 + k) for k, (lat, n, a) in enumerate(spec)]
    rl = I.R_CUT + skin
    ctx, x0, arrs = make_ctx(reps, prec, 2, 256)
    L0 = spec[0][1] * spec[0][2]
    assert int(2.0 * L0 / rl) == ncell
    for sigma in (0.05, 0.4):
        pos = I.displaced(arrs["x0"], sigma, seed=11)
        x = E.to_soa(pos)
        got = []
        for lds in (True, False):
            ctx.set_list_builder(lds)
            ctx.neigh_build(x, skin, cap if lds or cap <= 3584 else 0)   # (the global builder's widest rows)
            nnb, nbr = ctx.copy_lists()
            got.append((nnb.cpu().numpy(), nbr.cpu().numpy()))
        assert np.array_equal(got[0][0], got[1][0])
        w = got[1][1].shape[1]
        assert np.array_equal(got[0][1][:, :w], got[1][1]) and (got[0][1][:, w:] == -1).all()
        nnb, nbr = got[0]
        off = 0
        for lat, n, a in spec:
            na = n ** 3 * (2 if lat == "bcc" else 4)
            L = n * a
            p = pos[off:off + na]
            d2 = np.zeros((na, na))
            for c in range(3):
                d = p[:, None, c] - p[None, :, c]
                d -= L * np.rint(d / L)
                d2 += d * d
            np.fill_diagonal(d2, 1e9)
            r = np.sqrt(d2)
            has = np.zeros((na, na), dtype=np.int32)
            for i in range(na):
                np.add.at(has[i], nbr[off + i, :nnb[off + i]] - off, 1)
            # the candidate test is widened, by less than 2e-3 A
            inside, outside = r < rl - 1e-9, r > rl + 2e-3
            assert (has[inside] == 1).all() and (has[outside] == 0).all() and has.max() <= 1
            off += na
        say(f"{case}, sigma {sigma}: mean row {nnb.mean():.1f}, max {nnb.max()}")
    ctx.close()


@pytest.mark.parametrize("prec,cells,n_rep,want", [
    (FP32, 4, 1, (16, 512)),      # 128 atoms
    (FP32, 11, 4, (8, 512)),      # 10,648 atoms: 2662 wavefronts at 16 lanes, 1331 at 8
    (FP32, 24, 7, (1, 512)),      # 193,536 atoms: 3024 wavefronts at one lane
    (FP64, 4, 1, (16, 64)),
    (FP64, 7, 2, (16, 64)),       # 1,372 atoms: 343 wavefronts
    (FP64, 14, 1, (16, 1024)),    # 5,488 atoms: 1372 wavefronts
])
def test_default_shape_by_size(prec, cells, n_rep, want):
    import torch

    import paper_2201_04622_amd.eamfe as E
    a = I.A_BCC_VERBATIM
    reps = [I.Replica("bcc", cells, a, 300.0, 5.0, 3 + k) for k in range(n_rep)]
    arrs = I.batch_arrays(reps)
    x = E.to_soa(I.displaced(arrs["x0"], 0.05, seed=5))
    out = []
    for shape in (None, (4, 256)):
        ctx = E.Context(0, prec)
        if shape:
            ctx.set_launch(*shape)
        ctx.eam_setup(I.synthetic_eam_knots())
        ctx.system_setup(reps, E.to_soa(arrs["x0"]))
        n_cu = torch.cuda.get_device_properties(0).multi_processor_count
        if n_cu == 256:
            assert ctx.get_launch() == (shape or want)
        ctx.neigh_build(x, 0.3, 0)
        f = torch.zeros_like(x)
        U = torch.zeros(n_rep, dtype=torch.float64, device="cuda")
        ctx.eam_forces(x, f, U)
        out.append((f.cpu().numpy(), U.cpu().numpy()))
        ctx.close()
    for qa, qb in zip(*out):
        if prec == FP32:
            assert np.array_equal(qa, qb)
        else:   # sums of under 1e3 terms in another order
            assert np.linalg.norm(qa - qb) <= 1e-12 * np.linalg.norm(qb)
