"""Both row builders on candidate streams longer than one register chunk, where
rows grow piece by piece: streams ending at and one past a piece (768) and a
chunk (1024), all-pairs boxes of such sizes, one replica whose cells are
dealt out to many wavefronts and many replicas that fill the chip, and rows that
overflow in the middle of a stream.  Rows of both builders are equal slot
for slot and hold exactly the brute-force pairs."""
import numpy as np
import pytest

from gpu_common import make_ctx, say
from paper_2201_04622_amd import inputs as I

pytestmark = pytest.mark.gpu
FP32 = 1


def _sites(n_cells, atoms):
    """A bcc crystal thinned to `atoms` (a stencil of a box of five cells per edge streams all of them)."""
    full = 2 * n_cells ** 3
    gone = np.random.default_rng(atoms).permutation(full)[:full - atoms]
    return I.Replica("bcc", n_cells, I.A_BCC_STABLE, 300.0, 5.0, atoms, vacancies=tuple(int(g) for g in gone))


def _brute(reps, pos, rl):
    """Which pairs are inside and outside the list radius, per replica."""
    off = 0
    for r in reps:
        p, L = pos[off:off + r.natoms], r.box
        d = p[:, None] - p[None]
        d -= L * np.rint(d / L)
        dist = np.sqrt((d * d).sum(-1))
        np.fill_diagonal(dist, 1e9)
        yield off, dist < rl - 1e-9, dist > rl + 2e-3   # the candidate test is widened by less than 2e-3 A
        off += r.natoms


def _check(reps, pos, skin, cap=0, builders=(True, False)):
    import paper_2201_04622_amd.eamfe as E
    ctx, _, _ = make_ctx(reps, FP32, 2, 256)
    x = E.to_soa(pos)
    got = []
    for lds in builders:
        ctx.set_list_builder(lds)
        ctx.neigh_build(x, skin, cap)
        nnb, nbr = ctx.copy_lists()
        got.append((nnb.cpu().numpy(), nbr.cpu().numpy()))
    ctx.close()
    nnb, nbr = got[0]
    for other in got[1:]:
        w = min(nbr.shape[1], other[1].shape[1])
        assert np.array_equal(nnb, other[0]) and np.array_equal(nbr[:, :w], other[1][:, :w])
    for off, inside, outside in _brute(reps, pos, I.R_CUT + skin):
        has = np.zeros(inside.shape, dtype=np.int32)
        for i in range(len(has)):
            np.add.at(has[i], nbr[off + i, :nnb[off + i]] - off, 1)
        assert (has[inside] == 1).all() and (has[outside] == 0).all() and has.max() <= 1
    return nnb


@pytest.mark.parametrize("atoms", [769, 1025, 1458])
@pytest.mark.parametrize("skin,cells", [(0.65, 5), (1.9, 4)])   # streams of all atoms; all-pairs rows
def test_pieces_of_a_stream(atoms, skin, cells):
    reps = [_sites(9, atoms)]
    assert int(2.0 * reps[0].box[0] / (I.R_CUT + skin)) == cells
    nnb = _check(reps, I.displaced(reps[0].sites(), 0.1, seed=3), skin)
    say(f"{atoms} atoms, {cells} cells per edge: mean row {nnb.mean():.1f}, max {nnb.max()}")


def test_two_pieces_exactly():
    for atoms in (1536, 1537):   # twice 768, and one more
        reps = [_sites(10, atoms)]
        _check(reps, I.displaced(reps[0].sites(), 0.1, seed=4), 1.4)   # five cells per edge


@pytest.mark.parametrize("n_rep", [1, 12])
@pytest.mark.parametrize("n", [9, 13])   # through LDS by default, and beyond it
def test_items_dealt_to_wavefronts(n, n_rep):
    reps = [I.Replica("bcc", n, I.A_BCC_STABLE, 300.0, 5.0, 7 + q) for q in range(n_rep)]
    pos = np.concatenate([I.displaced(r.sites(), 0.08, seed=20 + q) for q, r in enumerate(reps)])
    if n_rep > 1 and n > 9:   # the brute force of a few is enough
        reps, pos = reps[:4], pos[:4 * reps[0].natoms]
    _check(reps, pos, 0.65)


@pytest.mark.parametrize("lds", [True, False])
def test_overflow_within_a_long_stream(lds):
    import paper_2201_04622_amd.eamfe as E
    reps = [I.Replica("bcc", 9, I.A_BCC_STABLE, 300.0, 5.0, 7)]
    pos = I.displaced(reps[0].sites(), 0.05, seed=9)
    ctx, _, _ = make_ctx(reps, FP32, 2, 256)
    ctx.set_list_builder(lds)
    x = E.to_soa(pos)
    with pytest.raises(E.EamfeError) as e:
        ctx.neigh_build(x, 0.65, 96)          # rows are about 250 long
    assert e.value.code == 6
    assert ctx.list_stats()[1:] == (96, 96)   # cut at the capacity
    nnb, nbr = (t.cpu().numpy() for t in ctx.copy_lists())
    ctx.neigh_build(x, 0.65, 0)
    full = ctx.copy_lists()[1].cpu().numpy()
    assert (nnb == 96).all() and np.array_equal(nbr, full[:, :96])
    ctx.close()


@pytest.mark.parametrize("atoms", [500, 1458])   # one chunk, and pieces
def test_more_members_than_a_wavefront_in_one_cell(atoms):
    reps = [_sites(9, atoms)]
    rng = np.random.default_rng(6)
    pos = I.displaced(reps[0].sites(), 0.1, seed=3)
    crowd = rng.permutation(atoms)[:140]
    # the crowd in the middle of one cell of edge 3.54 A (five per box edge)
    pos[crowd] = 1.5 * reps[0].box / 5 + rng.uniform(-1.0, 1.0, (140, 3))
    nnb = _check(reps, pos, 0.65)
    assert nnb[crowd].min() >= 139
