"""md_build_neighbors entry by entry: the lists of every atom, in order, against the candidate
order written out in numpy (stencil cell, then position in the cell; FP64 minimum image without
fused multiply-adds), where the build changes its form or its path:

  grids of 2 (both images of a pair in one cell), 3, 4 and more cells per axis, walled axes,
  cells of one atom, of more than 64 and with more candidates than fit the staging
  pairs at exactly r_ns (decided in FP64), lists longer than the LDS slots, max_neigh overflow
  positions that left their cells since the binning
"""
import numpy as np
import pytest

import mdinputs as mi

pytestmark = pytest.mark.gpu


def _stencil(c, nc, periodic):
    """Cells along one axis in stencil order (None: no cell)."""
    if periodic and nc < 3:
        return [t if t < nc else None for t in range(3)]
    out = []
    for q in (c - 1, c, c + 1):
        out.append(q % nc if periodic else (q if 0 <= q < nc else None))
    return out


def _model(pos, cell_start, box, nc, r_ns):
    lo, ln, per = box.as_arrays()
    inv = np.where(per != 0, 1.0 / ln, 0.0)
    rns2 = r_ns * r_ns
    lists = [None] * len(pos)
    for c in np.ndindex(*nc):
        a = (c[0] * nc[1] + c[1]) * nc[2] + c[2]
        atoms = np.arange(cell_start[a], cell_start[a + 1])
        if not len(atoms):
            continue
        st = [_stencil(c[k], nc[k], per[k]) for k in range(3)]
        cand = [np.arange(cell_start[q], cell_start[q + 1])
                for x in st[0] for y in st[1] for z in st[2]
                if x is not None and y is not None and z is not None
                for q in [(x * nc[1] + y) * nc[2] + z]]
        cand = np.concatenate(cand)
        for i in atoms:
            d = pos[cand] - pos[i]
            for k in range(3):
                if per[k]:
                    d[:, k] = d[:, k] - ln[k] * np.rint(d[:, k] * inv[k])
            r2 = (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]
            lists[i] = cand[(r2 < rns2) & (cand != i)]
    return lists


def _check(pos, box, r_ns, lanes=4, max_neigh=128, move=None):
    from paper_2511_22951_amd import _native as N
    from paper_2511_22951_amd import md
    import torch
    plan = md.Plan([box], [len(pos)], r_ns)
    st = md.State(plan, pos, None, N.MD_FP64)
    nl = md.NeighborList(plan.n_atoms, max_neigh, lanes)
    nl.neigh.fill_(-1)
    md.md_bin_cells(st)
    if move is not None:
        st.pos[:, :3] += torch.as_tensor(move(st.n), device="cuda")
    md.md_build_neighbors(st, nl)
    p = st.pos[:, :3].cpu().numpy()
    want = _model(p, st.cell_start.cpu().numpy(), box, plan.cells_per_axis[0], r_ns)
    got = nl.host_lists()
    longest = max(len(w) for w in want)
    status, info = st.read_flags()
    assert info["max_nneigh"] == longest
    assert bool(info["flags"] & N.FLAG_NEIGH_OVERFLOW) == (longest > nl.max_neigh)
    for i, (g, w) in enumerate(zip(got, want)):
        assert np.array_equal(g, w[:nl.max_neigh]), i
    return longest


def _crystal(cells, a, sigma, seed=1, periodic=(1, 1, 1)):
    pos, box = mi.fcc_lattice(*cells, a)
    pos = pos + np.random.default_rng(seed).normal(0.0, sigma, pos.shape)
    box = mi.Box(box.lo, box.len, periodic)
    pos = mi.wrap_into_box(pos, box)
    lo, ln, per = box.as_arrays()
    return np.where(per, pos, np.clip(pos, lo, lo + ln)), box


@pytest.mark.parametrize("lanes", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("cells", [(4, 4, 4), (5, 6, 8), (9, 7, 5)])
def test_thermal_crystals(cells, lanes):
    """2 x 2 x 2, 3 x 3 x 4 and 5 x 4 x 3 cells of 5.8 A and more."""
    _check(*_crystal(cells, 3.615, 0.1), 5.8, lanes)


@pytest.mark.parametrize("periodic", [(0, 0, 0), (1, 0, 1), (0, 1, 1), (1, 1, 0)])
def test_walled_axes(periodic):
    _check(*_crystal((6, 5, 8), 3.615, 0.1, periodic=periodic), 5.8)


def test_pairs_at_the_radius():
    """A perfect lattice whose third shell is the search radius to the last bit and beside it."""
    a = 4.0
    pos, box = mi.fcc_lattice(6, 6, 7, a)
    for r in (a * np.sqrt(1.5), np.nextafter(a * np.sqrt(1.5), 0.0),
              np.nextafter(a * np.sqrt(1.5), 9.0), a * np.sqrt(1.5) * (1 + 1e-7)):
        _check(pos, box, float(r))


def test_cells_as_wide_as_the_radius():
    pos, box = _crystal((5, 5, 5), 3.6, 0.05)  # 18 A: three cells of exactly 6 A
    _check(pos, box, 6.0)


def test_sparse_gas():
    """About one atom per cell, many cells empty."""
    box = mi.Box((-3.0, 2.0, 0.0), (40.0, 31.0, 55.0), (1, 1, 1))
    pos = np.random.default_rng(3).uniform(0.0, 1.0, (300, 3)) * box.len + box.lo
    assert _check(pos, box, 5.0, lanes=2) < 20


@pytest.mark.parametrize("lanes,max_neigh", [(1, 256), (4, 256), (2, 130), (8, 96)])
def test_dense_lists(lanes, max_neigh):
    """About 150 neighbours: past the LDS slots of an atom, and past max_neigh."""
    longest = _check(*_crystal((8, 6, 6), 3.615, 0.1), 7.2, lanes, max_neigh)
    assert 130 < longest < 256


def test_more_candidates_than_the_staging_holds():
    """About 300 neighbours, 2000 candidates and 75 atoms per cell (lists of up to 400)."""
    box = mi.Box((0.0, 0.0, 0.0), (24.0, 25.0, 30.0), (1, 1, 1))
    pos = np.random.default_rng(4).uniform(0.0, 1.0, (4000, 3)) * box.len
    assert _check(pos, box, 5.0, lanes=2, max_neigh=512) > 130


def test_uneven_density():
    """A dense slab in a thin gas: cells on both sides of the staging limit in one launch."""
    rng = np.random.default_rng(5)
    box = mi.Box((0.0, 0.0, 0.0), (20.0, 20.0, 80.0), (1, 1, 0))
    thin = rng.uniform(0.0, 1.0, (800, 3)) * box.len
    dense = rng.uniform(0.0, 1.0, (2500, 3)) * (20.0, 20.0, 12.0) + (0.0, 0.0, 30.0)
    _check(np.concatenate([thin, dense]), box, 5.0, lanes=4, max_neigh=512)


@pytest.mark.parametrize("scale", [0.1, 1.0, 4.0])
def test_positions_moved_since_the_binning(scale):
    """The lists hold the pairs within r_ns among the binned stencils, whatever the positions."""
    rng = np.random.default_rng(6)
    _check(*_crystal((6, 7, 8), 3.615, 0.1), 5.8,
           move=lambda n: rng.normal(0.0, scale, (n, 3)))


@pytest.mark.parametrize("lanes", [1, 4])
def test_batch_of_uneven_boxes(lanes):
    """About 370, 870 and 1700 candidates per cell in one launch: the lists of each box alone."""
    from paper_2511_22951_amd import md
    boxes = [_crystal(c, a, 0.1, seed) for c, a, seed in
             [((6, 6, 6), 3.95, 6), ((6, 6, 6), 3.45, 7), ((5, 5, 5), 3.45, 8), ((9, 7, 6), 3.7, 9)]]

    def lists(sel):
        plan = md.Plan([b for _, b in sel], [len(p) for p, _ in sel], 5.8)
        st = md.State(plan, np.concatenate([p for p, _ in sel]), None, 0)
        nl = md.NeighborList(plan.n_atoms, 128, lanes)
        md.md_bin_cells(st)
        md.md_build_neighbors(st, nl)
        st.check_flags()
        return nl.host_lists()

    got = lists(boxes)
    first = 0
    for p, b in boxes:
        for i, w in enumerate(lists([(p, b)])):
            assert np.array_equal(got[first + i] - first, w), (first, i)
        first += len(p)


def _gas(cells, n, seed, r_ns=5.0, edge=5.3):
    """n atoms anywhere in a periodic box of the given cells, several boxes' worth of seeds."""
    box = mi.Box((0.0, 0.0, 0.0), tuple(edge * c for c in cells), (1, 1, 1))
    pos = np.random.default_rng(seed).uniform(0.0, 1.0, (n, 3)) * box.len
    return pos, box, r_ns


@pytest.mark.parametrize("cells,n", [((3, 3, 3), 14), ((3, 3, 3), 27), ((4, 4, 4), 32),
                                     ((3, 4, 5), 40), ((4, 3, 3), 64)])
def test_dilute_periodic_gases(cells, n):
    """A few atoms on the smallest grids of the matrix form: the runs of stencil cells that
    follow one another in memory begin and end at empty cells, at the first atom and at wraps."""
    for seed in range(24):
        _check(*_gas(cells, n, seed), lanes=1 + seed % 2)


def test_first_cell_of_the_box_after_its_image():
    """Cell (1, 1, 0) reads (0, 0, 2) through the boundary, then (0, 0, 0), which starts at atom 0
    without an image, with (0, 1, 0) and (0, 1, 1) empty and (0, 1, 2) next in memory."""
    e = 5.3
    box = mi.Box((0.0, 0.0, 0.0), (3 * e, 3 * e, 3 * e), (1, 1, 1))
    at = {(0, 0, 0): [(4.9, 4.8, 0.4), (4.5, 4.9, 0.9)], (0, 0, 2): [(4.7, 4.7, 15.5)],
          (0, 1, 2): [(5.0, 5.6, 15.4), (5.1, 6.0, 15.0)], (1, 1, 0): [(5.5, 5.5, 0.2), (5.7, 5.4, 1.0)]}
    pos = np.array([x for cell in at for x in at[cell]])
    cell = np.repeat(list(at), [len(at[c]) for c in at], axis=0)
    assert np.array_equal(np.floor(pos / e).astype(int), cell)
    for lanes in (1, 4):
        assert _check(pos, box, 5.0, lanes) == len(pos) - 1


@pytest.mark.parametrize("cells", [3, 4])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("sign", [1, -1])
def test_own_atom_moved_out_of_its_cell(cells, axis, sign):
    """An atom that left its cell for the far side of the next one, and one of the cell on the
    other side: 2.2 cell edges apart, 0.8 through the boundary of a three-cell axis."""
    w = 6.2
    box = mi.Box((0.0, 0.0, 0.0), (cells * w,) * 3, (1, 1, 1))
    a = np.full(3, 1.5 * w)  # the centre of cell (1, 1, 1)
    b = a.copy()
    b[axis] -= sign * 1.2 * w
    pos = np.stack([a, b])
    cell = np.floor(pos / w).astype(int) % cells
    order = np.lexsort(cell.T[::-1])

    def move(n):
        d = np.zeros((2, 3))
        d[0, axis] = sign * w
        return d[order]

    assert _check(pos, box, 5.8, move=move) == (1 if cells == 3 else 0)


# Grids of more than 8192 cells go by blocks that take several cells in turn where atoms are fewer
# than cells or the rebuild is conditional: beside that size, with chunks of 2 and of 64 cells, past
# 64 x 8192 cells (blocks stride), with two cells on an axis and walls (the FP64 form in the loop)
@pytest.mark.parametrize("cells,n,periodic", [
    ((16, 16, 32), 3000, (1, 1, 1)), ((16, 19, 27), 3000, (1, 1, 1)), ((16, 19, 27), 8207, (1, 0, 1)),
    ((16, 19, 27), 8208, (1, 1, 1)), ((2, 3, 1021), 4000, (1, 1, 1)), ((2, 5, 900), 6000, (1, 0, 0)),
    ((70, 85, 90), 2000, (1, 1, 1))])
def test_large_sparse_grids(cells, n, periodic):
    pos, box, r_ns = _gas(cells, n, seed=n)
    _check(pos, mi.Box(box.lo, box.len, periodic), r_ns, lanes=2)


def test_more_cells_than_blocks_of_one_launch():
    """17.6 million cells (a block each would be 2^32 threads and more): pairs found by brute force."""
    from paper_2511_22951_amd import _native as N
    from paper_2511_22951_amd import md
    pos, box, r_ns = _gas((260, 260, 260), 300, seed=1)
    pos[150:] = pos[:150] + np.random.default_rng(2).normal(0.0, 2.0, (150, 3))
    pos[:3] = ((0.1, 0.2, 0.3), (1377.9, 0.3, 0.2), (1377.8, 1377.5, 1377.9))  # the corners
    pos = mi.wrap_into_box(pos, box)
    plan = md.Plan([box], [len(pos)], r_ns)
    assert plan.n_cells > 1 << 24
    st = md.State(plan, pos, None, N.MD_FP64)
    nl = md.NeighborList(plan.n_atoms, 64, 2)
    md.md_bin_cells(st)
    md.md_build_neighbors(st, nl)
    st.check_flags()
    p, ln = st.pos[:, :3].cpu().numpy(), np.asarray(box.len)
    d = p[None] - p[:, None]
    d -= ln * np.rint(d / ln)
    near = (d * d).sum(-1) < r_ns * r_ns
    np.fill_diagonal(near, False)
    assert near.sum() > 200
    for i, got in enumerate(nl.host_lists()):
        assert np.array_equal(np.sort(got), np.flatnonzero(near[i])), i


@pytest.mark.parametrize("shape", [(18, 18, 18), (4, 40, 60)])
def test_conditional_rebuild_of_a_large_grid(shape):
    """9261 and 12,696 cells, two and three atoms each: nothing is written before a drift exceeds
    half the skin, and the lists of the moved positions after."""
    from paper_2511_22951_amd import _native as N
    from paper_2511_22951_amd import md
    import torch
    pos, box = _crystal(shape, 3.615, 0.1)
    plan = md.Plan([box], [len(pos)], 3.0)
    assert plan.n_cells > 8192 and plan.n_atoms > plan.n_cells
    vel = np.random.default_rng(3).normal(0.0, 1.0, pos.shape)
    st = md.State(plan, pos, vel, N.MD_FP64)
    nl = md.NeighborList(plan.n_atoms, 32, 2)
    md.md_bin_cells(st)
    md.md_build_neighbors(st, nl)
    st.check_flags()
    nl.neigh.fill_(-1)
    for half_skin, moves in ((1.0, False), (1e-6, True)):
        md.md_verlet_step(st, N.MD_KICK_DRIFT, 1e-2, 1.0 / 40.0, half_skin=half_skin)
        md.md_bin_cells(st, N.MD_IF_FLAGGED)
        md.md_build_neighbors(st, nl, N.MD_IF_FLAGGED)
        assert bool((nl.neigh == -1).all()) != moves
    assert st.check_flags()["n_rebuilds"] == 2
    p = st.pos[:, :3].cpu().numpy()
    want = _model(p, st.cell_start.cpu().numpy(), box, plan.cells_per_axis[0], 3.0)
    for i, (g, w) in enumerate(zip(nl.host_lists(), want)):
        assert np.array_equal(g, w), i


@pytest.mark.parametrize("scale", [0.0, 0.02, 2.0])
@pytest.mark.parametrize("periodic", [(1, 1, 1), (1, 0, 1)])
def test_dense_cells_of_few_per_axis(scale, periodic):
    """2250 candidates per cell on 3 x 3 x 4 cells: the FP64 form by the stencil's images, or by the
    minimum image where positions left their cells since the binning."""
    box = mi.Box((1.0, -2.0, 0.0), (15.6, 16.5, 21.0), periodic)
    rng = np.random.default_rng(12)
    pos = rng.uniform(0.0, 1.0, (3000, 3)) * box.len + box.lo
    _check(pos, box, 5.0, lanes=2, max_neigh=512, move=lambda n: rng.normal(0.0, scale, (n, 3)))
