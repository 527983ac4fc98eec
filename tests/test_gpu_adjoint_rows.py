"""The adjoint by per-atom rows (4 lanes per atom and more, coefficients that fit) against the
adjoint by bins (2 lanes, the same snapshots): coefficient counts of the smallest splines, around
one and two columns per lane and past the rows' limit, with and without the density Jacobian,
tiles full and with remainders.  Both sum the same terms in FP64 in different orders: within
1e-12 of the largest entry of each function's gradient.  The LJ pass with a list addressed with 64
bits (streamed) against the same list in 32 bits: the same bits."""
from types import SimpleNamespace

import numpy as np
import pytest

import mdinputs as mi

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _snapshots(big=False):
    """Three boxes (17 tiles), or one more of 250 tiles: past 256, where the adjoint without the
    Jacobian goes by rows too."""
    rng = np.random.default_rng(21)
    out = []
    for cells in ((4, 4, 4), (5, 5, 5), (4, 4, 5)) + (((20, 20, 10),) if big else ()):
        pos, box = mi.fcc_lattice(*cells, 3.7)
        out.append(SimpleNamespace(pos=mi.wrap_into_box(pos + rng.normal(0, 0.08, pos.shape), box),
                                   box=box))
    return out


def _potential(n):
    from paper_2511_22951_amd import md
    r_lo, r_cut = 1.5, 5.5
    r = r_lo + (np.arange(n) - 1) * (r_cut - r_lo) / (n - 3)
    e = (np.arange(n) - 1) * 4.0 / (n - 3)
    return md.EAMPotential(np.exp(-2.0 * r) - 0.1 * np.exp(-r), np.exp(-r), 0.1 * e * e - e, r_lo,
                           (r_cut - r_lo) / (n - 3), 0.0, 4.0 / (n - 3), r_cut)


@pytest.mark.parametrize("jac", [False, True])
@pytest.mark.parametrize("n", [6, 7, 63, 64, 65, 100, 128, 129, 300])
def test_gradient_by_rows(n, jac):
    from paper_2511_22951_amd import fm
    snaps, pot = _snapshots(not jac), _potential(n)
    rng = np.random.default_rng(n)
    cot = [rng.normal(size=s.pos.shape) for s in snaps]
    grads = {}
    for lanes in (2, 4, 8, 16):
        batch = fm.SnapshotBatch(snaps, 5.8, lanes=lanes, density_jacobian=jac)
        batch.forces(pot)
        try:
            g = batch.backward(pot, batch.to_current_order(np.concatenate(cot)))
        except Exception as err:  # the bins of many waves do not fit: refused, as ever
            assert lanes > 4 and n > 128 and "status -1" in str(err)
            continue
        batch.state.check_flags()
        grads[lanes] = g.cpu().numpy()
    assert 4 in grads
    for lanes, g in grads.items():
        for k in range(3):
            want = grads[2][k * n:(k + 1) * n]
            scale = np.max(np.abs(want))
            assert scale > 0.0
            assert np.max(np.abs(g[k * n:(k + 1) * n] - want)) <= 1e-12 * scale, (lanes, k)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_coefficients_no_pair_reads(bad):
    """A non-finite rho coefficient below every distance: both ways leave it out."""
    from paper_2511_22951_amd import fm
    snaps, pot = _snapshots(True), _potential(64)
    pot.coef[1][:2] = bad
    cot = np.random.default_rng(3).normal(size=(sum(len(s.pos) for s in snaps), 3))
    grads = []
    for lanes in (2, 4):
        batch = fm.SnapshotBatch(snaps, 5.8, lanes=lanes, density_jacobian=False)
        batch.forces(pot)
        grads.append(batch.backward(pot, batch.to_current_order(cot)).cpu().numpy())
    assert np.all(np.isfinite(grads[0]))
    assert np.max(np.abs(grads[1] - grads[0])) <= 1e-12 * np.max(np.abs(grads[0]))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("lanes", [1, 4])
def test_lj_streamed_list(lanes, prec):
    from paper_2511_22951_amd import md
    pos, box = mi.fcc_lattice(8, 8, 8, 5.26)
    pos = mi.wrap_into_box(pos + np.random.default_rng(2).normal(0, 0.1, pos.shape), box)
    plan = md.Plan([box], [len(pos)], 8.8)
    out = []
    for max_neigh in (128, 65536):  # 2^18 and 2^27 entries
        st = md.State(plan, pos, None, prec)
        nl = md.NeighborList(plan.n_atoms, max_neigh, lanes)
        md.md_bin_cells(st)
        md.md_build_neighbors(st, nl)
        md.md_lj_forces(st, md.lj_params(0.0104, 3.4, 8.5), nl)
        st.check_flags()
        out.append(st.force.clone())
    assert torch.equal(out[0], out[1]) and float(out[0].abs().max()) > 0


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("lanes", [1, 4])
def test_lj_list_past_32_bits(lanes, prec):
    """2048 atoms with room for 524,288 neighbours each, 2^30 entries: addressed with 64 bits and
    streamed, the same bits as an ordinary list's."""
    from paper_2511_22951_amd import md
    pos, box = mi.fcc_lattice(8, 8, 8, 5.26)
    pos = mi.wrap_into_box(pos + np.random.default_rng(2).normal(0, 0.1, pos.shape), box)
    plan = md.Plan([box], [len(pos)], 8.8)
    out = []
    for max_neigh in (128, 1 << 19):
        st = md.State(plan, pos, None, prec)
        nl = md.NeighborList(plan.n_atoms, max_neigh, lanes)
        md.md_bin_cells(st)
        md.md_build_neighbors(st, nl)
        md.md_lj_forces(st, md.lj_params(0.0104, 3.4, 8.5), nl)
        st.check_flags()
        out.append(st.force.clone())
        del nl
    assert torch.equal(out[0], out[1]) and float(out[0].abs().max()) > 0


def test_lj_streamed_by_what_is_read():
    """878,080 atoms read 7e7 entries (streamed), as 7 x 14 x 7 copies of a box of 1280 atoms, which is
    not: every copy has its forces, to the rounding of the sums (the copies' positions are rounded
    to the larger box, FP64)."""
    from paper_2511_22951_amd import md
    lj = md.lj_params(0.0104, 3.4, 8.5)
    small, box = mi.fcc_lattice(5, 8, 8, 5.26)
    small = mi.wrap_into_box(small + np.random.default_rng(2).normal(0, 0.1, small.shape), box)
    copies = (7, 14, 7)
    L = np.asarray(box.len)
    shift = np.stack(np.meshgrid(*[range(c) for c in copies], indexing="ij"), -1).reshape(-1, 3)
    big = (small[None] + shift[:, None] * L).reshape(-1, 3)
    out = []
    for pos, b in ((small, box), (big, mi.Box((0.0, 0.0, 0.0), tuple(L * copies), (1, 1, 1)))):
        plan = md.Plan([b], [len(pos)], 8.8)
        st = md.State(plan, mi.wrap_into_box(pos, b), None, 0)
        nl = md.NeighborList(plan.n_atoms, 128, 1)
        md.md_bin_cells(st)
        md.md_build_neighbors(st, nl)
        md.md_lj_forces(st, lj, nl)
        st.check_flags()
        out.append(st.forces())
    assert len(big) * (4 * 4.19 * len(big) / plan.n_cells + 32) >= 1 << 28
    # positions up to 589 A: 2^-44 A of rounding each, times the slope of the pair force (below 1 eV / A^2
    # at the closest pair, 3.24 A: 24 eps / s^2 (26 (s/r)^14 - 7 (s/r)^8)) and 90 pairs
    assert np.abs(out[1].reshape(-1, len(small), 3) - out[0]).max() < 90 * 2.0 ** -43
