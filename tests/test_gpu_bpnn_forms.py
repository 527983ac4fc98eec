"""GPU parity of md_bpnn_forces with the oracle over the symmetry-function sets its two forms
take (shared squarings and an exponential table, or library exp and powers), and over the
numbers of neighbours and atoms where its pair enumeration and its split over wavefronts change.

Tolerances are those of the default set's parity test: forces 1e-10 (Frobenius), atomic
energies 1e-11 of the largest.
"""
import numpy as np
import pytest

import mdinputs as mi
from oracle import bpnn

pytestmark = pytest.mark.gpu


def _params(zetas, lams, etas, n_g2=8):
    p = mi.bpnn_params()
    combos = [(z, l, e) for e in etas for z in zetas for l in lams]
    g4 = np.array(combos, np.float64).reshape(-1, 3)
    rng = np.random.default_rng(5)
    ng = n_g2 + len(g4)
    w = rng.normal(0.0, 1.0, (ng, 10)) / np.sqrt(ng)
    w[:n_g2] /= 10.0
    w[n_g2:] /= 100.0
    p.update(g2_eta=p["g2_eta"][:n_g2], g4_zeta=g4[:, 0], g4_lambda=g4[:, 1], g4_eta=g4[:, 2],
             w01=w)
    return p


SETS = {
    "default": mi.bpnn_params(),
    "one_zeta_one_sign": _params([2.0], [1.0], [0.01, 0.05]),
    "minus_sign_only": _params([1.0, 8.0], [-1.0], [0.02]),
    "no_zero_eta_unsorted": _params([16.0, 1.0, 4.0], [-1.0, 1.0], [0.06, 0.004, 0.03]),
    "zero_eta_last": _params([2.0, 1.0], [1.0, -1.0], [0.05, 0.01, 0.0]),
    "eight_etas": _params([1.0, 4.0], [1.0, -1.0], [0.0, 0.01, 0.02, 0.03, 0.05, 0.07, 0.09, 0.11]),
    "repeated_functions": _params([1.0, 1.0, 2.0], [1.0, -1.0], [0.01, 0.01]),
    "table_limit": _params([1.0, 2.0], [1.0], [0.1185, -0.1185]),
    "past_table_limit": _params([1.0, 2.0], [1.0], [0.1186, 0.4]),
    "odd_zeta": _params([1.0, 3.0, 16.0], [1.0, -1.0], [0.0, 0.03]),
    "fractional_zeta": _params([1.5, 4.0], [1.0, -1.0], [0.01, 0.03]),
    "five_zetas": _params([1.0, 2.0, 4.0, 8.0, 16.0], [1.0], [0.0, 0.02]),
    "seven_etas_odd_zeta": _params([1.0, 3.0], [1.0, -1.0],
                                   [0.0, 0.01, 0.02, 0.03, 0.05, 0.07, 0.09]),
    "no_radial": _params([1.0, 2.0, 4.0], [1.0, -1.0], [0.01], n_g2=0),
    "radial_only": _params([], [], [], n_g2=8),
}


def _gpu(pos, box, p):
    import torch
    from paper_2511_22951_amd import _native as N
    from paper_2511_22951_amd import md
    plan = md.Plan([box], [len(pos)], p["r_cut"] + 0.3)
    st = md.State(plan, pos, None, N.MD_FP64)
    nl = md.NeighborList(plan.n_atoms, 256, 4)
    md.md_bin_cells(st)
    md.md_build_neighbors(st, nl)
    e = torch.empty(st.n, dtype=torch.float64, device="cuda")
    ev = md.ev_buffer(1, 1)
    md.md_bpnn_forces(st, md.BPNNPotential(p), nl, ev=ev, ev_cap=1, e_atom=e)
    st.check_flags()
    return st.forces(), e.cpu().numpy()[st._order()], md.ev_values(ev)[0, 0]


def _compare(pos, box, p):
    f, e, rec = _gpu(pos, box, p)
    E, eo, fo, w = bpnn.forces(pos, box, p)
    assert np.linalg.norm(f - fo) <= 1e-10 * np.linalg.norm(fo)
    assert np.abs(e - eo).max() <= 1e-11 * np.abs(eo).max()
    return rec, E, w


@pytest.mark.parametrize("name", list(SETS))
def test_symmetry_function_sets(name):
    s = mi.bpnn_copper(cells=4)
    rec, E, w = _compare(s.pos, s.box, SETS[name])
    assert abs(rec[0] - E) <= 1e-11 * abs(E)
    assert np.abs(rec[1:7] - w).max() <= 1e-10 * np.abs(w).max()


# neighbours per atom: a cluster of n atoms all within the cutoff has n - 1; 0 and 1 have no
# pairs, 2 one pair, 63..65 cross the wavefront, 127 and 128 the most that are kept (forces and
# energies: the records' resolution of 2^-36 eV is coarser than a virial of two atoms needs)
@pytest.mark.parametrize("neighbours", [0, 1, 2, 3, 11, 12, 63, 64, 65, 127, 128])
def test_neighbour_counts(neighbours):
    rng = np.random.default_rng(neighbours)
    n = neighbours + 1
    grid = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), -1).reshape(-1, 3)
    grid = grid[np.argsort(((grid - 2.5) ** 2).sum(1), kind="stable")][:n]
    pos = 12.0 + 0.85 * grid + rng.normal(0.0, 0.02, (n, 3))  # (all within 6 A of each other)
    assert n == 1 or max(np.linalg.norm(pos - q, axis=1).max() for q in pos) < 6.0
    box = mi.Box((0.0, 0.0, 0.0), (30.0, 30.0, 30.0), (1, 1, 1))
    p = mi.bpnn_params()
    if neighbours:
        _compare(pos, box, p)
    else:
        f, e, _ = _gpu(pos, box, p)
        eo = bpnn.forces(pos, box, p)[1]
        assert np.all(f == 0.0) and np.abs(e - eo).max() <= 1e-11 * np.abs(eo).max()


def test_several_atoms_per_wavefront():
    """19,200 atoms (two per wavefront) as 5 x 5 x 3 copies of a displaced 256-atom box: every
    copy has that box's forces and energies."""
    s = mi.bpnn_copper(cells=4)
    p = s.extra["bpnn"]
    f1, e1, _ = _gpu(s.pos, s.box, p)
    L = np.asarray(s.box.len)
    shifts = np.stack(np.meshgrid(range(5), range(5), range(3), indexing="ij"), -1).reshape(-1, 3)
    pos = np.concatenate([s.pos + L * k for k in shifts])
    box = mi.Box((0.0, 0.0, 0.0), tuple(L * (5, 5, 3)), (1, 1, 1))
    f, e, rec = _gpu(mi.wrap_into_box(pos, box), box, p)
    f, e = f.reshape(len(shifts), -1, 3), e.reshape(len(shifts), -1)
    assert np.abs(f - f1).max() <= 1e-10 * np.abs(f1).max()
    assert np.abs(e - e1).max() <= 1e-11 * np.abs(e1).max()
    assert abs(rec[0] - len(shifts) * e1.sum()) <= 1e-11 * abs(rec[0])


@pytest.mark.parametrize("zeta", [512.0, 1024.0, 1024.5])
@pytest.mark.parametrize("lams", [[1.0], [-1.0], [1.0, -1.0]])
def test_powers_near_the_largest_double(zeta, lams):
    """2^zeta at and past the range of a double, which only a pair of neighbours in one direction
    reaches: a centred tetrahedron has none, and most lanes have no pair at all."""
    c = np.array([[0.0, 0.0, 0.0], [1.0, 1.0, 1.0], [1.0, -1.0, -1.0], [-1.0, 1.0, -1.0],
                  [-1.0, -1.0, 1.0]])
    pos = 12.0 + 1.3 * c + np.random.default_rng(8).normal(0.0, 0.02, c.shape)
    box = mi.Box((0.0, 0.0, 0.0), (24.0, 24.0, 24.0), (1, 1, 1))
    _compare(pos, box, _params([zeta, 2.0], lams, [0.0, 0.01]))
