"""GPU parity of md_atom_observables (EAM) with the oracle at every list layout and on both sides
of the limit of coefficients kept in LDS, in a batch of two boxes with ragged tiles, and its
table-range flag.  Tolerances are those of the one-layout test: energies 1e-12, virials 1e-11 of
the largest entry.
"""
import numpy as np
import pytest

import mdinputs as mi
from oracle import core

pytestmark = pytest.mark.gpu


def _state(systems, lanes):
    from paper_2511_22951_amd import _native as N
    from paper_2511_22951_amd import md
    plan = md.Plan([s.box for s in systems], [len(s.pos) for s in systems], mi.EAM_CU.r_cut + 0.3)
    st = md.State(plan, np.concatenate([s.pos for s in systems]), None, N.MD_FP64)
    nl = md.NeighborList(plan.n_atoms, 128, lanes)
    md.md_bin_cells(st)
    md.md_build_neighbors(st, nl)
    return st, nl


@pytest.mark.parametrize("lanes,K", [(1, 2000), (2, 2000), (4, 2000), (8, 2000), (16, 2000),
                                     (2, 4), (4, 4094), (4, 4095)])
def test_layouts_and_table_sizes(lanes, K):
    from paper_2511_22951_amd import md
    systems = [mi.eam_copper(cells=5, seed=3), mi.eam_copper(cells=4, seed=4)]
    # (four samples: a coarse potential, but a valid spline)
    table = mi.tabulate_eam(mi.EAM_CU, K=K)
    st, nl = _state(systems, lanes)
    e, w, rf = md.md_atom_observables(st, nl, eam=md.EAMPotential.from_table(table))
    o = np.argsort(st.id.cpu().numpy(), kind="stable")
    e, w = e.cpu().numpy()[o], w.cpu().numpy().T[o]
    pot = core.EAMPotential.from_table(table)
    r = [core.eam(s.pos, s.box, pot) for s in systems]
    eo, wo = np.concatenate([q.e_atom for q in r]), np.concatenate([q.w_atom for q in r])
    assert np.abs(e - eo).max() < 1e-12 * np.abs(eo).max()
    assert np.abs(w - wo).max() < 1e-11 * np.abs(wo).max()


@pytest.mark.parametrize("K", [2000, 4095])
def test_pair_below_the_table_is_flagged(K):
    from paper_2511_22951_amd import _native as N
    from paper_2511_22951_amd import md
    s = mi.eam_copper(cells=4)
    pot = md.EAMPotential.from_table(mi.tabulate_eam(mi.EAM_CU, K=K, rho_hi=1e6))
    for close in (False, True):
        if close:
            s.pos = s.pos.copy()
            s.pos[7] = s.pos[6] + (0.9, 0.0, 0.0)  # the tables start at 1 A
        st, nl = _state([s], 4)
        md.md_atom_observables(st, nl, eam=pot)
        assert bool(st.read_flags()[1]["flags"] & N.FLAG_TABLE_RANGE) == close


@pytest.mark.parametrize("n", [2002, 4097])
@pytest.mark.parametrize("lanes", [1, 4])
def test_atoms_at_one_place(n, lanes):
    """Two atoms at one place, splines that reach r = 0 (the same coefficients on both sides: no
    fit, no extrapolation), on both sides of the limit of coefficients kept in LDS: energies,
    densities and F' are finite and reach their neighbours' virials; only the two atoms' own
    virials have no value."""
    from paper_2511_22951_amd import md
    s = mi.eam_copper(cells=4)
    s.pos = s.pos.copy()
    s.pos[7] = s.pos[6]
    h, e_h = 5.5 / (n - 3), 40.0 / (n - 3)
    x, rho = (np.arange(n) - 1) * h, (np.arange(n) - 1) * e_h
    c = (np.exp(-x) - 0.02 * x, np.exp(-0.7 * x), 0.01 * rho * rho - 0.5 * rho)
    st, nl = _state([s], lanes)
    e, w, rf = md.md_atom_observables(st, nl, eam=md.EAMPotential(*c, 0.0, h, 0.0, e_h, 5.5))
    st.check_flags()
    o = np.argsort(st.id.cpu().numpy(), kind="stable")
    e, w, rf = e.cpu().numpy()[o], w.cpu().numpy().T[o], rf.cpu().numpy()[:, o]
    f = [core.SplineFunc(q, 0.0, d) for q, d in zip(c, (h, h, e_h))]
    r = core.eam(s.pos, s.box, core.EAMPotential(*f, 5.5))
    pair = np.isin(np.arange(len(e)), (6, 7))
    for got, want in ((e, r["e_atom"]), (rf[0], r["rhobar"]), (rf[1], r["fp"])):
        assert np.abs(got - want).max() < 1e-12 * np.abs(want).max()
    assert np.isnan(w[pair]).all() and np.isnan(r["w_atom"][pair]).all()
    assert np.abs(w - r["w_atom"])[~pair].max() < 1e-11 * np.abs(r["w_atom"][~pair]).max()
