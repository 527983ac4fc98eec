"""md_nlist.block = 0 against every explicit workgroup size, at the atom counts where the choice
changes (256 and 512 tiles of 64 atoms at 4 and 2 lanes) and beside them, for each lane count:
forces bit for bit (an atom's sum does not know its workgroup), records to the fixed-point quantum
of 2^-36 eV per tile plus 1e-12 (FP64) or 1e-6 (FP32 tile partials) of the largest component."""
import numpy as np
import pytest

import mdinputs as mi
from tests.gpu_util import displaced, evv, md_ev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape,lanes", [((4, 4, 4), 1), ((4, 4, 4), 4), ((13, 13, 13), 2),
                                         ((16, 16, 16), 4), ((16, 16, 17), 4), ((16, 16, 32), 4),
                                         ((16, 17, 32), 4), ((16, 16, 16), 8), ((16, 16, 17), 8),
                                         ((6, 6, 6), 16), ((32, 32, 16), 2)])
def test_chosen_block(shape, lanes, prec):
    from paper_2511_22951_amd import md
    if prec and lanes == 16:
        pytest.skip("FP32 passes are not run at 16 lanes")
    pos, box = displaced(0, 3.615, 0.05, 11, shape=shape)
    plan = md.Plan([box], [len(pos)], 5.8)
    st = md.State(plan, pos, None, prec)
    nl = md.NeighborList(plan.n_atoms, 128, lanes)
    md.md_bin_cells(st)
    md.md_build_neighbors(st, nl)
    pot = md.EAMPotential.from_table(mi.tabulate_eam(mi.EAM_CU))
    table = pot.table(prec)
    lj = md.lj_params(0.167, 2.3, 5.5)

    def run(block):
        nl.set_block(block)
        out = []
        for call in (lambda ev: md.md_eam_forces(st, pot, nl, table=table, ev=ev),
                     lambda ev: md.md_lj_forces(st, lj, nl, ev=ev)):
            ev = md_ev(1)
            call(ev)
            st.check_flags()
            out.append((st.force.clone(), evv(ev)[0]))
        return out

    want = run(0)
    tiles = (len(pos) + 63) // 64
    for block in (256, 512, 1024):
        if block < 64 * lanes:
            continue
        for (f, e), (f0, e0) in zip(run(block), want):
            assert torch.equal(f, f0), block
            tol = (1e-6 if prec else 1e-12) * np.max(np.abs(e0)) + tiles * 2.0 ** -36
            assert np.all(np.abs(e - e0) <= tol), (block, e, e0)


@pytest.mark.parametrize("shape", [(16, 16, 64), (16, 16, 65), (4, 4, 4)])
@pytest.mark.parametrize("lanes", [2, 4, 8])
def test_chosen_block_coarse_table(shape, lanes):
    """A table of 61 intervals, at most a 1024-thread workgroup per CU (1024 tiles at 4 lanes) and
    more: forces bit for bit those of every explicit workgroup size."""
    from paper_2511_22951_amd import md
    pos, box = displaced(0, 3.615, 0.05, 11, shape=shape)
    plan = md.Plan([box], [len(pos)], 5.8)
    st = md.State(plan, pos, None, 0)
    nl = md.NeighborList(plan.n_atoms, 128, lanes)
    md.md_bin_cells(st)
    md.md_build_neighbors(st, nl)
    pot = md.EAMPotential.from_table(mi.tabulate_eam(mi.EAM_CU, K=62))
    table = pot.table(0)
    forces = []
    for block in (0, 256, 512, 1024):
        if block and block < 64 * lanes:
            continue
        nl.set_block(block)
        md.md_eam_forces(st, pot, nl, table=table)
        st.check_flags()
        forces.append(st.force.clone())
    assert all(torch.equal(f, forces[0]) for f in forces) and float(forces[0].abs().max()) > 0
