"""md_bin_cells against numpy (wrap, cell, stable order by cell and id; FP64, operation by
operation, so every array is compared exactly) on each of its routes: one block (at most 32 tiles,
64 where the rebuild is conditional, and 4096 cells), four launches, and grids past 131,072 cells;
at the sizes beside those limits, in batches, and called again on its own result."""
import numpy as np
import pytest

import mdinputs as mi

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _expect(plan, pos, vel, ids):
    cell = np.empty(len(pos), np.int64)
    x = pos.copy()
    for r in range(plan.n_rep):
        d = plan.host_domains[r]
        s = slice(plan.atom_off[r], plan.atom_off[r + 1])
        c = 0
        for a in range(3):
            if d.periodic[a]:
                y = x[s, a] - d.len[a] * np.floor((x[s, a] - d.lo[a]) / d.len[a])
                x[s, a] = np.where(y >= d.lo[a] + d.len[a], d.lo[a], y)
            k = np.clip(np.floor((x[s, a] - d.lo[a]) * d.inv_w[a]), 0, d.nc[a] - 1)
            c = c * d.nc[a] + k.astype(np.int64)
        cell[s] = c + d.cell_off
    order = np.lexsort((ids, cell))
    start = np.searchsorted(cell[order], np.arange(plan.n_cells + 1))
    return x[order], vel[order], ids[order], start


def _compare(st, plan, want):
    x, v, i, start = want
    assert np.array_equal(st.id.cpu().numpy(), i)
    assert np.array_equal(st.pos[:, :3].cpu().numpy(), x)
    assert np.array_equal(st.pos_ref.t().cpu().numpy(), x)
    assert np.array_equal(st.vel.t().cpu().numpy(), v)
    assert np.array_equal(st.cell_start.cpu().numpy(), start)


# atoms of each box, edge per box (A), periodic
CASES = [([1], 20.0, (1, 1, 1)), ([63, 65, 1], 25.0, (1, 0, 1)), ([2048], 40.0, (1, 1, 1)),
         ([2049], 40.0, (0, 1, 1)), ([64] * 32, 24.0, (1, 1, 1)), ([1] * 33, 24.0, (1, 1, 1)),
         ([4096], 50.0, (1, 1, 0)), ([4097], 50.0, (1, 1, 1)), ([500], 92.5, (1, 1, 1)),
         ([500], 98.0, (1, 1, 1)), ([30000, 7, 9000], 90.0, (1, 1, 1)), ([9000], 293.0, (1, 1, 1)),
         ([9000], 300.0, (0, 1, 1))]


@pytest.mark.parametrize("counts,edge,periodic", CASES)
def test_every_route(counts, edge, periodic):
    from paper_2511_22951_amd import _native as N
    from paper_2511_22951_amd import md
    rng = np.random.default_rng(len(counts) + counts[0])
    boxes = [mi.Box((-1.0, 2.0, 0.5), (edge, edge * 1.03, edge * 0.99), periodic) for _ in counts]
    n = sum(counts)
    lo, ln, per = boxes[0].as_arrays()
    # periodic axes: some positions outside the box; the others inside
    u = rng.uniform(0.0, 1.0, (n, 3))
    pos = lo + ln * np.where(per != 0, 1.4 * u - 0.2, u)
    vel = rng.normal(0.0, 1.0, (n, 3))
    ids = rng.permutation(n).astype(np.int32)
    plan = md.Plan(boxes, counts, 5.8)
    st = md.State(plan, pos, vel, N.MD_FP64, ids=ids)
    for trip in range(2):  # again on its own result: the histogram was left empty
        md.md_bin_cells(st)
        want = _expect(plan, pos, vel, ids)
        _compare(st, plan, want)
        pos, vel, ids = want[:3]
    info = st.check_flags()
    assert info["n_rebuilds"] == 2
    # conditional: nothing until a drift exceeds half the skin
    big = vel * 100.0
    st.vel.copy_(torch.as_tensor(big.T.copy()))
    md.md_bin_cells(st, N.MD_IF_FLAGGED)
    _compare(st, plan, (pos, big, ids, want[3]))
    assert st.check_flags()["n_rebuilds"] == 2
    md.md_verlet_step(st, N.MD_KICK_DRIFT, 1e-3, 1.0 / 40.0, half_skin=1e-6)
    moved = st.pos[:, :3].cpu().numpy()
    md.md_bin_cells(st, N.MD_IF_FLAGGED)
    if all(periodic):
        _compare(st, plan, _expect(plan, moved, big, ids))
        assert st.check_flags()["n_rebuilds"] == 3
