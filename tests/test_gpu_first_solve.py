"""Solves in which nearly every particle misses its first count, as the first of
a run: one walk of the group replaces the rows by wider sets, from which the
iteration counts.  Irregular sets against the oracle, exact: rows that hold
the wider sets, rows that many of them overflow, and rows too short for any."""
import numpy as np
import pytest

import oracle as O
from paper_1905_03344_amd import inputs
from test_gpu_parity import _gather_rows_flat, compare_cells, compare_neighbors

pytestmark = pytest.mark.gpu


def _uniform(n, periodic):
    rng = np.random.default_rng(n)
    ic = inputs.clumpy(n_clumps=1, per_clump=n - 8, n_background=8, seed=3)
    for a in (ic.x, ic.y, ic.z):
        a[:] = rng.random(n)
    ic.periodic, ic.box_lo, ic.box_hi = periodic, (0.0,) * 3, (1.0,) * 3
    ic.h[:] = inputs.initial_h(float(n))
    return ic


@pytest.mark.parametrize("list_stride", [108, 120, 136, 288])
@pytest.mark.parametrize("scale,periodic", [(0.93, (0, 0, 0)), (0.88, (1, 0, 1))])
def test_first_solve_matches_oracle(scale, periodic, list_stride):
    from paper_1905_03344_amd.state import Simulation
    ic = _uniform(200003, periodic)
    ic.h[:] *= scale
    print(f"first solve n {ic.n} scale {scale} rows of {list_stride}", flush=True)
    st = O.State(ic.copy())
    st.keep_gather = True
    st.evaluate(method=1)
    sim = Simulation(ic, extra_per_particle=128, list_stride=list_stride)
    sim.evaluate()
    _, stats = sim.sync()
    compare_cells(sim, st)
    compare_neighbors(sim, st)
    np.testing.assert_array_equal(_gather_rows_flat(sim), st.lidx)
    assert stats.nonconverged == st.nonconv
    assert stats.h_counts > 1.875 * ic.n   # (nearly all missed)


@pytest.mark.parametrize("search_div", [1, 3, 4])
def test_first_solve_search_div(search_div):
    """Cells of other widths: the walks of one particle take none below half a
    radius.  The same sets."""
    from paper_1905_03344_amd.state import Simulation
    ic = inputs.square_patch(24, 8)
    ic.h[:] *= 0.8
    print(f"search_div {search_div}", flush=True)
    st = O.State(ic.copy())
    st.keep_gather = True
    st.evaluate(method=1)
    sim = Simulation(ic, extra_per_particle=128, search_div=search_div)
    sim.evaluate()
    sim.sync()
    compare_cells(sim, st)
    compare_neighbors(sim, st)
    np.testing.assert_array_equal(_gather_rows_flat(sim), st.lidx)
