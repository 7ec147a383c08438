"""The neighbour search does not depend on the unit of length: the same set in
units of 2^k gives the same counts, flags and rows, and h in that unit, bit for
bit (powers of two scale FP64 exactly)."""
import numpy as np
import pytest

from paper_1905_03344_amd import inputs

pytestmark = pytest.mark.gpu

BASE = {}


def _search(n_side, k, prefilter):
    from paper_1905_03344_amd.state import Simulation
    ic = inputs.square_patch(n_side, 5)
    for a in (ic.x, ic.y, ic.z, ic.h):
        a *= 2.0 ** k
    ic.box_lo, ic.box_hi = (tuple(2.0 ** k * v for v in b) for b in (ic.box_lo, ic.box_hi))
    sim = Simulation(ic, walk_prefilter=prefilter, extra_per_particle=256, max_level=4)
    sim.build_cells()
    sim.find_neighbors()
    _, st = sim.sync()
    nc, idx = sim.gather_dense()
    idx = np.where(np.arange(idx.shape[0])[:, None] < nc[None, :], idx, -1)
    off, csr = (t.cpu().numpy() for t in sim.interaction_csr_device())
    return {"id": sim.numpy("id"), "h": np.ldexp(sim.numpy("h"), -k), "nc": nc, "idx": idx,
            "flags": sim.numpy("flags"), "counts": st.h_counts, "off": off, "csr": csr}


@pytest.mark.parametrize("prefilter", [0, 1])
@pytest.mark.parametrize("n_side", [17, 47])
@pytest.mark.parametrize("k", [-200, -70, 70, 200])
def test_unit_of_length(k, n_side, prefilter):
    print(f"unit 2^{k} n {n_side}^3 prefilter {prefilter}", flush=True)
    if n_side not in BASE:
        BASE[n_side] = _search(n_side, 0, 0)
    a = _search(n_side, k, prefilter)
    for f, v in BASE[n_side].items():
        np.testing.assert_array_equal(v, a[f], err_msg=f)
