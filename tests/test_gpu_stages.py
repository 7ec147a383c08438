"""Stage timing: the first counts are a stage of their own, inside the walk's and
the h iteration's, in both forms."""
import numpy as np
import pytest

from paper_1905_03344_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("learned", [False, True])
def test_first_counts_stage(learned):
    from paper_1905_03344_amd import ffi
    from paper_1905_03344_amd.state import Simulation
    sim = Simulation(inputs.square_patch(50, 3),
                     h_mode=ffi.SPH_H_LEARNED if learned else ffi.SPH_H_PLAIN)
    if learned:
        w = inputs.mlp_init(3)
        w["W3"] = 0.0 * w["W3"]
        w["b3"] = np.array([0.3], dtype=np.float32)   # every try misses
        sim.set_mlp(w, np.array([0.0] * 6 + [1.0] * 6))
    sim.evaluate()
    sim.step(0.0)
    sim.sync()
    ffi.sph_timing(sim.ctx, True)
    for _ in range(4):
        sim.step(0.0)
    sim.sync()
    t = ffi.sph_timing_read(sim.ctx, first=True)
    assert "hfirst" not in ffi.sph_timing_read(sim.ctx)
    ffi.sph_timing(sim.ctx, False)
    ms = {k: v[0] / 4 for k, v in t.items()}
    print({k: round(v, 4) for k, v in ms.items()}, flush=True)
    assert all(t[k][1] == 4 for k in ("hfirst", "hwalk", "hsolve"))
    assert 0.0 < ms["hfirst"] < ms["hwalk"] < ms["hsolve"]
    # the plain form's walk has the tail in it, the learned one's the tries alone
    # (an event record more on either side)
    if learned:
        assert ms["hwalk"] - ms["hfirst"] < 0.05
    else:
        assert ms["hwalk"] - ms["hfirst"] > 0.05
