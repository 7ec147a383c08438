"""Learned misses counted again by a walk of their group (from 100,000 particles
on, groups with at least 24 misses): bit for bit the plain iteration, in every
try-shell mode, from tries far above (rows that overflow) and far below."""
import numpy as np
import pytest

from paper_1905_03344_amd import inputs

pytestmark = pytest.mark.gpu

FIELDS = ("id", "h", "nc", "rho", "divv", "ax", "ay", "az", "du", "x", "vx", "u")


def constant_model(y):
    """Weights that predict log(h_new / h) = y everywhere."""
    w = inputs.mlp_init(3)
    w["W3"] = 0.0 * w["W3"]
    w["b3"] = np.array([y], dtype=np.float32)
    return w, np.array([0.0] * 6 + [1.0] * 6)


def _run(ic, y=None, steps=2, **kw):
    from paper_1905_03344_amd import ffi
    from paper_1905_03344_amd.state import Simulation
    sim = Simulation(ic, h_mode=ffi.SPH_H_PLAIN if y is None else ffi.SPH_H_LEARNED, **kw)
    if y is not None:
        sim.set_mlp(*constant_model(y))
    sim.evaluate()
    stats = []
    for _ in range(steps):
        sim.step(0.0)
        stats.append(sim.sync()[1])
    return sim, stats


@pytest.fixture(scope="module", params=["fp64", "mixed"])
def plain(request):
    from paper_1905_03344_amd import ffi
    ic = inputs.square_patch(48, 77)
    prec = ffi.SPH_FP64 if request.param == "fp64" else ffi.SPH_MIXED
    return ic, prec, _run(ic, precision=prec)[0]


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("y", [0.5, -0.5])
def test_all_missed_is_plain(plain, y, mode):
    ic, prec, ref = plain
    print(f"all missed: y {y} mode {mode} precision {prec}", flush=True)
    sim, stats = _run(ic, y, precision=prec, learned_try_shell=mode)
    for f in FIELDS:
        np.testing.assert_array_equal(ref.numpy(f), sim.numpy(f), err_msg=f)
    valid = np.arange(sim.params.list_stride)[:, None] < sim.numpy("nc")[None, :]
    np.testing.assert_array_equal(ref.gather_dense()[1][valid], sim.gather_dense()[1][valid])
    for s in stats:
        assert s.learned_fallback == ic.n and s.learned_accepted == 0
    assert not np.any(sim.numpy("flags") & 2)


def test_never_counts_misses_together():
    """The misses of a run under NEVER take no longer than under ALWAYS (each
    counted by a walk of its own they took 1.36 times as long)."""
    import torch
    from paper_1905_03344_amd import ffi
    ic = inputs.square_patch(80, 5)
    ms = {}
    for mode in (ffi.SPH_TRY_SHELL_NEVER, ffi.SPH_TRY_SHELL_ALWAYS):
        sim, _ = _run(ic, -0.02, steps=2, learned_try_shell=mode)
        ffi.sph_timing(sim.ctx, True)
        for _ in range(5):
            sim.step(0.0)
        _, st = sim.sync()
        t = ffi.sph_timing_read(sim.ctx)
        torch.cuda.synchronize()
        ms[mode] = t["hsolve"][0] / 5
        assert st.learned_fallback > 0.5 * 5 * ic.n
    print(f"h iteration, ms per step: {ms}", flush=True)
    assert ms[ffi.SPH_TRY_SHELL_NEVER] < 1.25 * ms[ffi.SPH_TRY_SHELL_ALWAYS]
