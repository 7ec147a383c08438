"""The full-shell rule of learned tries (a try in the band is a miss where more
than 48 particles lie in |r - 2h| < 2h/24) against counts of scipy's tree."""
import numpy as np
import pytest

from paper_1905_03344_amd import inputs

pytestmark = pytest.mark.gpu


def zero_model():
    """Weights that predict no change: tries are at h_prev."""
    w = inputs.mlp_init(3)
    w["W3"] = 0.0 * w["W3"]
    w["b3"] = 0.0 * w["b3"]
    return w, np.array([0.0] * 6 + [1.0] * 6)


def sheet(tiles=32):
    """A sheet in a periodic unit box, tiles x tiles squares of 17 particles,
    16 in the lower half and one in the upper: half a tile is a Morton cell, so
    that one particle in 17 has no others in its group.  (In a plane a sixth
    of the neighbours are in the shell.)"""
    rng = np.random.default_rng(17)
    n = 17 * tiles * tiles
    ic = inputs.clumpy(n_clumps=1, per_clump=n - 8, n_background=8, seed=1)
    tx, ty = np.divmod(np.arange(n) // 17, tiles)
    up = np.arange(n) % 17 == 16
    f = 0.02 + 0.96 * rng.random((2, n))
    ic.x[:] = (tx + f[0]) / tiles
    ic.y[:] = (ty + 0.5 * (up + f[1])) / tiles
    ic.z[:] = 0.25 + 1e-5 * rng.random(n)
    for a in (ic.vx, ic.vy, ic.vz):
        a[:] = 0.0
    ic.periodic, ic.box_lo, ic.box_hi = (1, 1, 1), (0.0,) * 3, (1.0,) * 3
    return ic


def exempt(x, h, key, defer):
    """Particles whose share of their 64 in index order is at most `defer`: the
    64 are split by radius (within 3 of the smallest), then by Morton prefix
    while they spread over more than 3 of the largest."""
    out = np.zeros(len(h), dtype=bool)
    for b in range(0, len(h), 64):
        pending = np.arange(b, min(b + 64, len(h)))
        while len(pending):
            g = pending
            while True:
                r = 2.0 * h[g]
                if r.max() > 3.0 * r.min():
                    g = g[r <= 3.0 * r.min()]
                    continue
                if np.ptp(x[g], axis=0).max() <= 3.0 * r.max() or len(g) <= 2:
                    break
                top = int(key[g].min()) ^ int(key[g].max())
                if top == 0:
                    break
                g = g[(key[g] ^ key[g[0]]) >> (top.bit_length() - 1) == 0]
            out[g] = len(g) <= defer
            pending = np.setdiff1d(pending, g)
    return out


@pytest.mark.parametrize("tiles", [32, 82])   # groups of up to 16 and of up to 64
@pytest.mark.parametrize("prefilter", [0, 1])
@pytest.mark.parametrize("n_target", [100, 260])
def test_counts_beyond_the_held_hits(n_target, prefilter, tiles):
    """260 neighbours: more particles within the shell's outer radius than a
    wave holds, about half of the shells full."""
    from scipy.spatial import cKDTree
    from paper_1905_03344_amd import ffi
    from paper_1905_03344_amd.state import Simulation
    ic = sheet(tiles)
    ic.h[:] = 0.5 * np.sqrt(n_target / (np.pi * ic.n))
    out = {}
    for mode in (ffi.SPH_TRY_SHELL_NEVER, ffi.SPH_TRY_SHELL_ALWAYS):
        print(f"shells n {ic.n} n_target {n_target} prefilter {prefilter} mode {mode}", flush=True)
        p = ffi.default_params()
        p.n_target = n_target
        sim = Simulation(ic, params=p, h_mode=ffi.SPH_H_LEARNED, learned_try_shell=mode,
                         list_stride=512, extra_per_particle=512, walk_defer_group=1,
                         walk_prefilter=prefilter)
        sim.set_mlp(*zero_model())
        sim.evaluate()
        h = sim.numpy("h")[np.argsort(sim.numpy("id"))]
        sim.step(1e-12)
        sim.sync()
        o = np.argsort(sim.numpy("id"))
        out[mode] = {f: sim.numpy(f)[o] for f in ("x", "y", "z", "flags")}
        out[mode]["h_prev"] = h
        x = np.stack([sim.numpy(f) for f in ("x", "y", "z")], axis=1)
        out[mode]["exempt"] = exempt(x, h[sim.numpy("id")], sim.numpy("key"), 1)[o]
    a, b = out[ffi.SPH_TRY_SHELL_NEVER], out[ffi.SPH_TRY_SHELL_ALWAYS]
    np.testing.assert_array_equal(a["h_prev"], b["h_prev"])
    X = np.stack([a["x"], a["y"], a["z"]], axis=1)
    tree = cKDTree(X, boxsize=1.0)
    ball = lambda f: tree.query_ball_point(X, 2.0 * a["h_prev"] * f, return_length=True)
    outer = ball(1.0 + 1.0 / 24.0)
    full = outer - ball(1.0 - 1.0 / 24.0) > 48
    took_a, took_b = (a["flags"] & 2) != 0, (b["flags"] & 2) != 0
    assert took_a.mean() > 0.9
    if n_target == 260:
        # (the input has both kinds)
        assert np.mean(outer > 257) > 0.9 and 0.05 < np.mean(full) < 0.95
    assert np.mean(b["exempt"]) < 0.01
    # exactly the tries with a full shell are misses
    np.testing.assert_array_equal(took_b, took_a & (~full | b["exempt"]))


def _cloud(n):
    """A power-law cloud: in many bands more than 48 particles in the shell."""
    rng = np.random.default_rng(31)
    ic = inputs.clumpy(n_clumps=1, per_clump=n - 8, n_background=8, seed=2)
    r = rng.random(n) ** 2.5
    u = rng.normal(size=(n, 3))
    u *= (r / np.linalg.norm(u, axis=1))[:, None]
    ic.x[:], ic.y[:], ic.z[:] = u[:, 0], u[:, 1], u[:, 2]
    for a in (ic.vx, ic.vy, ic.vz):
        a[:] = 0.0
    ic.h[:] = np.maximum(0.5 * (100.0 / n) ** 0.4 * np.maximum(r, 1e-3) ** 0.87, 1e-5)
    return ic


def test_auto_follows_the_solve_before():
    """AUTO at 140,003 particles: a first step, whose tries (2% above h_prev) miss
    by more than a tenth, as NEVER, and a second one (tries at h_prev) as ALWAYS
    from the same state; sph_evaluate and new weights start afresh."""
    from paper_1905_03344_amd import ffi
    from paper_1905_03344_amd.state import Simulation
    NEVER, ALWAYS, AUTO = (ffi.SPH_TRY_SHELL_NEVER, ffi.SPH_TRY_SHELL_ALWAYS,
                           ffi.SPH_TRY_SHELL_AUTO)
    ic = _cloud(140003)
    # y = 0.02 where the feature dt c / h is large, 0 where it is small
    w, norm = zero_model()
    for k in ("W1", "W2", "W3"):
        w[k] = 0.0 * w[k]
    w["W1"][0, 5], w["W2"][0, 0], w["W3"].reshape(-1)[0] = 1.0, 4.0, 0.02
    norm[11] = 1e-10
    far, near = 1e-8, 1e-18

    def make(mode, like=None):
        sim = Simulation(ic, h_mode=ffi.SPH_H_LEARNED, learned_try_shell=mode, list_stride=256,
                         extra_per_particle=1024)
        sim.set_mlp(w, norm)
        if like is not None:
            for f in ffi.CARRIED_F64 + ffi.CARRIED_I32:
                sim.field(f).copy_(like.field(f))
            sim.d_dt.copy_(like.d_dt)
        return sim

    def state(sim):
        sim.sync()
        return {f: sim.numpy(f).copy() for f in ("id", "h", "nc", "flags", "rho", "ax", "du")}

    def same(a, b):
        return all(np.array_equal(a[f], b[f]) for f in a)

    sims = {m: make(m) for m in (NEVER, ALWAYS, AUTO)}
    first = {}
    for m, sim in sims.items():
        print(f"first step, mode {m}", flush=True)
        sim.evaluate()
        sim.step(far)
        first[m] = state(sim)
    miss = 1.0 - np.mean((first[AUTO]["flags"] & 2) != 0)
    assert 0.1 < miss < 0.9
    assert same(first[AUTO], first[NEVER]) and not same(first[AUTO], first[ALWAYS])
    auto = sims[AUTO]
    twins = {m: make(m, like=auto) for m in (NEVER, ALWAYS)}
    fresh, weights = make(AUTO, like=auto), make(AUTO, like=auto)
    keep = {f: auto.field(f).clone() for f in ffi.CARRIED_F64 + ffi.CARRIED_I32}
    keep_dt = auto.d_dt.clone()
    print("second step", flush=True)
    auto.step(near)
    second = state(auto)
    for m, sim in twins.items():
        sim.step(near)
        assert same(second, state(sim)) == (m == ALWAYS)
    # the state put back: sph_evaluate, or new weights, and the next solve is
    # a first one
    for restart in ("evaluate", "weights"):
        auto.step(far)
        auto.sync()
        for f, v in keep.items():
            auto.field(f).copy_(v)
        auto.d_dt.copy_(keep_dt)
        other = fresh if restart == "evaluate" else weights
        if restart == "evaluate":
            auto.evaluate()
            other.evaluate()
        else:
            auto.set_mlp(w, norm)
        auto.step(near)
        other.step(near)
        assert same(state(auto), state(other)), restart
