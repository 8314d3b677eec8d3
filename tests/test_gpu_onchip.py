"""GPU parity of predation models advanced inside one workgroup's LDS: the
edges of what is taken there, and what leaves it for global memory (all results
are whole numbers: equal to the oracle's, stale fields included)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FIELDS = ("x", "y", "e", "alive")


def _far_countdown(S):
    S.grass.reshape(-1)[::7] = 255
    S.grass.reshape(-1)[3] = 300


def _off_grid(S):
    S.sheep["x"][:3] = (-1, 5000, 70)
    S.wolves["y"][1] = -7


def _stale(S):
    dead = S.sheep["alive"] == 0
    S.sheep["x"][dead] = np.arange(int(dead.sum())) % 64
    S.sheep["e"][dead] = -5
    S.wolves["alive"][::3] = 0


def _stale_wide(S):
    S.sheep["y"][np.flatnonzero(S.sheep["alive"] == 0)[:5]] = 1 << 20


def _rich(S):
    S.sheep["e"][:9] = (20000, 2 ** 30, -1, -20000, 0, 1, 16384, 16385, -16385)


def _holes(S):
    S.sheep["alive"][::2] = 0
    S.wolves["alive"][:-1] = 0


# name: (parameters, change of the initial state)
CASES = {
    "one cell": (dict(W=1, H=1, cap_s=70, cap_w=65, n_s0=40, n_w0=30), None),
    "narrow": (dict(W=256, H=3, cap_s=700, cap_w=200, n_s0=300, n_w0=60), None),
    "tall": (dict(W=5, H=256, cap_s=700, cap_w=200, n_s0=300, n_w0=60), None),
    "too wide": (dict(W=257, H=9, cap_s=700, cap_w=200, n_s0=300, n_w0=60), None),
    "too tall": (dict(W=9, H=257, cap_s=700, cap_w=200, n_s0=300, n_w0=60), None),
    "R 1": (dict(R=1), None),
    "R 200": (dict(R=200), None),
    "R 201": (dict(R=201), None),
    # the LDS holds 236 rows of 64 slots beside the cells; 1.5 slots a cell, and one more
    "largest of one launch": (dict(W=170, H=170, cap_s=14080), None),
    "one row more": (dict(W=170, H=170, cap_s=14144), None),
    "slots a cell": (dict(cap_s=4096, cap_w=2048), None),
    "a slot more": (dict(cap_s=4096, cap_w=2049), None),
    "1024 slots": (dict(W=5, H=5, cap_s=900, cap_w=124, n_s0=300, n_w0=60), None),
    "full species": (dict(cap_s=400, cap_w=100, T_s=2 ** 31, T_w=2 ** 31), None),
    "no wolves": (dict(n_w0=0), None),
    "no agents": (dict(n_s0=0, n_w0=0), None),
    # more contested agents than are listed in LDS, and more contested cells than the table holds
    "crowded cells": (dict(W=16, H=8, cap_s=3000, cap_w=900, n_s0=3000, n_w0=900), None),
    "crowded table": (dict(cap_s=9000, cap_w=4000, n_s0=9000, n_w0=4000), None),
    "far countdowns": (dict(), _far_countdown),
    "stale fields": (dict(), _stale),
    "wide stale fields": (dict(), _stale_wide),
    "large energies": (dict(), _rich),
    "holes": (dict(), _holes),
    "gains past 16 bits": (dict(gain_s=8192, gain_w=8192, n_w0=300), None),
    "gains too large": (dict(gain_s=8193), None),
    "matched by rank": (dict(multi_prey=1), None),
    # room for 156 rows of 64 slots beside the cells, outgrown after a few steps
    "outgrown": (dict(W=256, H=256, R=3, cap_s=40000, cap_w=3000, n_s0=7500, n_w0=600,
                      T_s=2 ** 31, T_w=2 ** 31), None),
}


def _state(orc, kw, change):
    P = orc.pred_params(seed=31, **kw)
    S = orc.predation_init(P)
    if change:
        change(S)
    return P, S


def _check(got, S, steps):
    for name in ("sheep", "wolves"):
        for f in FIELDS:
            a, b = got[name][f].cpu().numpy(), getattr(S, name)[f]
            assert np.array_equal(a, b), (name, f, np.flatnonzero(a != b)[:5], steps)
    assert np.array_equal(got["grass"].cpu().numpy(), S.grass), ("grass", steps)


@pytest.mark.parametrize("name", CASES)
def test_one_model(abm, orc, name):
    kw, change = CASES[name]
    P, S = _state(orc, kw, change)
    m = abm.predation_init(abm.predation_params(seed=31, **kw))
    m.grass.copy_(torch.from_numpy(S.grass))
    for sp in ("sheep", "wolves"):
        for f in FIELDS:
            getattr(m, sp)[f].copy_(torch.from_numpy(getattr(S, sp)[f]))
    for steps in (1, 2, 60, 270):
        if P.cap_s > 10000 and steps > 60:
            continue
        stats = torch.full((steps, 8), -9, dtype=torch.int64, device="cuda")
        m.run(steps, stats)
        rows = orc.predation_run(P, S, steps)
        exp = np.array([[r[k] for k in abm.STAT_NAMES] for r in rows])
        assert np.array_equal(stats.cpu().numpy(), exp), (name, steps)
        _check(dict(grass=m.grass, sheep=m.sheep, wolves=m.wolves), S, steps)


@pytest.mark.parametrize("copies", [1, 3])
@pytest.mark.parametrize("name", CASES)
def test_batched(abm, orc, name, copies):
    """The model among others, run in launches of 1, 7 and 60 steps."""
    kw, change = CASES[name]
    P, S = _state(orc, kw, change)
    other = dict(W=12, H=30, cap_s=60, cap_w=30, n_s0=30, n_w0=10)
    params = [abm.predation_params(seed=31, **kw) for _ in range(copies)] + [
        abm.predation_params(seed=5 + k, **other) for k in range(2)]
    b = abm.BatchedPredation(params, 10000)
    b.init()
    cells = P.W * P.H
    for c in range(copies):
        b.ready[c * cells:(c + 1) * cells].copy_(torch.from_numpy(S.grass.reshape(-1)))
        for sp, flat, cap in (("sheep", b.sheep, P.cap_s), ("wolves", b.wolves, P.cap_w)):
            for f in FIELDS:
                flat[f][c * cap:(c + 1) * cap].copy_(torch.from_numpy(getattr(S, sp)[f]))
    others = [orc.pred_params(seed=5 + k, **other) for k in range(2)]
    states = [orc.predation_init(o) for o in others]
    updates = 0
    for steps in (1, 7, 60):
        b.run(steps)
        updates += sum(r["live_s"] + r["live_w"] for r in orc.predation_run(P, S, steps))
        countdown = b.grass_countdown()
        desc = b.descriptors()
        for c in range(copies):
            grass, sheep, wolves = b.model_state(c, countdown)
            _check(dict(grass=grass.reshape(S.grass.shape), sheep=sheep, wolves=wolves), S, steps)
            assert desc[c].step == S.step and desc[c].updates == updates
            assert desc[c].live_s == int(np.count_nonzero(S.sheep["alive"]))
        for k in range(2):
            orc.predation_run(others[k], states[k], steps)
            grass, sheep, wolves = b.model_state(copies + k, countdown)
            _check(dict(grass=grass.reshape(states[k].grass.shape), sheep=sheep, wolves=wolves),
                   states[k], steps)
    assert torch.equal(b.claims.view(torch.int64), torch.full_like(b.claims.view(torch.int64), -1))


def test_agents_off_the_grid(abm, orc):
    """They move, pay and breed but take part in no cell, whichever path runs
    the model: one workgroup, the general one (a larger capacity), a batch's."""
    P, S = _state(orc, {}, _off_grid)
    out = []
    for cap in (P.cap_s, 40000):
        m = abm.predation_init(abm.predation_params(seed=31, cap_s=cap))
        for sp in ("sheep", "wolves"):
            for f in FIELDS:
                a = getattr(S, sp)[f]
                getattr(m, sp)[f].zero_()
                getattr(m, sp)[f][:a.size].copy_(torch.from_numpy(a))
        m.run(9)
        out.append((m.grass, m.sheep, m.wolves))
    for lds in (True, False):
        b = abm.BatchedPredation([abm.predation_params(seed=31)], 9, lds=lds)
        b.init()
        for sp in ("sheep", "wolves"):
            for f in FIELDS:
                getattr(b, sp)[f].copy_(torch.from_numpy(getattr(S, sp)[f]))
        b.run(9)
        out.append(b.model_state(0, b.grass_countdown()))
    for grass, sheep, wolves in out[1:]:
        assert torch.equal(grass.reshape(-1), out[0][0].reshape(-1))
        for f in FIELDS:
            assert torch.equal(sheep[f][:P.cap_s], out[0][1][f])
            assert torch.equal(wolves[f], out[0][2][f])


# agents off the grid send the model to global memory
@pytest.mark.parametrize("off_grid", [False, True])
def test_cells_that_never_grow(abm, orc, off_grid):
    """Countdowns of 2^31 - 1 set in the middle of a run: no cell of them is eaten,
    whichever path runs the model."""
    P, S = _state(orc, {}, None)
    orc.predation_run(P, S, 3)
    S.grass.reshape(-1)[::3] = 2 ** 31 - 1
    if off_grid:
        _off_grid(S)
    got = []
    for cap in (P.cap_s, 40000):
        m = abm.predation_init(abm.predation_params(seed=31, cap_s=cap))
        m.run(3)
        m.grass.copy_(torch.from_numpy(S.grass))
        for sp in ("sheep", "wolves"):
            for f in FIELDS:
                a = getattr(S, sp)[f]
                getattr(m, sp)[f][:a.size].copy_(torch.from_numpy(a))
        stats = torch.zeros((80, 8), dtype=torch.int64, device="cuda")
        m.run(80, stats)
        got.append([m.grass, stats] + [getattr(m, sp)[f][:getattr(S, sp)[f].size]
                                       for sp in ("sheep", "wolves") for f in FIELDS])
    assert int((got[0][0] == 2 ** 31 - 81).sum()) == (P.W * P.H + 2) // 3
    for a, b in zip(*got):
        assert torch.equal(a, b)
    if not off_grid:
        orc.predation_run(P, S, 80)
        _check(dict(grass=got[0][0], sheep=dict(zip(FIELDS, got[0][2:6])),
                    wolves=dict(zip(FIELDS, got[0][6:]))), S, 80)


# path: (grid, one model or how the batch is run); 257 cells do not fit the chip
LIVE_PATHS = {
    "chip": (dict(), None),
    "general": (dict(W=257, H=16), None),
    "batch on the chip": (dict(), dict(max_steps=7)),
    "batch": (dict(W=257, H=16), dict(max_steps=7)),
    "batch, claims in global memory": (dict(), dict(max_steps=7, lds=False)),
    "launches": (dict(W=257, H=16), dict(max_steps=7, team_size=2)),
    "teams": (dict(W=257, H=16), dict(max_steps=1 << 20, team_size=2)),
}


@pytest.mark.parametrize("multi_prey", [0, 1])
@pytest.mark.parametrize("path", LIVE_PATHS)
def test_any_nonzero_value_is_live(abm, orc, path, multi_prey):
    """Live agents' values are kept (2 becomes 1), whichever path runs the model."""
    grid, how = LIVE_PATHS[path]
    kw = dict(grid, multi_prey=multi_prey)
    P, S = _state(orc, kw, None)
    for sp in (S.sheep, S.wolves):
        live = np.flatnonzero(sp["alive"])
        sp["alive"][live] = np.resize([-1, 7, 2, -2 ** 31, 2 ** 31 - 1, 1], live.size)
    params = abm.predation_params(seed=31, **kw)
    if how is None:
        m = abm.predation_init(params)
        flat = (m.sheep, m.wolves)
    else:
        how = dict(how)
        b = abm.BatchedPredation([params], 14, team_min_size=1, lds=how.pop("lds", True),
                                 team_size=how.pop("team_size", 1))
        b.init()
        flat = (b.sheep, b.wolves)
    for d, sp in zip(flat, (S.sheep, S.wolves)):
        for f in FIELDS:
            d[f].copy_(torch.from_numpy(sp[f]))
    for part in range(1 if how and how["max_steps"] > 14 else 2):
        if how is None:
            m.run(7)
            got = dict(grass=m.grass, sheep=m.sheep, wolves=m.wolves)
        else:
            b.run(**how)
            grass, sheep, wolves = b.model_state(0, b.grass_countdown())
            got = dict(grass=grass.reshape(S.grass.shape), sheep=sheep, wolves=wolves)
        orc.predation_run(P, S, 14 if how and how["max_steps"] > 14 else 7)
        for sp in (S.sheep, S.wolves):
            sp["alive"][sp["alive"] == 2] = 1
        _check(got, S, part)


@pytest.mark.parametrize("path", [p for p, (_, how) in LIVE_PATHS.items() if how])
def test_cells_grown_since_ever(abm, orc, path):
    """A batch's cells whose step is -2^31 are grown at every step."""
    grid, how = LIVE_PATHS[path]
    how = dict(how)
    P, S = _state(orc, grid, None)
    b = abm.BatchedPredation([abm.predation_params(seed=31, **grid)], 10, team_min_size=1,
                             lds=how.pop("lds", True), team_size=how.pop("team_size", 1))
    b.init()
    b.run(3)
    orc.predation_run(P, S, 3)
    b.ready[::2] = -2 ** 31
    S.grass.reshape(-1)[::2] = 0
    b.run(**how)
    orc.predation_run(P, S, 7)
    # (the countdown of a cell grown at -2^31 is not asked for: it is not a step)
    ready = torch.where(b.ready == -2 ** 31, 0, b.ready)
    grass = (ready - 10).clamp(min=0).cpu().numpy().reshape(S.grass.shape)
    assert np.array_equal(grass, S.grass)
    _, sheep, wolves = b.model_state(0, b.ready)
    for d, sp in ((sheep, S.sheep), (wolves, S.wolves)):
        for f in FIELDS:
            assert np.array_equal(d[f].cpu().numpy(), sp[f]), f


# the regrowth bytes are rebased several times in 600 steps; dead slots between live ones hold
# what no agent could, and keep it until a child is put there
@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("R", [1, 30, 200])
def test_far_countdowns_and_odd_dead_slots(abm, orc, R, batched):
    kw = dict(R=R, T_s=10 ** 8, n_s0=300)
    P, S = _state(orc, kw, None)
    S.grass.reshape(-1)[::5] = np.resize([254, 255, 256, 300, 454, 455, 479, 480, 510, 700,
                                          10 ** 9, 2 ** 31 - 1], S.grass.reshape(-1)[::5].size)
    g = np.random.default_rng(R)
    for sp in (S.sheep, S.wolves):
        sp["alive"][g.random(sp["alive"].size) < 0.4] = 0
        dead = np.flatnonzero(sp["alive"] == 0)
        for f in ("x", "y", "e"):
            sp[f][dead] = g.integers(-2 ** 31, 2 ** 31, dead.size)
    params = abm.predation_params(seed=31, **kw)
    if batched:
        b = abm.BatchedPredation([params], 600)
        b.init()
        b.ready.copy_(torch.from_numpy(S.grass.reshape(-1)))
        flat = (b.sheep, b.wolves)
    else:
        m = abm.predation_init(params)
        m.grass.copy_(torch.from_numpy(S.grass))
        flat = (m.sheep, m.wolves)
    for d, sp in zip(flat, (S.sheep, S.wolves)):
        for f in FIELDS:
            d[f].copy_(torch.from_numpy(sp[f]))
    for steps in (3, 597):
        if batched:
            b.run(steps)
            grass, sheep, wolves = b.model_state(0, b.grass_countdown())
            got = dict(grass=grass.reshape(S.grass.shape), sheep=sheep, wolves=wolves)
        else:
            stats = torch.zeros((steps, 8), dtype=torch.int64, device="cuda")
            m.run(steps, stats)
            got = dict(grass=m.grass, sheep=m.sheep, wolves=m.wolves)
        rows = orc.predation_run(P, S, steps)
        if not batched:
            assert np.array_equal(stats.cpu().numpy(), [[r[k] for k in abm.STAT_NAMES] for r in rows])
        _check(got, S, steps)


def test_one_model_replayed_from_a_graph(abm, orc):
    """Captured calls replayed with other work between them."""
    P, S = _state(orc, {}, None)
    m = abm.predation_init(abm.predation_params(seed=31))
    m.run(1)
    orc.predation_run(P, S, 1)
    torch.cuda.synchronize()
    keep = {sp: {f: getattr(m, sp)[f].clone() for f in FIELDS} for sp in ("sheep", "wolves")}
    grass = m.grass.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        m.run(5)
    orc.predation_run(P, S, 5)
    for _ in range(4):
        m.grass.copy_(grass)
        for sp in ("sheep", "wolves"):
            for f in FIELDS:
                getattr(m, sp)[f].copy_(keep[sp][f])
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        _check(dict(grass=m.grass, sheep=m.sheep, wolves=m.wolves), S, 5)


# more models than CUs (two share one), and than twice as many (four do); some of every size
# class, some that outgrow the smaller ones during a run, runs of 1, 6 and 30 steps
@pytest.mark.parametrize("n", [300, 700])
def test_size_classes(abm, orc, n):
    g = np.random.default_rng(n)
    kws = []
    for k in range(n):
        side = int(g.choice([8, 20, 60, 100, 140])) if k % 40 else 220
        cells = side * side
        grows = k % 5 == 0
        kws.append(dict(W=side, H=side + k % 3, seed=k, cap_s=4 * cells, cap_w=cells,
                        n_s0=cells // 8, n_w0=cells // 40, R=2 if grows else 30,
                        T_s=2 ** 31 if grows else 171798691))
    b = abm.BatchedPredation([abm.predation_params(**kw) for kw in kws], 100)
    b.init()
    states = [(orc.pred_params(**kw),) for kw in kws]
    states = [(p, orc.predation_init(p)) for (p,) in states]
    updates = np.zeros(n, np.int64)
    for steps in (1, 6, 30):
        b.run(steps)
        countdown, desc = b.grass_countdown(), b.descriptors()
        check = range(n) if steps < 30 else range(0, n, 7)
        for m, (p, s) in enumerate(states):
            if m not in check:
                continue
            updates[m] += sum(r["live_s"] + r["live_w"] for r in orc.predation_run(p, s, steps))
            grass, sheep, wolves = b.model_state(m, countdown)
            _check(dict(grass=grass.reshape(s.grass.shape), sheep=sheep, wolves=wolves), s,
                   (m, steps))
            assert desc[m].step == s.step and desc[m].updates == updates[m]
