"""GPU parity of the batched (segmented) primitives: every segment of a packed
collection must end exactly as the single-collection oracle leaves it alone,
with its own counts.  Segment layouts include empty segments, one-slot
segments, segments straddling lane and tile boundaries, and one segment
spanning many tiles."""
import numpy as np
import pytest
import torch

from paper_2508_16508_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _layout(seed, n_seg, max_len):
    g = np.random.default_rng(seed)
    lens = g.integers(0, max_len + 1, size=n_seg)
    lens[g.random(n_seg) < 0.15] = 0          # empty segments
    lens[g.random(n_seg) < 0.10] = 1
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)


LAYOUTS = [
    ("one", lambda: np.array([0, 50_000], dtype=np.int64)),
    ("uneven", lambda: _layout(1, 300, 2000)),
    ("tiny", lambda: _layout(2, 2000, 40)),
    ("large+small", lambda: np.concatenate([[0], np.cumsum([3, 70_001, 0, 8192, 1, 40_000, 0])])
     .astype(np.int64)),
]


@pytest.mark.parametrize("name,mk", LAYOUTS)
@pytest.mark.parametrize("p,qf", [(0.05, 1.0), (0.5, 0.5), (0.9, 1.5)])
def test_select_update_batched(abm, orc, name, mk, p, qf):
    so = mk()
    n_seg, n = so.size - 1, int(so[-1])
    A = 3
    attrs = W.int32_rows(n + 3, A, n)
    mask = W.bernoulli_mask(n + 4, p, n)
    # records per segment: qf x selected slots of that segment
    q = [int(qf * int(mask[so[m]:so[m + 1]].sum())) for m in range(n_seg)]
    ro = np.concatenate([[0], np.cumsum(q)]).astype(np.int64)
    recs = W.int32_rows(n + 5, A, int(ro[-1]))
    exp = attrs.copy()
    ea, ed = [], []
    for m in range(n_seg):
        out, a_, d_ = orc.select_update(attrs[:, so[m]:so[m + 1]], mask[so[m]:so[m + 1]],
                                        recs[:, ro[m]:ro[m + 1]])
        exp[:, so[m]:so[m + 1]] = out
        ea.append(a_)
        ed.append(d_)
    d_attrs = dev(attrs)
    applied, dropped = abm.select_update_batched(d_attrs, dev(so), dev(mask), dev(recs), dev(ro))
    assert np.array_equal(host(d_attrs), exp)
    assert list(host(applied)[:n_seg]) == ea
    assert list(host(dropped)[:n_seg]) == ed


@pytest.mark.parametrize("name,mk", LAYOUTS)
def test_add_and_remove_batched(abm, orc, name, mk):
    so = mk()
    n_seg, n = so.size - 1, int(so[-1])
    A = 2
    attrs = W.int32_rows(n + 7, A, n)
    alive = (1 - W.bernoulli_mask(n + 8, 0.3, n)).astype(np.int32)
    q = [int(0.8 * int((alive[so[m]:so[m + 1]] == 0).sum())) + (m % 3) for m in range(n_seg)]
    ro = np.concatenate([[0], np.cumsum(q)]).astype(np.int64)
    recs = W.int32_rows(n + 9, A, int(ro[-1]))
    exp, exp_alive = attrs.copy(), alive.copy()
    ea, ed = [], []
    for m in range(n_seg):
        out, al, a_, d_ = orc.add_agents(attrs[:, so[m]:so[m + 1]], alive[so[m]:so[m + 1]],
                                         recs[:, ro[m]:ro[m + 1]])
        exp[:, so[m]:so[m + 1]] = out
        exp_alive[so[m]:so[m + 1]] = al
        ea.append(a_)
        ed.append(d_)
    d_attrs, d_alive = dev(attrs), dev(alive)
    added, dropped = abm.add_agents_batched(d_attrs, d_alive, dev(so), dev(recs), dev(ro))
    assert np.array_equal(host(d_attrs), exp)
    assert np.array_equal(host(d_alive), exp_alive)
    assert list(host(added)[:n_seg]) == ea and list(host(dropped)[:n_seg]) == ed
    # then remove with a kill mask
    kill = W.bernoulli_mask(n + 10, 0.4, n)
    exp_alive2 = exp_alive.copy()
    er = []
    for m in range(n_seg):
        al, r_ = orc.remove_agents(exp_alive[so[m]:so[m + 1]], kill[so[m]:so[m + 1]])
        exp_alive2[so[m]:so[m + 1]] = al
        er.append(r_)
    removed = abm.remove_agents_batched(d_alive, dev(so), dev(kill))
    assert np.array_equal(host(d_alive), exp_alive2)
    assert list(host(removed)[:n_seg]) == er


def test_resolve_conflicts_batched(abm, orc):
    g = np.random.default_rng(5)
    n_seg = 200
    nc = g.integers(0, 300, size=n_seg)
    nt = g.integers(0, 50, size=n_seg)
    co = np.concatenate([[0], np.cumsum(nc)]).astype(np.int64)
    to = np.concatenate([[0], np.cumsum(nt)]).astype(np.int64)
    target = np.concatenate([g.integers(-1, t + 1, size=c) for c, t in zip(nc, nt)]).astype(np.int32)
    prio = g.integers(0, 6, size=int(co[-1])).astype(np.uint32)
    active = (g.random(int(co[-1])) < 0.85).astype(np.uint8)
    best, winner, won = abm.resolve_conflicts_batched(
        dev(co), dev(target), dev(prio.view(np.int32)).view(torch.uint32), dev(to),
        active=dev(active))
    hb, hw, hwon = host(best), host(winner), host(won)
    for m in range(n_seg):
        eb, ew, ewon = orc.resolve_conflicts(target[co[m]:co[m + 1]], prio[co[m]:co[m + 1]],
                                             int(nt[m]), active=active[co[m]:co[m + 1]])
        assert np.array_equal(hb[to[m]:to[m + 1]], eb), m
        assert np.array_equal(hw[to[m]:to[m + 1]], ew), m
        assert np.array_equal(hwon[co[m]:co[m + 1]], ewon), m


# segments of one or a few slots (several starts in one 16-byte chunk), lengths around the 32
# slots of a line and the 8192 of a tile, empty segments, packed lengths of any remainder mod 4
@pytest.mark.parametrize("rem", [0, 1, 2, 3])
@pytest.mark.parametrize("kind", ["ones", "few", "lines", "tiles", "holes"])
def test_segment_starts_inside_lines(abm, orc, kind, rem):
    g = np.random.default_rng(len(kind) * 7 + rem)
    lens = {"ones": np.ones(9000, np.int64), "few": g.integers(1, 6, 5000),
            "lines": g.integers(30, 35, 600), "tiles": g.choice([8191, 8192, 8193], 5),
            "holes": g.choice([0, 0, 0, 1, 2, 70, 3000], 400)}[kind]
    lens = np.append(lens, 4 - (int(lens.sum()) - rem) % 4)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n, A = int(off[-1]), 3
    q = g.integers(0, np.maximum(1, lens) + 2)
    roff = np.concatenate([[0], np.cumsum(q)]).astype(np.int64)
    attrs = g.integers(-9, 9, (A, n)).astype(np.int32)
    recs = g.integers(100, 10 ** 6, (A, max(1, int(roff[-1])))).astype(np.int32)
    mask = (g.random(n) < 0.6).astype(np.uint8) * 7
    alive = (g.random(n) < 0.5).astype(np.int32) * 3
    kill = (g.random(n) < 0.3).astype(np.uint8)
    dev = lambda a: torch.from_numpy(a).cuda()
    d_attrs, d_alive = dev(attrs), dev(alive)
    ap, dr = abm.select_update_batched(d_attrs, dev(off), dev(mask), dev(recs), dev(roff))
    rm = abm.remove_agents_batched(d_alive, dev(off), dev(kill))
    ad, dd = abm.add_agents_batched(d_attrs, d_alive, dev(off), dev(recs), dev(roff))
    ap, dr, rm, ad, dd = (t.cpu().numpy() for t in (ap, dr, rm, ad, dd))
    e_attrs, e_alive = attrs.copy(), alive.copy()
    for m in range(len(lens)):
        s, r = slice(off[m], off[m + 1]), recs[:, roff[m]:roff[m + 1]]
        sel = np.flatnonzero(mask[s])[:r.shape[1]]
        e_attrs[:, s][:, sel] = r[:, :sel.size]
        assert (int(ap[m]), int(dr[m])) == (sel.size, r.shape[1] - sel.size), m
        gone = (kill[s] != 0) & (e_alive[s] != 0)
        e_alive[s][gone] = 0
        assert int(rm[m]) == int(gone.sum()), m
        free = np.flatnonzero(e_alive[s] == 0)[:r.shape[1]]
        e_attrs[:, s][:, free] = r[:, :free.size]
        e_alive[s][free] = 1
        assert (int(ad[m]), int(dd[m])) == (free.size, r.shape[1] - free.size), m
    assert np.array_equal(d_attrs.cpu().numpy(), e_attrs)
    assert np.array_equal(d_alive.cpu().numpy(), e_alive)


def test_records_far_from_the_first(abm):
    """Two segments of one tile whose records lie 2^28 and more apart."""
    far = 2 ** 28 + 100
    recs = torch.zeros((1, far + 40), dtype=torch.int32, device="cuda")
    recs[0, :8] = torch.arange(8, device="cuda")
    recs[0, far:far + 40] = 1000 + torch.arange(40, device="cuda")
    off = torch.tensor([0, 10, 20, 90], device="cuda")
    roff = torch.tensor([0, far - 164, far, far + 40], device="cuda")   # the second starts at 2^28 - 64
    attrs = torch.full((1, 90), -1, dtype=torch.int32, device="cuda")
    mask = torch.ones(90, dtype=torch.uint8, device="cuda")
    ap, _ = abm.select_update_batched(attrs, off, mask, recs, roff)
    a = attrs[0].cpu()
    assert ap.tolist() == [10, 10, 40]
    assert a[:10].tolist() == [0, 1, 2, 3, 4, 5, 6, 7, 0, 0] and a[10:20].tolist() == [0] * 10
    assert a[20:60].tolist() == list(range(1000, 1040)) and a[60:].tolist() == [-1] * 30


def test_empty_offsets_are_refused(abm):
    """No offset at all is not a number of segments: the call's own error."""
    none = torch.zeros(0, dtype=torch.int64, device="cuda")
    rows = torch.zeros((1, 8), dtype=torch.int32, device="cuda")
    alive = torch.zeros(8, dtype=torch.int32, device="cuda")
    mask = torch.zeros(8, dtype=torch.uint8, device="cuda")
    for call in (lambda: abm.select_update_batched(rows, none, mask, rows, none),
                 lambda: abm.add_agents_batched(rows, alive, none, rows, none),
                 lambda: abm.remove_agents_batched(alive, none, mask)):
        with pytest.raises(abm.AbmError):
            call()
