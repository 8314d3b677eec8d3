"""GPU parity of sort_agents (stable LSD radix sort + gather) and
select_agents (stable partition) against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2508_16508_amd import workloads as W

pytestmark = pytest.mark.gpu


def _keys(kind, n, g):
    if kind == "full":
        return g.integers(-2 ** 31, 2 ** 31, size=n, dtype=np.int64).astype(np.int32)
    if kind == "few":
        return g.integers(-3, 4, size=n).astype(np.int32)       # long runs of equal keys
    if kind == "equal":
        return np.full(n, 7, dtype=np.int32)
    if kind == "sorted":
        return np.sort(g.integers(-1000, 1000, size=n)).astype(np.int32)
    if kind == "reversed":
        return np.sort(g.integers(-1000, 1000, size=n))[::-1].astype(np.int32).copy()
    if kind == "extremes":
        return g.choice(np.array([-2 ** 31, -1, 0, 1, 2 ** 31 - 1], dtype=np.int32), size=n)
    raise ValueError(kind)


@pytest.mark.parametrize("n", [1, 100, 4096, 4097, 3 * 4096 + 17, 1 << 20])
@pytest.mark.parametrize("kind", ["full", "few", "equal", "sorted", "reversed", "extremes"])
@pytest.mark.parametrize("descending", [False, True])
def test_sort_matches_oracle(abm, orc, n, kind, descending):
    g = np.random.default_rng(n + len(kind) + descending)
    key = _keys(kind, n, g)
    attrs = W.int32_rows(n + 1, 3, n)
    alive = (g.random(n) < 0.5).astype(np.int32)
    eo, ea, ep = orc.sort_agents(attrs, key, descending=descending, alive=alive)
    d_attrs = torch.from_numpy(attrs).cuda()
    d_alive = torch.from_numpy(alive).cuda()
    perm = abm.sort_agents(d_attrs, torch.from_numpy(key).cuda(), descending, alive=d_alive)
    torch.cuda.synchronize()
    assert np.array_equal(perm.cpu().numpy()[:n], ep)
    assert np.array_equal(d_attrs.cpu().numpy(), eo)
    assert np.array_equal(d_alive.cpu().numpy(), ea)


@pytest.mark.parametrize("n_attrs,with_alive", [(0, True), (1, False), (1, True), (2, True),
                                                (4, True), (8, False), (8, True), (16, True)])
@pytest.mark.parametrize("n", [6, 4099, 70001])
def test_sort_column_groups(abm, orc, n_attrs, with_alive, n):
    """Every record size (1 to 17 columns: records of 1 to 32 words) and
    every length mod 4."""
    g = np.random.default_rng(100 * n_attrs + n + with_alive)
    key = _keys("few", n, g)
    attrs = W.int32_rows(n_attrs + 3, max(n_attrs, 1), n)[:n_attrs]
    alive = (g.random(n) < 0.5).astype(np.int32)
    eo, ea, ep = orc.sort_agents(attrs, key, alive=alive if with_alive else None)
    d_attrs = torch.from_numpy(np.ascontiguousarray(attrs)).cuda()
    d_alive = torch.from_numpy(alive).cuda()
    perm = abm.sort_agents(d_attrs, torch.from_numpy(key).cuda(),
                           alive=d_alive if with_alive else None)
    torch.cuda.synchronize()
    assert np.array_equal(perm.cpu().numpy()[:n], ep)
    assert np.array_equal(d_attrs.cpu().numpy(), eo)
    if with_alive:
        assert np.array_equal(d_alive.cpu().numpy(), ea)
    else:
        assert np.array_equal(d_alive.cpu().numpy(), alive)


def test_sort_microbench_size(abm, orc):
    """2^24 agents x 8 attributes, full-range keys (the select_update
    workload's collection)."""
    n = 1 << 24
    g = np.random.default_rng(24)
    key = _keys("full", n, g)
    attrs = W.int32_rows(5, 8, n)
    _, _, ep = orc.sort_agents(attrs[:1], key)
    d_attrs = torch.from_numpy(attrs).cuda()
    perm = abm.sort_agents(d_attrs, torch.from_numpy(key).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(perm.cpu().numpy(), ep)
    sample = g.integers(0, n, size=4096)
    got = d_attrs.cpu().numpy()
    assert np.array_equal(got[:, sample], attrs[:, ep[sample]])


@pytest.mark.parametrize("n", [1, 64, 4097, 1 << 16, 1 << 24, (1 << 24) + 12345])
@pytest.mark.parametrize("p", [0.0, 0.001, 0.5, 1.0])
def test_select_agents_matches_oracle(abm, orc, n, p):
    cond = W.bernoulli_mask(n + 7, p, n) if 0 < p < 1 else np.full(n, int(p), dtype=np.uint8)
    eo, ec = orc.select_agents(cond)
    order, count = abm.select_agents(torch.from_numpy(cond).cuda())
    torch.cuda.synchronize()
    assert int(count.item()) == ec
    assert np.array_equal(order.cpu().numpy()[:n], eo)


# the last size of the single launch (15 tiles of 4096 flags) and the first past it
@pytest.mark.parametrize("n", [4096, 15 * 4096 - 1, 15 * 4096, 15 * 4096 + 1])
@pytest.mark.parametrize("p", [0.0, 0.5, 1.0])
def test_select_agents_around_the_single_launch(abm, orc, n, p):
    cond = (np.random.default_rng(n).random(n) < p).astype(np.uint8) * 255
    eo, ec = orc.select_agents(cond)
    order, count = abm.select_agents(torch.from_numpy(cond).cuda())
    assert int(count.item()) == ec
    assert np.array_equal(order.cpu().numpy()[:n], eo)


@pytest.mark.parametrize("offset", [1, 3, 8])
@pytest.mark.parametrize("n", [5, 4096 * 3 + 9])
def test_select_agents_unaligned_flags(abm, orc, offset, n):
    """Flags that do not start on a 16-byte boundary, with values other than
    0 and 1 (any nonzero byte is true)."""
    g = np.random.default_rng(offset * 7 + n)
    flags = (g.random(n + offset) < 0.3).astype(np.uint8) * g.integers(1, 256, size=n + offset,
                                                                       dtype=np.int64).astype(
        np.uint8)
    cond = flags[offset:]
    eo, ec = orc.select_agents(cond)
    order, count = abm.select_agents(torch.from_numpy(flags).cuda()[offset:])
    torch.cuda.synchronize()
    assert int(count.item()) == ec
    assert np.array_equal(order.cpu().numpy()[:n], eo)


def test_empty_collection(abm, orc):
    """n = 0: nothing to sort, the count is 0."""
    attrs = torch.zeros((3, 0), dtype=torch.int32, device="cuda")
    perm = abm.sort_agents(attrs, torch.zeros(0, dtype=torch.int32, device="cuda"),
                           alive=torch.zeros(0, dtype=torch.int32, device="cuda"))
    order, count = abm.select_agents(torch.zeros(0, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert int(count.item()) == 0 and perm.numel() >= 0 and order.numel() >= 0
    assert orc.select_agents(np.zeros(0, dtype=np.uint8))[1] == 0


def test_sort_rejects_small_workspace_and_bad_counts(abm):
    key = torch.zeros(5000, dtype=torch.int32, device="cuda")
    attrs = torch.zeros((1, 5000), dtype=torch.int32, device="cuda")
    small = abm.sort_workspace(100)
    with pytest.raises(abm.AbmError):
        abm.sort_agents(attrs, key, ws=small)
    with pytest.raises(abm.AbmError):
        abm.select_agents(torch.zeros(5000, dtype=torch.uint8, device="cuda"), ws=small)
    # enough for select_agents and for 2 columns, not for the records of 9
    ws0 = abm.sort_workspace(5000, n_cols=0)
    abm.select_agents(torch.zeros(5000, dtype=torch.uint8, device="cuda"), ws=ws0)
    abm.sort_agents(torch.zeros((2, 5000), dtype=torch.int32, device="cuda"), key, ws=ws0)
    with pytest.raises(abm.AbmError):
        abm.sort_agents(torch.zeros((8, 5000), dtype=torch.int32, device="cuda"), key,
                        alive=torch.zeros(5000, dtype=torch.int32, device="cuda"), ws=ws0)
    with pytest.raises(ValueError):
        abm.sort_workspace(5000, n_cols=18)
