"""Runs of neighbours at every length: what does not fill a load step, a batch of steps or a run of 64, rows whose run
crosses from the local to the halo table, wavefronts whose short rows differ in length, at every number of lanes a table
row can take; items taken by a team of wavefronts, as a launch this small does by itself where a row takes 8 lanes or
more, and one after the other by one (items_per_wave given).  Reference: the sum in float64, row by row.
"""
import numpy as np
import pytest
import torch

from paper_2209_06800_amd import binding

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def _graph(n, top, rng):
    """Row v of the first half has v mod (top + 1) neighbours anywhere; the others are only gathered."""
    lens = np.concatenate([np.arange(n // 2) % (top + 1), np.zeros(n - n // 2, dtype=np.int64)])
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    row = np.repeat(np.arange(n), lens)
    col = rng.integers(0, n - 1, ptr[-1])
    return ptr, (col + (col >= row)).astype(np.int32)               # no self-loops


@pytest.mark.parametrize("short_max,per_wave", [(-1, 0), (-1, 2), (16, 0), (200, 0)])
@pytest.mark.parametrize("dim,bf16", [(3, False), (16, False), (30, False), (64, False), (75, False), (128, False), (210, False), (300, False),
                                      (5, True), (32, True), (60, True), (128, True), (250, True), (400, True)])
def test_runs_of_every_length(dim, bf16, short_max, per_wave):
    rng = np.random.default_rng(dim + short_max)
    n, top = 600, 149
    ptr, col = _graph(n, top, rng)
    x = torch.from_numpy(rng.standard_normal((n, dim)).astype(np.float32)).cuda()
    if bf16:
        x = x.bfloat16()
    bounds = np.array([0, 400, n], dtype=np.int64)                  # owned rows 0..399, some neighbours on the other side
    part = binding.mgg_build_partition(ptr, col, 2, 0, bounds, short_max=short_max)
    part.set_option("items_per_wave", per_wave)
    e = part.export()
    halo = torch.from_numpy(e["halo_gid"].astype(np.int64)).cuda()
    xd = x.double().cpu()
    for mode in ("gin", "gcn"):
        got = binding.mgg_aggregate(part, mode, x[:400].contiguous(), x[halo].contiguous(), eps=0.25).double().cpu()
        dinv = torch.from_numpy(1.0 / np.sqrt(np.diff(ptr) + 1.0))
        for v in range(400):
            nb = torch.from_numpy(col[ptr[v]:ptr[v + 1]].astype(np.int64))
            if mode == "gin":
                want, scale = xd[nb].sum(0) + 1.25 * xd[v], xd[nb].abs().sum(0) + 1.25 * xd[v].abs()
            else:
                w = dinv[nb][:, None] * dinv[v]
                want, scale = (w * xd[nb]).sum(0) + dinv[v] ** 2 * xd[v], (w * xd[nb].abs()).sum(0) + dinv[v] ** 2 * xd[v].abs()
            # at most one rounding per term on the way, and four for factors, self term and row factor
            assert ((got[v] - want).abs() <= (len(nb) + 5) * U * scale).all(), (mode, v)


@pytest.mark.parametrize("per_wave", [0, 1])
@pytest.mark.parametrize("dim,bf16", [(16, False), (64, False), (100, False), (200, False), (128, True)])
def test_a_row_that_is_not_gathered_does_not_count(dim, bf16, per_wave):
    """Lanes without a neighbour of their own gather a row that exists and drop it: an infinity there reaches only the
    rows whose neighbour it is."""
    rng = np.random.default_rng(dim)
    n, top = 600, 70
    ptr, col = _graph(n, top, rng)
    x = torch.from_numpy(rng.standard_normal((n, dim)).astype(np.float32)).cuda()
    bad = [0, 1, 399, 450]
    x[bad] = float("inf")
    if bf16:
        x = x.bfloat16()
    part = binding.mgg_build_partition(ptr, col, 2, 0, np.array([0, 400, n], dtype=np.int64))
    part.set_option("items_per_wave", per_wave)
    halo = torch.from_numpy(part.export()["halo_gid"].astype(np.int64)).cuda()
    for mode in ("gin", "gcn"):
        got = binding.mgg_aggregate(part, mode, x[:400].contiguous(), x[halo].contiguous()).cpu()
        for v in range(400):
            touched = v in bad or bool(np.isin(col[ptr[v]:ptr[v + 1]], bad).any())
            assert bool(torch.isinf(got[v]).all()) if touched else bool(torch.isfinite(got[v]).all()), (mode, v)


@pytest.mark.parametrize("rows,team", [(40, 8), (600, 4), (1500, 2)])
@pytest.mark.parametrize("dim,bf16", [(16, False), (30, False), (64, False), (100, False), (200, False), (128, True), (300, True)])
def test_teams_of_every_size(dim, bf16, rows, team):
    """Launches that take teams of 8, 4 and 2 wavefronts, with rows cut at 512 neighbours of each list beside whole ones,
    against float64 and against one wavefront per item: equal up to the order of the sums."""
    rng = np.random.default_rng(dim)
    n, own = 3000, 2600
    lens = np.zeros(n, dtype=np.int64)
    lens[:rows] = rng.integers(17, 600, rows)
    lens[rng.permutation(rows)[:3]] = 4500                             # 3900 local and 600 remote neighbours, or about that
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    row = np.repeat(np.arange(n), lens)
    col = rng.integers(0, n - 1, ptr[-1])
    col = (col + (col >= row)).astype(np.int32)
    x = torch.from_numpy(rng.standard_normal((n, dim)).astype(np.float32)).cuda()
    if bf16:
        x = x.bfloat16()
    part = binding.mgg_build_partition(ptr, col, 2, 0, np.array([0, own, n], dtype=np.int64), xcd_min_deg=-1)
    assert part.info.n_split_rows >= 3 and part.info.n_split_items > 20
    assert binding.mgg_aggregate_plan(part, "gcn", dim, bf16=bf16).team == team
    halo = torch.from_numpy(part.export()["halo_gid"].astype(np.int64)).cuda()
    xl, xh, xd = x[:own].contiguous(), x[halo].contiguous(), x.double().cpu().numpy()
    for mode in ("gin", "gcn"):
        want, scale = _sums(ptr, col, own, xd, mode, 0.5)
        bound = (lens[:own, None] + 6) * U * scale
        for per_wave in (0, 2):
            part.set_option("items_per_wave", per_wave)
            assert (binding.mgg_aggregate_plan(part, mode, dim, bf16=bf16).team > 1) == (per_wave == 0)
            got = binding.mgg_aggregate(part, mode, xl, xh, eps=0.5).double().cpu().numpy()
            assert (np.abs(got - want) <= bound).all(), (mode, per_wave)


@pytest.mark.parametrize("dim,bf16", [(80, False), (256, True)])
def test_fine_schedule(dim, bf16):
    """A share large enough for the schedule that regroups rows of 128 neighbours on: in the partition's own buffer and in
    a layer's workspace there is room for its partial sums, in the fixed array of the static call there is not, and a
    workspace that holds those of the other schedule is still enough.  Both against float64; a partition without the
    second schedule gives the same bits in all of them."""
    rng = np.random.default_rng(8)
    n, own = 60000, 34000
    lens = np.concatenate([rng.integers(100, 256, own // 2), rng.integers(256, 440, own // 2), np.zeros(n - own, dtype=np.int64)])
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    row = np.repeat(np.arange(n), lens)
    col = rng.integers(0, n - 1, ptr[-1])
    col = (col + (col >= row)).astype(np.int32)
    bounds = np.array([0, own, n], dtype=np.int64)
    part = binding.mgg_build_partition(ptr, col, 2, 0, bounds, fine_min_neighbours=0)
    one = binding.mgg_build_partition(ptr, col, 2, 0, bounds, fine_min_neighbours=-1)
    need = binding.mgg_aggregate_scratch_bytes(part, dim)
    assert ptr[-1] > 8 << 20 and need == binding.mgg_aggregate_scratch_bytes(one, dim) and part.info.n_fine_split_items > 0
    static_fits = need <= 64 << 20
    assert static_fits == (dim == 80)
    assert [binding.mgg_aggregate_plan(part, "gcn", dim, bf16=bf16, scratch_bytes=b).fine for b in (None, 64 << 20)] == [1, 0]
    x = torch.from_numpy(rng.standard_normal((n, dim)).astype(np.float32)).cuda()
    if bf16:
        x = x.bfloat16()
    halo = torch.from_numpy(part.export()["halo_gid"].astype(np.int64)).cuda()
    xl, xh, xd = x[:own].contiguous(), x[halo].contiguous(), x.double().cpu().numpy()
    w = torch.eye(dim, device="cuda", dtype=x.dtype)
    full = binding.mgg_layer_workspace_bytes(part, "gcn", [w], ["none"])
    least = binding.mgg_layer_workspace_least_bytes(part, "gcn", [w], ["none"])
    assert least == binding.mgg_layer_workspace_bytes(one, "gcn", [w], ["none"]) and least < full <= least + 2 * need
    layer = lambda p, room: binding.mgg_layer_forward(p, mode, xl, xh, [w], ["none"], workspace=torch.empty(room, dtype=torch.uint8, device="cuda"))
    for mode in ("gin", "gcn"):
        want, scale = _sums(ptr, col, own, xd, mode, 0)
        bound = (lens[:own, None] + 6) * U * scale
        got, coarse = binding.mgg_aggregate(part, mode, xl, xh), binding.mgg_aggregate(one, mode, xl, xh)
        for g in (got, coarse):
            assert (np.abs(g.double().cpu().numpy() - want) <= bound).all(), mode
        assert not torch.equal(got, coarse), mode                    # another order of the sums: the two schedules
        if static_fits:
            assert torch.equal(coarse, binding.mgg_aggregate_static(one, mode, xl, xh))
            static = binding.mgg_aggregate_static(part, mode, xl, xh)
            assert (np.abs(static.double().cpu().numpy() - want) <= bound).all() and not torch.equal(got, static), mode
            assert torch.equal(layer(part, full), got) and torch.equal(layer(part, least), static), mode
        assert torch.equal(layer(one, full), layer(one, least)), mode
    with pytest.raises(binding.MggError):
        layer(part, least - 512)


def test_slabs_in_chunks():
    """Rows of 1 KB, a table whose 256-byte slabs fit the L2s and more ids than 128 MB: the launch walks chunks of the work
    through all slabs.  Against the same slabs asked for, which are walked in one chunk: the same bits."""
    rng = np.random.default_rng(4)
    n, dim = 60000, 256
    lens = rng.integers(0, 600, n)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    row = np.repeat(np.arange(n), lens)
    col = rng.integers(0, n - 1, ptr[-1])
    col = (col + (col >= row)).astype(np.int32)
    assert ptr[-1] * 8 >= 128 << 20
    x = torch.from_numpy(rng.standard_normal((n, dim)).astype(np.float32)).cuda()
    part = binding.mgg_build_partition(ptr, col)
    plan = binding.mgg_aggregate_plan(part, "gcn", dim)
    assert (plan.slab_bytes, plan.n_slabs, plan.n_chunks) == (256, 4, 4)
    got = binding.mgg_aggregate(part, "gcn", x)
    part.set_option("col_slab_bytes", 256)
    assert binding.mgg_aggregate_plan(part, "gcn", dim).n_chunks == 1
    assert torch.equal(got, binding.mgg_aggregate(part, "gcn", x))


def _sums(ptr, col, own, x, mode, eps):
    """Aggregate rows 0 .. own - 1 in float64, and the sums of the magnitudes."""
    import scipy.sparse as sp
    n = ptr.size - 1
    adj = sp.csr_matrix((np.ones(col.size), col, ptr), shape=(n, n))[:own]
    if mode == "gcn":
        dinv = 1.0 / np.sqrt(np.diff(ptr) + 1.0)
        adj, self_w = sp.diags(dinv[:own]) @ adj @ sp.diags(dinv), dinv[:own, None] ** 2
    else:
        self_w = 1.0 + eps
    return adj @ x + self_w * x[:own], adj @ np.abs(x) + np.abs(self_w) * np.abs(x[:own])


@pytest.mark.parametrize("lds", [0, 1])
@pytest.mark.parametrize("wpb,per_wave,ps,dist,xcd_min_deg", [(1, 1, 0, 0, 0), (1, 3, 16, 2, 40), (2, 2, 7, 3, 0), (4, 1, 0, 0, 40), (4, 5, 0, 1, 0), (8, 2, 0, 0, 20), (16, 3, 5, 4, 0),
                                                              (16, 1, 0, 0, 40)])
@pytest.mark.parametrize("dim,bf16", [(12, False), (64, False), (100, False), (128, True)])
def test_items_of_every_queue(dim, bf16, wpb, per_wave, ps, dist, xcd_min_deg, lds):
    """One wavefront per item, several items one after the other, at every kind of workgroup: queues that end inside a
    wavefront's items, rows without local or without remote neighbours, empty rows between them; halo rows through
    registers and through LDS; both lists in one launch and in two."""
    rng = np.random.default_rng(wpb * 100 + per_wave + dim)
    n, own = 900, 500
    lens = rng.integers(0, 90, n)
    lens[::7] = 0
    lens[rng.permutation(own)[:12]] = rng.integers(200, 700, 12)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    row = np.repeat(np.arange(n), lens)
    col = rng.integers(0, n, ptr[-1])
    col = np.where(row % 5 == 1, col % own, np.where(row % 5 == 2, own + col % (n - own), col))     # local only, remote only
    col = np.where(col == row, (col + 1) % own, col).astype(np.int32)
    x = torch.from_numpy(rng.standard_normal((n, dim)).astype(np.float32)).cuda()
    if bf16:
        x = x.bfloat16()
    xd = x.double().cpu().numpy()
    part = binding.mgg_build_partition(ptr, col, 2, 0, np.array([0, own, n], dtype=np.int64), wpb=wpb, ps=ps, dist=dist, xcd_min_deg=xcd_min_deg, short_max=-1 if wpb == 1 else 0)
    part.set_option("items_per_wave", per_wave)
    part.set_option("lds_halo", lds)
    plan = binding.mgg_aggregate_plan(part, "gcn", dim, bf16=bf16)
    assert (plan.team, plan.wpb, plan.items_per_wave, plan.lds_halo) == (1, wpb, per_wave, int(lds and wpb <= 8))
    halo = torch.from_numpy(part.export()["halo_gid"].astype(np.int64)).cuda()
    for mode in ("gin", "gcn"):
        want, scale = _sums(ptr, col, own, xd, mode, 0.25)
        for two in (0, 1):
            part.set_option("split_phases", two)
            got = binding.mgg_aggregate(part, mode, x[:own].contiguous(), x[halo].contiguous(), eps=0.25).double().cpu().numpy()
            # one rounding per term on the way, four for factors, self term and row factor, one where two launches meet
            assert (np.abs(got - want) <= (lens[:own, None] + 6) * U * scale).all(), (mode, two)


@pytest.mark.parametrize("classes", [False, True])
@pytest.mark.parametrize("rows", [1, 7, 8, 9, 15, 16, 17, 31, 33, 50])
def test_teams_take_every_item_of_every_queue(rows, classes):
    """One workgroup per item, queue by queue: lists that end inside a group of a queue, padded lists of regrouped rows, slabs."""
    rng = np.random.default_rng(rows)
    n = 2000
    lens = np.zeros(n, dtype=np.int64)
    lens[rng.permutation(n)[:rows]] = rng.integers(300, 900, rows)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    row = np.repeat(np.arange(n), lens)
    col = rng.integers(0, n - 1, ptr[-1])
    col = (col + (col >= row)).astype(np.int32)
    part = binding.mgg_build_partition(ptr, col, xcd_min_deg=0 if classes else -1, hot_phases=-1)
    for dim in (64, 300):
        x = torch.from_numpy(rng.standard_normal((n, dim)).astype(np.float32)).cuda()
        assert binding.mgg_aggregate_plan(part, "gcn", dim).team > 1
        want, scale = _sums(ptr, col, n, x.double().cpu().numpy(), "gcn", 0)
        out = torch.full((n, dim), float("nan"), device="cuda")
        got = binding.mgg_aggregate(part, "gcn", x, out=out).double().cpu().numpy()
        assert (np.abs(got - want) <= (lens[:, None] + 6) * U * scale).all()
