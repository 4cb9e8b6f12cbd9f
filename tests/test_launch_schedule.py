"""The schedule as the kernels read it, on the CPU: the neighbour stream in the order of the work, the two item tables over
it (whole and cut rows, and the fine schedule that regroups rows of 128 neighbours too), the short rows and the
partial-sum slots.  Reference: the canonical row lists of the same partition, which the builder tests compare with the oracle.
"""
import numpy as np
import pytest

from paper_2209_06800_amd import binding, inputs

HALO = np.uint32(1 << 31)


def _graph(n, top, seed, hubs=0):
    """Directed rows of 0 .. top neighbours, `hubs` of them with up to 3000; duplicates, no self-loops."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, top + 1, n)
    lens[:n // 4] = rng.integers(0, 20, n // 4)
    lens[rng.permutation(n)[:hubs]] = rng.integers(600, 3000, hubs)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    row = np.repeat(np.arange(n), lens)
    col = rng.integers(0, n - 1, ptr[-1])
    return ptr, (col + (col >= row)).astype(np.int32)


def _runs(beg, length):
    """Positions of runs [beg, beg + length), one after the other."""
    return np.repeat(beg - np.concatenate([[0], np.cumsum(length)[:-1]]), length) + np.arange(length.sum())


def _check_cover(part, e, l, items, which):
    """Every (row, neighbour, table) once in these items and the short rows; slots of cut rows in order."""
    info = part.info
    nnz = int(info.nnz_local + info.nnz_remote)
    it = items[items[:, 0] >= 0].astype(np.int64)
    assert np.all(items[items[:, 0] < 0][:, 3:5] == [0, -1])                    # padding: nothing to do
    row, beg, nl, n, slot, rbeg = it[:, :6].T
    assert np.all(nl >= 0) and np.all(n >= nl) and np.all(beg >= 0) and np.all(beg + nl <= nnz)
    assert np.all(rbeg >= 0) and np.all(rbeg + n - nl <= nnz)
    sh = l["launch_short"].astype(np.int64)
    assert np.array_equal(sh[:, 0], e["short_rows"]) and np.all(sh[:, 2] <= sh[:, 3])
    pos = np.concatenate([_runs(beg, nl), _runs(rbeg, n - nl), _runs(sh[:, 1], sh[:, 3])])
    assert np.array_equal(np.sort(pos), np.arange(nnz)), which                  # each place of the stream once
    rows = np.concatenate([np.repeat(row, nl), np.repeat(row, n - nl), np.repeat(sh[:, 0], sh[:, 3])])
    remote = np.concatenate([np.zeros(nl.sum()), np.ones((n - nl).sum()), (np.arange(sh[:, 3].sum()) - np.repeat(np.cumsum(sh[:, 3]) - sh[:, 3], sh[:, 3]) >=
                                                                          np.repeat(sh[:, 2], sh[:, 3]))]).astype(bool)
    got = l["launch_cols"][pos]
    assert np.array_equal(got >= HALO, remote), which                           # the bit says the table that the counts say
    key = rows * (1 << 33) + (got & ~HALO).astype(np.int64) * 2 + remote
    n_own = int(info.n_own)
    want = np.concatenate([np.repeat(np.arange(n_own), np.diff(e[f"{k}_row_ptr"])) * (1 << 33) + e[f"{k}_col"].astype(np.int64) * 2 + b
                           for b, k in enumerate(("local", "remote"))])
    assert np.array_equal(np.sort(key), np.sort(want)), which
    # cut rows: the slots of a SplitRow are its items', contiguous and nobody else's
    sr = l["launch_split_rows"].astype(np.int64)
    if which == "coarse":
        sr = sr[:info.n_split_rows]
    cut = slot >= 0
    owner = np.full(int(sr[:, 2].sum()), -1)
    for r, first, count, _ in sr:
        assert np.all(owner[first:first + count] == -1)
        owner[first:first + count] = r
    assert np.all(owner >= 0) and np.array_equal(np.sort(slot[cut]), np.arange(owner.size)), which
    assert np.array_equal(owner[slot[cut]], row[cut]) and np.unique(sr[:, 0]).size == sr.shape[0]
    whole = np.concatenate([row[~cut], sr[:, 0], sh[:, 0]])
    assert np.array_equal(np.sort(whole), np.arange(n_own)), which              # every row is written once
    return it, pos


@pytest.mark.parametrize("parts,part_id,wpb,seed,bags", [(1, 0, 0, 1, False), (2, 0, 1, 2, False), (3, 1, 4, 3, False), (2, 1, 16, 4, False), (1, 0, 2, 5, True)])
def test_launch_arrays_hold_every_neighbour_once(parts, part_id, wpb, seed, bags):
    n = 2400
    ptr, col = _graph(n, 330, seed, hubs=30)
    kw = dict(host_only=True, wpb=wpb, hot_phases=-1, fine_min_neighbours=1)
    if bags:
        part = binding.mgg_build_bags(ptr, col, n, 200, 900, **kw)
    else:
        part = binding.mgg_build_partition(ptr, col, parts, part_id, **kw)
    info, e, l = part.info, part.export(), part.export_launch()
    assert info.n_fine_items > 0 and info.n_fine_split_items > 0 and info.n_short_rows > 0
    assert int(info.nnz_local + info.nnz_remote) >= 1 << 18 or parts > 1       # laid out by several threads, too
    assert info.n_fine_split_items <= 2 * info.n_split_items
    _, _ = _check_cover(part, e, l, l["launch_items"], "coarse")
    it, _ = _check_cover(part, e, l, l["launch_fine_items"], "fine")
    # the coarse table is the exported one, item by item, and its stream runs front to back in the queue of each XCD
    li = l["launch_items"].astype(np.int64)
    assert np.array_equal(li[:, 0], e["item_row"]) and np.array_equal(li[:, 4], e["item_slot"])
    assert np.array_equal(li[:, 2], e["item_lend"] - e["item_lbeg"]) and np.array_equal(li[:, 3] - li[:, 2], e["item_rend"] - e["item_rbeg"])
    xcd = (np.arange(li.shape[0]) // info.wpb) % 8
    queue = np.concatenate([np.nonzero(xcd == x)[0] for x in range(8)])
    begs = np.concatenate([li[queue, 1], l["launch_short"][:, 1]])
    ends = np.concatenate([li[queue, 1] + li[queue, 3], l["launch_short"][:, 1] + l["launch_short"][:, 3]])
    assert begs[0] == 0 and np.array_equal(begs[1:], ends[:-1])
    # the fine table: rows of 128 to 255 are pieces of one class on its XCD (or the rest of the row), the others as they were
    fi = l["launch_fine_items"].astype(np.int64)
    assert fi.shape[0] % (8 * info.wpb) == 0
    deg = np.diff(e["local_row_ptr"]) + np.diff(e["remote_row_ptr"])
    cls = np.concatenate([e["src_class_local"], e["src_class_halo"]])
    n_local = e["src_class_local"].size
    for i, (row, beg, nl, cnt, slot, rbeg) in enumerate(fi[:, :6]):
        if row < 0 or not 128 <= deg[row] < 256:
            continue
        place = np.concatenate([np.arange(beg, beg + nl), np.arange(rbeg, rbeg + cnt - nl)])
        u = l["launch_cols"][place]
        c = cls[np.where(u >= HALO, (u & ~HALO) + n_local, u).astype(np.int64)]
        count = np.bincount(cls[np.concatenate([e["local_col"][e["local_row_ptr"][row]:e["local_row_ptr"][row + 1]],
                                                n_local + e["remote_col"][e["remote_row_ptr"][row]:e["remote_row_ptr"][row + 1]]])], minlength=8)
        if np.all(c == c[0]) and count[c[0]] >= info.min_piece:
            assert c[0] == (i // info.wpb) % 8 and count[c[0]] == c.size
        else:
            assert np.all(count[c] < info.min_piece)
    other = {tuple(r[[0, 1, 2, 3, 4]]) for r in li if r[0] >= 0 and not 128 <= deg[r[0]] < 256}
    assert other == {tuple(r[[0, 1, 2, 3, 4]]) for r in fi if r[0] >= 0 and not 128 <= deg[r[0]] < 256}
    # the factor beside every neighbour is that neighbour's
    if not bags:
        u = l["launch_cols"]
        d = np.where(u >= HALO, e["deg_halo"][np.minimum(u & ~HALO, max(int(info.num_halo) - 1, 0))] if info.num_halo else 0, e["deg_own"][np.minimum(u, info.n_own - 1)])
        assert np.array_equal(l["launch_wts"], (1.0 / np.sqrt(d + 1.0)).astype(np.float32))


def test_the_fine_schedule_is_for_large_shares_with_the_default_cuts():
    ptr, col = _graph(1500, 330, 7, hubs=20)
    build = lambda **kw: binding.mgg_build_partition(ptr, col, host_only=True, hot_phases=-1, **kw).info
    nnz = int(ptr[-1])
    assert build().n_fine_items == 0                                            # 2^23 neighbours by default
    assert build(fine_min_neighbours=nnz).n_fine_items > 0 and build(fine_min_neighbours=nnz + 1).n_fine_items == 0
    for kw in (dict(xcd_min_deg=256), dict(min_piece=16), dict(xcd_min_deg=-1)):
        assert build(fine_min_neighbours=1, **kw).n_fine_items == 0, kw
    info = build(fine_min_neighbours=-1)
    assert (info.n_fine_items, info.n_fine_split_rows, info.n_fine_split_items) == (0, 0, 0)


# ---- what a launch is: mgg_aggregate_plan ------------------------------------------------------------------------
def _lists(lens, n_table, seed=0):
    """A directed graph of max(len(lens), n_table) nodes whose first rows have these lengths."""
    rng = np.random.default_rng(seed)
    lens = np.concatenate([lens, np.zeros(max(0, n_table - len(lens)), dtype=np.int64)]).astype(np.int64)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    row = np.repeat(np.arange(lens.size), lens)
    col = rng.integers(0, lens.size - 1, ptr[-1])
    return ptr, (col + (col >= row)).astype(np.int32)


def test_plan_says_which_schedule_runs():
    """The fine schedule runs from the scratch on that holds its partial sums, the coarse one below; a partition built
    without it has one schedule whatever the scratch.  Narrow rows do not pay for it and ask for no room."""
    ptr, col = _graph(1500, 330, 7, hubs=20)
    part = binding.mgg_build_partition(ptr, col, host_only=True, hot_phases=-1, fine_min_neighbours=1)
    one = binding.mgg_build_partition(ptr, col, host_only=True, hot_phases=-1, fine_min_neighbours=-1)
    for dim in (36, 64, 100, 602):
        need = binding.mgg_aggregate_scratch_bytes(part, dim)
        full = need + int(part.info.n_fine_split_items) * (-(-dim // 8) * 8) * 4
        assert binding.mgg_aggregate_plan(part, "gcn", dim).fine == 1
        assert [binding.mgg_aggregate_plan(part, "gcn", dim, scratch_bytes=b).fine for b in (need, full - 1, full)] == [0, 0, 1]
        assert binding.mgg_aggregate_plan(one, "gcn", dim).fine == 0 and need == binding.mgg_aggregate_scratch_bytes(one, dim)
    for dim, bf16, fine in ((1, False, 0), (16, False, 0), (32, False, 0), (33, False, 1), (7, True, 0), (64, True, 0), (128, True, 0), (129, True, 1), (256, True, 1)):
        assert binding.mgg_aggregate_plan(part, "gcn", dim, bf16=bf16).fine == fine, (dim, bf16)
    # 16 lanes of bf16: on large tables with many neighbours
    for table, more, want in ((380000, 0, 0), (400000, 0, 1), (400000, -2000, 0)):
        lens = np.concatenate([np.full(25000, 200), np.full(29500 + more, 512)])
        ptr, col = _lists(lens, table)
        big = binding.mgg_build_partition(ptr, col, host_only=True, hot_phases=-1)
        assert big.info.n_fine_items > 0 and (ptr[-1] >= 20000000) == (more == 0)
        assert [binding.mgg_aggregate_plan(big, "gcn", d, bf16=True).fine for d in (64, 128, 256)] == [0, want, 1]


def test_plan_checks_its_arguments():
    part = binding.mgg_build_partition(*_graph(40, 20, 1), host_only=True)
    for kw in (dict(dim=0), dict(dim=8, ld=4), dict(dim=8, base_align=3), dict(dim=8, base_align=0)):
        with pytest.raises(binding.MggError) as err:
            binding.mgg_aggregate_plan(part, "gcn", **kw)
        assert err.value.status == binding.ERR_INVALID_ARG, kw
    lib = binding.lib()
    assert lib.mgg_aggregate_plan(None, 0, 0, 8, 8, 16, 0, None) == binding.ERR_INVALID_ARG
    assert lib.mgg_aggregate_plan(part.handle, 0, 0, 8, 8, 16, 0, None) == binding.ERR_INVALID_ARG
    with pytest.raises(binding.MggError):
        binding.mgg_aggregate_plan(part, "gcn", 2 ** 31 - 8)                    # beyond 65535 slabs of 4 KB


@pytest.mark.parametrize("dim,ld,bf16,align,lanes,per_lane", [(1, 1, False, 256, 4, 1), (3, 3, False, 4, 4, 1), (3, 4, False, 16, 4, 1), (16, 16, False, 256, 4, 1),
                                                              (20, 20, False, 256, 8, 1), (75, 75, False, 4, 32, 1), (64, 64, False, 256, 16, 1),
                                                              (5, 5, True, 2, 8, 1), (128, 128, True, 256, 16, 1), (260, 260, False, 256, 32, 1)])
def test_plan_lanes_of_a_row(dim, ld, bf16, align, lanes, per_lane):
    part = binding.mgg_build_partition(*_graph(40, 20, 1), host_only=True)
    plan = binding.mgg_aggregate_plan(part, "gcn", dim, ld=ld, bf16=bf16, base_align=align)
    assert (plan.lanes_per_row, plan.vectors_per_lane) == (lanes, per_lane)
    assert plan.n_slabs == -(-dim * (2 if bf16 else 4) // plan.slab_bytes)


@pytest.mark.parametrize("bags,per,table,slab_bytes", [(200000, 1, 8000, 512), (200000, 1, 8400, 256), (1000, 30, 200000, 256), (1000, 1, 4000, 512), (1000, 1, 1 << 20, 256),
                                                       (150000, 1, 1100000, 512), (100, 2000, 60000, 512), (100, 2000, 140000, 256), (100, 2000, 300000, 512)])
def test_slabs_go_by_the_rows_of_the_tables(bags, per, table, slab_bytes):
    """What has to stay in L2 is the tables, not the bags that a bag partition owns: the whole of them for short bags, which
    have no source classes, an eighth for long ones."""
    rng = np.random.default_rng(3)
    ptr = np.arange(bags + 1, dtype=np.int64) * per
    idx = rng.integers(0, table, bags * per).astype(np.int32)
    for lo, hi in ((0, table), (0, table // 2)):                                # all rows local; half of them served from the halo table
        part = binding.mgg_build_bags(ptr, idx, table, lo, hi, host_only=True, hot_phases=-1)
        rows = int(part.info.n_local_rows + part.info.num_halo)
        if per <= 32:
            want = 256 if rows * 512 > 4 << 20 and rows * 256 <= 256 << 20 else 512
        else:
            want = 256 if (rows // 8 + 1) * 512 > 8 << 20 and (rows // 8 + 1) * 256 <= 8 << 20 else 512
        assert want == slab_bytes or rows < table
        assert binding.mgg_aggregate_plan(part, "gin", 256).slab_bytes == want, (lo, hi)


@pytest.mark.parametrize("wpb", [1, 2, 4, 8, 16])
def test_a_given_number_of_wavefronts_is_kept(wpb):
    """wpb is a knob and an axis of the parameter search: a launch that a team would take by itself has the workgroups that
    were asked for, and several wpb are several launches."""
    ptr, col = _graph(1500, 330, 7, hubs=20)
    free = binding.mgg_aggregate_plan(binding.mgg_build_partition(ptr, col, host_only=True), "gcn", 64)
    assert free.team > 1 and free.wpb == free.team
    part = binding.mgg_build_partition(ptr, col, host_only=True, wpb=wpb)
    plan = binding.mgg_aggregate_plan(part, "gcn", 64)
    assert (plan.team, plan.wpb) == (1, wpb)
    part.set_option("items_per_wave", 2)
    assert binding.mgg_aggregate_plan(part, "gcn", 64).wpb == wpb


def test_plan_of_halo_rows_through_lds_and_of_two_launches():
    """Staged rows are requested 8 KB at a time: pieces stay as large as the coarse schedule leaves them.  Tables it cannot
    stage (rows off 16 bytes, 4 GB and more, no halo, workgroups beyond 8 wavefronts, several chunks a lane) take registers."""
    ptr, col = _graph(1500, 330, 7, hubs=20)
    kw = dict(host_only=True, hot_phases=-1, fine_min_neighbours=1)
    part = binding.mgg_build_partition(ptr, col, 2, 0, **kw)
    assert binding.mgg_aggregate_plan(part, "gcn", 64).fine == 1
    part.set_option("lds_halo", 1)
    plan = binding.mgg_aggregate_plan(part, "gcn", 64)
    assert (plan.lds_halo, plan.fine, plan.team) == (1, 0, 1)
    rows = max(int(part.info.n_local_rows), int(part.info.num_halo))
    wide = -(-2 ** 32 // (4 * rows)) // 4 * 4 + 4
    for dim, more in ((64, dict(base_align=8)), (63, dict(ld=63)), (64, dict(ld=wide))):
        plan = binding.mgg_aggregate_plan(part, "gcn", dim, **more)
        assert (plan.lds_halo, plan.fine) == (0, 1), more
    assert binding.mgg_aggregate_plan(part, "gcn", 64, ld=wide - 8).lds_halo == 1
    part.set_option("col_slab_bytes", 1)
    assert [binding.mgg_aggregate_plan(part, "gcn", d).lds_halo for d in (256, 260)] == [1, 0]
    two = binding.mgg_build_partition(ptr, col, 2, 0, **kw)
    two.set_option("split_phases", 1)                               # every piece is walked and added up twice
    assert binding.mgg_aggregate_plan(two, "gcn", 64).fine == 0
    alone = binding.mgg_build_partition(ptr, col, **kw)
    alone.set_option("split_phases", 1)                             # no halo: one launch
    assert binding.mgg_aggregate_plan(alone, "gcn", 64).fine == 1
    many = binding.mgg_build_partition(ptr, col, 2, 0, wpb=16, **kw)
    for p in (alone, many):
        p.set_option("lds_halo", 1)
        assert binding.mgg_aggregate_plan(p, "gcn", 64).lds_halo == 0


@pytest.mark.parametrize("lens,short,dim,bf16,team", [
    ((150, 255, 64), 0, 128, False, 8), ((150, 255, 64), 10000, 128, False, 4), ((150, 255, 64), 100000, 128, False, 1),    # short rows keep the chip busy
    ((1500, 2500, 300), 2000, 128, False, 2), ((1500, 2500, 300), 100000, 128, False, 1),
    ((17, 31, 2000), 0, 256, True, 1), ((60, 75, 3000), 0, 64, False, 1),                                                # every item is short
    ((60, 120, 300), 0, 64, False, 2), ((60, 120, 5000), 0, 64, False, 1), ((400, 511, 900), 0, 64, False, 2)])
def test_teams_are_for_launches_that_wait_for_their_longest_item(lens, short, dim, bf16, team):
    """The rule counts all the loads of a launch, those of its short rows too, against the chain behind the longest item."""
    rng = np.random.default_rng(1)
    lo, hi, rows = lens
    ptr, col = _lists(np.concatenate([rng.integers(lo, hi + 1, rows), rng.integers(1, 14, short)]), 4000)
    part = binding.mgg_build_partition(ptr, col, host_only=True, xcd_min_deg=-1)
    assert binding.mgg_aggregate_plan(part, "gcn", dim, bf16=bf16).team == team


def test_chunked_slabs_by_table_and_ids():
    """256-byte slabs, chunk by chunk, where a class of them fits one L2 and the ids are more than 128 MB; not on rows off line
    boundaries, nor where the table is small and the ids stay in the Infinity Cache in any case."""
    nnz = 17 << 20
    for rows, gcn_slab in ((12000, 512), (16000, 256)):
        lens = np.full(rows, nnz // rows + 1)
        ptr, col = _lists(lens, rows)
        part = binding.mgg_build_partition(ptr, col, host_only=True)
        plan = lambda mode, dim, **kw: binding.mgg_aggregate_plan(part, mode, dim, **kw)
        gcn = plan("gcn", 256)
        assert (gcn.slab_bytes, gcn.n_slabs) == (gcn_slab, 1024 // gcn_slab) and (gcn.n_chunks > 1) == (gcn_slab == 256)
        assert gcn.n_chunks == (1 if gcn_slab == 512 else -(-int(ptr[-1]) * 8 // (36 << 20)))
        for other in (plan("gin", 256), plan("gcn", 256, ld=257), plan("gcn", 256, base_align=64), plan("gcn", 300)):      # half the ids; off lines
            assert (other.slab_bytes, other.n_chunks) == (512, 1)
        assert plan("gcn", 128).n_slabs == 1


@pytest.mark.parametrize("parts,part_id", [(1, 0), (3, 1)])
def test_large_partition_bit_exact_against_oracle(parts, part_id):
    """Counted, filled and laid out by several threads: hubs, empty rows, duplicates and self-loops."""
    import oracle
    rng = np.random.default_rng(5)
    n = 6000
    lens = rng.integers(0, 200, n)
    lens[rng.permutation(n)[:60]] = rng.integers(2000, 9000, 60)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = (rng.random(ptr[-1]) ** 2 * n).astype(np.int32)
    assert ptr[-1] >= 6 << 17
    bounds = np.linspace(0, n, parts + 1).astype(np.int64)
    want = oracle.build_partition(ptr, col, parts, part_id, bounds)
    got = binding.mgg_build_partition(ptr, col, parts, part_id, bounds, host_only=True).export()
    for key in ("local_row_ptr", "local_col", "remote_row_ptr", "remote_col", "halo_gid", "halo_peer_ptr", "deg_own", "deg_halo"):
        assert np.array_equal(got[key].astype(np.int64), want[key].astype(np.int64)), key
    for bad in ([123456], [900000 - 1, 7, 654321], [int(ptr[-1]) - 1]):         # the first one is named, whichever thread meets it
        wrong = col.copy()
        bad = [b % int(ptr[-1]) for b in bad]
        wrong[bad] = [n + i for i in range(len(bad))]
        with pytest.raises(binding.MggError, match=f"column {wrong[min(bad)]} at position {min(bad)} ") as err:
            binding.mgg_build_partition(ptr, wrong, parts, part_id, bounds, host_only=True)
        assert err.value.status == binding.ERR_BAD_GRAPH


@pytest.mark.parametrize("dims", [(100, 40), (64, 64), (40, 24, 24), (130, 7)])
@pytest.mark.parametrize("order", ["agg_first", "update_first", "auto"])
def test_the_least_workspace_is_the_coarse_schedules(dims, order):
    """A share with a fine schedule asks for a workspace that holds its partial sums; the least is what the same share
    without one asks for, and what one of the fine schedule adds is the partial sums it has more."""
    import torch
    ptr, col = _graph(1500, 330, 7, hubs=20)
    kw = dict(host_only=True, hot_phases=-1)
    fine = binding.mgg_build_partition(ptr, col, 2, 0, fine_min_neighbours=1, **kw)
    one = binding.mgg_build_partition(ptr, col, 2, 0, fine_min_neighbours=-1, **kw)
    layer = (["gcn"], [torch.zeros(a, b) for a, b in zip(dims, dims[1:])], ["none"] * (len(dims) - 1))
    ask = lambda f, p: f(p, layer[0][0], layer[1], layer[2], order=order)
    least = ask(binding.mgg_layer_workspace_least_bytes, fine)
    assert least == ask(binding.mgg_layer_workspace_bytes, one) == ask(binding.mgg_layer_workspace_least_bytes, one)
    more = ask(binding.mgg_layer_workspace_bytes, fine) - least
    extra = [int(fine.info.n_fine_split_items) * (-(-d // 8) * 8) * 4 if -(-d // 8) * 8 > 32 else 0 for d in dims[:2]]
    assert any(abs(more - x) < 256 for x in extra)


def test_groups_of_short_rows_per_wavefront():
    """Two where the launch keeps 8192 workgroups, rows of a graph take 16 lanes or more and their ids therefore come with the
    group before; one for fewer lanes, for bags and below that."""
    rng = np.random.default_rng(2)
    for rows, want in ((120000, 1), (140000, 2)):                              # 4 rows a wavefront, 2 wavefronts a workgroup
        ptr, col = _lists(rng.integers(1, 5, rows), rows)
        part = binding.mgg_build_partition(ptr, col, host_only=True)
        plan = lambda dim, **kw: binding.mgg_aggregate_plan(part, "gcn", dim, **kw).short_per_wave
        assert (plan(64), plan(128), plan(16), plan(32), plan(128, bf16=True)) == (want, 2, 1, 1, want)
        bags = binding.mgg_build_bags(ptr, col, rows, 0, rows, host_only=True)
        assert binding.mgg_aggregate_plan(bags, "gin", 128).short_per_wave == 1
        part.set_option("short_per_wave", 5)
        assert plan(16) == 5
