"""The plan of a plain launch (which kernel, shape and segments a call takes), on the CPU."""
import pytest

from tests import plan


# The segments cover the iterations exactly, each with rows of its own, also where their number
# of rows added to the iterations passes 2^32.
@pytest.mark.parametrize("u32", [False, True])
@pytest.mark.parametrize("n", [1, 7, 16, 128, 1024, 4096, 4099, 65536, 100003, 262147])
def test_segments_cover_the_iterations(n, u32):
    counts = {1, 2, 23, 24, 63, 64, 65, 100, 257, 10000, 2**31, 2**32 - 2**24, 2**32 - 2**24 + 1,
              2**32 - 10**6, 2**32 - 2, 2**32 - 1}
    for iters in sorted(counts):
        for out in (0, 8):
            p = plan.query(n, iters, u32=u32, out=out)
            assert p["segs"] >= 1 and p["seg_rows"] >= 1, (iters, p)
            assert (p["segs"] - 1) * p["seg_rows"] < iters <= p["segs"] * p["seg_rows"], (iters, p)


# Served batches: one wave per item up to 192 MiB, above that the grouped order (the sweep order
# of the batch API holds a compute unit for itself, which costs batches that run side by side).
@pytest.mark.parametrize("values,per_item,group", [
    (16, 1, 0), (1 << 23, 1, 0), ((1 << 23) + 16, 1, 0), (3 << 23, 1, 0), ((3 << 23) + 16, 0, 32),
    (1 << 26, 0, 32), ((1 << 26) + 16, 0, 32), (2 * 10**9, 0, 32)])
def test_served_order(values, per_item, group):
    c = plan.served(values)
    assert (c["per_item"], c["group"]) == (per_item, group)
    assert c["values_per_lane"] == 16 and c["waves_per_block"] == 4


# The batch API's own order: items up to 2^26 values (half lines up to 2^25); above, the sweep
# order or, without memory for its anchors, groups, launched without a graph all the same.
UPLOAD, SWEEP = 2, 1


@pytest.mark.parametrize("anchors", [False, True])
def test_batch_order(anchors):
    for values, rows in [(1, 8), (1 << 25, 8), ((1 << 25) + 1, 16), (1 << 26, 16)]:
        c = plan.batch(values, anchors)
        assert (c["per_item"], c["row_values"], c["group"], c["use_graph"]) == (1, rows, 0, UPLOAD)
    c = plan.batch((1 << 26) + 1, anchors)
    assert (c["per_item"], c["use_graph"]) == (0, UPLOAD)
    assert (c["group"], c["values_per_lane"], c["pace_gbs"]) == \
        ((SWEEP, 8, 7000) if anchors else (32, 16, 6250))


def test_anchors_of_growing_batches_are_seldom_allocated():
    # Batches of 512 MiB up to 256 GiB, each a little larger than the one before.
    have = allocated = 0
    values = (1 << 26) + 1
    while values <= 1 << 35:
        need = -(-values // 8192)
        if need > have:
            allocated += 1
            have = plan.anchor_room(need)
            assert need <= have <= max(2 * need, 1 << 17)
        values += values // 100
    assert allocated <= 6


# With the states in place (after a capture, or without memory for a second buffer) a call stays
# in one segment and unstaged, and keeps to its row schedule wherever its rows are 16-byte aligned.
@pytest.mark.parametrize("u32,n,iters,out", [
    (False, 4096, 100, 0), (False, 4096, 10000, 0), (False, 4098, 10000, 0), (False, 65536, 1000, 0),
    (False, 262146, 500, 0), (False, (1 << 20) + 2, 256, 0), (False, 1 << 20, 256, 16),
    (True, 4096, 10000, 0), (True, 4100, 10000, 16), (True, (1 << 20) + 4, 256, 0),
    (True, 65536, 2000, 0), (False, 4099, 10000, 0), (False, (1 << 20) + 3, 256, 0),
    (True, (1 << 20) + 4, 256, 4)])
def test_in_place_plans(u32, n, iters, out):
    away = plan.query(n, iters, u32=u32, out=out)
    p = plan.query(n, iters, u32=u32, out=out, in_place=True)
    assert away["segs"] > 1 or away["shift"]
    assert (p["segs"], p["seg_rows"], p["shift"]) == (1, iters, 0)
    size = 4 if u32 else 8
    assert p["scheduled"] == int(n * size % 16 == 0 and out % 16 == 0)


# A plan that is in place anyway is the same with and without that condition.
@pytest.mark.parametrize("u32", [False, True])
@pytest.mark.parametrize("star", [False, True])
def test_in_place_changes_no_other_plan(u32, star):
    same = 0
    for n in (100, 4096, 4099, 65536, 114688, 262144, 262147, 1 << 20, (1 << 20) + 2, 1 << 24):
        for iters in (1, 2, 5, 13, 63, 64, 400, 5000):
            for out in (0, 16, 8):
                a = plan.query(n, iters, u32=u32, star=star, out=out)
                if a["segs"] == 1 and not a["shift"]:
                    assert a == plan.query(n, iters, u32=u32, star=star, out=out, in_place=True)
                    same += 1
    assert same > 100


# Staged rows: the words after a row's last whole chunk are read inside the wavefront's stage, for
# every number of columns left and every offset of the row in its line.
@pytest.mark.parametrize("chunk,line,columns", [(2, 16, 128), (2, 16, 256), (4, 32, 256),
                                                (4, 32, 512)])
def test_staged_row_ends_stay_inside_the_stage(chunk, line, columns):
    assert plan.stage_tail_faults(chunk, line, columns) == 0


# Many segments run at most at a rate that they hold; a lower rate that the caller has set stays.
@pytest.mark.parametrize("u32,n,iters,most", [
    (False, 4099, 10000, 6000), (False, 16387, 10000, 6500), (False, 131073, 2000, 7500),
    (True, 65537, 1000, 6000), (True, 131073, 2000, 6500), (True, 25600, 6553, 6750),
    (False, 4096, 10000, 7500), (False, 1 << 22, 256, 7500)])
def test_rates_of_segments(u32, n, iters, most):
    for pace in (1000, 5000, 6000, 7000, 7500, 20000):
        p = plan.query(n, iters, u32=u32, launch=(512, 2, 1, pace))
        assert p["scheduled"]
        assert p["pace_gbs"] == (min(pace, most) if most < 7500 else pace)


@pytest.mark.parametrize("m", [1, 49, 4096, 2**28, 2**30 - 3, 2**30 - 2, 2**30, 2**32 - 1])
def test_batch_tables_are_uploaded_whole(m):
    # 128 bytes before the records, 64 bytes each.
    assert plan.table_chunks(m) * 16 == 128 + 64 * m


# The headline shape runs as configured: scheduled, in place, one segment of unstaged rows. (The
# committed counters are of that launch.)
def test_headline_plan():
    for launch in [(512, 2, 1, 7000), (512, 2, 1, 7500), (256, 4, 1, 7500), (256, 1, 1, 7000)]:
        p = plan.query(1 << 26, 256, launch=launch)
        assert (p["block"], p["chunks"], p["nontemporal"], p["pace_gbs"]) == launch
        assert p["scheduled"] and not p["shift"] and (p["segs"], p["seg_rows"]) == (1, 256)


# Without a schedule, rows run where they lie and as configured, but for wide rows of outputs well
# beyond the cache, which are staged.
@pytest.mark.parametrize("launch", [(256, 1, 1, 0), (128, 2, 0, 0), (1024, 4, 0, 0)])
def test_unscheduled_plans(launch):
    for u32, n, iters in [(False, 39239, 1207), (False, 75649, 3269), (True, 9215, 16422),
                          (True, 167153, 837), (False, 448631, 97), (False, 2648055, 13),
                          (False, 4099, 10000), (False, 4096, 10000)]:
        p = plan.query(n, iters, u32=u32, launch=launch)
        assert not p["scheduled"] and not p["shift"] and p["segs"] == 1, (n, iters)
        assert (p["block"], p["chunks"], p["nontemporal"], p["pace_gbs"]) == launch
    assert plan.query(1000003, 256, launch=launch)["shift"]


# Rows of 1,280 wavefronts and more in one segment keep to their schedule above 64 MiB; shorter
# ones, and segments, run free while the cache holds their output.
@pytest.mark.parametrize("u32,n,iters,free", [
    (False, 65536, 300, True), (False, 131072, 180, True), (False, 4096, 1000, True),
    (False, 179200, 40, True), (False, 179200, 60, False), (False, 332800, 71, False),
    (True, 486400, 97, False), (False, 332800, 20, True), (False, 131072, 250, False)])
def test_free_running_rows(u32, n, iters, free):
    p = plan.query(n, iters, u32=u32)
    assert p["scheduled"] and p["chunks"] == 1 and (p["pace_gbs"] == 0) == free


# Rows off the lines that the cache puts together, 16-byte aligned: narrow rows in one chunk, with
# normal stores (a launch of one chunk too), others as configured.
@pytest.mark.parametrize("u32,star,n,iters,narrow", [
    (False, False, 128002, 190, True), (False, False, 179202, 118, True),
    (False, False, 332802, 71, True), (False, True, 332802, 71, True),
    (True, False, 486404, 97, True), (True, True, 800004, 60, True),
    (False, False, 600002, 40, False), (True, True, 1200004, 40, False)])
def test_rows_off_the_lines_in_the_cache(u32, star, n, iters, narrow):
    p = plan.query(n, iters, u32=u32, star=star)
    assert p["scheduled"] and not p["shift"] and p["segs"] == 1
    assert (p["block"], p["chunks"], p["nontemporal"]) == ((256, 1, 0) if narrow else (512, 2, 1))
    p = plan.query(n, iters, u32=u32, star=star, launch=(1024, 1, 1, 7500))
    assert p["scheduled"] and (p["chunks"], p["nontemporal"]) == (1, 0)
    # On the lines, or staged, the stores are as configured.
    assert plan.query(n & ~31, iters, u32=u32, star=star)["nontemporal"]
    assert plan.query(n, 4 * iters, u32=u32, star=star)["nontemporal"]


# Rows that are not 16-byte aligned stay where they lie somewhat beyond the cache's size, as far as
# that is faster; aligned ones do not.
@pytest.mark.parametrize("u32,star,n,iters,staged", [
    (False, False, 179201, 216, False), (False, True, 332801, 116, False),
    (False, False, 179201, 418, True), (False, False, 537601, 72, True),
    (False, False, 7040001, 6, False), (False, False, 7040001, 9, True),
    (False, False, 102401, 400, True), (True, False, 2304001, 33, False),
    (True, True, 2304001, 46, True), (True, False, 19200001, 5, False),
    (True, False, 300001, 250, True), (False, False, 332802, 116, True),
    (True, False, 2304004, 33, True)])
def test_where_staging_begins(u32, star, n, iters, staged):
    p = plan.query(n, iters, u32=u32, star=star)
    assert bool(p["shift"]) == staged
    if not staged:
        assert p["segs"] == 1 and not p["scheduled"] and (p["block"], p["chunks"]) == (512, 2)


# Short rows: segments from 64 iterations on, off the lines from where their jumps pay.
@pytest.mark.parametrize("u32,star,n,least", [
    (False, False, 4096, 64), (True, True, 4096, 64), (False, False, 1001, 48),
    (False, True, 1001, 32), (True, False, 1001, 28), (True, True, 1001, 24),
    (False, False, 4098, 48)])
def test_where_segments_begin(u32, star, n, least):
    assert plan.query(n, least - 1, u32=u32, star=star)["segs"] == 1
    p = plan.query(n, least, u32=u32, star=star)
    assert p["segs"] > 1 and p["seg_rows"] >= 8


# Rows on 64-byte halves of lines run as rows on the lines do.
@pytest.mark.parametrize("u32,star,n,iters", [
    (False, False, 4096, 1000), (False, False, 131072, 500), (False, True, 179200, 250),
    (True, True, 1075200, 200), (False, False, 1 << 20, 256), (True, False, 19200000, 10)])
def test_half_lines(u32, star, n, iters):
    p = plan.query(n + (16 if u32 else 8), iters, u32=u32, star=star)
    q = plan.query(n, iters, u32=u32, star=star, out=64)
    assert q == plan.query(n, iters, u32=u32, star=star)
    assert p["scheduled"] and not p["shift"]
    assert all(p[k] == q[k] for k in ("block", "chunks", "pace_gbs"))


# Few iterations of so many states that the cache holds one copy of them and not two stay in place.
@pytest.mark.parametrize("u32,n,most", [
    (False, 32000002, 12), (False, 25600001, 4), (True, 28160004, 12), (False, 40000001, 2),
    (False, 40000002, 1), (True, 51200004, 1)])
def test_few_iterations_of_many_states(u32, n, most):
    for iters in (most, most + 1):
        p = plan.query(n, iters, u32=u32)
        assert bool(p["shift"]) == (iters > most), iters
        assert p["shift"] or p["segs"] == 1
