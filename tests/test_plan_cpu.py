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
