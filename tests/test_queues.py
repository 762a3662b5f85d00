"""Which walker and which queues a plan's gather slices get (emb_debug_queue_text, host only)."""
import pytest

import paper_2507_01676_amd as embx


def queues(rows, E, dtype, stats, B, workers=256, **opts):
    """(head of the text as a dict, runs as tuples)"""
    lines = embx.queue_text(rows, E, dtype, stats, B, workers, **opts).splitlines()
    f = lines[0].split()
    return dict(zip(f[::2], f[1::2])), [tuple(x if i == 1 else int(x) for i, x in enumerate(ln.split())) for ln in lines[1:]]


def tables(n, mean, most=0):
    return [1000 + 40 * t for t in range(n)], [{"mean_pooling": mean, "max_pooling": most}] * n


@pytest.mark.parametrize("batch", [64, 1000, 4096, 30000])
@pytest.mark.parametrize("bag", [2.0, 3.0, 4.0, 8.0, 12.0, 30.0])
@pytest.mark.parametrize("E", [8, 16, 24, 32, 64])
def test_half_precision_rows_take_slots_with_weights_on_two_lanes_only(E, bag, batch):
    rows, stats = tables(26, bag)
    head, runs = queues(rows, E, "f16", stats, batch)
    assert head["kernel"] == "lookup_kernel" and head["walker"] == "sw"
    multi = [r for r in runs if r[1] == "multi"]
    if E >= 24:
        assert head["weighted"] == "sw"
    if E <= 16 and batch == 30000:
        assert head["weighted"] == "slots"
    assert all((r[6] > 0) == (head["weighted"] == "slots") for r in multi)
    if head["weighted"] == "slots":   # the sub-wavefronts keep chunks of their own size
        assert {r[6] for r in multi} <= {32, 64} and max(r[5] for r in multi) <= 64


@pytest.mark.parametrize("E,lanes", [(4, 2), (8, 2), (16, 4), (32, 8)])
def test_single_precision_rows_take_slots_where_the_slices_hold_bags(E, lanes):
    rows, stats = tables(26, 8.0)
    head, _ = queues(rows, E, "f32", stats, 8192)   # 32 bags per slice: half of 32 SWs and more
    assert head["lanes"] == str(lanes) and head["walker"] == "slots"
    rows, stats = tables(26, 30.0)
    head, _ = queues(rows, E, "f32", stats, 800)    # 3 bags per slice
    assert head["walker"] == "sw"


def test_wave_mode_slices_do_not_decide_for_the_others():
    # every bag is long: nothing is left for slots
    rows, stats = tables(5, 40.0)
    head, runs = queues(rows, 32, "f32", stats, 1100)
    assert {r[1] for r in runs} == {"wave"} and head["walker"] == "sw"
    # a table of long bags in slices of two holds most lookups; the others' slices hold enough bags
    rows, stats = tables(26, 2.0)
    stats = [{"mean_pooling": 100.0, "max_pooling": 0}] + stats[1:]
    head, runs = queues(rows, 32, "f32", stats, 512)
    assert {(r[1], r[2] == 0) for r in runs} == {("wave", True), ("multi", False)} and head["walker"] == "slots"
    # ... and size their chunks by their own lookups alone: 342 bags of 4 on a worker, 2.7 bags per
    # sub-wavefront of 16 wavefronts
    rows, stats = tables(24, 4.0)
    stats = [{"mean_pooling": 100.0, "max_pooling": 0}] * 4 + stats[4:]
    _, runs = queues(rows, 32, "f32", stats, 1024)
    assert {(r[4], r[5]) for r in runs if r[1] == "multi"} == {(3, 2 * 8)}


@pytest.mark.parametrize("E,sws,most", [(8, 32, 2), (16, 16, 4), (32, 8, 4)])
@pytest.mark.parametrize("bag", [0.2, 1.0, 2.0, 3.0, 4.0, 5.0, 8.0, 9.0, 40.0])
def test_a_slots_chunk_fills_a_step(E, sws, most, bag):
    """However short the queue: a step holds 8 lookups per sub-wavefront."""
    rows, stats = tables(26, bag)
    for batch in (sws, 300, 2500, 20000):
        head, runs = queues(rows, E, "f32", stats, batch, workers=32)
        if head["walker"] == "slots":
            bags = {r[5] for r in runs if r[1] == "multi"}
            least = max(1, min(most, int(8 // max(1.0, bag))))
            assert bags <= {sws * m for m in range(least, most + 1)}, (batch, bags)


@pytest.mark.parametrize("E,dtype,bytes_", [(4, "f32", 16), (8, "f16", 16), (8, "f32", 32), (16, "f16", 32)])
def test_long_bags_of_16_byte_rows_take_one_lane(E, dtype, bytes_):
    for bag in (150.0, 255.0, 256.0, 5000.0):
        rows, stats = tables(4, bag)
        head, runs = queues(rows, E, dtype, stats, 8)
        assert {r[1] for r in runs} == {"wave"} and head["lanes"] == "2"
        assert head["wave_lanes"] == ("1" if bytes_ == 16 and bag >= 256 else "2")
    rows, stats = tables(26, 8.0)
    assert queues(rows, E, dtype, stats, 8192)[0]["wave_lanes"] == "2"
