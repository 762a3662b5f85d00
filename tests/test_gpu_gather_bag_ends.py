"""Where bags end inside the steps of the gather walkers: lengths around one instruction (64 / G
lookups of G-lane rows), around the groups of four instructions that a short step skips, and
around a whole step; runs of empty bags; the most bags a chunk takes; rows and weights that
are infinite or NaN, which belong to their own bag only; and a narrow table past 4 GiB.  Wide
rows (gather_kernel) and narrow ones (lookup_kernel, mostly by sub-wavefronts; in matrix slots:
test_gpu_slots.py).
Integer tables, bit-exact against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import pool as OP

from gpu_helpers import host_tables, log, to_device, upload_tables

pytestmark = pytest.mark.gpu

WIDE = [(64, "f32"), (96, "f32"), (256, "f32"), (128, "f16"), (192, "f16"), (200, "f32")]
NARROW = [(4, "f32"), (8, "f32"), (16, "f32"), (24, "f32"), (32, "f32"), (8, "f16"), (16, "f16"), (24, "f16"),
          (32, "f16"), (64, "f16")]
SHAPES = WIDE + NARROW


def length_patterns(g):
    """Bag lengths of one table: every remainder around the kernel's units."""
    yield np.arange(0, 70)                                            # every length up to a step and past it
    yield np.array([16, 15, 17, 32, 31, 33, 48, 47, 49, 64, 63, 65, 128, 127, 129, 1, 0, 0, 0, 1] * 3)
    yield (g.random(200) < 0.2).astype(np.int64)                      # mostly empty, several ends per instruction
    yield np.concatenate([np.zeros(70, np.int64), [900], np.zeros(70, np.int64), [1]])
    yield g.integers(0, 4, size=333)


def plan_and_batch(E, dtype, seed, rows, stated_pooling):
    import paper_2507_01676_amd as embx
    g = np.random.default_rng(seed)
    lens = list(length_patterns(g))
    B = max(len(x) for x in lens)
    lens = [np.concatenate([x, np.zeros(B - len(x), np.int64)]) for x in lens]
    T = len(lens)
    c = W.Config(170, "bag ends", E, dtype, -1.0, 1.0, B, [W.TableSpec(m, "fixed", 1, 1, 1, "uniform") for m in rows])
    c.value_seeds = [W.value_seed(170, t) for t in range(T)]
    off = np.zeros(T * B + 1, np.int64)
    np.cumsum(np.concatenate(lens), out=off[1:])
    idx = np.concatenate([g.integers(0, m, size=int(x.sum())) for m, x in zip(rows, lens)])
    stats = [{"mean_pooling": stated_pooling or max(0.1, float(x.mean())), "max_pooling": 0} for x in lens]
    plan = embx.Plan(rows, E, dtype, stats, B)
    assert plan.info()["kernel"] == ("gather_kernel" if (E, dtype) in WIDE else "lookup_kernel")
    return c, plan, W.Batch(B, T, idx, off), g


@pytest.mark.parametrize("stated_pooling", [0.0, 1.0, 40.0])   # (chunks of a few bags up to the most)
@pytest.mark.parametrize("E,dtype", SHAPES)
def test_every_bag_end_is_found(E, dtype, stated_pooling):
    import torch
    log(f"bag ends, E{E} {dtype}, stated pooling {stated_pooling}")
    rows = [7, 50_000, 300, 9, 2_000]
    c, plan, batch, g = plan_and_batch(E, dtype, 5, rows, stated_pooling)
    batch.indices[g.random(batch.indices.size) < 0.02] = -1           # out of range: adds nothing, is counted
    hw = host_tables(c, W.VAL_INTEGER)
    plan.bind(upload_tables(hw))
    idx, off = to_device(batch)
    psw = g.integers(-3, 4, size=batch.indices.size).astype(np.float32)
    for w in (None, psw):
        out = torch.full((batch.B, batch.T, E), float("nan"), device="cuda")
        plan.lookup(idx, off, batch.B, out, weights=None if w is None else torch.from_numpy(w).cuda())
        torch.cuda.synchronize()
        ref, _, bad = OP.pool_reference(hw, batch.indices, batch.offsets, batch.B, psw=w)
        assert np.array_equal(out.cpu().numpy(), ref)
        assert plan.check_errors() == bad


@pytest.mark.parametrize("E,dtype", SHAPES)
def test_infinities_and_nans_stay_in_their_bag(E, dtype):
    import torch
    log(f"non-finite rows and weights, E{E} {dtype}")
    rows = [40, 50, 60, 70, 80]
    c, plan, batch, g = plan_and_batch(E, dtype, 6, rows, 0.0)
    hw = host_tables(c, W.VAL_INTEGER)
    for t, w in enumerate(hw):
        w[3, :] = np.inf
        w[5, ::2] = np.nan
        w[8, 1::2] = -np.inf
    plan.bind(upload_tables(hw))
    idx, off = to_device(batch)
    psw = g.integers(1, 4, size=batch.indices.size).astype(np.float32)
    psw[g.random(psw.size) < 0.02] = np.inf
    psw[g.random(psw.size) < 0.02] = np.nan
    with np.errstate(invalid="ignore"):
        for w in (None, psw):
            out = torch.full((batch.B, batch.T, E), 7.5, device="cuda")
            plan.lookup(idx, off, batch.B, out, weights=None if w is None else torch.from_numpy(w).cuda())
            torch.cuda.synchronize()
            ref, _, _ = OP.pool_reference(hw, batch.indices, batch.offsets, batch.B, psw=w)
            assert np.array_equal(out.cpu().numpy(), ref, equal_nan=True)


def test_narrow_rows_of_a_table_beyond_4_gib():
    import torch

    import paper_2507_01676_amd as embx
    E, rows, B = 16, 70_000_000, 600
    log(f"one table of {rows * E * 4 / 2**30:.2f} GiB, rows of {E * 4} bytes")
    w = torch.empty((rows, E), device="cuda")
    embx.fill_table(w, 0, 99, mode=W.VAL_INTEGER)
    g = np.random.default_rng(3)
    lens = g.integers(0, 9, size=B)
    off = np.zeros(B + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    idx = g.integers(0, rows, size=int(off[-1]))
    idx[::7] = rows - 1 - idx[::7] % 1000
    idx[5::50] = rows
    plan = embx.Plan([rows], E, "f32", [{"mean_pooling": 4.0, "max_pooling": 8}], B).bind([w])
    d_idx, d_off = to_device(W.Batch(B, 1, idx, off))
    got = plan.lookup(d_idx, d_off, B).cpu().numpy()
    ok = idx < rows
    vals = np.zeros((idx.size, E), np.float32)
    vals[ok] = W.table_rows_at(0, idx[ok], E, "f32", seed=99, mode=W.VAL_INTEGER)
    ref, _, _ = OP.pool_reference([vals], np.arange(idx.size, dtype=np.int64), off, B)
    assert np.array_equal(got, ref)
    assert plan.check_errors() == int((~ok).sum())


@pytest.mark.parametrize("pooling", ["sum", "mean"])
@pytest.mark.parametrize("E,dtype", [(64, "f32"), (96, "f32"), (256, "f32"), (128, "f16"), (256, "f16")])
def test_chunks_longer_than_the_rebase_distance(monkeypatch, E, dtype, pooling):
    """Positions inside a chunk are 32 bits wide and rebased every 2^30 lookups; in the test
    build every 96 (100 rounded down to whole steps): bags that end on, beside, a few lookups
    past and far past such a point."""
    import importlib.util

    import torch

    import paper_2507_01676_amd as embx
    log(f"rebased positions, E{E} {dtype} {pooling}")
    monkeypatch.setenv("EMBX_LIBRARY", embx.LIB_PATH.replace("libembx.so", "libembx_far.so"))
    monkeypatch.setenv("EMBX_GATHER_STEPS", "12")
    spec = importlib.util.spec_from_file_location("embx_far", embx.__file__)
    far = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(far)
    g = np.random.default_rng(11)
    lens = [np.concatenate([[95, 1, 1, 96, 97, 0, 0, 94, 0, 2, 98, 3, 5, 350, 0, 1000, 5], np.zeros(13, np.int64)]),
            g.integers(0, 70, size=30), np.full(30, 96), np.full(30, 25), np.full(30, 1)]
    rows = [7, 5_000, 300, 9, 2_000]
    B, T = 30, len(rows)
    c = W.Config(171, "rebase", E, dtype, -1.0, 1.0, B, [W.TableSpec(m, "fixed", 1, 1, 1, "uniform") for m in rows])
    c.value_seeds = [W.value_seed(171, t) for t in range(T)]
    off = np.zeros(T * B + 1, np.int64)
    np.cumsum(np.concatenate(lens), out=off[1:])
    idx = np.concatenate([g.integers(0, m, size=int(x.sum())) for m, x in zip(rows, lens)])
    idx[g.random(idx.size) < 0.02] = -1
    # one worker and a stated pooling of 1: chunks of several bags, far more lookups than stated
    stats = [{"mean_pooling": 1.0, "max_pooling": 0}] * T
    hw = host_tables(c, W.VAL_INTEGER)
    plan = far.Plan(rows, E, dtype, stats, B, num_workers=1, pooling=pooling).bind(upload_tables(hw))
    info = plan.info()
    assert info["kernel"] == "gather_kernel" and info["gather_steps"] == 12
    d_idx, d_off = to_device(W.Batch(B, T, idx, off))
    for w in (None, g.integers(-3, 4, size=idx.size).astype(np.float32)):
        out = torch.full((B, T, E), float("nan"), device="cuda")
        plan.lookup(d_idx, d_off, B, out, weights=None if w is None else torch.from_numpy(w).cuda())
        torch.cuda.synchronize()
        ref, mag, bad = OP.pool_reference(hw, idx, off, B, psw=w, pooling=pooling)
        if pooling == "sum":
            assert np.array_equal(out.cpu().numpy(), ref)
        else:   # a division by the length as a multiplication: two roundings of half an ulp
            assert OP.pooled_error(out.cpu().numpy(), ref, mag) <= 2.0 ** -22
        assert plan.check_errors() == bad


@pytest.mark.parametrize("pooling", ["sum", "mean"])
@pytest.mark.parametrize("E,dtype", [(4, "f32"), (8, "f16"), (8, "f32"), (16, "f16")])
def test_long_bags_of_the_narrowest_rows(E, dtype, pooling):
    """A wavefront per bag: 64 one-lane sub-wavefronts on 16-byte rows, 32 of two lanes on
    32-byte ones; lengths around a round of them, a step of 8 rounds, and several steps."""
    import torch

    import paper_2507_01676_amd as embx
    log(f"long bags, E{E} {dtype} {pooling}")
    g = np.random.default_rng(13)
    lens = np.array([511, 512, 513, 1, 0, 1024, 5000, 63, 64, 65, 31, 32, 33, 255, 256, 257, 0, 2049, 7, 1025])
    rows, B = [7, 50_000, 900], lens.size
    c = W.Config(172, "long bags", E, dtype, -1.0, 1.0, B, [W.TableSpec(m, "fixed", 1, 1, 1, "uniform") for m in rows])
    c.value_seeds = [W.value_seed(172, t) for t in range(len(rows))]
    off = np.zeros(len(rows) * B + 1, np.int64)
    np.cumsum(np.concatenate([g.permutation(lens) for _ in rows]), out=off[1:])
    n = off[::B]
    idx = np.concatenate([g.integers(0, m, size=int(n[t + 1] - n[t])) for t, m in enumerate(rows)])
    idx[g.random(idx.size) < 0.02] = -1
    hw = host_tables(c, W.VAL_INTEGER)
    plan = embx.Plan(rows, E, dtype, [{"mean_pooling": float(lens.mean()), "max_pooling": 0}] * 3, B, pooling=pooling,
                     num_workers=3).bind(upload_tables(hw))
    assert {ln.split()[1] for ln in plan.queues().splitlines()[1:]} == {"wave"}
    d_idx, d_off = to_device(W.Batch(B, len(rows), idx, off))
    for w in (None, g.integers(-3, 4, size=idx.size).astype(np.float32)):
        out = torch.full((B, len(rows), E), float("nan"), device="cuda")
        plan.lookup(d_idx, d_off, B, out, weights=None if w is None else torch.from_numpy(w).cuda())
        torch.cuda.synchronize()
        # sums of up to 5000 integers: exact below 2^24, which 64 partial sums stay under and the totals may not
        ref, mag, bad = OP.pool_reference(hw, idx, off, B, psw=w, pooling=pooling)
        assert OP.pooled_error(out.cpu().numpy(), ref, mag) <= 2.0 ** -20
        assert plan.check_errors() == bad
