"""Narrow rows summed in matrix slots by whole wavefronts (lookup_kernel's Slots): every plan
here is asked which walker it got.  Few workers, so that a slice holds bags for the
sub-wavefronts of a chunk; fp32 rows of 2, 4 and 8 lanes, full and with idle lanes, and fp16
rows of 2, whose weighted lookups of at least half the plan's batch go there."""
import numpy as np
import pytest

import workloads as W
from oracle import pool as OP

from gpu_helpers import host_tables, log, to_device, upload_tables
from test_gpu_gather_bag_ends import length_patterns

pytestmark = pytest.mark.gpu

SHAPES = [(4, "f32"), (8, "f32"), (12, "f32"), (16, "f32"), (24, "f32"), (32, "f32"), (8, "f16"), (16, "f16")]


def slots_plan(rows, E, dtype, stats, B, weights, **opts):
    import paper_2507_01676_amd as embx
    plan = embx.Plan(rows, E, dtype, stats, B, num_workers=2, **opts).bind(weights)
    f = plan.queues().splitlines()[0].split()
    head = dict(zip(f[::2], f[1::2]))
    assert head["kernel"] == "lookup_kernel" and head["weighted"] == "slots", head
    assert head["walker"] == ("slots" if dtype == "f32" else "sw"), head
    return plan


def patterns_batch(seed, rows, B):
    g = np.random.default_rng(seed)
    lens = [np.resize(x, B) for x in length_patterns(g)]
    off = np.zeros(len(rows) * B + 1, np.int64)
    np.cumsum(np.concatenate(lens), out=off[1:])
    idx = np.concatenate([g.integers(0, m, size=int(x.sum())) for m, x in zip(rows, lens)])
    stats = [{"mean_pooling": max(0.1, float(x.mean())), "max_pooling": 0} for x in lens]
    return idx, off, stats, g


def config(E, dtype, rows, B):
    c = W.Config(180, "slots", E, dtype, -1.0, 1.0, B, [W.TableSpec(m, "fixed", 1, 1, 1, "uniform") for m in rows])
    c.value_seeds = [W.value_seed(180, t) for t in range(len(rows))]
    return c


def look_up(plan, idx, off, B, E, w):
    import torch
    d_idx, d_off = to_device(W.Batch(B, plan.T, idx, off))
    out = torch.full((B, plan.T, E), float("nan"), device="cuda")
    plan.lookup(d_idx, d_off, B, out, weights=None if w is None else torch.from_numpy(w).cuda())
    torch.cuda.synchronize()
    return out.cpu().numpy()


ROWS = [7, 50_000, 300, 9, 2_000]


@pytest.mark.parametrize("pooling", ["sum", "mean"])
@pytest.mark.parametrize("E,dtype", SHAPES)
def test_bag_ends(E, dtype, pooling):
    log(f"slots: bag ends, E{E} {dtype} {pooling}")
    B = 1500   # (chunks of one to all slots)
    hw = host_tables(config(E, dtype, ROWS, B), W.VAL_INTEGER)
    idx, off, stats, g = patterns_batch(5, ROWS, B)
    plan = slots_plan(ROWS, E, dtype, stats, B, upload_tables(hw), pooling=pooling)
    for run in (B, B // 2, 333, 97, 1):   # (a runtime batch below the plan's)
        idx, off, _, g = patterns_batch(run, ROWS, run)
        idx[g.random(idx.size) < 0.02] = -1   # adds nothing, is counted
        for w in (None, g.integers(-3, 4, size=idx.size).astype(np.float32)):
            got = look_up(plan, idx, off, run, E, w)
            ref, mag, bad = OP.pool_reference(hw, idx, off, run, pooling=pooling, psw=w)
            if pooling == "sum":
                assert np.array_equal(got, ref)
            else:   # exact sums times a rounded reciprocal, against a rounded quotient: three half ulps
                assert OP.pooled_error(got, ref, mag) <= 2.0 ** -22
            assert plan.check_errors() == bad


def fma_in_order(rows, idx, off, psw):
    """x * w + acc per lookup in order, rounded once to fp32 (products of two fp32 are exact in
    80-bit floats; their sum's first rounding is 2^-40 of the second's)."""
    n = np.diff(off)
    acc = np.zeros((n.size, rows.shape[1]), np.float32)
    for k in range(int(n.max())):
        on = np.nonzero(n > k)[0]
        x = rows[idx[off[on] + k]].astype(np.longdouble)
        if psw is not None:
            x = x * psw[off[on] + k].astype(np.longdouble)[:, None]
        acc[on] = (x + acc[on].astype(np.longdouble)).astype(np.float32)
    return acc


@pytest.mark.parametrize("values", ["uniform", "wide", "subnormal"])
@pytest.mark.parametrize("E,dtype", SHAPES)
def test_each_sum_is_a_chain_of_fmas(E, dtype, values):
    """Bit for bit, at ordinary values, over 60 binary orders and below the normal numbers."""
    import torch
    log(f"slots: fma chains, E{E} {dtype} {values}")
    g = np.random.default_rng(E)
    m, B = 200, 300
    half = dtype == "f16"
    w = g.uniform(-1, 1, (m, E)).astype(np.float32)
    if values == "wide":
        w = np.ldexp(w, g.integers(-8, 8, (m, E)) if half else g.integers(-30, 30, (m, E))).astype(np.float32)
    if values == "subnormal":
        w = np.ldexp(w, g.integers(-24, -10, (m, E)) if half else g.integers(-148, -120, (m, E))).astype(np.float32)
    if half:
        w = w.astype(np.float16)
    lens = g.integers(0, 12, size=B)
    off = np.zeros(B + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    idx = g.integers(0, m, size=int(off[-1]))
    plan = slots_plan([m], E, dtype, [{"mean_pooling": 5.5, "max_pooling": 11}], B, [torch.from_numpy(w).cuda()])
    psw = g.uniform(0.5, 2, idx.size).astype(np.float32)
    if values == "subnormal":
        psw[::3] = np.ldexp(psw[::3], -20)
        if half:
            psw = np.ldexp(psw, -118)
    for p in (None, psw):
        got = look_up(plan, idx, off, B, E, p)[:, 0]
        ref = fma_in_order(w, idx, off, p)
        if p is not None or not half:   # (sums of halves alone are normal numbers)
            assert np.any((ref != 0) & (np.abs(ref) < 1.1e-38)) == (values == "subnormal")
        assert np.array_equal(got, ref), np.argwhere(got != ref)[:5]


@pytest.mark.parametrize("pooling", ["sum", "mean"])
@pytest.mark.parametrize("E,dtype", SHAPES)
def test_infinities_and_nans_stay_in_their_bag(E, dtype, pooling):
    log(f"slots: non-finite rows, weights and sums, E{E} {dtype} {pooling}")
    B, rows = 1500, [40, 50, 60, 70, 80]
    hw = host_tables(config(E, dtype, rows, B), W.VAL_INTEGER)
    for w in hw:
        w[3, :] = np.inf
        w[5, ::2] = np.nan
        w[8, 1::2] = -np.inf
    idx, off, stats, g = patterns_batch(6, rows, B)
    idx[g.random(idx.size) < 0.7] = 0   # (some chunks are finite, some not)
    idx[g.random(idx.size) < 0.02] = -1
    plan = slots_plan(rows, E, dtype, stats, B, upload_tables(hw), pooling=pooling)
    psw = g.integers(1, 4, size=idx.size).astype(np.float32)
    psw[g.random(psw.size) < 0.02] = np.inf
    psw[g.random(psw.size) < 0.02] = np.nan
    with np.errstate(invalid="ignore"):
        for w in (None, psw):
            got = look_up(plan, idx, off, B, E, w)
            p = None if w is None else np.where(idx >= 0, w, 0)   # the weight of an invalid id is ignored
            ref, _, bad = OP.pool_reference(hw, idx, off, B, psw=p, pooling=pooling)
            same = np.isclose(got, ref, rtol=2.0 ** -22 if pooling == "mean" else 0, atol=0, equal_nan=True)
            assert same.all(), np.argwhere(~same)[:5]
            assert plan.check_errors() == bad


def test_rows_of_a_table_beyond_4_gib():
    import torch

    import paper_2507_01676_amd as embx
    E, rows, B = 16, 70_000_000, 600
    log(f"slots: one table of {rows * E * 4 / 2**30:.2f} GiB, rows of {E * 4} bytes")
    w = torch.empty((rows, E), device="cuda")
    embx.fill_table(w, 0, 99, mode=W.VAL_INTEGER)
    g = np.random.default_rng(3)
    lens = g.integers(0, 9, size=B)
    off = np.zeros(B + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    idx = g.integers(0, rows, size=int(off[-1]))
    idx[::7] = rows - 1 - idx[::7] % 1000
    idx[5::50] = rows
    plan = slots_plan([rows], E, "f32", [{"mean_pooling": 4.0, "max_pooling": 8}], B, [w])
    ok = idx < rows
    vals = np.zeros((idx.size, E), np.float32)
    vals[ok] = W.table_rows_at(0, idx[ok], E, "f32", seed=99, mode=W.VAL_INTEGER)
    for p in (None, g.integers(-3, 4, size=idx.size).astype(np.float32)):
        got = look_up(plan, idx, off, B, E, p)
        ref, _, _ = OP.pool_reference([vals], np.arange(idx.size, dtype=np.int64), off, B, psw=p)
        assert np.array_equal(got, ref)
        assert plan.check_errors() == int((~ok).sum())


@pytest.mark.parametrize("E,dtype", SHAPES)
def test_beside_a_single_lookup_queue(E, dtype):
    """Tables of at most one lookup per bag (one of which holds more at run time after all)
    beside multi-lookup ones."""
    log(f"slots beside single-lookup bags, E{E} {dtype}")
    B, rows = 333, [7, 50_000, 300, 9, 2_000]
    hw = host_tables(config(E, dtype, rows, B), W.VAL_INTEGER)
    g = np.random.default_rng(9)
    lens = [np.ones(B, int), g.poisson(8, B), g.integers(0, 2, B), g.poisson(3, B), np.where(np.arange(B) % 50, 1, 4)]
    off = np.zeros(len(rows) * B + 1, np.int64)
    np.cumsum(np.concatenate(lens), out=off[1:])
    idx = np.concatenate([g.integers(0, m, size=int(x.sum())) for m, x in zip(rows, lens)])
    idx[g.random(idx.size) < 0.02] = 1 << 40
    stats = [{"mean_pooling": max(1.0, float(x.mean())), "max_pooling": p} for x, p in zip(lens, (1, 30, 1, 15, 1))]
    plan = slots_plan(rows, E, dtype, stats, B, upload_tables(hw))
    queues = {ln.split()[1] for ln in plan.queues().splitlines()[1:]}
    assert queues == {"single", "multi"}
    for w in (None, g.integers(-3, 4, size=idx.size).astype(np.float32)):
        got = look_up(plan, idx, off, B, E, w)
        ref, _, bad = OP.pool_reference(hw, idx, off, B, psw=w)
        assert np.array_equal(got, ref)
        assert plan.check_errors() == bad


@pytest.mark.parametrize("E,dtype", [(4, "f32"), (16, "f32"), (8, "f16"), (32, "f16"), (128, "f32")])
def test_a_plan_has_the_queues_of_the_host_text(E, dtype):
    import paper_2507_01676_amd as embx
    log(f"queues of a device plan, E{E} {dtype}")
    rows = [1000 + 40 * t for t in range(12)]
    stats = [{"mean_pooling": m, "max_pooling": 1 if m == 1.0 else 0} for m in (1.0, 3.0, 8.0, 700.0) * 3]
    plan = embx.Plan(rows, E, dtype, stats, 2000, num_workers=64)
    assert plan.queues() == embx.queue_text(rows, E, dtype, stats, 2000, 64)
