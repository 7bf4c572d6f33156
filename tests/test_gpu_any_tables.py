"""The pooling kernel for any tables: rows that are no power of two of
sixteen-byte vectors (groups of lanes left over), rows of more than 64 vectors
(pooled 64 at a time, stored directly, a narrow last block), bag lengths at the
edges of a row group, of the loads in flight and of the staging slot, sum,
weighted sum and mean, element by element against the oracle; and index checks:
bags of invalid offsets or rows among valid ones, with rows of one vector block
and of several."""
import numpy as np
import pytest

import oracle
import synth
from synth import device as sdev
from tests.gpu_util import check_full, make_plan, new_buffers, run, say

pytestmark = pytest.mark.gpu

VECS = [3, 5, 7, 12, 21, 24, 33, 63, 65, 96, 130]


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


def _inputs(dtype, vecs, L, rows, B, R, C, weighted, seed):
    elt = 4 if dtype == synth.F32 else 2
    rng = np.random.default_rng([2305, 6942, 66, seed])
    off = np.zeros(len(L) + 1, np.int64)
    off[1:] = np.cumsum(L)
    idx = rng.integers(0, rows, int(off[-1])).astype(np.int32)
    tabs = []
    for v in vecs:
        x = rng.standard_normal((rows, v * 16 // elt)).astype(np.float32)
        tabs.append(x if dtype == synth.F32 else x.astype(np.float16) if dtype == synth.F16
                    else synth.gen.f32_to_bf16_bits(x))
    wts = rng.random(int(off[-1]), dtype=np.float32) if weighted else None
    w = synth.Workload("any", 9, len(vecs), (rows,) * len(vecs), tuple(v * 16 // elt for v in vecs), dtype, B, R, C,
                       "fixed:1", "uniform", weighted, "normal")
    return synth.Inputs(w, np.asarray(L, np.int64), off, idx, wts, tabs)


@pytest.mark.parametrize("mode", ["sum", "weighted", "mean"])
@pytest.mark.parametrize("kind", ["edges", "slot"])
@pytest.mark.parametrize("dtype", [synth.F32, synth.F16, synth.BF16])
@pytest.mark.parametrize("widest", [130, 32])  # with and without rows of more than 32 vectors
def test_any_width(widest, dtype, kind, mode):
    import torch
    B, R, C = 42, 2, 21
    rng = np.random.default_rng([2305, 6942, 67, dtype, kind == "slot"])
    L = []
    vecs = [v for v in VECS if v <= widest]
    for v in vecs:
        G = max(1, 64 // v)
        L.append(rng.choice([0, 1, G - 1, G, G + 1, 8 * G - 1, 8 * G, 8 * G + 1], B) if kind == "edges"
                 else rng.choice([0, 1, 127, 129, 447, 448, 449, 511, 512, 513, 700], B))
    inp = _inputs(dtype, vecs, np.concatenate(L), 90, B, R, C, mode == "weighted", dtype)
    w = inp.w
    say("any tables", widest, dtype, kind, mode)
    dev = sdev.to_device(inp)
    s64, a64, _ = oracle.pool_inputs(inp, mean=mode == "mean")
    outs = []
    for opts in (dict(), dict(bags_per_run=3, waves_per_wg=1, stream_rows=0, check_indices=1),
                 dict(bags_per_run=21, persistent_wgs_per_cu=1, release_mode=0), dict(rows_in_flight=4),
                 dict(rows_in_flight=16, waves_per_wg=16), dict(bags_per_run=21, waves_per_wg=1)):
        plan = make_plan(w, pooling_mode=int(mode == "mean"), **opts)
        for fused in (True, False):
            send, _, flags = new_buffers(w)
            run(plan, w, dev, send, flags, fused=fused)
            torch.cuda.synchronize()
            got = send.cpu().numpy()
            check_full(inp, got, s64, a64)
            assert np.all(flags.cpu().numpy() == 1)
            outs.append(got)
        assert plan.status_ex() == (0, -1, 0, -1)
        plan.close()
    for o in outs[1:]:
        assert np.array_equal(o.view(np.uint32), outs[0].view(np.uint32))


@pytest.mark.parametrize("what", ["offsets", "rows", "both"])
@pytest.mark.parametrize("vec", [4, 5, 70])
def test_invalid_bags_among_valid_ones(vec, what):
    """Bags of decreasing offsets, offsets past the end and rows out of range
    are reported (the lowest one) and every other bag is whole; rows out of
    range are left out of their bag."""
    import torch
    B, rows = 40, 50
    rng = np.random.default_rng([2305, 6942, 68, vec])
    inp = _inputs(synth.F32, [vec], rng.integers(1, 9, B), rows, B, 1, 20, False, vec)
    w, off, idx = inp.w, inp.offsets.copy(), inp.indices.copy()
    nnz = int(off[-1])
    if what != "rows":
        off[13] = off[15] + 2   # bag 13 runs backwards, bag 12 takes in the rows up to it
        off[31] = nnz + 5       # bags 30 and 31 touch an offset past the end
    bad_rows = []
    if what != "offsets":
        bad_rows = [int(inp.offsets[7]), int(inp.offsets[21])]
        idx[bad_rows[0]], idx[bad_rows[1]] = rows, -1
    want = np.zeros((B, w.dims[0]), np.float64)
    bad = []
    for b in range(B):
        lo, hi = int(off[b]), int(off[b + 1])
        if not 0 <= lo <= hi <= nnz:
            bad.append(b)
            continue
        ok = [k for k in range(lo, hi) if 0 <= idx[k] < rows]
        if len(ok) < hi - lo:
            bad.append(b)
        want[b] = inp.host_tables[0][idx[ok]].astype(np.float64).sum(0)
    say("invalid bags", vec, what, bad)
    inp2 = synth.Inputs(w, inp.lengths, off, idx, None, inp.host_tables)
    dev = sdev.to_device(inp2)
    for opts in (dict(), dict(bags_per_run=1, waves_per_wg=1), dict(bags_per_run=20, waves_per_wg=1)):
        plan = make_plan(w, check_indices=1, **opts)
        send, _, flags = new_buffers(w)
        run(plan, w, dev, send, flags)
        torch.cuda.synchronize()
        assert plan.status_ex() == (0, -1, 0, min(bad))
        # at most 9 + 9 rows of |values| < 8 a bag, rounded once each
        assert np.abs(send.cpu().numpy() - want).max() <= 18 * 18 * 8 * 2.0 ** -24
        plan.close()


@pytest.mark.parametrize("dtype", [synth.F32, synth.F16, synth.BF16])
@pytest.mark.parametrize("vec", [4, 5, 70])
def test_rows_left_out_whatever_their_weight(vec, dtype):
    """A row out of range adds nothing to its bag, also where its weight is
    infinite or not a number."""
    import torch
    B, rows = 24, 50
    rng = np.random.default_rng([2305, 6942, 69, vec, dtype])
    inp = _inputs(dtype, [vec], rng.integers(1, 9, B), rows, B, 1, 12, True, vec)
    left_out = _inputs(dtype, [vec], inp.lengths, rows, B, 1, 12, True, vec)
    assert np.array_equal(inp.indices, left_out.indices)
    for b, (row, weight) in {3: (rows, np.inf), 11: (-1, np.nan), 19: (rows + 7, -np.inf)}.items():
        k = int(inp.offsets[b])
        inp.indices[k], inp.weights[k] = row, weight
        left_out.indices[k], left_out.weights[k] = 0, 0.0
    say("rows left out", vec, dtype)
    dev = sdev.to_device(inp)
    plan = make_plan(inp.w, check_indices=1)
    send, _, flags = new_buffers(inp.w)
    run(plan, inp.w, dev, send, flags)
    torch.cuda.synchronize()
    assert plan.status_ex() == (0, -1, 0, 3)
    check_full(left_out, send.cpu().numpy())
    plan.close()


@pytest.mark.parametrize("dtype", [synth.F32, synth.F16, synth.BF16])
@pytest.mark.parametrize("vec", [3, 6, 12, 20, 24, 65, 72, 80, 96])
def test_short_weighted_bags_add_in_sequence(vec, dtype):
    """Weighted bags of fewer than seven lookups of a table whose rows are no
    power of two of vectors: fma(w, x, sum) row after row, bit for bit, in every
    column block of a row.  In 64 bits a product and its sum with the one before
    are exact here: weights are multiples of 2^-24, values of 2^-4 (below 8, so
    exact in every storage type), sums stay below 2^6."""
    import torch
    B, rows = 56, 50
    L = np.tile(np.arange(8), 7)
    inp = _inputs(dtype, [vec], L, rows, B, 1, 28, True, vec)
    tab = np.clip(np.round(np.random.default_rng([2305, 6942, 70, vec]).standard_normal((rows, inp.w.dims[0])) * 16),
                  -127, 127) / 16
    inp.host_tables[0] = (tab.astype(np.float16) if dtype == synth.F16 else tab.astype(np.float32)
                          if dtype == synth.F32 else synth.gen.f32_to_bf16_bits(tab.astype(np.float32)))
    say("short weighted bags", vec, dtype)
    dev = sdev.to_device(inp)
    plan = make_plan(inp.w)
    send, _, flags = new_buffers(inp.w)
    run(plan, inp.w, dev, send, flags)
    torch.cuda.synchronize()
    got = send.cpu().numpy()
    for b in range(B):
        if L[b] > 6:
            continue
        acc = np.zeros(inp.w.dims[0], np.float32)
        for k in range(int(inp.offsets[b]), int(inp.offsets[b + 1])):
            acc = (acc.astype(np.float64) + float(inp.weights[k]) * tab[inp.indices[k]]).astype(np.float32)
        assert np.array_equal(acc.view(np.uint32), got[b].view(np.uint32)), b
    plan.close()
