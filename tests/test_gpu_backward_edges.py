"""The embedding backward at the edges of its passes: a run's output around the
sizes where waves leave early (one wave, the workgroup) and where a pass takes
1, 2, 4 or 8 elements a thread, runs whose weights just fit LDS and do not,
empty runs, widths of one float4 and of no power of two; sum, weighted and mean,
bit for bit against the oracle, with a guard past the last value."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import make_plan, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


def _check(dims, lengths, mode, **opts):
    import torch
    T, B = len(dims), len(lengths) // len(dims)
    rng = np.random.default_rng([2305, 6942, 71, T, B, int(sum(lengths))])
    off = np.zeros(T * B + 1, np.int64)
    off[1:] = np.cumsum(lengths)
    wts = rng.random(max(1, int(off[-1])), dtype=np.float32)[: int(off[-1])] if mode == "weighted" else None
    g = rng.standard_normal((B, sum(dims))).astype(np.float32)
    w = synth.Workload("bwd", 9, T, (10,) * T, tuple(dims), synth.F32, B, 1, B, "fixed:1", "uniform",
                       mode == "weighted", "normal")
    plan = make_plan(w, pooling_mode=int(mode == "mean"), **opts)
    want = oracle.backward(dims, off, wts, g, B, 1, mean=mode == "mean")
    values = torch.full((want.size + 64,), float("nan"), device="cuda")
    d = None if wts is None else torch.from_numpy(wts if wts.size else np.zeros(1, np.float32)).cuda()
    plan.backward(torch.from_numpy(g).cuda(), torch.from_numpy(off).cuda(), d, B, 1, values)
    torch.cuda.synchronize()
    got = values.cpu().numpy()
    assert np.array_equal(got[: want.size].view(np.uint32), want.view(np.uint32))
    assert np.isnan(got[want.size:]).all(), "stores past the last value"
    plan.close()


@pytest.mark.parametrize("mode", ["sum", "weighted", "mean"])
@pytest.mark.parametrize("dim", [4, 12, 128])
@pytest.mark.parametrize("waves", [1, 2, 16])
def test_run_output_sizes(waves, dim, mode):
    say("backward run sizes", waves, dim, mode)
    step, V = 64 * waves, dim // 4
    edges = [0, 1, 63, 64, 65] + [m * step + d for m in (1, 2, 4, 8, 12, 16) for d in (-1, 0, 1)]
    per_run = sorted({max(0, -(-n // V)) for n in edges})  # lookups whose float4s reach each edge
    lengths = []
    for r in per_run:  # three bags a run: part, none, rest
        lengths += [r // 3, 0, r - r // 3]
    _check([dim], lengths, mode, backward_bags_per_run=3, backward_waves_per_wg=waves)


@pytest.mark.parametrize("rows", [2047, 2048, 2049, 5000])
def test_weights_around_their_lds_slots(rows):
    say("backward weights", rows)
    _check([8, 20], [rows, 0, 7, 0, rows - 5, 5] * 2, "weighted", backward_bags_per_run=2)


@pytest.mark.parametrize("per_bag", [1, 144, 145, 300])
@pytest.mark.parametrize("waves", [1, 16])
def test_weights_beside_rows_that_nearly_fill_lds(waves, per_bag):
    """Fourteen rows of 1024 floats a run leave 2018 words for its weights (none
    with one wave)."""
    say("backward full LDS", waves, per_bag)
    _check([1024], [per_bag] * 28, "weighted", backward_bags_per_run=16, backward_waves_per_wg=waves)


@pytest.mark.parametrize("mode", ["sum", "weighted", "mean"])
def test_every_bag_empty(mode):
    say("backward empty", mode)
    _check([16, 64], [0] * 24, mode)
