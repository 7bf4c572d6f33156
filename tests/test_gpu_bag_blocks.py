"""Bags that share a wave's loads: lengths at the edges of a row group (G rows
a load), of the loads in flight and of the 512-index staging slot, empty bags
first, last and between, for every power-of-two row width and storage type,
sum, weighted sum and mean, against the oracle; and the same bags pooled one to
a run, which must not change a bit."""
import numpy as np
import pytest

import oracle
import synth
from synth import device as sdev
from tests.gpu_util import check_full, make_plan, new_buffers, run, say

pytestmark = pytest.mark.gpu

KINDS = {
    "one_row": lambda rng, n, G: np.ones(n, np.int64),
    "few": lambda rng, n, G: rng.integers(0, 4, n),
    "edges": lambda rng, n, G: rng.choice([0, 1, G - 1, G, G + 1, 2 * G, 8 * G - 1, 8 * G, 8 * G + 1], n),
    "all_empty": lambda rng, n, G: np.zeros(n, np.int64),
    "slot": lambda rng, n, G: rng.choice([0, 127, 128, 129, 511, 512, 513, 700], n),
}


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("mode", ["sum", "weighted", "mean"])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("dtype", [synth.F32, synth.F16, synth.BF16])
def test_bags_sharing_a_wave(dtype, kind, mode):
    import torch
    elt = 4 if dtype == synth.F32 else 2
    vecs = [1, 2, 4, 8, 16, 32, 64]
    T, B, R, C = len(vecs), 42, 2, 21
    rng = np.random.default_rng([2305, 6942, 55, dtype, sorted(KINDS).index(kind)])
    L = np.concatenate([KINDS[kind](rng, B, 64 // v) for v in vecs]).astype(np.int64)
    if kind == "edges":
        L[0] = L[-1] = 0
    off = np.zeros(T * B + 1, np.int64)
    off[1:] = np.cumsum(L)
    rows = 300
    idx = rng.integers(0, rows, int(off[-1])).astype(np.int32)
    tabs = []
    for v in vecs:
        x = rng.standard_normal((rows, v * 16 // elt)).astype(np.float32)
        tabs.append(x if dtype == synth.F32 else x.astype(np.float16) if dtype == synth.F16
                    else synth.gen.f32_to_bf16_bits(x))
    wts = rng.random(int(off[-1]), dtype=np.float32) if mode == "weighted" else None
    w = synth.Workload("blocks", 9, T, (rows,) * T, tuple(v * 16 // elt for v in vecs), dtype, B, R, C, "fixed:1",
                       "uniform", mode == "weighted", "normal")
    inp = synth.Inputs(w, L, off, idx, wts, tabs)
    say("bag blocks", dtype, kind, mode)
    dev = sdev.to_device(inp)
    if dev.indices.numel() == 0:
        dev.indices = torch.zeros(1, dtype=torch.int32, device="cuda")
    s64, a64, _ = oracle.pool_inputs(inp, mean=mode == "mean")
    outs = []
    for opts in (dict(), dict(bags_per_run=1, waves_per_wg=1), dict(bags_per_run=21, waves_per_wg=1, stream_rows=0),
                 dict(bags_per_run=7, waves_per_wg=3, persistent_wgs_per_cu=1)):
        plan = make_plan(w, pooling_mode=int(mode == "mean"), **opts)
        send, _, flags = new_buffers(w)
        run(plan, w, dev, send, flags)
        torch.cuda.synchronize()
        got = send.cpu().numpy()
        check_full(inp, got, s64, a64)
        assert np.all(flags.cpu().numpy() == 1)
        outs.append(got)
        plan.close()
    for o in outs[1:]:
        assert np.array_equal(o.view(np.uint32), outs[0].view(np.uint32)), "bags sharing a wave changed a bit"
