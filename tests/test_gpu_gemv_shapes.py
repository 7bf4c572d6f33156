"""GEMV + AllReduce at the edges of its launch shapes: rows of V sixteen-byte
vectors around the limits where lanes are shared between rows (V <= 32), where
16, 8 or 4 rows go at once (64, 128, 256) and where x moves to LDS (above), few
output rows (workgroups split to single rows), ragged tiles, unequal ranks,
every storage type; against the oracle and bitwise equal fused and unfused."""
import pytest

import synth
from tests.gpu_util import say
from tests.test_gpu_gemv_ar import _run

pytestmark = pytest.mark.gpu

VECS = [1, 2, 3, 8, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 600]


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", [synth.F32, synth.F16, synth.BF16])
@pytest.mark.parametrize("V", VECS)
def test_row_lengths(V, dtype):
    e = 4 if dtype == synth.F32 else 8
    say("gemv row length", V, dtype)
    _run(3, 333, [V * e, max(1, V // 2) * e, V * e], dtype, seed=V)
    _run(1, 130, [V * e], dtype, seed=V + 1, integer=True)


@pytest.mark.parametrize("M", [1, 2, 7, 63, 64, 65, 129])
@pytest.mark.parametrize("V", [5, 64, 256, 1025])
def test_few_rows(V, M):
    say("gemv few rows", V, M)
    _run(1, M, [V * 4], synth.F32, seed=M)
    _run(2, M, [V * 8, V * 8], synth.F16, seed=M, waves_per_wg=1)
    _run(2, M, [V * 8, 8], synth.BF16, seed=M, waves_per_wg=4, tile_rows=100, wgs_per_rank=1)
    _run(2, M, [V * 8, 8], synth.BF16, seed=M, reduce_mode=1)
