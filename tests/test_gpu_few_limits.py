"""Steps of 5 to 8 rows on both sides of the line between the few-row kernel and
the matrix-core kernels, against the fp64 oracle: the row counts that have a
version of the few-row kernel of their own (5, 6) and those that share one (7, 8)."""
import pytest
import torch

from synth import workloads as wl
from tests.gpu_util import check, run_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1805_09863_amd as kb
    kb.lib()
    return kb


@pytest.mark.parametrize("dt,H,V,kernel", [
    ("f32", 256, 26000, "few"), ("f32", 256, 26004, "dma"), ("f32", 260, 26004, "reg"),
    ("bf16", 1024, 3000, "few"), ("bf16", 128, 36000, "few"), ("bf16", 1024, 17008, "dma"), ("bf16", 1000, 17008, "reg"),
])
@pytest.mark.parametrize("rows", [[5], [3, 3], [5, 2], [1, 5, 2]])
def test_limits(kb, rows, dt, H, V, kernel):
    n = sum(rows)
    assert kb.kbest_plan(kb.KB_BF16 if dt == "bf16" else kb.KB_F32, n, H, V, 5)["kernel"] == kernel
    inp = wl.make_step(H=H, V=V, k=5, rows_per_sentence=rows, dtype=dt, seed=4700 + n, name=f"few_limit_{dt}_{n}x{H}x{V}")
    check(inp, run_step(kb, inp, row_lse=True))
