"""Selection where its kernels change over: up to 384 positions in one launch, more in two."""
import numpy as np
import pytest

from tests.gpu_common import need_gpu, note
from tests.test_gpu_select import _costs, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,D", [(51, 4), (16, 15), (257, 0), (86, 2), (17, 15), (33, 30), (24, 15), (55, 6), (455, 17), (8192 // 64, 63)])
@pytest.mark.parametrize("kind", ["mixed", "ties"])
def test_select_rank_edges(B, D, kind):
    need_gpu()
    rng = np.random.default_rng(B * 64 + D)
    conf = (rng.random((B, D)) ** 0.3 if kind == "mixed" else rng.choice([0.0, 0.5, 1.0], size=(B, D))).astype(np.float32)
    draft = rng.integers(0, 151936, size=(B, D + 1)).astype(np.int32)
    ctx = rng.integers(0, 8192, size=B).astype(np.int32)
    budgets = sorted({B, B * (D + 1), *rng.integers(B, B * (D + 1) + 1, size=9).tolist()})
    note(f"select rank edges {kind} B={B} D={D}")
    check(conf, draft, ctx, budgets, _costs(rng, budgets))
