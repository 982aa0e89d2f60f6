"""Selection where its kernels change over: one launch while at most 512 positions have to be
counted (those that score 1 by definition come first) and at most 1024 exist, else two."""
import numpy as np
import pytest

from paper_2607_14647_amd import lib as L
from tests.gpu_common import need_gpu, note
from tests.test_gpu_rs import check_select
from tests.test_gpu_select import _costs, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,D", [(51, 4), (16, 15), (257, 0), (86, 2), (17, 15), (33, 30), (24, 15), (55, 6), (455, 17), (8192 // 64, 63),
                                 (34, 15), (35, 15), (512, 1), (513, 1), (1024, 0), (1025, 0), (8, 63), (2000, 2)])
@pytest.mark.parametrize("kind", ["mixed", "ties"])
def test_select_rank_edges(B, D, kind):
    need_gpu()
    rng, *args = _inputs(B, D, kind)
    note(f"select rank edges {kind} B={B} D={D}")
    check(*args, _costs(rng, args[-1]))


def _inputs(B, D, kind):
    rng = np.random.default_rng(B * 64 + D)
    conf = (rng.random((B, D)) ** 0.3 if kind == "mixed" else rng.choice([0.0, 0.5, 1.0], size=(B, D))).astype(np.float32)
    draft = rng.integers(0, 151936, size=(B, D + 1)).astype(np.int32)
    ctx = rng.integers(0, 8192, size=B).astype(np.int32)
    budgets = sorted({B, B * (D + 1), *rng.integers(B, B * (D + 1) + 1, size=9).tolist()})
    return rng, conf, draft, ctx, budgets


# the same with shifted scores, of which depths 0 and 1 score 1
@pytest.mark.parametrize("B,D", [(36, 15), (37, 15), (512, 1), (513, 1), (256, 3), (257, 3), (400, 0), (18, 30), (3, 2)])
@pytest.mark.parametrize("kind", ["mixed", "ties"])
def test_select_rs_rank_edges(B, D, kind):
    need_gpu()
    rng, conf, draft, ctx, budgets = _inputs(B, D, kind)
    note(f"select_rs rank edges {kind} B={B} D={D}")
    check_select(conf, draft, ctx, L.RS_SCAN, budgets, _costs(rng, budgets))
    check_select(conf, draft, ctx, L.RS_FIXED, budgets[len(budgets) // 2:][:1], [1.0])
