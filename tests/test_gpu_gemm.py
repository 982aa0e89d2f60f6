"""GEMM edges of the verify layer against the float64 oracle: row, column and k remainders.

Tolerances as for the layer parity tests (2e-2 row-relative, bf16 activations)."""
import dataclasses

import pytest

from paper_2607_14647_amd import workload as wl
from tests.gpu_common import need_gpu
from tests.test_gpu_layer import _layer_parity

pytestmark = pytest.mark.gpu

_C1 = wl.CONFIGS[1]


def _cfg(cid, B, K, D=15, **layer):
    return dataclasses.replace(_C1, cid=cid, B=B, D=D, budgets=(K,), layer=dataclasses.replace(_C1.layer, **layer))


CASES = {
    # k loops that start past k = 0 (8208 columns: 33 blocks of 256 over the eighths) with a last
    # slice of 40 and of 8 k in their middle; column and row tiles with remainders
    "k_tail": _cfg(101, 12, 150, hidden=1000, inter=4104),
    # grouped expert GEMMs with the same remainders, every expert at a start of its own
    "k_tail_moe": _cfg(102, 12, 150, hidden=1000, inter=0, n_exp=9, top_k=2, exp_inter=200, rope_theta=1e6),
}


@pytest.mark.parametrize("name", list(CASES))
def test_gemm_edges(name):
    need_gpu()
    _layer_parity(CASES[name], name, 0)
