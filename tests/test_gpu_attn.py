"""Edges of the split-KV attention and its merge against the float64 oracle (layer parity tolerances)."""
import dataclasses

import pytest

from paper_2607_14647_amd import workload as wl
from tests.gpu_common import need_gpu
from tests.test_gpu_layer import _layer_parity

pytestmark = pytest.mark.gpu

_C1 = wl.CONFIGS[1]


def _cfg(cid, B, K, ctx, D=15, **layer):
    return dataclasses.replace(_C1, cid=cid, B=B, D=D, budgets=(K,), ctx=ctx,
                               layer=dataclasses.replace(_C1.layer, **layer))


CASES = {
    # 128-key chunks, 33 to 47 per request: more than the merge reads in one round
    "many_chunks": _cfg(111, 2, 20, ("uniform", 4200, 6000)),
    # exactly 8, 16 and 32 chunks of 128 keys, one key less and one more
    "chunk_edges": _cfg(112, 2, 9, ("uniform", 1023, 1025), D=4),
    # 256-key chunks; three query heads a group, so pairs do not fill the last workgroup
    "odd_heads": _cfg(113, 9, 31, ("uniform", 0, 1500), D=4, n_q=9, n_kv=3, hidden=264),
    # 97 to 128 query rows an item: both row blocks of every wave, head dimension 128
    "two_blocks": _cfg(114, 3, 48, ("uniform", 100, 700), n_q=16, n_kv=2, head_dim=128),
}


@pytest.mark.parametrize("name", list(CASES))
def test_attention_edges(name):
    need_gpu()
    _layer_parity(CASES[name], name, 0)
