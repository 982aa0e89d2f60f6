"""Edges of the split-KV attention and its merge against the float64 oracle (layer parity tolerances)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import layer as olay
from oracle import select as osel
from paper_2607_14647_amd import runner
from paper_2607_14647_amd import workload as wl
from tests import test_gpu_layer
from tests.gpu_common import X_RTOL, need_gpu, note, row_rel_err, workload
from tests.test_gpu_layer import _layer_parity

pytestmark = pytest.mark.gpu

_C1 = wl.CONFIGS[1]


def _cfg(cid, B, K, ctx, D=15, **layer):
    return dataclasses.replace(_C1, cid=cid, B=B, D=D, budgets=(K,), ctx=ctx,
                               layer=dataclasses.replace(_C1.layer, **layer))


CASES = {
    # 128-key chunks, 33 to 47 per request: more than the merge reads in one round
    "many_chunks": _cfg(111, 2, 20, ("uniform", 4200, 6000)),
    # two requests of 8 chunks of 128 keys, the last one key short (chunk counts at the merge's
    # edges: test_merge_chunk_counts)
    "chunk_edges": _cfg(112, 2, 9, ("uniform", 1023, 1025), D=4),
    # 256-key chunks; three query heads a group, so pairs do not fill the last workgroup
    "odd_heads": _cfg(113, 9, 31, ("uniform", 0, 1500), D=4, n_q=9, n_kv=3, hidden=264),
    # 97 to 128 query rows an item: both row blocks of every wave, head dimension 128
    "two_blocks": _cfg(114, 3, 48, ("uniform", 100, 700), n_q=16, n_kv=2, head_dim=128),
    # 129 to 256 query rows an item, sixteen waves: all 256 of them, and ragged kept counts that
    # leave waves without rows; one and several chunks
    "wide_64": _cfg(116, 3, 96, ("uniform", 20, 700), D=31, n_q=16, n_kv=2),
    "wide_128": _cfg(117, 3, 96, ("uniform", 20, 700), D=31, n_q=8, n_kv=1, head_dim=128),
    "wide_ragged_64": _cfg(118, 4, 37, ("uniform", 0, 200), D=16, n_q=8, n_kv=1),
    "wide_ragged_128": _cfg(119, 5, 77, ("uniform", 100, 900), D=23, n_q=16, n_kv=2, head_dim=128),
    "wide_block_64": _cfg(120, 2, 128, ("uniform", 300, 500), D=63, n_q=4, n_kv=1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_attention_edges(name):
    need_gpu()
    _layer_parity(CASES[name], name, 0)


def test_merge_chunk_counts(monkeypatch):
    """Chunk counts at the edges of the merge's rounds of 8 loads and 32 weights."""
    need_gpu()
    cfg = _cfg(121, 8, 24, ("uniform", 1, 1), D=4, n_kv=1)
    st, w, _ = workload(cfg, 0, with_kv=False)
    st = dict(st, ctx_len=np.array([1023, 1024, 1025, 2048, 2049, 4095, 4096, 4097], dtype=np.int32))
    kv = wl.make_kv(cfg, 0, st["ctx_len"])
    max_ctx = int(kv["cap"].max())
    assert cfg.B * cfg.layer.n_kv * -(-max_ctx // 128) <= 288          # 128-key chunks
    assert [-(-L // 128) for L in st["ctx_len"].tolist()] == [8, 8, 9, 16, 17, 32, 32, 33]
    monkeypatch.setattr(test_gpu_layer, "workload", lambda c, seed: (st, w, kv))
    _layer_parity(cfg, "merge_chunk_counts", 0)


def test_scores_past_two_to_the_31():
    """Queries and keys of 2^22 the usual size: scores of about 2^38, finite in float32, whose
    softmax is one key.  Rows where bf16 activations alone change that key (the two oracles
    differ) are only required to be finite; at least half are compared."""
    need_gpu()
    cfg = _cfg(115, 4, 24, ("uniform", 100, 700))
    st, w, kv = workload(cfg, 0)
    ly = cfg.layer
    w, kv = dict(w), dict(kv)
    qk = (ly.n_q + ly.n_kv) * ly.head_dim
    big = w["w_qkv"].copy()
    big[:qk] = wl.bf16_round(wl.bf16_to_f32(big[:qk]) * np.float32(2.0 ** 22))
    w["w_qkv"], kv["k"] = big, wl.bf16_round(wl.bf16_to_f32(kv["k"]) * np.float32(2.0 ** 22))
    vs = runner.VerifyStep(cfg, w, st, kv)
    K = cfg.budgets[0]
    vs.select([K], [1.0])
    vs.verify()
    torch.cuda.synchronize()
    sel = osel.select(st["conf"], st["draft"], st["ctx_len"], [K], [1.0])
    args = (ly, olay.prepare_weights(w), kv, sel["cu"], sel["packed_tok"], sel["packed_pos"], sel["packed_req"],
            st["ctx_len"], cfg.D)
    ref, ref16 = olay.verify_layer(*args)["x_out"], olay.verify_layer(*args, act_bf16=True)["x_out"]
    x = vs.x.cpu().numpy()[:K]
    ok = row_rel_err(ref16, ref) <= X_RTOL
    ex = row_rel_err(x[ok], ref16[ok])
    note(f"scores past 2^31: {ok.sum()}/{K} rows compared, {np.isfinite(x).all(axis=1).sum()} finite, max rel err {ex.max():.2e}")
    assert np.isfinite(x).all()
    assert ok.sum() >= K // 2 and ex.max() <= X_RTOL
