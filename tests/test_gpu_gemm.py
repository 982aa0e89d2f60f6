"""GEMM edges of the verify layer against the float64 oracle: row, column and k remainders.

Tolerances as for the layer parity tests (2e-2 row-relative, bf16 activations)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import layer as olay
from oracle import select as osel
from paper_2607_14647_amd import lib as L
from paper_2607_14647_amd import workload as wl
from tests.gpu_common import LOGIT_RTOL, ROUTER_GAP, X_RTOL, need_gpu, note, row_rel_err, workload
from tests.test_gpu_layer import _gpu_run, _layer_parity, _oracle

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
    # one and two k slices (fewer than the rings hold) and a last row tile of one row
    "k_short": _cfg(104, 129, 129, D=0, hidden=64, inter=72),
    "k_short_moe": _cfg(105, 129, 129, D=0, hidden=64, inter=0, n_exp=5, top_k=2, exp_inter=8, rope_theta=1e6),
}


@pytest.mark.parametrize("name", list(CASES))
def test_gemm_edges(name):
    need_gpu()
    _layer_parity(CASES[name], name, 0)


# 1024 rows of a layer whose QKV and down projections split k (in four): 128 x 128 tiles at 64 live
# rows; down takes 128 x 256 at 320 and 256 x 256 at 576 and 1024, QKV 128 x 256 at 1024 (chosen on
# the device from the live rows)
_TILES = _cfg(103, 64, 320, hidden=4096, n_q=8, n_kv=2, head_dim=128, inter=4096)


def test_tile_choice_keeps_bits():
    """A row's residual is the same bits whichever tile shape its batch's row count selects (the
    full-size tests hold 256 and 768 rows of every tile's shapes against the oracle)."""
    need_gpu()
    st, w, kv = workload(_TILES, 0)
    runs = [_gpu_run(_TILES, st, w, kv, [K], [1.0])[0] for K in (64, 320, 576, 1024)]
    full, cf = runs[-1].x.cpu().numpy(), runs[-1].host("cu")
    for vs in runs[:-1]:
        x, cu = vs.x.cpu().numpy(), vs.host("cu")
        for i in range(_TILES.B):
            n = cu[i + 1] - cu[i]
            assert np.array_equal(x[cu[i]: cu[i + 1]], full[cf[i]: cf[i] + n]), i


# 8192 rows of a layer that splits no k (31, 30 and 4 slices): QKV takes 128 x 128 tiles at 512 live
# rows, 128 x 256 at 1024 and 256 x 256 from 1600 on; O and down 128 x 128 up to 1600, 128 x 256 at
# 3000 and 256 x 256 at 8192
_UNSPLIT = _cfg(108, 512, 3000, hidden=1984, n_q=15, n_kv=15, head_dim=128, inter=256)


def test_unsplit_tile_choice_keeps_bits():
    """The fused RoPE and cache append and the in-place residual add in every tile: residual rows and
    appended keys and values of one run against those of all rows kept, bit for bit, and the first
    requests of one run against the oracle."""
    need_gpu()
    cfg = dataclasses.replace(_UNSPLIT, ctx=("uniform", 0, 8))
    st, w, kv = workload(cfg, 0)
    ly, ctx = cfg.layer, st["ctx_len"]
    full = _gpu_run(cfg, st, w, kv, [cfg.B * (cfg.D + 1)], [1.0])[0]
    xf, cf = full.x.cpu().numpy(), full.host("cu")
    kf, vf = (full.kv[n].cpu().numpy() for n in "kv")
    for K in (512, 1024, 1600, 3000):
        vs = _gpu_run(cfg, st, w, kv, [K], [1.0])[0]
        x, cu = vs.x.cpu().numpy(), vs.host("cu")
        rows = np.concatenate([cf[i] + np.arange(cu[i + 1] - cu[i]) for i in range(cfg.B)])
        assert len(rows) == K and np.array_equal(x[:K], xf[rows]), K
        for mine, theirs in ((vs.kv["k"].cpu().numpy(), kf), (vs.kv["v"].cpu().numpy(), vf)):
            for i in range(cfg.B):
                cap, n = int(kv["cap"][i]), int(cu[i + 1] - cu[i])
                at = slice(kv["base"][i], kv["base"][i] + ly.n_kv * cap * ly.head_dim)
                a, b = (t[at].reshape(ly.n_kv, cap, ly.head_dim)[:, : ctx[i] + n] for t in (mine, theirs))
                assert np.array_equal(a, b), (K, i)
        if K == 3000:
            sel = osel.select(st["conf"], st["draft"], ctx, [K], [1.0])
            assert np.array_equal(cu, sel["cu"])
            lay = olay.verify_layer(ly, olay.prepare_weights(w), kv, sel["cu"], sel["packed_tok"], sel["packed_pos"],
                                    sel["packed_req"], ctx, cfg.D, requests=range(32))
            ex = row_rel_err(x[: cu[32]], lay["x_out"][: cu[32]])
            note(f"unsplit tiles: {cu[32]} rows of {K} against the oracle, max rel err {ex.max():.2e}")
            assert ex.max() <= X_RTOL


# experts of more than one 128-row tile: four of them with about 300 of 1200 assignments each, or
# one of sixteen that every row takes (its first component is large in every row) and fifteen small ones
_EXPERTS = {
    "all_large": (_cfg(106, 40, 600, hidden=256, inter=0, n_exp=4, top_k=2, exp_inter=200, rope_theta=1e6), False),
    "one_large": (_cfg(107, 20, 300, hidden=256, inter=0, n_exp=16, top_k=2, exp_inter=200, rope_theta=1e6), True),
}


@pytest.mark.parametrize("name", list(_EXPERTS))
def test_experts_of_several_row_tiles(name):
    need_gpu()
    cfg, skew = _EXPERTS[name]
    st, w, kv = workload(cfg, 0)
    w = dict(w)
    if skew:
        w["embed"], w["w_router"] = w["embed"].copy(), w["w_router"].copy()
        w["embed"][:, 0] = wl.bf16_round(np.float32([0.25]))[0]
        w["w_router"][:, 0] = 0
        w["w_router"][0, 0] = wl.bf16_round(np.float32([2.0]))[0]
    K = cfg.budgets[0]
    vs, _ = _gpu_run(cfg, st, w, kv, [K], [1.0])
    _, lay, _, _ = _oracle(cfg, st, olay.prepare_weights(w), kv, K)
    n = np.bincount(lay["router_ids"].ravel(), minlength=cfg.layer.n_exp)
    ok = lay["router_gap"] > ROUTER_GAP
    ex = row_rel_err(vs.x.cpu().numpy()[:K][ok], lay["x_out"][ok])
    note(f"experts {name}: rows per expert {n.tolist()}, {ok.sum()}/{K} rows compared, max rel err {ex.max():.2e}")
    assert n.max() > 256 and ok.sum() > K // 2
    assert ex.max() <= X_RTOL


@pytest.mark.parametrize("temperature", [0.0, 1.0])
def test_small_vocabulary_head_keeps_bits(temperature):
    """An LM head in 128 x 128 tiles (65 column tiles, 67 MB of weights) at 16 live rows, one task per CU
    (two row tiles, weights streamed) and more (five, not streamed): the bits of a row depend on neither
    the cache policy nor the row blocks that have no live row; logits against float64."""
    need_gpu()
    H, V, B, D = 4096, 8200, 40, 15
    rows = B * (D + 1)
    g = torch.Generator(device="cuda").manual_seed(5)
    w = (torch.randn(V, H, device="cuda", generator=g) * 0.02).bfloat16()
    x = torch.randn(rows, H, device="cuda", generator=g)
    gain = torch.ones(H, device="cuda", dtype=torch.bfloat16)
    req = torch.arange(rows, device="cuda", dtype=torch.int32) % B
    pos = torch.arange(rows, device="cuda", dtype=torch.int32) // B
    ws = L.workspace(L.workspace_bytes(2, L.LayerCfg(hidden=H, vocab=V), B, D))
    outs = {}
    for K in (16, 256, 600):
        cu = torch.full((B + 1,), K, device="cuda", dtype=torch.int32)
        tok = torch.full((rows,), -1, device="cuda", dtype=torch.int32)
        best, lse = (torch.full((rows,), -7.0, device="cuda") for _ in range(2))
        logits = torch.full((rows, V), -7.0, device="cuda")
        if temperature > 0.0:
            L.lm_head_sample(H, V, B, D, cu, req, pos, x, gain, 1e-5, w, temperature, 11, tok, ws, max_score=best,
                             logits=logits, lse=lse)
        else:
            L.lm_head_argmax(H, V, B, D, cu, x, gain, 1e-5, w, tok, ws, max_logit=best, logits=logits)
        torch.cuda.synchronize()
        outs[K] = (tok, best, lse, logits)
        assert (tok[K:] == -1).all() and (logits[K:] == -7.0).all()
    for K in (16, 256):
        for a, b in zip(outs[K], outs[600]):
            assert torch.equal(a[:K], b[:K]), K
    h = x[:600].double() / torch.sqrt((x[:600].double() ** 2).mean(dim=1, keepdim=True) + 1e-5)
    err = row_rel_err(outs[600][3][:600].cpu().numpy(), (h @ w.double().t()).cpu().numpy())
    note(f"small vocabulary head T={temperature}: max rel err {err.max():.2e}")
    assert err.max() <= LOGIT_RTOL
