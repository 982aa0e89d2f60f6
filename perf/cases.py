"""Performance cases of the D-cut verify step, measured through the library's public calls.

A case is one call of the library (or one whole step) at sizes its users run: the layer and LM-head
shapes of `paper_2607_14647_amd.workload.CONFIGS`, the batch sizes of the startup cost table (1 to 64,
and the batch-128 MoE and batch-256 ragged configurations), and generic smaller layers in the drawn
cases.  Inputs are made on the GPU from the seed: unit-variance keys and values, embedding-scale
residuals, N(0, 0.02^2) weights, Beta(a, 1) confidences.  `exact` recomputes a case in float64 with
plain torch and numpy.
"""
import math

import numpy as np
import torch

from paper_2607_14647_amd import lib as L
from paper_2607_14647_amd import workload as wl

DENSE = dict(hidden=4096, n_q=32, n_kv=8, head_dim=128, inter=14336, n_exp=0, top_k=0, exp_inter=0)
MOE = dict(hidden=2048, n_q=32, n_kv=4, head_dim=128, inter=0, n_exp=128, top_k=8, exp_inter=768)
TINY = dict(hidden=256, n_q=4, n_kv=2, head_dim=64, inter=688, n_exp=0, top_k=0, exp_inter=0)
# generic smaller layers for the drawn cases: 64- and 128-wide heads, group sizes 4 and 8, widths
# that are no multiple of a GEMM tile
LAYERS = [
    DENSE,
    MOE,
    dict(hidden=2048, n_q=32, n_kv=8, head_dim=64, inter=8192, n_exp=0, top_k=0, exp_inter=0),
    dict(hidden=3072, n_q=24, n_kv=8, head_dim=128, inter=8200, n_exp=0, top_k=0, exp_inter=0),
    dict(hidden=1024, n_q=16, n_kv=2, head_dim=128, inter=2816, n_exp=0, top_k=0, exp_inter=0),
    dict(hidden=1024, n_q=16, n_kv=4, head_dim=64, inter=0, n_exp=32, top_k=4, exp_inter=512),
]
EPS, THETA = 1e-5, 500000.0
W_STD, KV_STD, X_STD = 0.02, 1.0, 0.05
X_STD_MOE = 0.25       # a residual several times what the routed MLP adds: a row whose 8th and 9th experts tie stays close


def listed():
    return [
        # the whole greedy step of a small draft-sized model: launch latency only
        dict(name="step_tiny_b4", kind="step", B=4, D=15, K=24, R=1, ctx_lo=64, ctx_hi=128, ctx_log=False,
             conf="u18", vocab=1024, logits=True, **TINY),
        # the benchmark's step: batch 64, adaptive budget over 16 candidates (256 rows are kept)
        dict(name="step_dense_b64", kind="step", B=64, D=15, K=256, R=16, ctx_lo=2048, ctx_hi=4096, ctx_log=False,
             conf="mix", vocab=128256, logits=False, **DENSE),
        # selection and packing alone at the ragged batch of 256
        dict(name="select_b256", kind="select", B=256, D=15, R=16, rs=False, ctx_lo=512, ctx_hi=8192, ctx_log=True,
             conf="lognormal"),
        # one request served alone, its block verified whole: the smallest batch of the cost table
        dict(name="layer_dense_b1", kind="layer", B=1, D=15, K=16, ctx_lo=2048, ctx_hi=4096, ctx_log=False,
             conf="u18", **DENSE),
        # batch 16 at half its rows
        dict(name="layer_dense_b16", kind="layer", B=16, D=15, K=128, ctx_lo=1024, ctx_hi=2048, ctx_log=False,
             conf="u18", **DENSE),
        # batch 64 pruned to a quarter of its rows: the layer of the benchmark's step, in the middle of a model
        dict(name="layer_dense_b64", kind="layer", B=64, D=15, K=256, ctx_lo=2048, ctx_hi=4096, ctx_log=False,
             conf="mix", **DENSE),
        # batch 64 without pruning (the comparison every deployment starts from; also the cost table's last bucket)
        dict(name="layer_dense_b64_full", kind="layer", B=64, D=15, K=1024, ctx_lo=2048, ctx_hi=4096, ctx_log=False,
             conf="mix", **DENSE),
        # batch 256 with ragged contexts, an odd budget
        dict(name="layer_dense_b256", kind="layer", B=256, D=15, K=771, ctx_lo=512, ctx_hi=8192, ctx_log=True,
             conf="lognormal", **DENSE),
        # routed MoE layer, batch 128
        dict(name="layer_moe_b128", kind="layer", B=128, D=15, K=768, ctx_lo=1024, ctx_hi=4096, ctx_log=False,
             conf="u18", **MOE),
        # greedy LM head of the MoE model at its batch: many rows, the widest vocabulary
        dict(name="head_argmax_b128", kind="head", B=128, D=15, K=768, hidden=2048, vocab=151936, temperature=0.0,
             logits=False, conf="u18"),
        # LM head at temperature 1 with the logits and log-partition that rejection sampling reads
        dict(name="head_sample_b64", kind="head", B=64, D=15, K=256, hidden=4096, vocab=128256, temperature=1.0,
             logits=True, conf="mix"),
        # rejection-sampling acceptance over full proposal distributions
        dict(name="accept_rs_b64", kind="accept_rs", B=64, D=15, K=256, vocab=128256, temperature=1.0, conf="mix"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "select", "layer", "layer", "layer", "head", "head", "accept", "accept_rs"])
    conf = rng.choice(["u18", "mix", "lognormal"])
    D = rng.choice([3, 4, 7, 9, 15, 15, 15, 16, 23, 31])
    if kind == "step":
        B = _log_int(rng, 1, 16)
        return dict(kind="step", B=B, D=D, K=rng.randint(B, B * (D + 1)), R=1, ctx_lo=rng.randint(0, 64),
                    ctx_hi=_log_int(rng, 65, 1000), ctx_log=False, conf=conf, vocab=_log_int(rng, 500, 30000),
                    logits=True, **TINY)
    if kind in ("select", "accept"):
        D = rng.choice([D, rng.randint(1, 63)])
        B = _log_int(rng, 1, min(1024, 8192 // (D + 1)))
        if kind == "accept":
            return dict(kind="accept", B=B, D=D, K=rng.randint(B, B * (D + 1)), vocab=32000, conf=conf)
        return dict(kind="select", B=B, D=D, R=rng.randint(1, 64), rs=rng.random() < 0.3, ctx_lo=0, ctx_hi=4096,
                    ctx_log=False, conf=conf)
    B = _log_int(rng, 1, 128 if kind == "layer" else 256)
    rows = B * (D + 1)
    K = _log_int(rng, B, max(B, min(rows, 1024)))
    if kind == "layer":
        ly = rng.choice(LAYERS)
        hi = _log_int(rng, 200, min(8192, 400000 // B))
        return dict(kind="layer", B=B, D=D, K=K, ctx_lo=_log_int(rng, 1, hi), ctx_hi=hi, ctx_log=rng.random() < 0.5,
                    conf=conf, **ly)
    if kind == "head":
        sample = rng.random() < 0.4
        H, V = rng.choice([256, 1000, 2048, 3072, 4096]), _log_int(rng, 2000, 152064)
        K = max(B, min(K, int(4e11 / (H * V))))
        return dict(kind="head", B=B, D=D, K=K, hidden=H, vocab=V,
                    temperature=rng.choice([0.5, 1.0, 1.3]) if sample else 0.0,
                    logits=sample and B <= 64 and rng.random() < 0.5, conf=conf)
    B = _log_int(rng, 1, 64)
    D = min(D, 16)
    return dict(kind="accept_rs", B=B, D=D, K=rng.randint(B, min(1024, B * (D + 1))), vocab=_log_int(rng, 1000, 128256),
                temperature=rng.choice([0.7, 1.0]), conf=conf)


# ------------------------------------------------------------------ inputs

def _gen(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 64 + tag)
    return g


def _normal(seed, tag, shape, std, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=_gen(seed, tag))


def _host_inputs(case, seed):
    """Confidences, contexts and draft tokens of the batch (host arrays)."""
    rng = np.random.default_rng([int(seed), 17])
    B, D = case["B"], case["D"]
    if case["conf"] == "u18":
        a = rng.uniform(1.0, 8.0, size=B)
    elif case["conf"] == "mix":
        a = np.where(rng.permutation(B) < B // 2, 6.0, 1.2)
    else:
        a = np.exp(0.5 + rng.standard_normal(B))
    conf = np.power(rng.random((B, D)), 1.0 / a[:, None]).astype(np.float32)
    lo, hi = case.get("ctx_lo", 0), case.get("ctx_hi", 1024)
    if case.get("ctx_log"):
        ctx = np.rint(np.exp(rng.uniform(math.log(max(lo, 1)), math.log(max(hi, 1)), size=B)))
    else:
        ctx = rng.integers(lo, hi + 1, size=B)
    draft = rng.integers(0, case.get("vocab", 32000), size=(B, D + 1))
    return conf, ctx.astype(np.int32), draft.astype(np.int32)


def _candidates(case, seed):
    """Candidate budgets and their step costs: the case's one budget, or R of them over the whole range with
    the step time of a row count that rises at every 256 rows (as the measured cost rows do)."""
    B, rows, R = case["B"], case["B"] * (case["D"] + 1), case.get("R", 1)
    if R == 1 and "K" in case:
        return [case["K"]], [1.0]
    if R == 16 and case["D"] == 15:
        budgets = [B * m for m in range(1, 17)]
    else:
        budgets = sorted(np.random.default_rng([int(seed), 19]).integers(B, rows + 1, size=R).tolist())
    return budgets, [0.23 + 0.30 * math.ceil(k / 256) + 0.0004 * k for k in budgets]


def _select_np(conf, draft, ctx, budgets, costs, rs=False):
    """Selection and packing in numpy: sequential float32 scores, (score desc, depth, request) order, exact
    integer benefits, first strict maximum of benefit / cost; with `rs`, shifted scores and the causal scan."""
    B, D = conf.shape
    D1, N = D + 1, B * (D + 1)
    s = np.ones((B, D1), dtype=np.float32)
    for k in range(1, D1):
        s[:, k] = s[:, k - 1] * conf[:, k - 1]
    if rs:
        s[:, 1:] = s[:, :-1].copy()
    i, k = np.divmod(np.arange(N), D1)
    order = np.lexsort((i, k, -s.reshape(-1).astype(np.float64)))
    units = np.floor(s.reshape(-1)[order].astype(np.float64) * 2.0 ** 40).astype(np.uint64)
    P = np.concatenate([np.zeros(1, dtype=np.uint64), np.cumsum(units, dtype=np.uint64)])
    benefit = np.array([P[K] for K in budgets], dtype=np.uint64)
    if rs:
        def cost(K):
            r = sum(1 for b in budgets if b <= K) - 1
            if r < 0:
                return costs[0]
            if r == len(budgets) - 1:
                return costs[r]
            return costs[r] + ((costs[r + 1] - costs[r]) * float(K - budgets[r])) / float(budgets[r + 1] - budgets[r])
        obj = lambda K: float(P[K]) * 2.0 ** -40 / cost(K)
        Kstar = next((K for K in range(B, N) if not obj(K + 1) > obj(K)), N)
        best = sum(1 for b in budgets if b <= Kstar) - 1
    else:
        best = int(np.argmax([float(p) * 2.0 ** -40 / c for p, c in zip(benefit, costs)]))
        Kstar = budgets[best]
    keep = np.bincount(i[order[:Kstar]], minlength=B).astype(np.int32)
    cu = np.concatenate([[0], np.cumsum(keep)]).astype(np.int32)
    tok, pos, req = (np.zeros(N, dtype=np.int32) for _ in range(3))
    for b in range(B):
        n = keep[b]
        tok[cu[b]: cu[b] + n] = draft[b, :n]
        pos[cu[b]: cu[b] + n] = ctx[b] + np.arange(n)
        req[cu[b]: cu[b] + n] = b
    return dict(keep_len=keep, cu=cu, packed_tok=tok, packed_pos=pos, packed_req=req,
                choice=np.array([Kstar, best], dtype=np.int32), benefit=benefit.astype(np.int64))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _shape(case):
    return wl.LayerShape(hidden=case["hidden"], n_q=case["n_q"], n_kv=case["n_kv"], head_dim=case["head_dim"],
                         inter=case["inter"], vocab=case.get("vocab", 32000), n_exp=case["n_exp"],
                         top_k=case["top_k"], exp_inter=case["exp_inter"], rms_eps=EPS, rope_theta=THETA)


def _weights(case, seed, embed=False, head=False):
    H, hd, E = case["hidden"], case.get("head_dim", 0), case.get("n_exp", 0)
    w = {}
    if embed:
        w["embed"] = _normal(seed, 1, (case["vocab"], H), X_STD)
    if head:
        w["final_norm"] = (1.0 + _normal(seed, 2, (H,), 0.1, torch.float32)).bfloat16()
        w["w_lm"] = _normal(seed, 3, (case["vocab"], H), W_STD)
    if hd:
        w["attn_norm"] = (1.0 + _normal(seed, 4, (H,), 0.1, torch.float32)).bfloat16()
        w["mlp_norm"] = (1.0 + _normal(seed, 5, (H,), 0.1, torch.float32)).bfloat16()
        w["w_qkv"] = _normal(seed, 6, ((case["n_q"] + 2 * case["n_kv"]) * hd, H), W_STD)
        w["w_o"] = _normal(seed, 7, (H, case["n_q"] * hd), W_STD)
        if E == 0:
            w["w_gate_up"] = _normal(seed, 8, (2 * case["inter"], H), W_STD)
            w["w_down"] = _normal(seed, 9, (H, case["inter"]), W_STD)
        else:
            w["w_router"] = _normal(seed, 10, (E, H), 1.0 / math.sqrt(H))
            w["w_exp_gate_up"] = _normal(seed, 11, (E, 2 * case["exp_inter"], H), W_STD)
            w["w_exp_down"] = _normal(seed, 12, (E, H, case["exp_inter"]), W_STD)
    return w


def _cache(case, seed, ctx):
    """One slab of the same capacity per request (a serving engine's fixed slots).  Request i's slab starts
    L_i slots before a regular grid, so that the slots the step appends, L_i to L_i + D, of every request and
    head form one strided view (`new_k`, `new_v`: zero before the call)."""
    B, D1, n_kv, hd = case["B"], case["D"] + 1, case["n_kv"], case["head_dim"]
    cap = int(ctx.max()) + D1
    slab = n_kv * cap * hd
    lead = int(ctx.max()) * hd
    base = lead + np.arange(B, dtype=np.int64) * slab - ctx.astype(np.int64) * hd
    out = dict(base=_dev(base), cap=torch.full((B,), cap, dtype=torch.int32, device="cuda"), cap_host=cap)
    for n, tag in (("k", 20), ("v", 21)):
        t = _normal(seed, tag, (lead + B * slab,), KV_STD)
        new = t.as_strided((B, n_kv, D1, hd), (slab, cap * hd, hd, 1), lead)
        new.zero_()
        out[n], out["new_" + n] = t, new
    return out


def _selection(case, seed):
    conf, ctx, draft = _host_inputs(case, seed)
    budgets, costs = _candidates(case, seed)
    return conf, ctx, draft, budgets, costs, _select_np(conf, draft, ctx, budgets, costs, case.get("rs", False))


def _head_x(case, seed):
    rows = case["B"] * (case["D"] + 1)
    return _normal(seed, 30, (rows, case["hidden"]), 1.0, torch.float32)


def _proposals(case, seed, sel):
    """Target logits of the kept rows, the drafter's proposal distributions (the target's logits blurred by
    noise, so that drafts survive at a realistic rate) and the drafts drawn from them."""
    B, D, V, T = case["B"], case["D"], case["vocab"], case["temperature"]
    rows, K = B * (D + 1), int(sel["cu"][-1])
    logits = torch.zeros(rows, V, device="cuda")
    logits[:K].normal_(0.0, 2.5, generator=_gen(seed, 40))
    lse = torch.zeros(rows, device="cuda")
    lse[:K] = torch.logsumexp(logits[:K].double() / T, dim=1).float()
    q = torch.empty(B, D, V, device="cuda").normal_(0.0, 0.7, generator=_gen(seed, 41))
    for i in range(B):
        n = int(sel["keep_len"][i]) - 1
        if n > 0:
            q[i, :n] += logits[int(sel["cu"][i]): int(sel["cu"][i]) + n] / T
        q[i] = torch.softmax(q[i], dim=1)
    z = torch.multinomial(q.view(B * D, V), 1, generator=_gen(seed, 42)).view(B, D) if D else None
    draft = torch.zeros(B, D + 1, dtype=torch.int32, device="cuda")
    if D:
        draft[:, 1:] = z.to(torch.int32)
    token = torch.zeros(rows, dtype=torch.int32, device="cuda")
    token[:K] = torch.randint(0, V, (K,), device="cuda", generator=_gen(seed, 43)).to(torch.int32)
    return logits, lse, q, draft, token


def prepare(case, seed):
    kind, B, D = case["kind"], case["B"], case["D"]
    rows = B * (D + 1)
    conf, ctx, draft, budgets, costs, sel = _selection(case, seed)
    i32 = dict(dtype=torch.int32, device="cuda")
    st = dict(case=case, B=B, D=D, conf=_dev(conf), ctx=_dev(ctx), draft=_dev(draft), budgets=budgets, costs=costs,
              err=torch.zeros(1, **i32))
    if kind in ("step", "select"):
        st["sel"] = L.select_outputs(B, D, len(budgets))
    else:
        st["sel"] = {k: _dev(v) for k, v in sel.items()}
    if kind in ("step", "layer"):
        kv = _cache(case, seed, ctx)
        ly = _shape(case)
        st.update(kv=kv, kvd=L.kv_desc(kv), cfg=L.layer_cfg(ly, kv["cap_host"]),
                  w=_weights(case, seed, embed=kind == "step", head=kind == "step"))
        st["lw"] = L.layer_weights(st["w"])
        st["x"] = torch.zeros(rows, case["hidden"], device="cuda")
        st["x_in"] = None if kind == "step" else _normal(
            seed, 31, (rows, case["hidden"]), X_STD_MOE if case["n_exp"] else X_STD, torch.float32)
        st["ws"] = L.workspace(L.workspace_bytes(1, st["cfg"], B, D))
    if kind == "head":
        st["w"] = _weights(case, seed, head=True)
        st["x"] = _head_x(case, seed)
    if kind in ("step", "head"):
        V = case["vocab"]
        hc = L.LayerCfg(hidden=case["hidden"], vocab=V)
        st.update(ws_lm=L.workspace(L.workspace_bytes(2, hc, B, D)), argmax=torch.zeros(rows, **i32),
                  max_logit=torch.zeros(rows, device="cuda"),
                  logits=torch.zeros(rows, V, device="cuda") if case["logits"] else None,
                  lse=torch.zeros(rows, device="cuda") if case["logits"] else None, seed=int(seed) + 5)
    if kind == "accept":
        st["argmax"] = _dev(_accept_argmax(case, seed, sel, draft, conf))
    if kind == "accept_rs":
        st["logits"], st["lse"], st["q"], st["draft"], st["token"] = _proposals(case, seed, sel)
        st["ws"] = L.workspace(L.workspace_bytes(4, L.LayerCfg(vocab=case["vocab"]), B, D))
        st["seed"] = int(seed) + 5
    st.update(accept_len=torch.zeros(B, **i32), next_tok=torch.zeros(B, **i32), total=torch.zeros(1, **i32))
    return st


def _accept_argmax(case, seed, sel, draft, conf):
    """Greedy tokens of the kept rows: the next draft with the probability of its confidence."""
    B, D = case["B"], case["D"]
    rng = np.random.default_rng([int(seed), 23])
    g = rng.integers(0, case["vocab"], size=(B, D + 1)).astype(np.int32)
    hit = rng.random((B, D)) < conf
    g[:, :D] = np.where(hit, draft[:, 1:], g[:, :D])
    out = np.zeros(B * (D + 1), dtype=np.int32)
    for i in range(B):
        out[sel["cu"][i]: sel["cu"][i + 1]] = g[i, : sel["keep_len"][i]]
    return out


# ------------------------------------------------------------------ one pass

def _run_select(st):
    if st["case"].get("rs"):
        L.select_rs(st["B"], st["D"], st["conf"], st["draft"], st["ctx"], L.RS_SCAN, st["budgets"], st["costs"],
                    st["sel"], st["err"])
    else:
        L.select(st["B"], st["D"], st["conf"], st["draft"], st["ctx"], st["budgets"], st["costs"], st["sel"], st["err"])


def _run_layer(st):
    L.verify_layer(st["cfg"], st["lw"], st["B"], st["D"], st["sel"], st["ctx"], st["kvd"], st["x"], st["ws"],
                   x_in=st["x_in"], dev_err=st["err"])


def _run_head(st):
    c, w = st["case"], st["w"]
    if c.get("temperature", 0.0) > 0.0:
        L.lm_head_sample(c["hidden"], c["vocab"], st["B"], st["D"], st["sel"]["cu"], st["sel"]["packed_req"],
                         st["sel"]["packed_pos"], st["x"], w["final_norm"], EPS, w["w_lm"], c["temperature"],
                         st["seed"], st["argmax"], st["ws_lm"], max_score=st["max_logit"], logits=st["logits"],
                         lse=st["lse"])
    else:
        L.lm_head_argmax(c["hidden"], c["vocab"], st["B"], st["D"], st["sel"]["cu"], st["x"], w["final_norm"], EPS,
                         w["w_lm"], st["argmax"], st["ws_lm"], max_logit=st["max_logit"], logits=st["logits"])


def run(st):
    """One pass.  Rows past the kept ones are never written and stay zero."""
    kind = st["case"]["kind"]
    if kind == "select":
        _run_select(st)
        return {k: st["sel"][k] for k in ("keep_len", "cu", "packed_tok", "packed_pos", "packed_req", "choice", "benefit")}
    if kind == "layer":
        _run_layer(st)
        return dict(x=st["x"], new_k=st["kv"]["new_k"], new_v=st["kv"]["new_v"])
    if kind == "head":
        _run_head(st)
        out = dict(token=st["argmax"], max_logit=st["max_logit"])
        if st["logits"] is not None:
            out["logits"] = st["logits"]
            if st["case"]["temperature"] > 0.0:
                out["lse"] = st["lse"]
        return out
    if kind == "accept":
        L.accept(st["B"], st["D"], st["draft"], st["sel"]["keep_len"], st["sel"]["cu"], st["argmax"],
                 st["accept_len"], st["next_tok"], st["total"])
        return dict(accept_len=st["accept_len"], next_tok=st["next_tok"], total=st["total"])
    if kind == "accept_rs":
        c = st["case"]
        L.accept_rs(st["B"], st["D"], c["vocab"], c["temperature"], st["seed"], st["draft"], st["q"],
                    st["sel"]["keep_len"], st["sel"]["cu"], st["sel"]["packed_pos"], st["logits"], st["lse"],
                    st["token"], st["accept_len"], st["next_tok"], st["total"], st["ws"], dev_err=st["err"])
        return dict(accept_len=st["accept_len"], next_tok=st["next_tok"], total=st["total"])
    _run_select(st)
    _run_layer(st)
    _run_head(st)
    L.accept(st["B"], st["D"], st["draft"], st["sel"]["keep_len"], st["sel"]["cu"], st["argmax"],
             st["accept_len"], st["next_tok"], st["total"])
    # the committed next token of a request is the argmax of one of its rows: it is in `token` (or in `logits`)
    out = dict(keep_len=st["sel"]["keep_len"], cu=st["sel"]["cu"], choice=st["sel"]["choice"], x=st["x"],
               new_k=st["kv"]["new_k"], new_v=st["kv"]["new_v"], max_logit=st["max_logit"],
               accept_len=st["accept_len"], total=st["total"])
    if st["logits"] is not None:
        out["logits"] = st["logits"]
    else:
        out["token"] = st["argmax"]
    return out


# ------------------------------------------------------------------ what a pass cannot do without

def _mean_ctx(case):
    lo, hi = case["ctx_lo"], case["ctx_hi"]
    if case.get("ctx_log") and hi > max(lo, 1):
        return (hi - max(lo, 1)) / math.log(hi / max(lo, 1))
    return (lo + hi) / 2


def work(case):
    kind, B, D, K = case["kind"], case["B"], case["D"], case.get("K", 0)
    D1 = D + 1
    by, fl = 0.0, 0.0
    if kind in ("step", "select"):
        n = B * D1
        kept = K if K else n / 2
        by += 4 * B * D + 4 * kept + 4 * B + 12 * kept + 8 * B + 8 * case["R"]
        fl += n * max(1.0, math.log2(n))
    if kind in ("step", "layer"):
        H, hd, nq, nkv = case["hidden"], case["head_dim"], case["n_q"], case["n_kv"]
        keys = B * _mean_ctx(case)
        attn_params = (nq + 2 * nkv) * hd * H + nq * hd * H
        by += 2 * attn_params + 4 * keys * nkv * hd + 4 * K * nkv * hd + 4 * H
        by += K * H * (2 if kind == "step" else 4) + 4 * K * H
        fl += 2 * K * attn_params + 4 * (K / B) * keys * nq * hd
        if case["n_exp"] == 0:
            by += 6 * case["inter"] * H
            fl += 6 * K * case["inter"] * H
        else:
            E, k = case["n_exp"], case["top_k"]
            used = E * (1.0 - (1.0 - k / E) ** K)
            by += 2 * E * H + 6 * used * case["exp_inter"] * H
            fl += 2 * K * E * H + 6 * K * k * case["exp_inter"] * H
    if kind in ("step", "head"):
        H, V = case["hidden"], case["vocab"]
        by += 2 * V * H + (4 * K * H if kind == "head" else 0) + 8 * K + (4 * K * V if case["logits"] else 0)
        fl += 2.0 * K * V * H
    if kind in ("step", "accept"):
        by += 8 * K + 12 * B
        fl += K
    if kind == "accept_rs":
        # about half the requests reject a draft: one row of logits and of proposals each
        V = case["vocab"]
        by += B * 0.5 * 8 * V + 12 * K
        fl += B * 0.5 * 20 * V
    return {"bytes": float(by), "flops": float(fl)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("select", "accept"):
        return "exact"
    if kind == "accept_rs":
        return {"rel": 1e-6, "differ": 0.01}
    if kind == "head":
        # the rows' float32 mean square in another order flips a few bf16 roundings of the normalised
        # rows (2^-9 each, about 1e-5 of them), then float32 sums in another order; tokens at near-ties
        return {"rel": 2e-4, "max": 5e-3, "differ": 0.01}
    if case["n_exp"]:
        # as below, and rows whose last routed expert is a near-tie may take the other one: against
        # float64, where every such row within 1e-3 flips, rel is 0.013
        return {"rel": 2e-2, "max": 0.9, "differ": 0.01}
    # bf16 activations between the GEMMs (2e-3 to 5e-3 against float64): a changed sum order flips
    # roundings that travel on
    return {"rel": 1e-2, "max": 0.3, "differ": 0.01}


# ------------------------------------------------------------------ the same in float64

def _rms(x, gain):
    return x / torch.sqrt((x * x).mean(dim=-1, keepdim=True) + EPS) * gain.double()


def _mm(x, w):
    """x w^T in float64, the weights converted a few thousand rows at a time."""
    return torch.cat([x @ w[r: r + 8192].double().t() for r in range(0, w.shape[0], 8192)], dim=1)


def _rope(x, pos):
    half = x.shape[-1] // 2
    inv = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / x.shape[-1])
    ang = pos.double()[:, None, None] * inv
    c, s = torch.cos(ang), torch.sin(ang)
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _layer64(case, st, sel, x):
    """x [K][H] float64 -> (residual after the layer, new_k, new_v)."""
    H, hd, nq, nkv, B = case["hidden"], case["head_dim"], case["n_q"], case["n_kv"], case["B"]
    K, w, kv, g = x.shape[0], st["w"], st["kv"], nq // nkv
    pos = _dev(sel["packed_pos"][:K])
    qkv = _mm(_rms(x, w["attn_norm"]), w["w_qkv"]).view(K, nq + 2 * nkv, hd)
    q, k, v = _rope(qkv[:, :nq], pos), _rope(qkv[:, nq: nq + nkv], pos), qkv[:, nq + nkv:]
    new_k = torch.zeros(kv["new_k"].shape, dtype=torch.float64, device="cuda")
    new_v = torch.zeros_like(new_k)
    att = torch.empty(K, nq, hd, dtype=torch.float64, device="cuda")
    base, cap, ctx = kv["base"].tolist(), kv["cap_host"], st["ctx"].tolist()
    for i in range(B):
        t0, t1 = int(sel["cu"][i]), int(sel["cu"][i + 1])
        d, n = t1 - t0, ctx[i]
        if d == 0:
            continue
        ki, vi = k[t0:t1].transpose(0, 1), v[t0:t1].transpose(0, 1)
        new_k[i, :, :d], new_v[i, :, :d] = ki, vi
        old = lambda t: t[base[i]: base[i] + nkv * cap * hd].view(nkv, cap, hd)[:, :n].double()
        kk, vv = torch.cat([old(kv["k"]), ki], dim=1), torch.cat([old(kv["v"]), vi], dim=1)
        qi = q[t0:t1].view(d, nkv, g, hd).permute(1, 2, 0, 3).reshape(nkv, g * d, hd)
        s = torch.matmul(qi, kk.transpose(1, 2).contiguous()) / math.sqrt(hd)
        depth = torch.arange(d, device="cuda").repeat(g)
        s = s.masked_fill(torch.arange(n + d, device="cuda")[None, :] > (n + depth)[:, None], -math.inf)
        o = torch.matmul(torch.softmax(s, dim=-1), vv.contiguous())
        att[t0:t1] = o.view(nkv, g, d, hd).permute(2, 0, 1, 3).reshape(d, nq, hd)
    y = x + _mm(att.view(K, nq * hd), w["w_o"])
    h = _rms(y, w["mlp_norm"])
    if case["n_exp"] == 0:
        gu = _mm(h, w["w_gate_up"])
        y = y + _mm(torch.nn.functional.silu(gu[:, : case["inter"]]) * gu[:, case["inter"]:], w["w_down"])
    else:
        top, ids = torch.topk(_mm(h, w["w_router"]), case["top_k"], dim=1)
        wt = torch.softmax(top, dim=1)
        out = torch.zeros_like(y)
        for e in range(case["n_exp"]):
            r, s = (ids == e).nonzero(as_tuple=True)
            if len(r):
                gu = _mm(h[r], w["w_exp_gate_up"][e])
                I = case["exp_inter"]
                out.index_add_(0, r, wt[r, s][:, None] * _mm(torch.nn.functional.silu(gu[:, :I]) * gu[:, I:], w["w_exp_down"][e]))
        y = y + out
    return y, new_k, new_v


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 over int64 tensors holding 32-bit counters: four tensors of 32-bit words."""
    M = 0xFFFFFFFF
    k0, k1 = seed & M, (seed >> 32) & M
    for r in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57      # products wrap in int64; the halves are right
        c0, c1, c2, c3 = ((p1 >> 32) & M) ^ c1 ^ k0, p1 & M, ((p0 >> 32) & M) ^ c3 ^ k1, p0 & M
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c0, c1, c2, c3


def _gumbel(req, pos, V, seed):
    """Gumbel noise of one row's V columns: counter (32 (c >> 7) + (c & 31), pos, req, 0), word (c >> 5) & 3."""
    n = torch.arange((V + 127) // 128 * 32, dtype=torch.int64, device="cuda")
    f = lambda v: torch.full_like(n, int(v))
    w = torch.stack(_philox(n, f(pos), f(req), f(0), seed))             # [4][blocks * 32]
    w = w.view(4, -1, 32).permute(1, 0, 2).reshape(-1)[:V]
    return -torch.log(-torch.log((w.double() + 0.5) / 2.0 ** 32))


def _head64(case, st, sel, x):
    """x [K][H] float64 -> (token, winning value, logits, log-partition)."""
    logits = _mm(_rms(x, st["w"]["final_norm"]), st["w"]["w_lm"])
    T = case.get("temperature", 0.0)
    if T <= 0.0:
        best, tok = logits.max(dim=1)
        return tok, best, logits, None
    tok, best = [], []
    for t in range(x.shape[0]):
        m, c = (logits[t] / T + _gumbel(sel["packed_req"][t], sel["packed_pos"][t], case["vocab"], st["seed"])).max(dim=0)
        tok.append(c)
        best.append(m)
    return torch.stack(tok), torch.stack(best), logits, torch.logsumexp(logits / T, dim=1)


def _rows(t, n):
    """t padded with zero rows to n."""
    return torch.cat([t, torch.zeros(n - t.shape[0], *t.shape[1:], dtype=t.dtype, device=t.device)])


def _accept_np(draft, sel, argmax):
    B = draft.shape[0]
    acc, nxt = np.zeros(B, dtype=np.int32), np.zeros(B, dtype=np.int32)
    for i in range(B):
        c, n = sel["cu"][i], sel["keep_len"][i] - 1
        miss = np.nonzero(draft[i, 1: n + 1] != argmax[c: c + n])[0]
        acc[i] = miss[0] if len(miss) else n
        nxt[i] = argmax[c + acc[i]]
    return acc, nxt, np.array([int((acc + 1).sum())], dtype=np.int32)


def _accept_rs64(case, st, sel):
    B, V, T, seed = case["B"], case["vocab"], case["temperature"], st["seed"]
    acc, nxt = np.zeros(B, dtype=np.int32), np.zeros(B, dtype=np.int32)
    draft, token = st["draft"].cpu().numpy(), st["token"].cpu().numpy()
    one = lambda v: torch.tensor([int(v)], dtype=torch.int64)
    for i in range(B):
        c, n = int(sel["cu"][i]), int(sel["keep_len"][i]) - 1
        for j in range(n):
            r, z = c + j, int(draft[i, j + 1])
            p = math.exp(float(st["logits"][r, z]) / T - float(st["lse"][r]))
            w = int(_philox(one(0), one(sel["packed_pos"][r]), one(i), one(1), seed)[0])
            if not (w + 0.5) / 2.0 ** 32 * float(st["q"][i, j, z]) < p:
                rest = torch.exp(st["logits"][r].double() / T - st["lse"][r].double()) - st["q"][i, j].double()
                score = torch.where(rest > 0, torch.log(rest.clamp_min(1e-300)) + _gumbel(i, sel["packed_pos"][r], V, seed), -math.inf)
                nxt[i] = int(score.argmax()) if bool((rest > 0).any()) else token[r]
                acc[i] = j
                break
        else:
            acc[i], nxt[i] = n, token[c + n]
    return dict(accept_len=acc, next_tok=nxt, total=np.array([int((acc + 1).sum())], dtype=np.int32))


def exact(case, seed):
    kind, rows = case["kind"], case["B"] * (case["D"] + 1)
    conf, ctx, draft, budgets, costs, sel = _selection(case, seed)
    if kind == "select":
        return sel
    if kind == "accept":
        a, n, t = _accept_np(draft, sel, _accept_argmax(case, seed, sel, draft, conf))
        return dict(accept_len=a, next_tok=n, total=t)
    st = prepare(case, seed)
    if kind == "accept_rs":
        return _accept_rs64(case, st, sel)
    K = int(sel["cu"][-1])
    if kind == "head":
        tok, best, logits, lse = _head64(case, st, sel, st["x"][:K].double())
        out = dict(token=_rows(tok.int(), rows), max_logit=_rows(best, rows))
        if case["logits"]:
            out["logits"] = _rows(logits, rows)
            if lse is not None:
                out["lse"] = _rows(lse, rows)
        return out
    x = st["w"]["embed"][_dev(sel["packed_tok"][:K]).long()].double() if kind == "step" else st["x_in"][:K].double()
    x, new_k, new_v = _layer64(case, st, sel, x)
    out = dict(x=_rows(x, rows), new_k=new_k, new_v=new_v)
    if kind == "layer":
        return out
    tok, best, logits, _ = _head64(case, st, sel, x)
    a, _, t = _accept_np(draft, sel, _rows(tok.int(), rows).cpu().numpy())
    out.update(keep_len=sel["keep_len"], cu=sel["cu"], choice=sel["choice"], max_logit=_rows(best, rows),
               accept_len=a, total=t)
    if case["logits"]:
        out["logits"] = _rows(logits, rows)
    else:
        out["token"] = _rows(tok.int(), rows)
    return out
