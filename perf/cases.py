"""Performance cases of the SentenceKV hot path: what a serving program has the library do, over the sizes it does it at.

  decode      one generated token: skv_decode_step for every layer, one sequence or a ragged batch
  token       one generated token with everything around it: mean-query update, decode step, attention over a resident
              window of recent tokens, merge of the two partial results, for every layer
  chain       the decode step through its four separate calls, the K/V pool in HBM or in pinned host memory
  prefill     one prompt: sentence segmentation and the mean-key table of every layer and head
  importance  one prompt: observation-window importance of every token
  retain      one prompt: top-k of the importance, compaction of the K/V pool, mean keys of the retained tokens

Inputs are synthetic: keys scatter around one centre per sentence, values and queries are normal, sentence lengths follow the
distributions named in a case.
"""
import math
import random

import numpy as np
import torch

import paper_2504_00970_amd as skv

DEV = "cuda:0"
D = 128                                   # head dimension
VOCAB, TERM_MOD = 131072, 20              # token ids; an id divisible by TERM_MOD ends a sentence
MEAN_LENGTH = {"lognormal": 25, "uniform": 24, "geometric": TERM_MOD}
TORCH_TYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
TABLE = {"f32": (4, torch.float32, skv.SKV_F32), "bf16": (2, torch.bfloat16, skv.SKV_BF16),
         "e4m3": (1, torch.uint8, skv.SKV_FP8_E4M3)}

# Largest pools of a case, in tokens x layers: K and V take 4096 bytes per token and layer at 8 bf16 heads.
MOST_DECODE, MOST_PROMPT, MOST_HOST = 1 << 22, 1 << 20, 1 << 16
MOST_BYTES, MOST_FLOPS = 1.7e9, 2.7e11    # what a drawn pass moves and computes: no more than the largest listed ones


def _case(name, kind, **kw):
    c = {"name": name, "kind": kind, "layers": 32, "q_heads": 32, "kv_heads": 8, "dtype": "bf16", "table": "f32", "batch": 1,
         "lengths": "lognormal"}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one layer of a short fp32 context, launched directly
        _case("decode_1x4k_f32", "decode", layers=1, dtype="f32", tokens_min=4096, tokens_max=4096, budget=512, lengths="uniform",
              graph=False),
        # the ordinary decode step: one sequence, 32 layers, recorded once and replayed for every token
        _case("decode_1x32k", "decode", tokens_min=32768, tokens_max=32768, budget=2048, graph=True),
        # a long context: thousands of buckets per head
        _case("decode_1x128k", "decode", tokens_min=131072, tokens_max=131072, budget=2048, graph=True),
        # a chat turn in an eager loop: four calls per layer and token, odd sizes, the smallest mean-key table
        _case("token_1x7351", "token", table="e4m3", tokens_min=7351, tokens_max=7351, budget=1000, window=257),
        # a few users at once, contexts from short to medium, eager loop, reduced table
        _case("decode_6x_ragged", "decode", table="bf16", batch=6, tokens_min=1900, tokens_max=21001, budget=1500, graph=False),
        # a ragged batch on the wide-group geometry
        _case("decode_16x_ragged", "decode", layers=4, q_heads=64, batch=16, tokens_min=8192, tokens_max=65536, budget=2048,
              graph=True),
        # a full serving batch
        _case("decode_64x32k", "decode", layers=2, batch=64, tokens_min=32768, tokens_max=32768, budget=2048, graph=True),
        # the offloaded store: retrieved rows cross PCIe into HBM, then attention over them
        _case("chain_host_32k", "chain", layers=2, tokens_min=32768, tokens_max=32768, budget=2048, pool="host"),
        # a short prompt: launches count
        _case("prefill_1531", "prefill", tokens_min=1531, tokens_max=1531, lengths="geometric"),
        # an ordinary prompt
        _case("prefill_32k", "prefill", tokens_min=32768, tokens_max=32768, lengths="geometric"),
        # which of its tokens matter, and the pool of those that do
        _case("importance_32k", "importance", tokens_min=32768, tokens_max=32768, window=32),
        _case("retain_32k", "retain", tokens_min=32768, tokens_max=32768, keep=4096, lengths="geometric"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: contexts of 1K to 128K tokens, 1 to 64 sequences, budgets of 128 to 8192 tokens."""
    kind = rng.choice(["decode"] * 6 + ["token", "chain", "prefill", "importance", "retain"])
    q_heads = rng.choice([32, 32, 32, 64, 64, 16, 8])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    c = {"kind": kind, "q_heads": q_heads, "kv_heads": 8, "dtype": dtype, "table": rng.choice(["f32", "f32", "bf16", "e4m3"]),
         "batch": 1, "lengths": rng.choice(["lognormal", "lognormal", "uniform", "geometric"])}
    share = 1 if dtype == "bf16" else 2
    if kind == "decode":
        c["batch"] = _log(rng, 1, 64)
        hi = _log(rng, 1024, min(131072, MOST_DECODE // share // c["batch"]))
        lo = hi if rng.random() < 0.3 else _log(rng, max(512, hi // 8), hi)
        c.update(tokens_min=lo, tokens_max=hi, budget=_log(rng, 128, 8192), graph=rng.random() < 0.5)
        most = MOST_DECODE // share // sum(_tokens(c))
    elif kind in ("token", "chain"):
        pool = "host" if kind == "chain" and rng.random() < 0.5 else "hbm"
        t = _log(rng, 1024, MOST_HOST // share if pool == "host" else 131072)
        c.update(tokens_min=t, tokens_max=t, budget=_log(rng, 128, 4096))
        if kind == "token":
            c["window"] = _log(rng, 64, 1024)
        else:
            c["pool"] = pool
        most = (MOST_HOST if pool == "host" else MOST_DECODE) // share // t
    else:
        t = _log(rng, 1024, 131072)
        c.update(tokens_min=t, tokens_max=t)
        if kind == "importance":
            c["window"] = rng.choice([8, 16, 32])
        if kind == "retain":
            c["keep"] = min(_log(rng, 256, 16384), t // 2)
        most = MOST_PROMPT // share // t
    one = work(dict(c, layers=1))
    c["layers"] = max(1, int(min(32, most, MOST_BYTES // one["bytes"], MOST_FLOPS // one["flops"])))
    return c


# ---- inputs ---------------------------------------------------------------------------------------------------------------

def _tokens(c):
    """Context length of each sequence: spread evenly from tokens_min to tokens_max."""
    n, lo, hi = c["batch"], c["tokens_min"], c["tokens_max"]
    return [hi] if n == 1 else [lo + (hi - lo) * i // (n - 1) for i in range(n)]


def _lengths(kind, total, rng):
    """Sentence lengths that add up to `total`; the last one is cut to fit."""
    n = total // 8 + 64
    if kind == "lognormal":
        x = np.clip(np.rint(20.0 * np.exp(0.7 * rng.standard_normal(n))), 3, 120)
    elif kind == "uniform":
        x = rng.integers(8, 41, n)
    else:
        x = rng.geometric(1.0 / TERM_MOD, n)
    x = x.astype(np.int64)
    end = np.cumsum(x)
    k = int(np.searchsorted(end, total))
    x = x[: k + 1]
    x[k] -= int(end[k]) - total
    return x


def _offsets(lengths):
    return np.concatenate([[0], np.cumsum(lengths)])


def _i32(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


def _normal(shape, dtype, gen):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(generator=gen)


def _keys(layers, heads, lengths, dtype, gen):
    """K [layers][heads][T][D]: the sentence's centre + 0.5 * noise."""
    of = torch.repeat_interleave(torch.arange(len(lengths), device=DEV), torch.as_tensor(lengths, device=DEV))
    K = torch.empty(layers, heads, len(of), D, dtype=dtype, device=DEV)
    for l in range(layers):
        for h in range(heads):
            centres = _normal((len(lengths), D), dtype, gen)
            K[l, h].normal_(std=0.5, generator=gen).add_(centres[of])
    return K


def _values(layers, heads, total, dtype, gen):
    V = torch.empty(layers, heads, total, D, dtype=dtype, device=DEV)
    for l in range(layers):
        for h in range(heads):
            V[l, h].normal_(generator=gen)
    return V


def _bitmap():
    """Terminator bitmap of the vocabulary: bit id % 32 of word id // 32."""
    ids = np.arange(0, VOCAB, TERM_MOD)
    words = np.zeros((VOCAB + 31) // 32, dtype=np.uint32)
    np.bitwise_or.at(words, ids // 32, np.uint32(1) << (ids % 32).astype(np.uint32))
    return torch.as_tensor(words.view(np.int32)).to(DEV)


def _token_stream(lengths, rng):
    """Token ids: every sentence but the open last one ends with a terminator, no other token is one."""
    tok = rng.integers(0, VOCAB // TERM_MOD, int(lengths.sum())) * TERM_MOD
    inside = np.ones(len(tok), dtype=bool)
    inside[np.cumsum(lengths)[:-1] - 1] = False
    tok[inside] += rng.integers(1, TERM_MOD, int(inside.sum()))
    return _i32(np.minimum(tok, VOCAB - 1))


class State:
    """What a program holds between calls."""


def prepare(case, seed):
    c, s = case, State()
    s.case = c
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind, L, Hq, H, B, dt = c["kind"], c["layers"], c["q_heads"], c["kv_heads"], c["batch"], TORCH_TYPE[c["dtype"]]
    _, table_type, table_code = TABLE[c["table"]]
    # a case's sentences are always the same ones, so that its shapes are; their order is the seed's
    lens = [rng.permutation(_lengths(c["lengths"], t, np.random.default_rng([t, i]))) for i, t in enumerate(_tokens(c))]
    rng.shuffle(lens)
    flat = np.concatenate(lens)
    s.T, s.S = int(flat.sum()), len(flat)
    budget = c.get("budget", 1)
    s.ctx = skv.Context(skv.Desc(n_layers=L, n_q_heads=Hq, n_kv_heads=H, kv_dtype=skv.dtype_code(dt), max_tokens=s.T,
                                 max_sentences=s.S, max_budget=max(budget, c.get("window", 1)), max_batch=B,
                                 semvec_dtype=table_code))
    if kind in ("prefill", "retain"):
        s.tok, s.bitmap = _token_stream(flat, rng), _bitmap()
        s.seg_id = torch.empty(s.T, dtype=torch.int32, device=DEV)
        s.off, s.len = torch.empty(s.S + 1, dtype=torch.int32, device=DEV), torch.empty(s.S, dtype=torch.int32, device=DEV)
        s.n_sent = torch.empty(4, dtype=torch.int32, device=DEV)
    s.K = _keys(L, H, flat, dt, gen)
    if kind == "prefill":
        return s
    if kind == "importance":
        N = c["window"]
        s.q_obs = _normal((L, Hq, N, D), dt, gen)
        s.alpha = torch.empty(L, s.T - N, device=DEV)
        s.work = torch.empty(s.ctx.token_importance_work_bytes(s.T, N), dtype=torch.uint8, device=DEV)
        return s
    s.V = _values(L, H, s.T, dt, gen)
    if kind == "retain":
        k = c["keep"]
        s.ctx.segment(s.tok, s.bitmap, VOCAB, s.seg_id, s.off, s.len, s.n_sent)
        s.alpha = _normal((L, s.T), torch.float32, gen).mul_(1.5).exp_()          # few tokens hold most of the weight
        s.keep = torch.empty(L, k, dtype=torch.int32, device=DEV)
        s.n_keep = torch.empty(L, dtype=torch.int32, device=DEV)
        s.r_off, s.r_len = (torch.empty(L, s.S + n, dtype=torch.int32, device=DEV) for n in (1, 0))
        s.K_ret, s.V_ret = (torch.empty(L, H, k, D, dtype=dt, device=DEV) for _ in range(2))
        s.table = torch.empty(L, H, s.S, D, dtype=table_type, device=DEV)
        return s

    # decode side: the table comes from the prompt, the queries from the model
    s.table = torch.empty(L, H, s.S, D, dtype=table_type, device=DEV)
    s.ctx.build_semvec(s.K, _i32(_offsets(flat)), s.S, s.table)
    s.cu_tok, s.cu_sent = _i32(_offsets([len_.sum() for len_ in lens])), _i32(_offsets([len(len_) for len_ in lens]))
    s.off, s.len = _i32(np.concatenate([_offsets(len_) for len_ in lens])), _i32(flat)
    s.budget = _i32([budget] * B)
    s.ctx.set_budget_hint(budget)
    q = _normal((L, B, Hq, D), dt, gen)
    s.out, s.lse = torch.zeros(L, B, Hq, D, device=DEV), torch.zeros(L, B, Hq, device=DEV)
    s.q_l, s.out_l, s.lse_l = list(q), list(s.out), list(s.lse)
    if kind == "decode" and c["graph"]:
        s.graph = _record(s)
    elif kind == "token":
        W = c["window"]
        s.tok_t, s.bitmap = _i32(rng.integers(0, VOCAB, 4)), _bitmap()
        s.q_sum, s.q_cnt = torch.zeros(L, B, Hq, D, device=DEV), torch.zeros(L, 4, dtype=torch.int32, device=DEV)
        s.q_bar = torch.zeros(L, B, Hq, D, dtype=dt, device=DEV)
        s.q_sum_l, s.q_cnt_l, s.q_bar_l = list(s.q_sum), list(s.q_cnt), list(s.q_bar)
        s.Kw_l, s.Vw_l = list(_normal((L, H, W, D), dt, gen)), list(_normal((L, H, W, D), dt, gen))
        s.n_win = _i32([W] * H)
        s.out_w, s.lse_w = torch.zeros(Hq, D, device=DEV), torch.zeros(Hq, device=DEV)
        s.out_r, s.lse_r = torch.zeros(Hq, D, device=DEV), torch.zeros(Hq, device=DEV)
    elif kind == "chain":
        if c["pool"] == "host":
            s.K, s.V = (torch.empty(x.shape, dtype=dt, pin_memory=True).copy_(x) for x in (s.K, s.V))
        s.score = torch.zeros(L, H, s.S, device=DEV)
        s.sel = torch.zeros(L, H, s.ctx.desc.max_sel, dtype=torch.int32, device=DEV)
        s.n_sel, s.n_tok = (torch.zeros(L, H, dtype=torch.int32, device=DEV) for _ in range(2))
        s.idx = torch.zeros(L, H, budget, dtype=torch.int32, device=DEV)
        s.K_sel, s.V_sel = (torch.zeros(L, H, budget, D, dtype=dt, device=DEV) for _ in range(2))
        s.per_layer = [list(x) for x in (s.score, s.sel, s.n_sel, s.idx, s.n_tok, s.K_sel, s.V_sel)]
    return s


# ---- passes ---------------------------------------------------------------------------------------------------------------

def _decode_layers(s):
    for l in range(s.case["layers"]):
        s.ctx.decode_step(l, s.case["batch"], s.q_l[l], s.q_l[l], s.K, s.V, s.T, s.table, s.S, s.cu_tok, s.cu_sent, s.off, s.len,
                          s.budget, s.out_l[l], s.lse_l[l])


def _record(s):
    """The launches of one token as a HIP graph."""
    _decode_layers(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.ctx.set_stream(torch.cuda.current_stream().cuda_stream)
        _decode_layers(s)
    s.ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    return g


def run(state):
    s, c = state, state.case
    kind, L = c["kind"], c["layers"]
    if kind == "decode":
        if c["graph"]:
            s.graph.replay()
        else:
            _decode_layers(s)
        return s.out, s.lse
    if kind == "token":
        for l in range(L):
            s.ctx.query_update(1, s.q_l[l], s.tok_t, s.bitmap, VOCAB, s.q_sum_l[l], s.q_cnt_l[l], s.q_bar_l[l])
            s.ctx.decode_step(l, 1, s.q_bar_l[l], s.q_l[l], s.K, s.V, s.T, s.table, s.S, s.cu_tok, s.cu_sent, s.off, s.len,
                              s.budget, s.out_r, s.lse_r)
            s.ctx.attend(s.q_l[l], s.Kw_l[l], s.Vw_l[l], s.n_win, c["window"], s.out_w, s.lse_w)
            s.ctx.merge_lse(c["q_heads"], s.out_r, s.lse_r, s.out_w, s.lse_w, s.out_l[l], s.lse_l[l])
        return s.out, s.lse, s.q_sum, s.q_cnt, s.q_bar
    if kind == "chain":
        for l, (score, sel, n_sel, idx, n_tok, K_sel, V_sel) in enumerate(zip(*s.per_layer)):
            s.ctx.score(l, s.q_l[l], s.table, s.S, score)
            s.ctx.select(score, s.off, s.len, s.S, c["budget"], sel, n_sel, idx, n_tok)
            s.ctx.gather(l, s.K, s.V, s.T, idx, n_tok, c["budget"], K_sel, V_sel, pool_in_host=c["pool"] == "host")
            s.ctx.attend(s.q_l[l], K_sel, V_sel, n_tok, c["budget"], s.out_l[l], s.lse_l[l])
        return s.score, s.sel, s.n_sel, s.idx, s.n_tok, s.K_sel, s.V_sel, s.out, s.lse
    if kind == "prefill":
        # the number of sentences shapes the table
        S = s.ctx.segment(s.tok, s.bitmap, VOCAB, s.seg_id, s.off, s.len, s.n_sent)
        table = torch.empty(L, c["kv_heads"], S, D, dtype=TABLE[c["table"]][1], device=DEV)
        s.ctx.build_semvec(s.K, s.off, S, table)
        return s.seg_id, s.off, s.len, table
    if kind == "importance":
        s.ctx.token_importance(s.q_obs, s.K, s.T, c["window"], s.alpha, s.work)
        return s.alpha
    s.ctx.retain(s.alpha, s.T, c["keep"], s.seg_id, s.S, s.keep, s.n_keep, s.r_off, s.r_len)
    s.ctx.compact_pool(s.K, s.V, s.T, s.keep, c["keep"], s.n_keep, s.K_ret, s.V_ret)
    s.ctx.build_semvec_layers(s.K_ret, s.r_off, s.S, s.table)
    return s.keep, s.n_keep, s.r_off, s.r_len, s.K_ret, s.V_ret, s.table


# ---- what a pass cannot do without ------------------------------------------------------------------------------------------

def work(case):
    c = case
    kind, L, Hq, H, e = c["kind"], c["layers"], c["q_heads"], c["kv_heads"], 4 if c["dtype"] == "f32" else 2
    T = _tokens(c)
    total, S = sum(T), sum(T) // MEAN_LENGTH[c["lengths"]] + 1
    table, pool = H * S * D * TABLE[c["table"]][0], H * total * D * e          # one layer
    if kind == "prefill":
        return {"bytes": L * (pool + table) + 8 * total + 8 * S, "flops": L * H * total * D}
    if kind == "importance":
        N = c["window"]
        return {"bytes": L * (pool + Hq * N * D * e + 4 * total), "flops": L * Hq * N * total * D * 2}
    if kind == "retain":
        k = c["keep"]
        return {"bytes": L * (4 * total + 4 * k + 8 * S + 4 * H * k * D * e + table) + 4 * total, "flops": L * H * k * D}
    rows = sum(min(c["budget"], t) for t in T) * H                             # retrieved rows of K (and of V) per layer
    heads = c["batch"] * Hq * D
    bytes_, flops = table + 8 * S + 2 * rows * D * e + heads * (e + 4), 2 * H * S * D + 4 * rows * (Hq // H) * D
    if kind == "token":
        bytes_ += 2 * H * c["window"] * D * e + heads * (2 * 4 + e)
        flops += 4 * Hq * c["window"] * D
    elif kind == "chain":
        bytes_ += 4 * H * S + 4 * rows + 2 * rows * D * e
    return {"bytes": L * bytes_, "flops": L * flops}


def tolerance(case):
    """bf16 attention rounds its weights to bf16; a selection can differ where two scores agree to the last bits."""
    kind, reduced = case["kind"], case["table"] != "f32"
    if kind in ("decode", "token", "chain"):
        return {"rel": 1e-2 if case["dtype"] == "bf16" else 2e-5, "differ": 0.01}
    if kind == "importance":
        return {"rel": 5e-5}
    # means are fp32 sums, rounded once to the table's type: a neighbouring value of the type now and then
    return {"rel": 2e-3 if reduced else 1e-5, "differ": 0.01 if case["table"] == "e4m3" else 0.0}
