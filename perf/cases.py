"""The work a user of this library has it do, as cases that can be timed: scoring the keys of a prompt, selecting and
gathering the survivors, projecting the pseudo queries, and decoding over the compact cache.

Every case is one kind of call with its sizes.  The stages of the eviction step are separate cases (a score case ends
with the scores, a select case starts from scores), because the retained positions follow the scores through a
comparison: two correct score passes may differ in the last bits and keep another one of two nearly equal keys, so the
scores have a tolerance while everything from the scores on is exact.

  listed()            the cases that are reported
  draw(rng)           one more case of the same ranges
  prepare(case, seed) what a program holds before the call: tensors, shape descriptor, workspace, output buffers
  run(state)          one pass through the public entry points
  work(case)          bytes and floating-point operations the pass cannot do without
  tolerance(case)     how far two correct results may be apart
"""
import math
import random

import torch

import paper_2603_11564_amd as D

HEAD_DIM = 128
THETA = 500000.0
SCALE = 1.0 / math.sqrt(HEAD_DIM)
POOL_WIDTH = 7


def _score(name, layers, q_heads, kv_heads, n_pseudo, batch, low, high, layout, extended=False):
    """rope of the pseudo queries + scores of every prompt key.  batch prompts of low..high keys each (low == high:
    a dense batch).  layout: "heads" = K as [layer][head][token][d], "tokens" = [layer][token][head][d].  extended: the
    pseudo tokens' own keys are part of the normaliser (three calls instead of one)."""
    return dict(name=name, kind="score", layers=layers, q_heads=q_heads, kv_heads=kv_heads, n_pseudo=n_pseudo,
                batch=batch, low=low, high=high, layout=layout, extended=extended)


def _select(name, layers, kv_heads, batch, low, high, budget, own_budgets, layout):
    """max-pool + top-k + gather of the retained K and V rows.  own_budgets: every prompt has a budget of its own."""
    return dict(name=name, kind="select", layers=layers, kv_heads=kv_heads, batch=batch, low=low, high=high,
                budget=budget, own_budgets=own_budgets, layout=layout)


def _decode(name, layers, batch, q_heads, kv_heads, budget, filled):
    """one decode step over the compact cache.  filled: every head holds `budget` rows; else the prompts of the batch
    kept between a quarter of it and all of it."""
    return dict(name=name, kind="decode", layers=layers, batch=batch, q_heads=q_heads, kv_heads=kv_heads, budget=budget,
                filled=filled)


def _queries(name, layers, batch, n_pseudo, hidden, q_heads, tokens):
    """which prompt tokens the pseudo tokens copy, and their rotated queries out of the layer's query projection."""
    return dict(name=name, kind="queries", layers=layers, batch=batch, n_pseudo=n_pseudo, hidden=hidden, q_heads=q_heads,
                tokens=tokens)


def listed():
    return [
        # a single layer over a short prompt: the smallest call, all latency
        _score("score_layer_1k", 1, 32, 8, 64, 1, 1024, 1024, "heads"),
        # a model that compresses layer by layer while it prefills an 8k prompt (an odd length), window of 32
        _score("score_layer_8k", 1, 32, 8, 32, 1, 8191, 8191, "heads"),
        # the benchmark's workload: all 32 layers of the 8B shape over a 32k prompt
        _score("score_8b_32k", 32, 32, 8, 64, 1, 32768, 32768, "heads"),
        # a packed ragged batch with a long observation window: 512 query rows per KV head
        _score("score_ragged_n128", 32, 32, 8, 128, 8, 4096, 16384, "tokens"),
        # 8 layers of the 70B-class shape over a 128k prompt (8 query heads per KV head)
        _score("score_70b_128k", 8, 64, 8, 64, 1, 131072, 131072, "heads"),
        # a serving batch of short prompts of any length; the pseudo tokens' keys are in the normaliser
        _score("score_extended_short", 32, 32, 8, 32, 16, 200, 2500, "tokens", extended=True),
        # selection and gather of one layer, as after a layer-by-layer score call: 8 heads only
        _select("select_layer_32k", 1, 8, 1, 32768, 32768, 983, False, "heads"),
        # the benchmark's selection and gather
        _select("select_8b_32k", 32, 8, 1, 32768, 32768, 983, False, "heads"),
        # heads longer than one workgroup holds, large budget
        _select("select_70b_128k", 8, 8, 1, 131072, 131072, 3932, False, "heads"),
        # decoding one token: a model calls this once per layer
        _decode("decode_layer", 1, 1, 32, 8, 983, True),
        # decoding one token of each of 50 sequences with a small budget
        _decode("decode_layer_batch", 1, 50, 32, 8, 256, False),
        # the queries of the pseudo tokens of one layer
        _queries("queries_layer", 1, 1, 64, 4096, 32, 8192),
    ]


def _unnamed(case):
    del case["name"]
    return case


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(("score", "score", "score", "select", "select", "decode", "queries"))
    kv_heads = rng.choice((8, 8, 8, 4, 2))
    group = rng.choice((4, 4, 8, 2, 1))
    if kind == "score":
        while True:
            layers = rng.choice((1, 1, 2, 8, 16, 32))
            batch = rng.choice((1, 1, 1, 2, 5, 8, 16))
            high = _log_int(rng, 128, 131072)
            low = high if rng.random() < 0.6 else max(1, high // rng.randint(2, 8))
            n_pseudo = rng.choice((16, 32, 32, 64, 64, 128, 37))
            keys = layers * kv_heads * batch * high
            # no more than the largest listed cases: keys read, and key-row products
            if keys <= 6.7e7 and keys * max(64, group * n_pseudo) <= 8.6e9:
                break
        return _unnamed(_score(None, layers, kv_heads * group, kv_heads, n_pseudo, batch, low, high,
                               rng.choice(("heads", "tokens")), rng.random() < 0.25))
    if kind == "select":
        while True:
            layers = rng.choice((1, 1, 2, 8, 16, 32))
            batch = rng.choice((1, 1, 2, 5, 8))
            high = _log_int(rng, 256, 131072)
            low = high if rng.random() < 0.6 else max(1, high // rng.randint(2, 8))
            budget = min(_log_int(rng, 64, 4096), high)
            # (the candidates of a head of more than 32768 keys: pieces x budget)
            if layers * kv_heads * batch * high <= 8.4e6:
                break
        return _unnamed(_select(None, layers, kv_heads, batch, low, high, budget, batch > 1 and rng.random() < 0.5,
                                rng.choice(("heads", "tokens"))))
    if kind == "decode":
        while True:
            layers, batch, budget = rng.choice((1, 1, 1, 2, 32)), _log_int(rng, 1, 64), _log_int(rng, 64, 4096)
            if layers * batch * kv_heads * budget <= 1 << 20:
                break
        return _unnamed(_decode(None, layers, batch, kv_heads * group, kv_heads, budget, rng.random() < 0.5))
    layers, batch, n_pseudo = rng.choice((1, 1, 1, 2, 8)), rng.choice((1, 1, 2, 4)), rng.choice((16, 32, 64, 37))
    hidden = rng.choice((1024, 2048, 4096, 5120))
    return _unnamed(_queries(None, layers, batch, n_pseudo, hidden, hidden // HEAD_DIM, _log_int(rng, 256, 16384) * batch))


def _lengths(case):
    """Prompt lengths of the batch: part of the case, not of the seed, so that a case is the same amount of work."""
    if case["low"] == case["high"]:
        return [case["high"]] * case["batch"]
    r = random.Random(case["low"] * 1000003 + case["high"])
    return [r.randint(case["low"], case["high"]) for _ in range(case["batch"])]


def _bf16(gen, *shape):
    """N(0, 1) in bf16."""
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)


def _prompt_tensor(case, gen, tokens):
    """Keys or values of all prompts, and the strides (layer, seq, head, token) of the layout."""
    layers, heads = case["layers"], case["kv_heads"]
    if case["layout"] == "heads":
        return _bf16(gen, layers, heads, tokens, HEAD_DIM), (heads * tokens * HEAD_DIM, 0, tokens * HEAD_DIM, HEAD_DIM)
    return _bf16(gen, layers, tokens, heads, HEAD_DIM), (tokens * heads * HEAD_DIM, 0, HEAD_DIM, heads * HEAD_DIM)


def _offsets(case, lengths):
    """cu_seqlens of a ragged batch, None for a dense one."""
    if case["low"] == case["high"]:
        return None
    cu = [0]
    for n in lengths:
        cu.append(cu[-1] + n)
    return torch.tensor(cu, dtype=torch.int32, device="cuda")


def _prepare_score(case, gen):
    layers, q_heads, kv_heads, n, batch = (case[k] for k in ("layers", "q_heads", "kv_heads", "n_pseudo", "batch"))
    lengths = _lengths(case)
    tokens = sum(lengths)
    k, k_strides = _prompt_tensor(case, gen, tokens)
    # a tenth of the keys is long (the heavy hitters of real prompts)
    heavy = torch.rand(k.shape[:3], generator=gen, device="cuda") < 0.1
    k.mul_(torch.where(heavy, 4.0, 1.0).to(torch.bfloat16)[..., None])
    # [layer][head][prompt][row][d]: the rotation is one call for the whole batch
    q_pre = _bf16(gen, layers, q_heads, batch, n, HEAD_DIM)
    s = dict(case=case, k=k, q_pre=q_pre, q=torch.empty_like(q_pre))
    s["positions"] = torch.cat([torch.arange(L, L + n, dtype=torch.int32) for L in lengths]).to("cuda")
    s["shape"] = D.make_shape(n_layers=layers, batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, n_pseudo=n,
                              total_tokens=tokens, cu_seqlens=_offsets(case, lengths), k_strides=k_strides,
                              q_strides=(q_heads * batch * n * HEAD_DIM, n * HEAD_DIM, batch * n * HEAD_DIM, HEAD_DIM),
                              scale=SCALE)
    s["workspace"] = torch.empty(max(D.workspace_bytes(s["shape"]), 256), dtype=torch.uint8, device="cuda")
    s["scores"] = torch.empty((layers, kv_heads, tokens), dtype=torch.float32, device="cuda")
    if case["extended"]:
        s["k_pseudo"] = _bf16(gen, layers, batch, kv_heads, n, HEAD_DIM)
        s["lse2"] = torch.empty((layers, batch, q_heads, n), dtype=torch.float32, device="cuda")
    return s


def _run_score(s):
    c = s["case"]
    rows, row_axis = c["batch"] * c["n_pseudo"], c["batch"] * c["n_pseudo"] * HEAD_DIM
    D.dapq_rope_apply(s["q_pre"], s["q"], s["positions"], rows, c["layers"] * c["q_heads"], HEAD_DIM, HEAD_DIM, row_axis,
                      THETA, 0)
    if not c["extended"]:
        D.dapq_score(s["shape"], s["q"], s["k"], s["scores"], s["workspace"])
        return {"q": s["q"], "scores": s["scores"]}
    n, h = c["n_pseudo"], c["kv_heads"]
    D.dapq_score_stats(s["shape"], s["q"], s["k"], s["lse2"], s["workspace"])
    D.dapq_score_stats_extend(s["shape"], s["q"], s["k_pseudo"],
                              (c["batch"] * h * n * HEAD_DIM, h * n * HEAD_DIM, n * HEAD_DIM, HEAD_DIM), s["lse2"])
    D.dapq_score_accumulate(s["shape"], s["q"], s["k"], s["lse2"], s["scores"], s["workspace"])
    return {"q": s["q"], "lse2": s["lse2"], "scores": s["scores"]}


def _prepare_select(case, gen):
    layers, kv_heads, batch, budget = (case[k] for k in ("layers", "kv_heads", "batch", "budget"))
    lengths = _lengths(case)
    tokens = sum(lengths)
    k, strides = _prompt_tensor(case, gen, tokens)
    v, _ = _prompt_tensor(case, gen, tokens)
    # what a score pass over 256 query rows leaves: most keys within an octave of the mean mass, a tenth of them above
    # it by several times, a few that hold a whole query's mass
    z = torch.randn((layers, kv_heads, tokens), generator=gen, device="cuda")
    u = torch.rand((layers, kv_heads, tokens), generator=gen, device="cuda")
    scores = 256.0 / max(lengths) * torch.exp(0.25 * z) * torch.where(u < 0.1, torch.exp(1.0 + z), 1.0)
    scores += (u > 1.0 - 16.0 / max(lengths)) * u
    s = dict(case=case, k=k, v=v, scores=scores)
    s["shape"] = D.make_shape(n_layers=layers, batch=batch, n_q_heads=kv_heads, n_kv_heads=kv_heads, n_pseudo=1,
                              total_tokens=tokens, cu_seqlens=_offsets(case, lengths), k_strides=strides,
                              v_strides=strides, scale=SCALE)
    n = D.topk_workspace_bytes(s["shape"], budget)
    s["workspace"] = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
    # a head that is neither short enough for one workgroup nor cut in pieces needs the pooled scores as a buffer
    longest = max(lengths) if case["low"] == case["high"] else tokens
    s["pooled"] = torch.empty_like(scores) if longest > 65536 and not n else None
    s["budgets"] = None
    if case["own_budgets"]:
        r = random.Random(budget)
        s["budgets"] = torch.tensor([r.randint(1, budget) for _ in lengths], dtype=torch.int32, device="cuda")
    s["idx"] = torch.zeros((layers, batch, kv_heads, budget), dtype=torch.int32, device="cuda")
    s["count"] = torch.zeros((layers, batch, kv_heads), dtype=torch.int32, device="cuda")
    s["k_out"] = torch.zeros((layers, batch, kv_heads, budget, HEAD_DIM), dtype=torch.bfloat16, device="cuda")
    s["v_out"] = torch.zeros_like(s["k_out"])
    return s


def _run_select(s):
    budget = s["case"]["budget"]
    D.dapq_pool_topk(s["shape"], s["scores"], POOL_WIDTH, budget, s["budgets"], s["idx"], s["count"], s["pooled"],
                     workspace=s["workspace"])
    D.dapq_gather(s["shape"], s["k"], s["v"], s["idx"], s["count"], budget, s["k_out"], s["v_out"])
    return {"idx": s["idx"], "count": s["count"], "k": s["k_out"], "v": s["v_out"]}


def _decode_counts(case):
    if case["filled"]:
        return [case["budget"]] * case["batch"]
    r = random.Random(case["budget"] * 101 + case["batch"])
    return [r.randint(max(1, case["budget"] // 4), case["budget"]) for _ in range(case["batch"])]


def _prepare_decode(case, gen):
    layers, batch, q_heads, kv_heads, budget = (case[k] for k in ("layers", "batch", "q_heads", "kv_heads", "budget"))
    counts = torch.tensor(_decode_counts(case), dtype=torch.int32, device="cuda")
    return dict(case=case, q=_bf16(gen, layers, batch, q_heads, HEAD_DIM),
                k=_bf16(gen, layers, batch, kv_heads, budget, HEAD_DIM), v=_bf16(gen, layers, batch, kv_heads, budget, HEAD_DIM),
                count=counts[None, :, None].expand(layers, batch, kv_heads).contiguous(),
                out=torch.empty((layers, batch, q_heads, HEAD_DIM), dtype=torch.float32, device="cuda"),
                shape=D.make_shape(n_layers=layers, batch=batch, n_q_heads=q_heads, n_kv_heads=kv_heads, n_pseudo=1,
                                   total_tokens=batch, scale=SCALE))


def _run_decode(s):
    D.dapq_decode_attention(s["shape"], s["q"], s["k"], s["v"], s["count"], s["case"]["budget"], s["out"])
    return s["out"]


def _prepare_queries(case, gen):
    layers, batch, n, hidden, q_heads, tokens = (case[k] for k in ("layers", "batch", "n_pseudo", "hidden", "q_heads", "tokens"))
    features, rows = q_heads * HEAD_DIM, batch * n
    desc = D.Qproj(n_layers=layers, rows=rows, hidden=hidden, n_q_heads=q_heads, head_dim=HEAD_DIM, total_tokens=tokens,
                   x_stride_layer=tokens * hidden, x_stride_token=hidden, w_stride_layer=features * hidden,
                   w_stride_row=hidden, q_stride_layer=q_heads * rows * HEAD_DIM, q_stride_head=rows * HEAD_DIM,
                   q_stride_row=HEAD_DIM)
    ints = dict(dtype=torch.int32, device="cuda")
    n_ws = D.pseudo_queries_workspace_bytes(desc)
    return dict(case=case, desc=desc, x=_bf16(gen, layers, tokens, hidden),
                w=_bf16(gen, layers, features, hidden).mul_(1.0 / math.sqrt(hidden)),
                token_idx=torch.empty((batch, n), **ints), positions=torch.empty((batch, n), **ints),
                q=torch.empty((layers, q_heads, rows, HEAD_DIM), dtype=torch.bfloat16, device="cuda"),
                workspace=torch.empty(n_ws, dtype=torch.uint8, device="cuda") if n_ws else None,
                shape=D.make_shape(n_layers=layers, batch=batch, n_q_heads=q_heads, n_kv_heads=q_heads, n_pseudo=n,
                                   total_tokens=tokens, scale=SCALE))


def _run_queries(s):
    first = min(4, s["case"]["n_pseudo"])
    D.dapq_pseudo_tokens(s["shape"], first, s["case"]["n_pseudo"] - first, s["token_idx"], s["positions"])
    D.dapq_pseudo_queries(s["desc"], s["x"], s["token_idx"], s["w"], s["positions"], THETA, 0, s["q"], s["workspace"])
    return {"token_idx": s["token_idx"], "positions": s["positions"], "q": s["q"]}


_PREPARE = {"score": _prepare_score, "select": _prepare_select, "decode": _prepare_decode, "queries": _prepare_queries}
_RUN = {"score": _run_score, "select": _run_select, "decode": _run_decode, "queries": _run_queries}


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return _PREPARE[case["kind"]](case, gen)


def run(state):
    return _RUN[state["case"]["kind"]](state)


def work(case):
    row = 2 * HEAD_DIM  # bytes of one bf16 row
    if case["kind"] == "score":
        keys = case["layers"] * case["kv_heads"] * sum(_lengths(case))
        rows = case["layers"] * case["q_heads"] * case["batch"] * case["n_pseudo"]
        per_key = case["q_heads"] // case["kv_heads"] * case["n_pseudo"]
        own = case["extended"] * case["layers"] * case["batch"] * case["kv_heads"] * case["n_pseudo"]
        return {"bytes": keys * (row + 4) + rows * 2 * row + own * row + case["extended"] * rows * 4,
                "flops": keys * per_key * 2 * HEAD_DIM}
    if case["kind"] == "select":
        heads, lengths = case["layers"] * case["kv_heads"], _lengths(case)
        kept = heads * sum(min(case["budget"], n) for n in lengths)
        return {"bytes": heads * sum(lengths) * 4 + kept * (4 + 4 * row), "flops": heads * sum(lengths) * (POOL_WIDTH - 1)}
    if case["kind"] == "decode":
        held = case["layers"] * case["kv_heads"] * sum(_decode_counts(case))
        heads = case["layers"] * case["batch"] * case["q_heads"]
        return {"bytes": held * 2 * row + heads * (row + 4 * HEAD_DIM),
                "flops": held * (case["q_heads"] // case["kv_heads"]) * 4 * HEAD_DIM}
    features, rows = case["q_heads"] * HEAD_DIM, case["batch"] * case["n_pseudo"]
    return {"bytes": case["layers"] * 2 * (features * case["hidden"] + rows * case["hidden"] + rows * features),
            "flops": case["layers"] * rows * 2 * features * case["hidden"]}


def tolerance(case):
    """About four times the largest distance from float64 evaluations of the listed cases (2-norm, single element)."""
    if case["kind"] == "select":
        return "exact"  # positions are decided by comparisons of the given scores, rows are copied
    if case["kind"] == "score":
        # fp32 sums of exponentials of fp32 logits (bf16 products are exact in fp32): 2.5e-6 and 1.0e-5 seen
        return {"rel": 1e-5, "max": 4e-5}
    if case["kind"] == "decode":
        return {"rel": 1e-6, "max": 1e-5}  # 2.7e-7 and 2.3e-6 seen
    # bf16 results of fp32 sums: an element whose sum sits at a rounding boundary moves by one step of bf16 before the
    # rotation (3.9e-5 and 8.1e-3 seen)
    return {"rel": 1.5e-4, "max": 3e-2}
