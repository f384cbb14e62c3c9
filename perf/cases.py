"""The calls this library is measured by: what programs that compress a KV cache at prefill time and
generate over the compressed cache have it do, through the public entry points.

A case is a dict of plain values.  ``kind`` is "compress" or "decode".

compress   Section 2.2 of the paper for ``groups`` layer groups of ``gamma`` layers: sequences of
           ``lens`` tokens with windows of ``wins`` tokens (one number a sequence), ``budget`` of the
           prefix kept, by one of these calls (``call``):
             group    wkv_compress_group, one layer group at a time, as prefill reaches it
             groups   wkv_compress_groups, all groups of a model at once
             stages   wkv_score, wkv_window_pool, wkv_topk_windows, then wkv_gather_group layer by layer
           ``lse``: the prefill attention hands its softmax normalisers over.  ``pyramid``: the groups
           have budgets of their own (Eq. 5-7).  ``keep_padding``: compact rows past n_keep are left
           alone.  ``layout``: "bhtd" or "bthd", the order of the axes of the full caches.
decode     one generated token through ``layers`` layers over compact caches of ``rows`` retained rows
           (one number a sequence) with room for 256 tokens more.  The row counters stay as they
           are (WKV_DECODE_KEEP_COUNT), so that the same step can be run again.  ``static``: the entry
           point that takes no workspace.

Shapes are those of the workloads in ``wkv_synth`` and of the head layouts that the tests run.
"""
import math

import torch

import paper_2503_17922_amd as W
import wkv_synth as S

_TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
_WKV = {"bf16": W.WKV_BF16, "f16": W.WKV_F16, "f32": W.WKV_F32}
_ROOM = 256              # rows a decode cache has for tokens to come
_PYRAMID_LAMBDA = 2.0    # Eq. 6: the first group keeps 1.5 times the mean, the last half of it


def _ints(text):
    return [int(x) for x in str(text).split()]


def _text(xs):
    return " ".join(str(x) for x in xs)


def _compress(name, lens, wins, **kw):
    c = dict(name=name, kind="compress", call="groups", dtype="bf16", groups=8, gamma=4, q_heads=32, kv_heads=8,
             head_dim=128, w_obs=32, lens=_text(lens), wins=_text(wins), budget=0.125, lse=False, pyramid=False,
             keep_padding=False, layout="bhtd")
    c.update(kw)
    return c


def _decode(name, rows, **kw):
    c = dict(name=name, kind="decode", dtype="bf16", layers=4, q_heads=32, kv_heads=8, head_dim=128, rows=_text(rows),
             layout="bhtd", static=False)
    c.update(kw)
    return c


def _mixed_batch():
    w = S.make_workload("c5")
    return w.seq_len, w.win


def listed():
    lens, wins = _mixed_batch()
    return [
        # the smallest call: a short prompt of a small model in fp32; launches and host work are all there is
        _compress("group_tiny_f32", [512], [8], call="group", dtype="f32", groups=1, gamma=2, q_heads=4, kv_heads=2,
                  head_dim=64, w_obs=8),
        # one layer group of a LLaMA-3-8B shaped model at an ordinary prompt length, localisation windows
        _compress("group_4k", [4096], [8], call="group", groups=1),
        # the same at a long prompt with aggregation windows
        _compress("group_16k_agg", [16384], [32], call="group", groups=1),
        # fp32 tensors (a reference run, or a model kept in fp32), stage by stage, each layer gathered as it is produced
        _compress("stages_4k_f32", [4096], [16], call="stages", dtype="f32", groups=1),
        # a whole model's prefill of 32K tokens: the benchmark's workload
        _compress("model_32k", [32768], [16]),
        # the same where the attention kernel kept the normalisers of the observation rows
        _compress("model_32k_lse", [32768], [16], lse=True),
        # eight query heads to a KV head (70B-class head layout), budgets per group, an odd length
        _compress("model_16k_64q", [16381], [16], q_heads=64, pyramid=True),
        # a serving batch of mixed lengths and task modes: the largest call
        _compress("batch_mixed", lens, wins, budget=0.12),
        # half-precision tensors in token-major layout, seven query heads to a KV head, odd lengths and a window size
        # that is no power of two; padding is left alone, as the decode step never reads it
        _compress("batch_ragged_f16", [9973, 2051, 5003], [24, 8, 24], dtype="f16", groups=4, gamma=2, q_heads=28,
                  kv_heads=4, budget=0.12, keep_padding=True, layout="bthd"),
        # generation for one user: a token through all 32 layers, bound by latency
        _decode("decode_1", [4128], layers=32),
        # generation at full batch: the layers of one group
        _decode("decode_64", [4128] * 64),
        # generation after prompts of mixed lengths, half precision, seven query heads to a KV head
        _decode("decode_mixed_f16", [3703, 541, 1288, 2017, 640, 3011, 905, 1776, 2560, 777, 1431], dtype="f16", q_heads=28,
                kv_heads=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = [(32, 8), (32, 8), (64, 8), (28, 4), (12, 2), (32, 32)]


def _draw_compress(rng):
    q, kv = rng.choice(_HEADS)
    call = rng.choice(["group", "groups", "groups", "stages"])
    groups = rng.choice([2, 4, 8]) if call == "groups" else 1
    batch = _log(rng, 1, 8)
    longest = _log(rng, 512, 32768)
    lens = [longest] + [_log(rng, max(512, longest // 8), longest) for _ in range(batch - 1)]
    sizes = rng.choice([[8, 32], [8, 32], [16], [64, 16], [24, 12]])
    w_obs = rng.choice([32, 32, 16, 8])
    return dict(kind="compress", call=call, dtype=rng.choice(["bf16"] * 6 + ["f16"] * 3 + ["f32"]), groups=groups,
                gamma=rng.choice([1, 2, 4]), q_heads=q, kv_heads=kv, head_dim=rng.choice([64, 128, 128]), w_obs=w_obs,
                lens=_text(lens), wins=_text(rng.choice(sizes) for _ in lens), budget=rng.choice([0.12, 0.125, 0.25]),
                lse=rng.random() < 0.2, pyramid=groups > 1 and rng.random() < 0.3, keep_padding=rng.random() < 0.4,
                layout=rng.choice(["bhtd", "bhtd", "bthd"]))


def _draw_decode(rng):
    q, kv = rng.choice(_HEADS)
    batch = _log(rng, 1, 64)
    longest = _log(rng, 64, 32768)
    rows = [longest] + [_log(rng, max(64, longest // 8), longest) for _ in range(batch - 1)]
    return dict(kind="decode", dtype=rng.choice(["bf16"] * 6 + ["f16"] * 3 + ["f32"]), layers=rng.choice([1, 4, 32]), q_heads=q,
                kv_heads=kv, head_dim=rng.choice([64, 128, 128]), rows=_text(rows), layout=rng.choice(["bhtd", "bhtd", "bthd"]),
                static=rng.random() < 0.25)


def draw(rng):
    """One more case of the same ranges, no dearer than the largest listed one."""
    largest = next(c for c in listed() if c["name"] == "batch_mixed")
    top, room = work(largest), _tensor_bytes(largest)
    while True:
        case = _draw_decode(rng) if rng.random() < 0.35 else _draw_compress(rng)
        w = work(case)
        flops = w["flops"] * (32 if case["dtype"] == "f32" else 1)       # fp32 inputs have no matrix instructions at that rate
        if w["bytes"] <= top["bytes"] and flops <= top["flops"] and _tensor_bytes(case) <= room:
            return case


# ---- sizes ---------------------------------------------------------------------------------------
def _esize(case):
    return 4 if case["dtype"] == "f32" else 2


def _budgets(case):
    """(windows to keep per group and sequence, windows the outputs have room for per sequence)"""
    lens, wins, n = _ints(case["lens"]), _ints(case["wins"]), case["groups"]
    per_group = [[0] * len(lens) for _ in range(n)]
    for b, (L, win) in enumerate(zip(lens, wins)):
        tokens = case["budget"] * L
        of_group = W.wkv_group_budgets(tokens * n, n, _PYRAMID_LAMBDA) if case["pyramid"] else [tokens] * n
        for g in range(n):
            per_group[g][b] = max(1, int(of_group[g]) // win)
    return per_group, [max(k[b] for k in per_group) for b in range(len(lens))]


def _kept_rows(case):
    """Rows kept per KV head, over all groups and sequences, and the rows of a compact cache."""
    per_group, most = _budgets(case)
    wins = _ints(case["wins"])
    kept = sum(k * win + case["w_obs"] for ks in per_group for k, win in zip(ks, wins))
    return kept, max(k * win for k, win in zip(most, wins)) + case["w_obs"]


def _tensor_bytes(case):
    row = case["kv_heads"] * case["head_dim"] * _esize(case)
    if case["kind"] == "decode":
        rows = _ints(case["rows"])
        return 2 * case["layers"] * len(rows) * (max(rows) + _ROOM) * row
    lens = _ints(case["lens"])
    return 2 * case["groups"] * case["gamma"] * len(lens) * (max(lens) + _kept_rows(case)[1]) * row


def work(case):
    e, d, hq, hkv = _esize(case), case["head_dim"], case["q_heads"], case["kv_heads"]
    if case["kind"] == "decode":
        rows = _ints(case["rows"])
        # every retained row of K and V once; the new rows read and appended; queries in, fp32 outputs out
        cache = 2 * sum(rows) * hkv * d * e
        new = len(rows) * (4 * hkv * d * e + hq * d * (e + 4))
        return {"bytes": case["layers"] * (cache + new), "flops": case["layers"] * 4 * (sum(rows) + len(rows)) * hq * d}
    lens = _ints(case["lens"])
    kept, nk = _kept_rows(case)
    row, layers = hkv * d * e, case["groups"] * case["gamma"]
    scored = case["groups"] * (sum(lens) * row + len(lens) * hq * case["w_obs"] * d * e)
    # K of a group's first layer has been read for the scores; every other tensor gives its kept rows
    read = kept * row * (2 * case["gamma"] - 1)
    written = kept * row * 2 * case["gamma"] if case["keep_padding"] else 2 * layers * len(lens) * nk * row
    index = 4 * case["groups"] * len(lens) * hkv * nk
    return {"bytes": scored + read + written + index,
            "flops": 2 * hq * case["w_obs"] * d * sum(lens) * case["groups"]}


def tolerance(case):
    # Selections are whole numbers and the compact caches are copies of rows; token and window scores (the
    # stage calls return them) and the decode step's output are sums in fp32.
    return {"rel": 1e-5} if case["kind"] == "decode" or case["call"] == "stages" else "exact"


# ---- inputs --------------------------------------------------------------------------------------
def _rand(gen, dtype, *shape):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(generator=gen)


def _cache(gen, dtype, layout, b, h, t, d):
    """A [b, h, t, d] view of normal values, laid out as `layout` says."""
    if layout == "bthd":
        return _rand(gen, dtype, b, t, h, d).transpose(1, 2)
    return _rand(gen, dtype, b, h, t, d)


def _strides(layout, h, t, d):
    return (t * h * d, d, h * d) if layout == "bthd" else (h * t * d, t * d, d)


def _plant(gen, k, u, lens, wins, n_windows, w_obs):
    """Attention of the observation queries goes to passages of the prompt that concern them: in as many
    windows of every KV head as the budget keeps, the keys lie along the queries' common direction u
    [B, H, d] (cosine 0.6 to 0.9).  The other windows score well below these, so that no selection hangs
    on the rounding of a sum."""
    heads, d = k.shape[1], k.shape[3]
    hh = torch.arange(heads, device="cuda")[:, None]
    for b, (L, win, n) in enumerate(zip(lens, wins, n_windows)):
        w = torch.rand((heads, (L - w_obs) // win), device="cuda", generator=gen).topk(n, dim=1).indices
        tok = (w[:, :, None] * win + torch.arange(win, device="cuda")).reshape(heads, -1)
        c = (0.6 + 0.3 * torch.rand((heads, n), device="cuda", generator=gen)).repeat_interleave(win, dim=1)[..., None]
        kb = k[b]
        kb[hh, tok] = (c * math.sqrt(d) * u[b][:, None] + (1 - c * c).sqrt() * kb[hh, tok].float()).to(k.dtype)


def _normalisers(q, k, lens, w_obs):
    """ln sum exp over the visible keys of every observation row, float32 [B, Hq, w_obs]."""
    B, hq, _, d = q.shape
    hkv = k.shape[1]
    g = hq // hkv
    out = torch.empty((B, hq, w_obs), dtype=torch.float32, device="cuda")
    for b, L in enumerate(lens):
        hidden = torch.arange(L, device="cuda")[None] > (L - w_obs + torch.arange(w_obs, device="cuda"))[:, None]
        for h in range(hkv):
            keys = k[b, h, :L].float().t().contiguous()
            x = (q[b, h * g:(h + 1) * g].float().reshape(g * w_obs, d) @ keys) / math.sqrt(d)
            x = x.view(g, w_obs, L).masked_fill_(hidden, -math.inf)
            out[b, h * g:(h + 1) * g] = torch.logsumexp(x, dim=-1)
    return out


def _prepare_compress(case, gen):
    dt, lens, wins = _TORCH[case["dtype"]], _ints(case["lens"]), _ints(case["wins"])
    B, hq, hkv, d, w_obs = len(lens), case["q_heads"], case["kv_heads"], case["head_dim"], case["w_obs"]
    n_groups, gamma, T = case["groups"], case["gamma"], max(lens)
    per_group, most = _budgets(case)
    # localisation keeps the mean of a window of 8, aggregation the upper half of a larger one
    problem = W.Problem(n_q_heads=hq, n_kv_heads=hkv, head_dim=d, w_obs=w_obs, seq_len=lens, win=wins,
                        top_p=[w if w == 8 else w // 2 for w in wins], k_windows=most, dtype=_WKV[case["dtype"]],
                        kv_strides=_strides(case["layout"], hkv, T, d),
                        flags=W.WKV_KEEP_PADDING if case["keep_padding"] else 0)
    dims = W.wkv_get_dims(problem)
    q, k, v, lse = [], [], [], []
    for layer in range(n_groups * gamma):
        k.append(_cache(gen, dt, case["layout"], B, hkv, T, d))
        v.append(_cache(gen, dt, case["layout"], B, hkv, T, d))
        if layer % gamma == 0:
            u = torch.nn.functional.normalize(_rand(gen, torch.float32, B, hkv, d), dim=-1)
            x = _rand(gen, torch.float32, B, hq, w_obs, d)
            x += 0.35 * math.sqrt(d) * u.repeat_interleave(hq // hkv, dim=1)[:, :, None]
            q.append(x.to(dt))
            _plant(gen, k[-1], u, lens, wins, per_group[layer // gamma], w_obs)
            if case["lse"]:
                lse.append(_normalisers(q[-1], k[-1], lens, w_obs))
    nk = dims.nkeep_max
    cache = torch.zeros((n_groups * gamma, 2, B, hkv, nk, d), dtype=dt, device="cuda")
    out = {"cache": cache, "win_idx": torch.zeros((n_groups, B, hkv, dims.k_max), dtype=torch.int32, device="cuda"),
           "tok_idx": torch.zeros((n_groups, B, hkv, nk), dtype=torch.int32, device="cuda"),
           "n_keep": torch.zeros((n_groups, B, hkv), dtype=torch.int32, device="cuda")}
    if case["call"] == "stages":
        out["t"] = torch.zeros((B, hkv, dims.t_stride), dtype=torch.float32, device="cuda")
        out["s"] = torch.zeros((B, hkv, dims.nw_max), dtype=torch.float32, device="cuda")
    ws = torch.empty(W.wkv_workspace_bytes(problem, n_groups), dtype=torch.uint8, device="cuda")
    return dict(case=case, problem=problem, q=q, k=k, v=v, lse=lse or None, k_out=[c[0] for c in cache], v_out=[c[1] for c in cache],
                out=out, ws=ws, per_group=per_group if case["pyramid"] else None)


def _prepare_decode(case, gen):
    dt, rows, layers = _TORCH[case["dtype"]], _ints(case["rows"]), case["layers"]
    B, hq, hkv, d = len(rows), case["q_heads"], case["kv_heads"], case["head_dim"]
    cap = max(rows) + _ROOM
    shape = W.DecodeShape(batch=B, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype=_WKV[case["dtype"]], capacity=cap,
                          cache_strides=_strides(case["layout"], hkv, cap, d), flags=W.WKV_DECODE_KEEP_COUNT)
    n_valid = torch.tensor(rows, dtype=torch.int32, device="cuda")[:, None].repeat(1, hkv).contiguous()
    cache = _cache(gen, dt, case["layout"], layers * 2 * B, hkv, cap, d).unflatten(0, (layers, 2, B))
    q = (2 * _rand(gen, torch.float32, layers, B, hq, d)).to(dt)          # logits of standard deviation 2
    new = _rand(gen, dt, layers, 2, B, hkv, d)
    out = torch.zeros((layers, B, hq, d), dtype=torch.float32, device="cuda")
    ws = None if case["static"] else torch.empty(W.wkv_decode_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    steps = [(q[i], new[i, 0], new[i, 1], cache[i, 0], cache[i, 1], n_valid, out[i]) for i in range(layers)]
    return dict(case=case, shape=shape, steps=steps, ws=ws, out={"out": out, "cache": cache, "n_valid": n_valid})


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return _prepare_decode(case, gen) if case["kind"] == "decode" else _prepare_compress(case, gen)


# ---- one pass ------------------------------------------------------------------------------------
def run(state):
    case, out, ws = state["case"], state["out"], state["ws"]
    if case["kind"] == "decode":
        for step in state["steps"]:
            if case["static"]:
                W.wkv_decode_step_static(state["shape"], *step)
            else:
                W.wkv_decode_step(state["shape"], *step, ws)
        return out
    problem, q, k, v, lse = state["problem"], state["q"], state["k"], state["v"], state["lse"]
    idx = (out["win_idx"], out["tok_idx"], out["n_keep"])
    if case["call"] == "groups":
        W.wkv_compress_groups(problem, case["groups"], case["gamma"], q, lse, k, v, state["k_out"], state["v_out"], *idx, ws,
                              k_windows_groups=state["per_group"])
    elif case["call"] == "group":
        W.wkv_compress_group(problem, case["gamma"], q[0], lse[0] if lse else None, k, v, state["k_out"], state["v_out"], *idx, ws)
    else:
        W.wkv_score(problem, q[0], k[0], lse[0] if lse else None, out["t"], ws)
        W.wkv_window_pool(problem, out["t"], out["s"])
        W.wkv_topk_windows(problem, out["s"], *idx)
        for i in range(case["gamma"]):
            W.wkv_gather_group(problem, k[i:i + 1], v[i:i + 1], out["tok_idx"], out["n_keep"], state["k_out"][i:i + 1],
                               state["v_out"][i:i + 1])
    return out
