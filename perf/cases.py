"""The work a user of this library has it do, as cases that can be timed and compared.

Four kinds of pass, each through the public entry points of paper_2510_07651_amd.binding:

  score       obc_score of one layer: the W window queries against the whole cache (prefill).
  evict       selection on scores at hand, then compaction of K and V (the cache manager's side).
  decode      one generated token through `layers` layers: the token's K/V rows are appended, its query accumulates
              scores and every head drops one token in place (one call per layer, or the three it stands for).
  accumulate  obc_score_accumulate of one query row over a long cache (decoding between two evictions).

A score case and the eviction that follows it are separate passes because selection turns a difference in the last
bit of a score near the budget into a shifted index list: each of them can be compared, their chain cannot.
Programs keep their workspaces and output buffers, so `prepare` makes those; lengths are passed on every call.
Inputs are random with the structure long contexts show: a few large key channels, sink tokens whose keys point along
the mean query, and keys that repeat a window query (needles).
"""
import math

import torch

from paper_2510_07651_amd import binding as obc

DEVICE = "cuda"
DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}
SINKS = 4
POOL = 5               # SnapKV's pooling width
NEEDLES = 64
RING = 61              # different tokens a decoding state cycles through


def _score(name, **kw):
    c = dict(name=name, kind="score", dtype="bf16", B=1, Hq=32, Hkv=8, d=128, N=8192, W=32, variant="joint",
             ragged=False, needles=False)
    c.update(kw)
    return c


def _evict(name, **kw):
    c = dict(name=name, kind="evict", dtype="bf16", B=1, Hkv=8, d=128, N=32768, budget=2048, mode="top", ragged=False)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest prefill call: one fp32 head, 512 tokens, every score.  Launches and the host path.
        _score("score_fp32_1head_512", dtype="fp32", Hq=1, Hkv=1, d=64, N=512, W=16, variant="all"),
        # An ordinary prompt of one Llama-3.1-8B-shaped layer, all three scores at once.
        _score("score_llama_8k_all", N=8192, variant="all"),
        # The benchmark's workload: the same layer, four prompts of 32K.
        _score("score_llama_b4_32k", B=4, N=32768),
        # A Qwen2.5-7B-shaped layer at its longest context: 448 window rows per KV head, needles in the haystack.
        _score("score_qwen_128k_all", Hq=28, Hkv=4, N=131072, W=64, variant="all", needles=True),
        # Prompts of different lengths in one padded batch (one layer of the 32-layer sweep).
        _score("score_llama_ragged_64k", B=2, N=65536, ragged=True),
        # Models kept in fp32, with a length that is no multiple of anything.
        _score("score_fp32_8k_odd", dtype="fp32", N=8111),
        # Small models have heads of 64 channels.
        _score("score_bf16_d64_16k", d=64, N=16384),
        # The eviction that follows the benchmark's scoring call.
        _evict("evict_top_b4_32k", B=4),
        # SnapKV's eviction (pooled scores, sinks and the recent window kept) of very long heads.
        _evict("evict_pooled_128k", Hkv=4, N=131072, budget=4096, mode="pooled"),
        # AdaKV's eviction: one budget ranked over all heads of a layer, ragged prompts.
        _evict("evict_adaptive_ragged_24k", B=2, N=24001, budget=1024, mode="adaptive", ragged=True),
        # Generating with a budget of 1024 tokens: one token through 32 layers, an eviction in each.
        dict(name="decode_1k_32layers", kind="decode", dtype="bf16", B=1, Hq=32, Hkv=8, d=128, N=1025, layers=32,
             variant="joint", calls="one"),
        # Generating on the full cache, scores kept up to date for a later eviction.
        dict(name="accumulate_b4_32k", kind="accumulate", dtype="bf16", B=4, Hq=32, Hkv=8, d=128, N=32768,
             variant="joint", ragged=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# (query heads per KV head, KV heads): multi-head, Llama-like, Qwen-like and wide groups
_HEADS = [(1, 8), (1, 32), (2, 8), (4, 8), (7, 4), (8, 4), (8, 8)]


def draw(rng):
    kind = rng.choice(["score"] * 5 + ["evict"] * 3 + ["decode"] * 2 + ["accumulate"])
    G, Hkv = rng.choice(_HEADS)
    if kind == "score":
        dtype, d = rng.choice([("bf16", 128)] * 4 + [("bf16", 64), ("fp32", 128), ("fp32", 64)])
        W = _log_int(rng, 8, 64)
        # (longest cache, most (window row, token) pairs, most tokens over all KV heads), within the listed cases
        top, pairs, tokens = ((131072, 1 << 27, 1 << 20) if (dtype, d) == ("bf16", 128) else
                              (16384, 1 << 24, 1 << 18) if dtype == "bf16" else (8192, 8000000, 1 << 18))
        N = max(W, min(_log_int(rng, 512, top), pairs // (G * Hkv * W), tokens // Hkv))
        B = rng.randint(1, max(1, min(4, pairs // (G * Hkv * W * N), tokens // (Hkv * N))))
        return dict(kind=kind, dtype=dtype, B=B, Hq=G * Hkv, Hkv=Hkv, d=d, N=N, W=W,
                    variant=rng.choice(["joint", "joint", "key", "value", "all", "attn", "vatp"]),
                    ragged=B > 1 and rng.random() < 0.5, needles=N >= 4096 and rng.random() < 0.3)
    if kind == "evict":
        Hkv = min(Hkv, 8)
        N = _log_int(rng, 1024, 131072)
        B = rng.randint(1, max(1, min(4, (1 << 20) // (Hkv * N))))
        mode = rng.choice(["top", "protected", "pooled", "adaptive"])
        # an eighth at most: the adaptive output is padded to the most one head may get, Hkv times as much
        budget = max(64, min(4096, int(N * rng.uniform(0.02, 0.12))))
        return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "fp32"]), B=B, Hkv=Hkv, d=rng.choice([128, 128, 64]), N=N,
                    budget=budget, mode=mode, ragged=B > 1 and rng.random() < 0.5)
    d = rng.choice([128, 128, 64])
    variant = rng.choice(["joint", "joint", "key", "value", "attn"])
    Hkv = min(Hkv, 8)
    if kind == "decode":
        N = _log_int(rng, 320, 4096)
        B = rng.randint(1, max(1, min(8, 4096 // N)))
        return dict(kind=kind, dtype="bf16", B=B, Hq=G * Hkv, Hkv=Hkv, d=d, N=N, layers=rng.choice([4, 8, 16]),
                    variant=variant, calls=rng.choice(["one", "one", "three"]))
    N = _log_int(rng, 2048, 65536)
    B = rng.randint(1, max(1, min(8, (1 << 20) // (Hkv * N))))
    return dict(kind=kind, dtype="bf16", B=B, Hq=G * Hkv, Hkv=Hkv, d=d, N=N, variant=variant,
                ragged=B > 1 and rng.random() < 0.5)


def _lengths(case):
    """True lengths of the sequences, spread over the upper three quarters of N; None when all are N."""
    if not case.get("ragged"):
        return None
    B, N = case["B"], case["N"]
    return [N - (3 * N // 4) * b // B for b in range(B)]


def _layer_inputs(case, gen, W):
    """q [B,Hq,W,d], k, v [B,Hkv,N,d] of one layer."""
    B, Hq, Hkv, N, d = (case[x] for x in ("B", "Hq", "Hkv", "N", "d"))
    dtype, G = DTYPES[case["dtype"]], case["Hq"] // case["Hkv"]
    q = torch.randn(B, Hq, W, d, generator=gen, device=DEVICE, dtype=dtype)
    k = torch.randn(B, Hkv, N, d, generator=gen, device=DEVICE, dtype=dtype)
    v = torch.randn(B, Hkv, N, d, generator=gen, device=DEVICE, dtype=dtype)
    channels = torch.randperm(d, generator=gen, device=DEVICE)[:4]
    k[..., channels] *= 8
    windows = q.view(B, Hkv, G * W, d)
    k[:, :, :SINKS] = 3 * windows.float().mean(dim=2, keepdim=True).to(dtype)
    if case.get("needles"):
        at = torch.randperm(N - SINKS, generator=gen, device=DEVICE)[:NEEDLES] + SINKS
        which = torch.randint(G * W, (NEEDLES,), generator=gen, device=DEVICE)
        k[:, :, at] = 2 * windows[:, :, which]
    return q, k, v


def _running_scores(shape, gen):
    """Scores accumulated over a prompt: positive, spread over orders of magnitude, sinks far above the rest."""
    s = torch.exp(1.5 * torch.randn(shape, generator=gen, device=DEVICE))
    s[..., :SINKS] *= 1e4
    return s


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(int(seed))
    return {"score": _prepare_score, "evict": _prepare_evict, "decode": _prepare_decode,
            "accumulate": _prepare_accumulate}[case["kind"]](case, gen)


def run(state):
    return {"score": _run_score, "evict": _run_evict, "decode": _run_decode,
            "accumulate": _run_accumulate}[state["kind"]](state)


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device=DEVICE) if nbytes else None


def _score_workspace(case, W):
    return _workspace(obc.obc_score_workspace_bytes(case["B"], case["N"], W, case["Hq"], case["Hkv"], case["d"],
                                                    obc.OBC_BF16 if case["dtype"] == "bf16" else obc.OBC_F32,
                                                    obc.VARIANT_CODES[case["variant"]]))


def _prepare_score(case, gen):
    q, k, v = _layer_inputs(case, gen, case["W"])
    shape = (case["B"], case["Hkv"], case["N"])
    return dict(kind="score", q=q, k=k, v=v, variant=case["variant"], lens=_lengths(case),
                workspace=_score_workspace(case, case["W"]),
                scores=torch.empty((3,) + shape if case["variant"] == "all" else shape, device=DEVICE))


def _run_score(s):
    return obc.obc_score(s["q"], s["k"], s["v"], s["variant"], seq_lens=s["lens"], scores=s["scores"],
                         workspace=s["workspace"])


def _prepare_accumulate(case, gen):
    q, k, v = _layer_inputs(case, gen, 1)
    return dict(kind="accumulate", q=q, k=k, v=v, variant=case["variant"], lens=_lengths(case),
                workspace=_score_workspace(case, 1), scores=_running_scores((case["B"], case["Hkv"], case["N"]), gen))


def _run_accumulate(s):
    return obc.obc_score(s["q"], s["k"], s["v"], s["variant"], seq_lens=s["lens"], scores=s["scores"],
                         workspace=s["workspace"], accumulate=True)


def _safeguard(case):
    """AdaKV's guaranteed share of a head's budget."""
    return int(0.2 * case["budget"])


def _adaptive_cap(case):
    return min(case["N"], case["Hkv"] * case["budget"] - (case["Hkv"] - 1) * _safeguard(case))


def _recent(case):
    return min(64, case["budget"] // 4)


def _prepare_evict(case, gen):
    B, Hkv, N, d, budget = (case[x] for x in ("B", "Hkv", "N", "d", "budget"))
    dtype = DTYPES[case["dtype"]]
    k = torch.randn(B, Hkv, N, d, generator=gen, device=DEVICE, dtype=dtype)
    v = torch.randn(B, Hkv, N, d, generator=gen, device=DEVICE, dtype=dtype)
    lens = _lengths(case)
    scores = _running_scores((B, Hkv, N), gen)
    if lens is not None:
        for b, n in enumerate(lens):
            scores[b, :, n:] = 0
    rows = budget
    if case["mode"] == "adaptive":
        rows = _adaptive_cap(case)
    out = torch.empty(2, B, Hkv, rows, d, device=DEVICE, dtype=dtype)
    s = dict(kind="evict", mode=case["mode"], k=k, v=v, scores=scores, lens=lens, budget=budget, recent=_recent(case),
             safe=_safeguard(case), workspace=_workspace(obc.obc_select_workspace_bytes(B, Hkv, N)),
             keep=torch.empty(B, Hkv, budget, device=DEVICE, dtype=torch.int32), k_out=out[0], v_out=out[1])
    if case["mode"] == "protected":
        s["scores_out"] = torch.empty(B, Hkv, budget, device=DEVICE)
    return s


def _run_evict(s):
    if s["mode"] == "adaptive":
        keep, counts = obc.obc_select_adaptive(s["scores"], s["budget"], s["safe"], seq_lens=s["lens"])
        k, v = obc.obc_compact(s["k"], s["v"], keep, s["k_out"], s["v_out"])
        return {"keep": keep, "counts": counts, "k": k, "v": v}
    if s["mode"] == "top":
        keep = obc.obc_select(s["scores"], s["budget"], seq_lens=s["lens"], keep_idx=s["keep"], workspace=s["workspace"])
    else:
        heavy = s["budget"] - SINKS - s["recent"]
        if s["mode"] == "pooled":
            keep = obc.obc_select_pooled(s["scores"], heavy, POOL, SINKS, s["recent"], seq_lens=s["lens"],
                                         keep_idx=s["keep"], workspace=s["workspace"])
        else:
            keep = obc.obc_select_protected(s["scores"], heavy, SINKS, s["recent"], seq_lens=s["lens"],
                                            keep_idx=s["keep"], workspace=s["workspace"])
    k, v = obc.obc_compact(s["k"], s["v"], keep, s["k_out"], s["v_out"])
    out = {"keep": keep, "k": k, "v": v}
    if s["mode"] == "protected":                  # running scores follow their tokens
        out["scores"] = obc.obc_compact_scores(s["scores"], keep, scores_out=s["scores_out"], n_out=s["budget"])
    return out


def _prepare_decode(case, gen):
    L, B, Hq, Hkv, N, d = (case[x] for x in ("layers", "B", "Hq", "Hkv", "N", "d"))
    dtype = DTYPES[case["dtype"]]
    kv = torch.randn(2, L, B, Hkv, N, d, generator=gen, device=DEVICE, dtype=dtype)
    new = torch.randn(RING, 2, L, B, Hkv, d, generator=gen, device=DEVICE, dtype=dtype)
    channels = torch.randperm(d, generator=gen, device=DEVICE)[:4]
    kv[0][..., channels] *= 8
    new[:, 0][..., channels] *= 8
    q = torch.randn(RING, L, B, Hq, 1, d, generator=gen, device=DEVICE, dtype=dtype)
    scores = _running_scores((L, B, Hkv, N), gen)
    scores[..., N - 1] = 0                        # the slot of the token to come
    code, var = obc.OBC_BF16, obc.VARIANT_CODES[case["variant"]]
    one = case["calls"] == "one"
    ws = (obc.obc_decode_step_workspace_bytes(B, N, Hq, Hkv, d, code, var) if one
          else obc.obc_score_workspace_bytes(B, N, 1, Hq, Hkv, d, code, var))
    dropped = (L, B, Hkv) if one else (L, B, Hkv, N - 1)
    return dict(kind="decode", kv=kv, slot=kv[:, :, :, :, N - 1], new=list(new), q=[list(x) for x in q], k=list(kv[0]),
                v=list(kv[1]), scores=scores, layer_scores=list(scores), workspace=_workspace(ws), one=one, step=0,
                variant=case["variant"], recent=N // 4, heavy=N - 1 - SINKS - N // 4,
                picked=torch.empty(dropped, device=DEVICE, dtype=torch.int32))


def _run_decode(s):
    at = s["step"] % RING
    s["step"] += 1
    s["slot"].copy_(s["new"][at])
    for layer, q in enumerate(s["q"][at]):
        k, v, scores, picked = s["k"][layer], s["v"][layer], s["layer_scores"][layer], s["picked"][layer]
        if s["one"]:
            obc.obc_decode_step(q, k, v, scores, s["variant"], SINKS, s["recent"], evicted=picked, workspace=s["workspace"])
        else:
            obc.obc_score(q, k, v, s["variant"], scores=scores, workspace=s["workspace"], accumulate=True)
            obc.obc_select_protected(scores, s["heavy"], SINKS, s["recent"], keep_idx=picked, workspace=False)
            obc.obc_compact_inplace(k, v, picked, scores=scores)
    return {"picked": s["picked"], "kv": s["kv"], "scores": s["scores"]}


def _row_flops(variant, d):
    """Of one (window row, token) pair: the logit; the attention output and the cross term where the score needs them."""
    return 2 * d * (1 if variant in ("value", "attn", "vatp") else 3)


def work(case):
    size = 2 if case["dtype"] == "bf16" else 4
    B, Hkv, N, d = (case[x] for x in ("B", "Hkv", "N", "d"))
    live = sum(_lengths(case) or [N] * B)
    row = d * size
    if case["kind"] == "evict":
        kept = B * Hkv * case["budget"]
        slots = B * Hkv * (_adaptive_cap(case) if case["mode"] == "adaptive" else case["budget"])
        follow = 8 * kept if case["mode"] == "protected" else 0
        return {"bytes": 4 * live * Hkv + 4 * slots + 2 * row * (kept + slots) + follow, "flops": 0}
    tensors = 1 if case["variant"] == "attn" else 2
    if case["kind"] == "score":
        planes = 3 if case["variant"] == "all" else 1
        rows = case["Hq"] * case["W"]
        return {"bytes": row * (tensors * live * Hkv + B * rows) + 4 * planes * B * Hkv * N,
                "flops": rows * live * _row_flops(case["variant"], d)}
    if case["kind"] == "accumulate":
        return {"bytes": row * (tensors * live * Hkv + B * case["Hq"]) + 8 * live * Hkv,
                "flops": case["Hq"] * live * _row_flops(case["variant"], d)}
    # decode: the cache is read, and the rows behind the dropped one (half of those that compete, and the recent
    # ones) move up by one
    heads = case["layers"] * B * Hkv
    moved = (N - N // 4) // 2 + N // 4
    return {"bytes": heads * (2 * row * N + 2 * row * moved + 8 * N + row * case["Hq"] // Hkv),
            "flops": heads * (case["Hq"] // Hkv) * N * _row_flops(case["variant"], d)}


def tolerance(case):
    if case["kind"] == "evict":
        return "exact"
    # fp32 sums throughout; bf16 inputs have their attention weights and outputs carried in bf16 pairs (16 bits)
    return {"rel": 1e-5 if case["dtype"] == "fp32" else 5e-5}
