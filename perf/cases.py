"""The work that users of this library have it do, as cases to time.

A case is either
  * one attention step of one layer over a batch ("kind": "step"): the four compute calls that a serving
    engine makes per layer with a plan it keeps for the iteration -- work items over the pool, the self
    block of the new tokens, the merge of the partials, the one-pass rows; or
  * a stretch of serving ("kind": "serve"): sessions that share a system prompt go through turns, and every
    turn and every decoded token builds its plan, attends and appends the new tokens' K/V to the pool;
    at the end the sessions' segments are released and evicted.

Shapes come from the repository's five named workloads and its tests and benchmark (the Llama-3-8B layer
shape with 32 query heads on 8 KV heads, the 70B shape with 64 on 8, the tiny one with 8 on 2), or are
those layers split over several GPUs (one KV head and its 8 query heads for 70B on 8 GPUs).  K, V and Q are
N(0, 1) in bf16, prefixes end in the middle of a segment, slots are scattered over the pool at random.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2508_17219_amd import binding as B

D = 128
SCALE = 1.0 / math.sqrt(D)

ONE_PASS = "one_pass"      # TL_PLAN_FUSE_ROWS: what the benchmark plans with
TAILS = "tails"            # TL_PLAN_FUSE_TAILS: shared runs are work items that are read once
THREE_STEP = "three_step"  # neither: partials, self block, merge
_FLAGS = {
    ONE_PASS: B.TL_PLAN_SELF_BLOCK | B.TL_PLAN_FUSE_ROWS,
    TAILS: B.TL_PLAN_SELF_BLOCK | B.TL_PLAN_FUSE_TAILS,
    THREE_STEP: B.TL_PLAN_SELF_BLOCK,
}

# A step: `n_req` requests of new_lo..new_hi new tokens and `n_decode` more of one new token; prefixes of
# prefix_lo..prefix_hi tokens ("spread": uniform, or lognormal about their geometric mean and clipped to
# them), the first `shared` segments the same for all; "zipf": every prefix is instead drawn with
# replacement from `zipf` popular segments.  `layout` seeds the lengths.
_STEP = dict(kind="step", q_heads=32, kv_heads=8, seg_len=256, n_req=0, new_lo=1, new_hi=1, n_decode=0, prefix_lo=0,
             prefix_hi=0, spread="uniform", shared=0, zipf=0, plan=ONE_PASS, out="bf16", layout=1)
# Serving: `n_req` sessions with a `shared`-segment system prompt; each of `turns` turns brings new_lo new
# tokens per session and then decodes `decode` tokens, all appended to the session's chain.
_SERVE = dict(kind="serve", q_heads=32, kv_heads=8, seg_len=256, n_req=1, new_lo=256, shared=16, turns=2, decode=4,
              out="bf16", layout=1)


def listed():
    return [
        # The tiny configuration: one short chunk on a short prefix, where launches and latency are everything.
        dict(_STEP, name="tiny", q_heads=8, kv_heads=2, seg_len=128, n_req=1, new_lo=32, new_hi=32, prefix_lo=512,
             prefix_hi=512),
        # One user's chat being decoded, 70B shape: the interactive latency of a lightly loaded server.
        dict(_STEP, name="decode_one", q_heads=64, n_decode=1, prefix_lo=15900, prefix_hi=15900),
        # A small decode batch; fp32 output, which the interface offers beside bf16.
        dict(_STEP, name="decode_16", q_heads=64, n_decode=16, prefix_lo=2000, prefix_hi=131072, spread="lognormal", out="fp32"),
        # The decode configuration: 256 requests, lognormal prefixes of median 16k, capped at 128k.
        dict(_STEP, name="decode_256", q_heads=64, n_decode=256, prefix_lo=2048, prefix_hi=131072, spread="lognormal"),
        # Decode of the 70B shape on one of 8 GPUs: one KV head is left of every layer.
        dict(_STEP, name="decode_one_kv_head", q_heads=8, kv_heads=1, n_decode=64, prefix_lo=2048, prefix_hi=131072,
             spread="lognormal"),
        # The prefill configuration: chunks of 512 on 8k..32k prefixes, 2k of them shared.
        dict(_STEP, name="prefill", n_req=16, new_lo=512, new_hi=512, prefix_lo=8192, prefix_hi=32768, shared=8),
        # One long prompt's chunk by itself (the batch is too small to fill the GPU).
        dict(_STEP, name="prefill_one", n_req=1, new_lo=512, new_hi=512, prefix_lo=32500, prefix_hi=32500),
        # Prompts at their start: ragged lengths, nothing cached yet, the causal block is all there is.
        dict(_STEP, name="prompt_start", n_req=8, new_lo=700, new_hi=4096),
        # Chunked prefill and decode in one batch, as schedulers mix them.
        dict(_STEP, name="mixed", n_req=4, new_lo=300, new_hi=600, n_decode=48, prefix_lo=1000, prefix_hi=16384, shared=8),
        # The multi-turn configuration in its middle with the hot system prompt read once for all sessions.
        dict(_STEP, name="multi_turn", n_req=64, new_lo=256, new_hi=256, prefix_lo=7168, prefix_hi=7168, shared=16, plan=TAILS),
        # The long-context configuration: 128k prefixes of popular 512-token segments, many of them repeated.
        dict(_STEP, name="long_context", seg_len=512, n_req=4, new_lo=2048, new_hi=2048, prefix_lo=131072,
             prefix_hi=131072, zipf=1000),
        # Plans, attention and appends of a few sessions as a server runs them.
        dict(_SERVE, name="serve", n_req=16, new_lo=250, turns=3, decode=6),
    ]


# (query heads, KV heads): the layer shapes above whole and split, multi-head attention, an odd group
_HEADS = [(32, 8), (32, 8), (64, 8), (64, 8), (8, 2), (8, 1), (16, 4), (28, 4), (16, 16)]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    limit_kv, limit_flops = 2.6e10, 6e12      # what the listed configurations cost at most
    for _ in range(1000):
        hq, hkv = rng.choice(_HEADS)
        out = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        common = dict(q_heads=hq, kv_heads=hkv, seg_len=rng.choice([64, 128, 256, 256, 512]), out=out, layout=rng.randrange(1 << 20))
        what = rng.choice(["decode", "decode", "chunk", "chunk", "start", "mixed", "serve"])
        if what == "decode":
            mid = _log_int(rng, 300, 60000)
            case = dict(_STEP, **common)
            case.update(n_decode=_log_int(rng, 1, 256), prefix_lo=max(1, mid // 8), prefix_hi=min(131072, mid * 8), spread="lognormal",
                        shared=rng.choice([0, 0, 0, 8]))
        elif what == "chunk":
            hi = _log_int(rng, 300, 40000)
            new = _log_int(rng, 2, 2048)
            case = dict(_STEP, **common)
            case.update(n_req=_log_int(rng, 1, 64), new_lo=max(1, new // 2), new_hi=new, prefix_lo=hi // 4, prefix_hi=hi,
                        shared=rng.choice([0, 8, 16]), plan=rng.choice([ONE_PASS, ONE_PASS, TAILS, THREE_STEP]))
        elif what == "start":
            new = _log_int(rng, 16, 8192)
            case = dict(_STEP, **common)
            case.update(n_req=_log_int(rng, 1, 16), new_lo=max(1, new // 4), new_hi=new, plan=rng.choice([ONE_PASS, THREE_STEP]))
        elif what == "mixed":
            hi = _log_int(rng, 1000, 32768)
            case = dict(_STEP, **common)
            case.update(n_req=rng.randint(1, 8), new_lo=64, new_hi=rng.randint(100, 1000), n_decode=_log_int(rng, 4, 200),
                        prefix_lo=hi // 8, prefix_hi=hi, shared=rng.choice([0, 8]))
        else:
            case = dict(_SERVE, **common)
            case.update(n_req=_log_int(rng, 1, 64), new_lo=_log_int(rng, 30, 500), shared=rng.choice([4, 8, 16]),
                        turns=rng.randint(1, 3), decode=rng.randint(0, 8))
        w = work(case)
        if w["bytes"] <= limit_kv and w["flops"] <= limit_flops:
            return case
    raise RuntimeError("no case within the limits")


# ---- structure of a case (lengths and segment lists; the same for every seed) ---------------------------
def _private(req, pos):
    return ((req + 1) << 32) | pos


def _step_layout(case):
    """(new tokens per request, segment-id list per request, fill of segments that are not full)."""
    rng = np.random.Generator(np.random.PCG64(case["layout"]))
    n, C = case["n_req"] + case["n_decode"], case["seg_len"]
    new = np.concatenate([rng.integers(case["new_lo"], case["new_hi"] + 1, size=case["n_req"]), np.ones(case["n_decode"], np.int64)])
    lo, hi = case["prefix_lo"], case["prefix_hi"]
    if case["zipf"]:
        p = 1.0 / np.arange(1, case["zipf"] + 1, dtype=np.float64) ** 1.1
        p /= p.sum()
        return new, [[int(x) for x in rng.choice(case["zipf"], size=hi // C, p=p)] for _ in range(n)], {}
    if case["spread"] == "lognormal":
        ln = np.clip(np.rint(rng.lognormal(math.log(math.sqrt(lo * hi)), 1.0, size=n)), lo, hi).astype(np.int64)
    else:
        ln = rng.integers(lo, hi + 1, size=n)
    lists, fills = [], {}
    for r in range(n):
        n_seg = -(-int(ln[r]) // C)
        ids = [p if p < case["shared"] else _private(r, p) for p in range(n_seg)]
        tail = int(ln[r]) - (n_seg - 1) * C
        if n_seg and tail < C:
            ids[-1] = _private(r, n_seg - 1)
            fills[ids[-1]] = tail
        lists.append(ids)
    return new, lists, fills


def work(case):
    """Every distinct KV token read once, queries read and outputs written once; a slot that a list names
    several times needs its products once."""
    hq, hkv = case["q_heads"], case["kv_heads"]
    out_size = 2 if case["out"] == "bf16" else 4
    kv_row = 2 * hkv * D * 2

    def rows(n_tok):
        return n_tok * (hq * D * (2 + out_size) + hq * 4 + kv_row)

    if case["kind"] == "step":
        new, lists, fills = _step_layout(case)
        C = case["seg_len"]
        pairs = 0
        seen = set()
        for lq, ids in zip(new.tolist(), lists):
            distinct = set(ids)
            pairs += lq * sum(fills.get(i, C) for i in distinct) + lq * (lq + 1) // 2
            seen |= distinct
        return {"bytes": float(kv_row * sum(fills.get(i, C) for i in seen) + rows(int(new.sum()))), "flops": 4.0 * hq * D * pairs}
    S, shared = case["n_req"], case["shared"] * case["seg_len"]
    total_bytes, pairs, hist = 0, 0, 0
    for _ in range(case["turns"]):
        for lq in [case["new_lo"]] + [1] * case["decode"]:
            pairs += S * (lq * (shared + hist) + lq * (lq + 1) // 2)
            total_bytes += kv_row * (shared + S * hist) + rows(S * lq) + S * lq * kv_row     # the append writes the rows
            hist += lq
    return {"bytes": float(total_bytes), "flops": 4.0 * hq * D * pairs}


def tolerance(case):
    """Probabilities and a bf16 output are rounded to 8 bits: against the same path in 64 bits the output of
    these cases is off by at most 2.4e-3 in the 2-norm."""
    return {"rel": 1e-2}


# ---- on the GPU ------------------------------------------------------------------------------------------
class _Handles:
    """The pool and plan of a case; given back with the state."""

    def __init__(self, pool, plan=None):
        self.pool, self.plan = pool, plan

    def __del__(self):
        if self.plan is not None:
            B.tl_plan_destroy(self.plan)
        B.tl_pool_destroy(self.pool)


def _pool_tensors(case, seed, ids, extra):
    """Pool tensors with N(0, 1) everywhere, the slots of the segments `ids` at random and the generator of what
    follows; `extra` slots stay free."""
    C, hkv = case["seg_len"], case["kv_heads"]
    n_slots = max(8, len(ids) + len(ids) // 16 + extra)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kv = [torch.empty((n_slots, C, hkv, D), dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(2)]
    return kv, np.random.Generator(np.random.PCG64(seed)).permutation(n_slots)[:len(ids)], gen


def _pool(case, seed, ids, fills, extra):
    kv, slots, gen = _pool_tensors(case, seed, ids, extra)
    C, n_slots = case["seg_len"], kv[0].shape[0]
    pool = B.tl_pool_create(n_slots, C, case["kv_heads"], D, kv[0], kv[1])
    B.tl_pool_adopt(pool, ids, slots, [fills.get(i, C) for i in ids])
    return pool, kv, gen


def _rows(gen, n, heads):
    return torch.empty((n, heads, D), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)


def _outputs(case, n_tok):
    dt = torch.bfloat16 if case["out"] == "bf16" else torch.float32
    return (torch.zeros((n_tok, case["q_heads"], D), dtype=dt, device="cuda"),
            torch.zeros((n_tok, case["q_heads"]), dtype=torch.float32, device="cuda"))


def _partials(rows, hq):
    return (torch.empty((max(rows, 1), hq, D), dtype=torch.float32, device="cuda"),
            torch.empty((max(rows, 1), hq), dtype=torch.float32, device="cuda"))


def _ptr(counts):
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)


def prepare(case, seed):
    return _prepare_step(case, seed) if case["kind"] == "step" else _prepare_serve(case, seed)


def run(state):
    return _run_step(state) if state["case"]["kind"] == "step" else _run_serve(state)


def _prepare_step(case, seed):
    new, lists, fills = _step_layout(case)
    ids = list(dict.fromkeys(i for l in lists for i in l))
    pool, kv, gen = _pool(case, seed, ids, fills, 0)
    plan = B.tl_plan_create(pool, case["q_heads"], _ptr(new), _ptr([len(l) for l in lists]),
                            np.array([i for l in lists for i in l], np.uint64), _FLAGS[case["plan"]])
    T, hq, hkv = int(new.sum()), case["q_heads"], case["kv_heads"]
    partial, partial_lse = _partials(B.tl_plan_get_info(plan).n_partial_rows, hq)
    out, lse = _outputs(case, T)
    return dict(case=case, handles=_Handles(pool, plan), kv=kv, q=_rows(gen, T, hq), k=_rows(gen, T, hkv), v=_rows(gen, T, hkv),
                partial=partial, partial_lse=partial_lse, out=out, lse=lse)


def _attend(pool, plan, s, q, k, v, out, lse, partial, partial_lse):
    bf16 = s["case"]["out"] == "bf16"
    B.tl_segment_attn(pool, plan, q, SCALE, partial, partial_lse)
    B.tl_causal_block(plan, q, k, v, SCALE, partial, partial_lse)
    B.tl_merge(plan, partial, partial_lse, out, bf16, lse)
    B.tl_fused_attn(pool, plan, q, k, v, SCALE, out, bf16, lse, prior_partial=partial, prior_lse=partial_lse)


def _run_step(s):
    h = s["handles"]
    _attend(h.pool, h.plan, s, s["q"], s["k"], s["v"], s["out"], s["lse"], s["partial"], s["partial_lse"])
    return s["out"], s["lse"]


def _serve_steps(case):
    return [lq for _ in range(case["turns"]) for lq in [case["new_lo"]] + [1] * case["decode"]]


def _prepare_serve(case, seed):
    S, hq, hkv, C = case["n_req"], case["q_heads"], case["kv_heads"], case["seg_len"]
    steps = _serve_steps(case)
    shared = list(range(case["shared"]))
    pool, kv, gen = _pool(case, seed, shared, {}, S * (-(-sum(steps) // C)))
    inputs = [(_rows(gen, S * lq, hq), _rows(gen, S * lq, hkv), _rows(gen, S * lq, hkv)) for lq in steps]
    outputs = [_outputs(case, S * lq) for lq in steps]
    return dict(case=case, handles=_Handles(pool), kv=kv, steps=steps, inputs=inputs, outputs=outputs)


def _run_serve(s):
    case, pool = s["case"], s["handles"].pool
    S, C = case["n_req"], case["seg_len"]
    shared = list(range(case["shared"]))
    chains = [[] for _ in range(S)]            # ids of every session's own segments
    hist = 0                                   # tokens in each chain
    plans = []
    for lq, (q, k, v), (out, lse) in zip(s["steps"], s["inputs"], s["outputs"]):
        n_list = len(shared) + len(chains[0])
        plan = B.tl_plan_create(pool, case["q_heads"], np.arange(S + 1, dtype=np.int32) * lq, np.arange(S + 1, dtype=np.int32) * n_list,
                                np.array([i for c in chains for i in shared + c], np.uint64), _FLAGS[ONE_PASS])
        _attend(pool, plan, s, q, k, v, out, lse, *_partials(B.tl_plan_get_info(plan).n_partial_rows, case["q_heads"]))
        plans.append(plan)                     # kept until the stream has used it
        has_tail = hist % C != 0
        n_new = -(-(hist + lq) // C) - len(chains[0])
        fresh = [[_private(r, len(chains[r]) + j) for j in range(n_new)] for r in range(S)]
        B.tl_pool_append_batch(pool, [c[-1] if has_tail else None for c in chains], fresh, [lq] * S, k, v)
        for c, f in zip(chains, fresh):
            c += f
        hist += lq
    # what the pool now holds of the sessions' chains, and the end of the sessions
    slots = B.tl_pool_lookup(pool, [i for c in chains for i in c])
    for c in chains:
        for i in c:
            B.tl_pool_release(pool, i)
    for _ in range(len(slots)):
        B.tl_pool_evict_lru(pool)
    torch.cuda.current_stream().synchronize()
    for plan in plans:
        B.tl_plan_destroy(plan)
    return [t for o in s["outputs"] for t in o] + s["kv"] + [slots]


# ---- the same numbers in 64 bits ---------------------------------------------------------------------------
def exact(case, seed):
    return _exact_step(case, seed) if case["kind"] == "step" else _exact_serve(case, seed)


def _exact_attend(q, k_pre, v_pre, mult, k_new, v_new):
    """Softmax attention of one request's new tokens q [n, hq, D] over prefix keys [L, hkv, D], key j counted
    mult[j] times (None: once), and over the new tokens up to the row's own; returns (O [n, hq, D], LSE [n, hq])."""
    n, hq, _ = q.shape
    hkv, L = k_new.shape[1], k_pre.shape[0]
    out = torch.empty((n, hq, D), dtype=torch.float64, device="cuda")
    lse = torch.empty((n, hq), dtype=torch.float64, device="cuda")
    extra = None if mult is None else torch.log(mult.double())
    step = max(1, (1 << 27) // ((L + n) * (hq // hkv)))          # tokens at a time: 1 GiB of scores
    for g in range(hkv):
        heads = slice(g * (hq // hkv), (g + 1) * (hq // hkv))
        k = torch.cat([k_pre[:, g], k_new[:, g]]).double()
        v = torch.cat([v_pre[:, g], v_new[:, g]]).double()
        for t in range(0, n, step):
            e = min(n, t + step)
            s = (q[t:e, heads].double().reshape(-1, D) @ k.t() * SCALE).view(e - t, -1, L + n)
            if extra is not None:
                s[:, :, :L] += extra
            later = torch.arange(n, device="cuda")[None, :] > torch.arange(t, e, device="cuda")[:, None]
            s[:, :, L:].masked_fill_(later[:, None, :], -math.inf)
            top = torch.logsumexp(s, dim=-1)
            lse[t:e, heads] = top
            s.sub_(top[..., None]).exp_()
            out[t:e, heads] = (s.view(-1, L + n) @ v).view(e - t, -1, D)
    return out, lse


def _exact_step(case, seed):
    new, lists, fills = _step_layout(case)
    C, hq, hkv = case["seg_len"], case["q_heads"], case["kv_heads"]
    ids = list(dict.fromkeys(i for l in lists for i in l))
    kv, slots, gen = _pool_tensors(case, seed, ids, 0)
    slot_of = dict(zip(ids, slots.tolist()))
    T = int(new.sum())
    q, k, v = _rows(gen, T, hq), _rows(gen, T, hkv), _rows(gen, T, hkv)
    outs, at = [], 0
    for lq, ids_r in zip(new.tolist(), lists):
        times = {}
        for i in ids_r:
            times[i] = times.get(i, 0) + 1
        token = [slot_of[i] * C + np.arange(fills.get(i, C)) for i in times]
        mult = [np.full(fills.get(i, C), m) for i, m in times.items()]
        index = torch.from_numpy(np.concatenate(token) if token else np.zeros(0, np.int64)).cuda()
        mult = torch.from_numpy(np.concatenate(mult)).cuda() if case["zipf"] else None
        pre = [x.view(-1, hkv, D)[index] for x in kv]
        outs.append(_exact_attend(q[at:at + lq], *pre, mult, k[at:at + lq], v[at:at + lq]))
        at += lq
    return torch.cat([o for o, _ in outs]), torch.cat([l for _, l in outs])


def _exact_serve(case, seed):
    S, hq, hkv, C = case["n_req"], case["q_heads"], case["kv_heads"], case["seg_len"]
    steps = _serve_steps(case)
    kv, slots, gen = _pool_tensors(case, seed, list(range(case["shared"])), S * (-(-sum(steps) // C)))
    inputs = [(_rows(gen, S * lq, hq), _rows(gen, S * lq, hkv), _rows(gen, S * lq, hkv)) for lq in steps]
    index = torch.from_numpy(slots.astype(np.int64)).cuda()
    seen = [[x[index].view(-1, hkv, D) for x in kv] for _ in range(S)]
    outs = []
    for lq, (q, k, v) in zip(steps, inputs):
        per = []
        for r in range(S):
            rows = slice(r * lq, (r + 1) * lq)
            per.append(_exact_attend(q[rows], *seen[r], None, k[rows], v[rows]))
            seen[r] = [torch.cat([x, y[rows]]) for x, y in zip(seen[r], (k, v))]
        outs += [torch.cat([o for o, _ in per]), torch.cat([l for _, l in per])]
    return outs + [None, None, None]           # the pool's rows are copies and the slots whole numbers
