"""The work that is timed: calls of the paged-KV attention library as a rollout engine makes them.

Each case is one engine step of a multi-turn rollout on one GPU, through `PagedKV`:

  decode          one generated token per task over its whole context (already appended)
  decode_append   the same with the token's K/V append fused in (every generated token)
  decode_shared   decode of GRPO groups whose trajectories share their prompt's pages
  extend          append of the new observation's K/V, then attention over the kept prefix
  extend_append   the same two steps fused in one call
  reprefill       append of a whole history and its full causal attention (evicted cache)

Lengths come from a case's own numbers (`lens` seeds them), so that the work of a case is
known without its inputs; values, page placement and outlier rows come from the seed.  The
model shapes and length laws are those of workloads/configs.py and workloads/traces.py.
"""
import math

import numpy as np
import torch

import paper_2608_10402_amd as tide

PAGE = 16
# (query heads, kv heads, head dim): the 7B-class, 8-kv-head and long-horizon layers, and
# the small, ungrouped and widest-group ones of the tests
HEADS = ((28, 4, 128), (32, 8, 128), (64, 8, 128), (8, 2, 64), (8, 8, 128), (32, 2, 64))
MOST_BYTES = 8.0e9   # a drawn case does no more than the largest listed ones
MOST_FLOPS = 11.0e12


def _case(name, kind, heads, tasks, ctx, new=(0, 0), lse=False, outliers=0.0, group=1, prompt=(0, 0),
          lens=1):
    """ctx: (law, lo, hi) of the kept prefix (decode: of the whole context; reprefill: of the
    history; decode_shared: of a trajectory's own keys).  new: lo, hi of the new tokens, spread
    over their logarithm.  group / prompt: GRPO group size and shared prompt lengths."""
    c = {"kind": kind, "hq": heads[0], "hkv": heads[1], "d": heads[2], "tasks": tasks, "law": ctx[0],
         "ctx_lo": ctx[1], "ctx_hi": ctx[2], "new_lo": new[0], "new_hi": new[1], "lse": lse,
         "outliers": outliers, "group": group, "prompt_lo": prompt[0], "prompt_hi": prompt[1],
         "lens": lens}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the tail of a rollout step: a few short trajectories still generate; every token is
        # one such call per layer, and its latency is the step's
        _case("decode_tiny", "decode_append", HEADS[0], 4, ("uniform", 300, 2000)),
        # one straggler with a long context
        _case("decode_one", "decode", HEADS[1], 1, ("uniform", 30001, 30001), lse=True),
        # an ordinary round of the WebShop-shaped step: many tasks of about 1.5k tokens
        _case("decode_round", "decode_append", HEADS[0], 175, ("uniform", 500, 3000)),
        # a full decode batch of resumed tasks
        _case("decode_batch", "decode", HEADS[1], 256, ("lognormal", 1024, 32768), lse=True),
        # long-horizon agents: the largest contexts a pool holds
        _case("decode_long", "decode_append", HEADS[2], 32, ("uniform", 32768, 98304)),
        # GRPO groups of 8 over a shared prompt
        _case("decode_group", "decode_shared", HEADS[1], 256, ("lognormal", 256, 16384), group=8,
              prompt=(2048, 6144)),
        # a small model's few short tasks: the smallest resume
        _case("extend_tiny", "extend", HEADS[3], 4, ("uniform", 37, 511), (5, 128)),
        # a scheduler round in which a few tasks' observations arrive
        _case("extend_round", "extend", HEADS[0], 6, ("uniform", 600, 3000), (150, 450)),
        # one task resumed alone with a long observation
        _case("extend_one", "extend_append", HEADS[0], 1, ("uniform", 12000, 12000), (801, 801)),
        # the headline resume: 64 agents of a 7B-class layer
        _case("extend_agent", "extend", HEADS[0], 64, ("uniform", 2048, 16384), (64, 2048)),
        # image observations: long extends over outlier keys, with the log-sum-exp returned
        _case("extend_image", "extend_append", HEADS[1], 16, ("uniform", 4096, 24576), (1024, 4096),
              lse=True, outliers=0.1),
        # histories whose cache was evicted
        _case("reprefill", "reprefill", HEADS[0], 16, ("uniform", 2048, 16384)),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    """One more case: a kind, a model shape, a batch and lengths over the listed ranges."""
    while True:
        kind = rng.choice(("decode", "decode_append", "decode_append", "decode_shared", "extend",
                           "extend", "extend_append", "reprefill"))
        heads = rng.choice(HEADS[:3] + HEADS)
        lse = rng.random() < 0.3
        lens = rng.randrange(1 << 30)
        if kind == "decode_shared":
            group = rng.randint(2, 16)
            lo = _log_int(rng, 64, 2048)
            c = _case("", kind, heads, group * _log_int(rng, 1, 32), ("lognormal", lo, lo * 8), lse=lse,
                      group=group, prompt=(_log_int(rng, 64, 4096), 6144), lens=lens)
        else:
            lo = _log_int(rng, 37, 32768)
            law = rng.choice(("uniform", "lognormal"))
            ctx = (law, lo, int(lo * rng.uniform(1.0, 8.0)))
            if kind.startswith("decode"):
                c = _case("", kind, heads, _log_int(rng, 1, 256), ctx, lse=lse, lens=lens)
            elif kind == "reprefill":
                c = _case("", kind, heads, _log_int(rng, 1, 32), ctx, lse=lse, lens=lens)
            else:
                n = _log_int(rng, 5, 2048)
                c = _case("", kind, heads, _log_int(rng, 1, 64), ctx, (n, int(n * rng.uniform(1.0, 4.0))),
                          lse=lse, outliers=rng.choice((0.0, 0.0, 0.1)), lens=lens)
        w = work(c)
        if w["bytes"] <= MOST_BYTES and w["flops"] <= MOST_FLOPS and _lengths(c)["total"].max() <= 98304 + 4096:
            return c


def _lengths(case):
    """Host lengths of every task: kept prefix, new tokens and their sum; groups' prompts."""
    rng = np.random.default_rng([2608, 10402, case["lens"]])
    n, lo, hi = case["tasks"], case["ctx_lo"], case["ctx_hi"]
    if case["law"] == "uniform":
        ctx = rng.integers(lo, hi, n, endpoint=True)
    else:  # lognormal around the range's geometric middle, clipped
        ctx = np.clip(np.rint(np.exp(rng.normal(math.log(math.sqrt(lo * hi)), 0.7, n))), lo, hi)
    ctx = ctx.astype(np.int32)
    kind = case["kind"]
    got = {"shared": None}
    if kind == "decode_shared":
        prompt = rng.integers(case["prompt_lo"], case["prompt_hi"], n // case["group"], endpoint=True)
        got["shared"] = (prompt // PAGE * PAGE).astype(np.int32)
        ctx = ctx + np.repeat(got["shared"], case["group"])
    if kind.startswith("decode"):
        prefix, new = ctx - 1, np.ones(n, np.int32)
    elif kind == "reprefill":
        prefix, new = np.zeros(n, np.int32), ctx
    else:
        prefix = ctx
        new = np.exp(rng.uniform(math.log(case["new_lo"]), math.log(case["new_hi"] + 1), n))
        new = np.clip(new.astype(np.int32), case["new_lo"], case["new_hi"])
    got.update(prefix=prefix.astype(np.int32), new=new.astype(np.int32),
               total=(prefix + new).astype(np.int32))
    return got


def work(case):
    """Each key and value read once (a shared prompt once per group), Q and the new rows read,
    O and the appended rows written; two products of 2 d flops per visible (query, key) pair."""
    ln = _lengths(case)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    p, e = ln["prefix"].astype(np.float64), ln["new"].astype(np.float64)
    keys = float((p + e).sum())
    if ln["shared"] is not None:
        keys -= float(ln["shared"].sum()) * (case["group"] - 1)
    rows = float(e.sum())
    kv = 2.0 * 2 * hkv * d
    nbytes = keys * kv + rows * hq * d * 2 * 2 + 4.0 * keys / PAGE + (rows * hq * 4 if case["lse"] else 0)
    if case["kind"] not in ("decode", "decode_shared"):
        nbytes += rows * kv  # the appended rows, written to the pool
    flops = 4.0 * d * hq * float((e * p + e * (e + 1) / 2).sum())
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """bf16 probabilities and outputs, fp32 sums: against 64 bits the outputs are off by
    2e-3 to 3e-3 (2-norm), and two correct orders differ by as much."""
    return {"rel": 1e-2, "max": 0.25}


class _State:
    pass


def prepare(case, seed):
    """A pool whose pages hold the kept contexts (scattered over 1.1 times the pages in use),
    its block table, and the call's new rows and queries."""
    dev = torch.device("cuda")
    ln = _lengths(case)
    hq, hkv, d, n = case["hq"], case["hkv"], case["d"], case["tasks"]
    rng = np.random.default_rng([int(seed), case["lens"]])
    pages = -(-ln["total"].astype(np.int64) // PAGE)
    used = int(pages.sum())
    pool = int(used * 1.1) + 1
    order = rng.permutation(pool).astype(np.int32)
    table = np.zeros((n, int(pages.max())), np.int32)
    at = 0
    for b in range(n):
        first = 0
        if ln["shared"] is not None and b % case["group"]:
            first = int(ln["shared"][b // case["group"]]) // PAGE
            table[b, :first] = table[b - b % case["group"], :first]
        k = int(pages[b]) - first
        table[b, first:first + k] = order[at:at + k]
        at += k
    s = _State()
    s.case, s.ln = case, ln
    s.kv = tide.PagedKV(pool, hq, hkv, d, table, 1.0 / math.sqrt(d), device=dev, fill_canary=False)
    gen = torch.Generator(device=dev)
    gen.manual_seed((int(seed) * 1000003 + 7) % (1 << 62))
    s.kv.k_pool.normal_(generator=gen)
    s.kv.v_pool.normal_(generator=gen)
    if case["outliers"] > 0:
        hit = torch.rand((pool, 1, PAGE, 1), generator=gen, device=dev) < case["outliers"]
        s.kv.k_pool.mul_(torch.where(hit, 4.0, 1.0).to(torch.bfloat16))
    rows = int(ln["new"].sum())
    s.q = torch.empty((rows, hq, d), dtype=torch.bfloat16, device=dev).normal_(generator=gen)
    s.k = s.v = s.lse = None
    if case["kind"] not in ("decode", "decode_shared"):
        s.k = torch.empty((rows, hkv, d), dtype=torch.bfloat16, device=dev).normal_(generator=gen)
        s.v = torch.empty((rows, hkv, d), dtype=torch.bfloat16, device=dev).normal_(generator=gen)
        if case["outliers"] > 0:
            hit = torch.rand((rows, 1, 1), generator=gen, device=dev) < case["outliers"]
            s.k.mul_(torch.where(hit, 4.0, 1.0).to(torch.bfloat16))
    if case["lse"]:
        s.lse = torch.empty((rows, hq), dtype=torch.float32, device=dev)
    s.zeros = np.zeros(n, np.int32)
    if ln["shared"] is not None:
        s.group_start = np.arange(0, n + 1, case["group"], dtype=np.int32)
    return s


def run(s):
    kv, ln, kind = s.kv, s.ln, s.case["kind"]
    if kind == "decode":
        out = kv.decode(s.q, ln["total"], lse=s.lse)
    elif kind == "decode_append":
        out = kv.decode_append(s.q, s.k, s.v, ln["total"], lse=s.lse)
    elif kind == "decode_shared":
        out = kv.decode_shared(s.q, ln["total"], s.group_start, ln["shared"], lse=s.lse)
    elif kind == "extend":
        kv.append(s.k, s.v, ln["prefix"], ln["new"])
        out = kv.extend(s.q, ln["prefix"], ln["new"], lse=s.lse)
    elif kind == "extend_append":
        out = kv.extend_append(s.q, s.k, s.v, ln["prefix"], ln["new"], lse=s.lse)
    else:
        kv.append(s.k, s.v, s.zeros, ln["total"])
        out = kv.prefill(s.q, ln["total"], lse=s.lse)
    got = {"out": out}
    if s.lse is not None:
        got["lse"] = s.lse
    if s.k is not None:
        got["k_pool"], got["v_pool"] = kv.k_pool, kv.v_pool
    return got


def exact(case, seed):
    """The definition in 64 bits: the new rows put into their slots, then softmax attention of
    every query row over the keys at or before its position, one (task, kv head) at a time."""
    s = prepare(case, seed)
    ln, hq, hkv, d = s.ln, case["hq"], case["hkv"], case["d"]
    g = hq // hkv
    table = s.kv.block_table.long()
    kp, vp = s.kv.k_pool, s.kv.v_pool
    rows = int(ln["new"].sum())
    out = torch.empty((rows, hq, d), dtype=torch.float64, device=kp.device)
    lse = torch.empty((rows, hq), dtype=torch.float64, device=kp.device)
    row0 = 0
    for b in range(case["tasks"]):
        p, e = int(ln["prefix"][b]), int(ln["new"][b])
        if s.k is not None:
            pos = torch.arange(p, p + e, device=kp.device)
            page = table[b, pos // PAGE]
            kp[page, :, pos % PAGE] = s.k[row0:row0 + e]
            vp[page, :, pos % PAGE] = s.v[row0:row0 + e]
        page = table[b, : -(-(p + e) // PAGE)]
        for h in range(hkv):
            k = kp[page, h].reshape(-1, d)[: p + e].double()
            v = vp[page, h].reshape(-1, d)[: p + e].double()
            kt = k.t().contiguous()
            step = max(1, (1 << 28) // ((p + e) * g))
            for r in range(0, e, step):
                m = min(step, e - r)
                end = p + r + m
                q = s.q[row0 + r:row0 + r + m, h * g:(h + 1) * g].double().reshape(-1, d)
                x = q.mm(kt[:, :end]).mul_(1.0 / math.sqrt(d)).view(m, g, end)
                if m > 1:
                    seen = torch.arange(end, device=x.device) <= torch.arange(p + r, end, device=x.device)[:, None]
                    x.masked_fill_(~seen[:, None, :], -math.inf)
                z = torch.logsumexp(x, -1)
                x.sub_(z[..., None]).exp_()
                out[row0 + r:row0 + r + m, h * g:(h + 1) * g] = x.view(m * g, end).mm(v[:end]).view(m, g, d)
                lse[row0 + r:row0 + r + m, h * g:(h + 1) * g] = z
        row0 += e
    got = {"out": out}
    if s.lse is not None:
        got["lse"] = lse
    if s.k is not None:
        got["k_pool"], got["v_pool"] = kp, vp
    return got
