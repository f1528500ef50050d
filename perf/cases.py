"""The calls whose speed this framework is judged by, as a serving program makes them.

A serving engine with agent-aware KV reuse calls this library for five things:

* prefill attention of the new suffix tokens of one or many agent invocations
  over their cached anchors in the paged pool (a miss recomputes its whole
  prompt), always with ``workspace="auto"`` as the benchmark does;
* paged decode attention, one token per sequence, from a handful of sequences
  to a full batch;
* cascade decode of a batch whose sequences share their agents' anchors;
* the write of new tokens' K/V into their pool slots;
* the swap of whole blocks with the CPU tier (offload of evicted blocks, reload
  of the predicted agent's anchor).

Every case is one such call (the swap: its two copies).  Shapes follow the
repository's configurations: 32 query / 8 KV heads of dimension 128 (8B class),
64 / 8 (70B class), one GPU's 8 / 1 shard of it, and head dimension 64; anchors
of 1.5k to 8k tokens, suffixes from a few tokens to 2k.  Lengths are drawn from
the case's own ``lens`` number, so they belong to the case and not to the
seed; the seed gives the values (N(0, 1) in bf16) and the scattered pool slots.
"""

import math
import random

import torch

from paper_2608_14624_amd import ops

BLOCK = 16
DEV = "cuda"


# --------------------------------------------------------------------------
# Cases
# --------------------------------------------------------------------------

def listed():
    return [
        # the next turn of one agent: a short message on a cached prompt (latency)
        dict(name="turn", op="prefill", hq=32, hkv=8, d=128, agents=1, inv=1, prefix_lo=3011,
             prefix_hi=3011, suffix_lo=83, suffix_hi=83, hit_pct=100, lens=1),
        # one invocation of the 8B shape, 2048 cached + 1024 new tokens
        dict(name="invocation_8b", op="prefill", hq=32, hkv=8, d=128, agents=1, inv=1,
             prefix_lo=2048, prefix_hi=2048, suffix_lo=1024, suffix_hi=1024, hit_pct=100, lens=1),
        # one agent's batch of the 70B-shape serving step
        dict(name="agent_70b", op="prefill", hq=64, hkv=8, d=128, agents=1, inv=4, prefix_lo=4096,
             prefix_hi=4096, suffix_lo=512, suffix_hi=512, hit_pct=100, lens=1),
        # the same agents on one GPU of an 8-way split by KV head
        dict(name="agent_70b_tp8", op="prefill", hq=8, hkv=1, d=128, agents=1, inv=3,
             prefix_lo=4096, prefix_hi=4096, suffix_lo=512, suffix_hi=512, hit_pct=100, lens=1),
        # a scheduler step's mix: 32 ragged invocations of 4 agents, a quarter of them misses
        dict(name="mixed_batch", op="prefill", hq=32, hkv=8, d=128, agents=4, inv=32,
             prefix_lo=1536, prefix_hi=3072, suffix_lo=256, suffix_hi=2048, hit_pct=75, lens=2),
        # head dimension 64
        dict(name="batch_d64", op="prefill", hq=32, hkv=8, d=64, agents=3, inv=7, prefix_lo=1500,
             prefix_hi=2500, suffix_lo=200, suffix_hi=900, hit_pct=100, lens=3),
        # decode of the few sequences a lightly loaded server holds (latency)
        dict(name="decode_few", op="decode", hq=32, hkv=8, d=128, batch=3, len_lo=2000,
             len_hi=6000, lens=4),
        # decode of a medium batch of unequal lengths
        dict(name="decode_medium", op="decode", hq=32, hkv=8, d=128, batch=24, len_lo=500,
             len_hi=9000, lens=5),
        # decode of a full batch, nothing shared
        dict(name="decode_full", op="decode", hq=32, hkv=8, d=128, batch=128, len_lo=4224,
             len_hi=10800, lens=6),
        # decode of a full batch of 8 agents' sequences, anchors shared
        dict(name="cascade", op="cascade", hq=32, hkv=8, d=128, agents=8, batch=128,
             shared_lo=4096, shared_hi=8192, own_lo=128, own_hi=4096, lens=7),
        # the K/V of a prefill step's tokens into the pool
        dict(name="write_back", op="write", hkv=8, d=128, tokens=8192),
        # 64 blocks evicted to the CPU tier and 64 blocks of the next anchor reloaded
        dict(name="swap", op="swap", hkv=8, d=128, blocks=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = [(32, 8, 128), (32, 8, 128), (64, 8, 128), (8, 1, 128), (4, 1, 128), (32, 8, 64), (8, 2, 64)]


def draw(rng):
    """One more case of the same ranges, at most as costly as the largest listed one."""
    most = {}
    for c in listed():
        w = work(c)
        for k in ("bytes", "flops"):
            most[k] = max(most.get(k, 0), w[k])
    while True:
        op = rng.choice(["prefill"] * 5 + ["decode"] * 3 + ["cascade", "cascade", "write", "swap"])
        hq, hkv, d = rng.choice(_HEADS)
        if op == "prefill":
            inv = _log_int(rng, 1, 32)
            p_lo = _log_int(rng, 64, 6000)
            s_lo = _log_int(rng, 1, 1024)
            c = dict(op=op, hq=hq, hkv=hkv, d=d, agents=rng.randint(1, min(inv, 8)), inv=inv,
                     prefix_lo=p_lo, prefix_hi=p_lo + rng.randint(0, p_lo), suffix_lo=s_lo,
                     suffix_hi=s_lo + rng.randint(0, 2 * s_lo),
                     hit_pct=rng.choice([100, 100, 75, 0]), lens=rng.randrange(1 << 20))
        elif op == "decode":
            lo = _log_int(rng, 200, 8000)
            c = dict(op=op, hq=hq, hkv=hkv, d=d, batch=_log_int(rng, 1, 160), len_lo=lo,
                     len_hi=lo + rng.randint(0, 2 * lo), lens=rng.randrange(1 << 20))
        elif op == "cascade":
            batch = _log_int(rng, 8, 160)
            lo = _log_int(rng, 500, 8000)
            own = _log_int(rng, 16, 1000)
            c = dict(op=op, hq=hq, hkv=hkv, d=d, agents=rng.randint(1, min(8, batch // 4)),
                     batch=batch, shared_lo=lo, shared_hi=lo + rng.randint(0, lo), own_lo=own,
                     own_hi=own + rng.randint(0, 4 * own), lens=rng.randrange(1 << 20))
        elif op == "write":
            c = dict(op=op, hkv=hkv, d=d, tokens=_log_int(rng, 100, 16384))
        else:
            c = dict(op=op, hkv=hkv, d=d, blocks=_log_int(rng, 4, 256))
        w = work(c)
        if all(w[k] <= most[k] for k in most):
            return c


# --------------------------------------------------------------------------
# Lengths (of the case alone)
# --------------------------------------------------------------------------

def _prefill_lengths(case):
    """Per agent its anchor length; per invocation (agent, hit, suffix length)."""
    r = random.Random(case["lens"])
    anchors = [r.randint(case["prefix_lo"], case["prefix_hi"]) for _ in range(case["agents"])]
    invs = []
    for i in range(case["inv"]):
        invs.append((i * case["agents"] // case["inv"], r.randrange(100) < case["hit_pct"],
                     r.randint(case["suffix_lo"], case["suffix_hi"])))
    return anchors, invs


def _decode_lengths(case):
    r = random.Random(case["lens"])
    return [r.randint(case["len_lo"], case["len_hi"]) for _ in range(case["batch"])]


def _cascade_lengths(case):
    """Per group its shared tokens (whole blocks); per sequence (group, own tokens)."""
    r = random.Random(case["lens"])
    shared = [r.randint(case["shared_lo"], case["shared_hi"]) // BLOCK * BLOCK
              for _ in range(case["agents"])]
    # own histories: log-uniform, so most are short and a few long
    seqs = [(i * case["agents"] // case["batch"], _log_int(r, case["own_lo"], case["own_hi"]))
            for i in range(case["batch"])]
    return shared, seqs


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.bfloat16)


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device=DEV)


def _pool(gen, used, hkv, d):
    """K and V pools with `used` blocks to hand out and some free ones, and
    the slots in a scattered order."""
    n = used + used // 9 + 1
    return (_normal(gen, n, hkv, BLOCK, d), _normal(gen, n, hkv, BLOCK, d),
            torch.randperm(n, generator=gen, device=DEV).to(torch.int32))


def _tables(rows, width):
    table = torch.zeros(len(rows), width, dtype=torch.int32, device=DEV)
    for r, parts in enumerate(rows):
        ids = torch.cat(parts)
        table[r, :ids.numel()] = ids
    return table


def _ceil(n):
    return -(-n // BLOCK)


class _Slots:
    def __init__(self, order):
        self.order, self.at = order, 0

    def take(self, n):
        self.at += n
        return self.order[self.at - n:self.at]


def _prefill_state(case, seed):
    anchors, invs = _prefill_lengths(case)
    gen = _gen(seed)
    hit_agents = {a for a, hit, _ in invs if hit}
    # an agent's whole anchor blocks are shared by its hits; the rest is private
    shared = {a: anchors[a] // BLOCK for a in hit_agents}
    total = [_ceil(anchors[a] + s) for a, _, s in invs]
    used = sum(shared.values()) + sum(
        n - (shared[a] if hit else 0) for n, (a, hit, _) in zip(total, invs))
    k, v, order = _pool(gen, used, case["hkv"], case["d"])
    slots = _Slots(order)
    anchor_slots = {a: slots.take(n) for a, n in sorted(shared.items())}
    rows, prefix, qlens = [], [], []
    for n, (a, hit, s) in zip(total, invs):
        if hit:
            rows.append([anchor_slots[a], slots.take(n - shared[a])])
            prefix.append(anchors[a])
            qlens.append(s)
        else:
            rows.append([slots.take(n)])
            prefix.append(0)
            qlens.append(anchors[a] + s)
    cu = [0]
    for s in qlens:
        cu.append(cu[-1] + s)
    q = _normal(gen, cu[-1], case["hq"], case["d"])
    return dict(q=q, k=k, v=v, tables=_tables(rows, max(total)), prefix=_i32(prefix), cu=_i32(cu),
                out=torch.empty_like(q), max_q=max(qlens),
                max_kv=max(p + s for p, s in zip(prefix, qlens)), scale=case["d"] ** -0.5,
                prefix_host=prefix, cu_host=cu)


def _decode_state(case, seed):
    lens = _decode_lengths(case)
    gen = _gen(seed)
    blocks = [_ceil(n) for n in lens]
    k, v, order = _pool(gen, sum(blocks), case["hkv"], case["d"])
    slots = _Slots(order)
    q = _normal(gen, len(lens), case["hq"], case["d"])
    return dict(q=q, k=k, v=v, tables=_tables([[slots.take(n)] for n in blocks], max(blocks)),
                lens=_i32(lens), out=torch.empty_like(q), max_len=max(lens),
                scale=case["d"] ** -0.5, lens_host=lens)


def _cascade_state(case, seed):
    shared, seqs = _cascade_lengths(case)
    gen = _gen(seed)
    used = sum(n // BLOCK for n in shared) + sum(_ceil(own) for _, own in seqs)
    k, v, order = _pool(gen, used, case["hkv"], case["d"])
    slots = _Slots(order)
    anchor = [slots.take(n // BLOCK) for n in shared]
    rows = [[anchor[g], slots.take(_ceil(own))] for g, own in seqs]
    lens = [shared[g] + own for g, own in seqs]
    sizes = [sum(1 for g, _ in seqs if g == a) for a in range(len(shared))]
    cu = [0]
    for n in sizes:
        cu.append(cu[-1] + n)
    q = _normal(gen, len(seqs), case["hq"], case["d"])
    max_shared, max_own = max(shared), max(own for _, own in seqs)
    need = ops.cs_cascade_decode_workspace_bytes(len(seqs), case["hq"], case["d"], max_shared, max_own)
    return dict(q=q, k=k, v=v, tables=_tables(rows, max(_ceil(n) for n in lens)), lens=_i32(lens),
                cu=_i32(cu), shared=_i32(shared), out=torch.empty_like(q), max_len=max(lens),
                max_seqs=max(sizes), max_shared=max_shared, max_own=max_own,
                scale=case["d"] ** -0.5, lens_host=lens,
                workspace=torch.empty(max(need, 16), dtype=torch.uint8, device=DEV))


def _write_state(case, seed):
    gen = _gen(seed)
    t, hkv, d = case["tokens"], case["hkv"], case["d"]
    k, v, order = _pool(gen, _ceil(t), hkv, d)
    at = torch.arange(t, device=DEV)
    slots = (order[:_ceil(t)][at // BLOCK] * BLOCK + at % BLOCK).to(torch.int32)
    # a padded batch: the last few rows are not stored
    slots[t - t // 50:] = -1
    return dict(k=k, v=v, k_new=_normal(gen, t, hkv, d), v_new=_normal(gen, t, hkv, d), slots=slots)


def _swap_state(case, seed):
    gen = _gen(seed)
    n, hkv, d = case["blocks"], case["hkv"], case["d"]
    k, v, order = _pool(gen, 2 * n, hkv, d)

    def host(fill):
        t = torch.empty(n, hkv, BLOCK, d, dtype=torch.bfloat16, pin_memory=True)
        t.copy_(fill) if fill is not None else t.zero_()
        return t

    return dict(k=k, v=v, victims=order[:n].clone(), targets=order[n:2 * n].clone(),
                host_k=host(_normal(gen, n, hkv, BLOCK, d)),
                host_v=host(_normal(gen, n, hkv, BLOCK, d)), evicted_k=host(None),
                evicted_v=host(None))


_STATES = dict(prefill=_prefill_state, decode=_decode_state, cascade=_cascade_state,
               write=_write_state, swap=_swap_state)


def prepare(case, seed):
    state = _STATES[case["op"]](case, seed)
    state["op"] = case["op"]
    return state


# --------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------

def run(s):
    op = s["op"]
    if op == "prefill":
        ops.cs_prefill_paged_attn(s["q"], s["k"], s["v"], s["tables"], s["prefix"], s["cu"],
                                  s["out"], max_q_len=s["max_q"], max_kv_len=s["max_kv"],
                                  scale=s["scale"], workspace="auto")
        return s["out"]
    if op == "decode":
        ops.cs_paged_decode_attn(s["q"], s["k"], s["v"], s["tables"], s["lens"], s["out"],
                                 max_seq_len=s["max_len"], scale=s["scale"])
        return s["out"]
    if op == "cascade":
        ops.cs_cascade_decode_attn(s["q"], s["k"], s["v"], s["tables"], s["lens"], s["cu"],
                                   s["shared"], s["out"], max_seq_len=s["max_len"],
                                   max_group_seqs=s["max_seqs"], max_shared_len=s["max_shared"],
                                   max_rest_len=s["max_own"], scale=s["scale"],
                                   workspace=s["workspace"])
        return s["out"]
    if op == "write":
        ops.cs_kv_write(s["k_new"], s["v_new"], s["slots"], s["k"], s["v"])
        return s["k"], s["v"]
    ops.cs_kv_offload(s["victims"], s["k"], s["v"], s["evicted_k"], s["evicted_v"])
    ops.cs_kv_prefetch(s["host_k"], s["host_v"], s["targets"], s["k"], s["v"])
    return s["k"], s["v"], s["evicted_k"], s["evicted_v"]


def work(case):
    """Bytes: each distinct K/V block, query and output once; flops: 4 D per
    (query head, query, visible key)."""
    op, d = case["op"], case["d"]
    kv = 4 * case["hkv"] * d                 # bytes of one token's K and V
    if op == "prefill":
        anchors, invs = _prefill_lengths(case)
        hit_agents = {a for a, hit, _ in invs if hit}
        keys = sum(anchors[a] for a in hit_agents)
        rows = pairs = 0
        for a, hit, s in invs:
            p, n = (anchors[a], s) if hit else (0, anchors[a] + s)
            keys += n
            rows += n
            pairs += n * p + n * (n + 1) // 2
        return dict(bytes=keys * kv + 4 * rows * case["hq"] * d, flops=4 * d * case["hq"] * pairs)
    if op in ("decode", "cascade"):
        if op == "decode":
            lens = _decode_lengths(case)
            keys = pairs = sum(lens)
        else:
            shared, seqs = _cascade_lengths(case)
            keys = sum(shared) + sum(own for _, own in seqs)
            pairs = sum(shared[g] + own for g, own in seqs)
            lens = seqs
        return dict(bytes=keys * kv + 4 * len(lens) * case["hq"] * d, flops=4 * d * case["hq"] * pairs)
    if op == "write":
        stored = case["tokens"] - case["tokens"] // 50
        return dict(bytes=2 * stored * kv, flops=0)
    return dict(bytes=4 * case["blocks"] * BLOCK * kv, flops=0)


def tolerance(case):
    if case["op"] in ("write", "swap"):
        return "exact"
    return {"rel": 1e-2, "max": 0.1}


# --------------------------------------------------------------------------
# The same results in 64 bits
# --------------------------------------------------------------------------

def _gather(pool, ids, n):
    """Tokens 0 .. n-1 of the blocks `ids` as float64 [hkv, n, d]."""
    x = pool[ids[:_ceil(n)].long()]                        # [blocks, hkv, 16, d]
    return x.permute(1, 0, 2, 3).reshape(x.shape[1], -1, x.shape[3])[:, :n].double()


def _attend(q, k, v, first, scale):
    """q [hq, s, d], k and v [hkv, n, d] in float64; row i sees keys 0 .. first + i."""
    hq, s, _ = q.shape
    g = hq // k.shape[0]
    out = torch.empty_like(q)
    at = torch.arange(k.shape[1], device=q.device)
    for h in range(hq):
        kt = k[h // g].t().contiguous()
        for i in range(0, s, 2048):
            rows = q[h, i:i + 2048]
            last = first + i + torch.arange(rows.shape[0], device=q.device)
            logits = (rows @ kt) * scale
            logits.masked_fill_(at[None, :] > last[:, None], -math.inf)
            out[h, i:i + 2048] = torch.softmax(logits, dim=1) @ v[h // g]
    return out


def exact(case, seed):
    s = prepare(case, seed)
    op = case["op"]
    if op == "prefill":
        out = torch.empty(s["q"].shape, dtype=torch.float64, device=DEV)
        for r, p in enumerate(s["prefix_host"]):
            a, b = s["cu_host"][r], s["cu_host"][r + 1]
            n = p + b - a
            k, v = _gather(s["k"], s["tables"][r], n), _gather(s["v"], s["tables"][r], n)
            out[a:b] = _attend(s["q"][a:b].transpose(0, 1).double(), k, v, p,
                               s["scale"]).transpose(0, 1)
        return out
    if op in ("decode", "cascade"):
        out = torch.empty(s["q"].shape, dtype=torch.float64, device=DEV)
        hkv = case["hkv"]
        g = case["hq"] // hkv
        for r, n in enumerate(s["lens_host"]):
            k, v = _gather(s["k"], s["tables"][r], n), _gather(s["v"], s["tables"][r], n)
            q = s["q"][r].double().reshape(hkv, g, -1)
            p = torch.softmax(torch.matmul(q, k.transpose(1, 2).contiguous()) * s["scale"], dim=2)
            out[r] = torch.matmul(p, v).reshape(case["hq"], -1)
        return out
    if op == "write":
        for pool, new in ((s["k"], s["k_new"]), (s["v"], s["v_new"])):
            stored = s["slots"] >= 0
            at = s["slots"][stored].long()
            pool[at // BLOCK, :, at % BLOCK] = new[stored]
        return s["k"], s["v"]
    evicted = [p[s["victims"].long()].cpu() for p in (s["k"], s["v"])]
    s["k"][s["targets"].long()] = s["host_k"].to(DEV)
    s["v"][s["targets"].long()] = s["host_v"].to(DEV)
    return (s["k"], s["v"], *evicted)
