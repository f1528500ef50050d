"""GPU parity of cascade decode in ranges: the launches whose workspace (that of
max_shared_len / 1024 chunks and max_rest_len / 1024 segments) has the room take
both halves as lists of 32-key units dealt to one-wave work-groups.

Sizes sit at the edges of the plan: shared prefixes of one block, of an odd
number of blocks (half a unit at the end) and of many units; groups of one
sequence, of exactly 64 stacked rows, one more, and several column blocks; query
groups that do not divide a column block; groups that share nothing, empty
groups and sequences without keys of their own; more than 64 groups and
sequences (a lane each); workspaces so small that the ranges are lengthened.
Every element is compared with the float64 oracle.
"""

import numpy as np
import pytest

import oracle
from gpu_util import MAX_ABS, MEAN_ABS, poison_slot_zero, poison_tails
from paper_2608_14624_amd.workload import Invocation, build_workload, decode_view

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).cuda()
    return torch.from_numpy(a).cuda()


def takes_ranges(batch, groups, max_seqs, hq, hkv, d, max_shared, max_rest, cus=256):
    """The rule of the launch: two estimates from the host's bounds."""
    g = hq // hkv
    parts = -(-max_shared // 1024) + -(-max_rest // 1024)
    width = min(64, -(-max_seqs * g // 16) * 16)
    room = (parts * batch * hq - (6 * batch + 9) // 2) // hkv - (
        (batch * g // width + groups + 2) * width + (batch + 2) * g)
    ranges = max(1, (4 if d == 128 else 8) * cus // hkv)
    shared = -(-batch * g // width) * max_shared / 32 / ranges
    distinct = min(shared, groups * max_shared / 32 / ranges)
    own = 0.4 * batch * max_rest / 32 / ranges
    if room <= 0:
        return False
    stretch = (shared * width + own * g) * ranges / ((shared + own) * room)
    return stretch <= (2 if g == 1 else 3) and (
        max(stretch, 1) * (0.8 * (shared + own) + 1.2 * width / 64 * shared) + 1.5 * (own + distinct)
        <= 0.95 * (21 + 1.1 * shared + 3 * own + 2.5 * distinct))


@pytest.mark.parametrize("expect,batch,groups,max_seqs,hq,hkv,d,max_shared,max_rest", [
    (True, 128, 8, 16, 32, 8, 128, 8000, 4096),
    (True, 16, 4, 4, 32, 8, 128, 10000, 4000),
    (True, 160, 4, 40, 32, 8, 64, 4000, 4000),
    # prefixes streamed once per column block, and little besides
    (False, 128, 1, 128, 32, 8, 128, 8000, 200),
    (False, 64, 1, 64, 32, 8, 128, 8000, 600),
    (False, 128, 1, 128, 64, 8, 128, 2300, 600),
    (False, 160, 4, 40, 32, 8, 64, 8000, 600),
    (False, 600, 1, 600, 4, 1, 128, 3500, 1500),
    # long ranges for want of room
    (False, 32, 8, 4, 16, 16, 128, 10000, 2500),
])
def test_launches_where_ranges_are_slower_run_in_chunks(expect, batch, groups, max_seqs, hq, hkv, d, max_shared,
                                                        max_rest):
    """A launch in ranges leaves its plan behind its partials, first the few units of
    a range; in chunks the place holds the mark set here, or the bits of a float."""
    from paper_2608_14624_amd import ops
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule is evaluated for 256 compute units")
    assert takes_ranges(batch, groups, max_seqs, hq, hkv, d, max_shared, max_rest) == expect
    bound = max_shared + max_rest
    bt = torch.zeros(batch, -(-bound // 16), dtype=torch.int32, device="cuda")
    pool = torch.ones(4, hkv, 16, d, dtype=torch.bfloat16, device="cuda")
    q = torch.ones(batch, hq, d, dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(q)
    sizes = [batch // groups] * groups
    cu = dev(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))
    need = ops.cs_cascade_decode_workspace_bytes(batch, hq, d, max_shared, max_rest)
    ws = torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")
    print(f"[case] cascade route B={batch} groups={groups} Hq={hq} Hkv={hkv} D={d} {max_shared}+{max_rest}", flush=True)
    ops.cs_cascade_decode_attn(q, pool, pool, bt, dev(np.full(batch, 48, np.int32)), cu,
                               dev(np.full(groups, 32, np.int32)), out, max_seq_len=bound, max_group_seqs=max_seqs,
                               max_shared_len=max_shared, max_rest_len=max_rest, scale=d ** -0.5, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(out, torch.ones_like(out))
    parts = -(-max_shared // 1024) + -(-max_rest // 1024)
    rows = (parts * batch * hq - (6 * batch + 9) // 2) // hkv
    at = 4 * (parts * batch * hq * d + 2 * rows * hkv)                     # the plan
    per = ws[at:at + 4].view(torch.int32).item()
    assert (0 < per < 1000) == expect


def build(groups, hq, hkv, d):
    """groups: list of (shared tokens, [own tokens of each sequence]), the
    shared part whole blocks; a group may be empty."""
    anchors, invs, cu, shared = [], [], [0], []
    for s, owns in groups:
        for own in owns:
            # an invocation needs a token: one with no keys of its own is
            # decoded at the last token of the shared part
            invs.append(Invocation(len(anchors), max(own, 1)))
        anchors.append(s)
        shared.append(s)
        cu.append(cu[-1] + len(owns))
    blocks = sum(s // 16 for s, _ in groups) + sum(-(-max(o, 1) // 16) for _, os in groups for o in os) + 3
    wl = build_workload("cascade_ranges", 91, anchors, invs, num_q_heads=hq, num_kv_heads=hkv,
                        head_dim=d, num_blocks=blocks)
    own = np.asarray([o for _, os in groups for o in os])
    q, seq_lens = decode_view(wl)
    seq_lens = np.where(own == 0, seq_lens - 1, seq_lens).astype(np.int32)
    return wl, q, seq_lens, np.asarray(cu, np.int32), np.asarray(shared, np.int32)


def lens(seed, n, lo, hi):
    return [int(x) for x in np.random.default_rng(seed).integers(lo, hi, size=n, endpoint=True)]


# name: groups, Hq, Hkv, D, parts of the workspace (through the host bounds)
CASES = {
    "one_group": ([(4096, lens(1, 16, 1, 900))], 32, 8, 128, 16),
    "agents": ([(1024 * i + 16 * i, lens(i, 5 + i, 1, 400 * i)) for i in range(1, 6)], 32, 8, 128, 12),
    "agents_d64": ([(1024 * i + 16 * i, lens(i, 5 + i, 1, 400 * i)) for i in range(1, 6)], 32, 8, 64, 16),
    "half_units_and_one_block": ([(16, [1, 33, 64]), (48, [5, 31]), (32, [32, 96, 1])], 8, 2, 128, 38),
    "64_rows_and_one_more": ([(2000, lens(3, 16, 1, 50)), (1520, lens(4, 17, 1, 50))], 32, 8, 128, 10),
    "column_blocks_group_3": ([(1600, lens(5, 70, 1, 60)), (800, [3])], 12, 4, 128, 8),
    "group_16": ([(3200, lens(6, 9, 1, 300)), (0, [700, 1])], 16, 1, 128, 60),
    "group_1": ([(2048, lens(7, 30, 1, 99))], 4, 4, 64, 18),
    "nothing_shared_and_empty_groups": ([(0, lens(8, 9, 1, 1500)), (640, []), (2048, [7, 600]), (0, [])],
                                        32, 8, 128, 13),
    "no_own_keys": ([(2064, [0, 0, 5]), (1040, [0, 2000])], 8, 2, 128, 63),
    "past_one_wave": ([(16 * (1 + i % 7), lens(i, 2, 1, 80)) for i in range(70)], 4, 2, 64, 11),
    "barely_enough_room": ([(1008, lens(9, 16, 1, 1000)), (800, lens(10, 16, 1, 1000))], 32, 8, 128, 8),
}


@pytest.mark.parametrize("poison", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_cascade_ranges_match_oracle(name, poison):
    from paper_2608_14624_amd import ops
    groups, hq, hkv, d, parts = CASES[name]
    wl, q, seq_lens, cu, shared = build(groups, hq, hkv, d)
    if poison:
        poison_slot_zero(wl)
        poison_tails(wl)
    max_seqs = max(len(o) for s, o in groups if s > 0)
    max_rest = int(max(int(seq_lens[i]) - int(shared[gr]) for gr in range(len(shared))
                       for i in range(cu[gr], cu[gr + 1])))
    chunks = -(-int(shared.max()) // 1024)
    max_rest = max(max_rest, (parts - chunks) * 1024)
    bound = max(int(seq_lens.max()), max_rest)
    bt = wl.block_tables
    if bound > bt.shape[1] * 16:
        bt = np.concatenate([bt, np.full((bt.shape[0], -(-bound // 16) - bt.shape[1]), -1, np.int32)], 1)
    assert takes_ranges(wl.batch, len(shared), max_seqs, hq, hkv, d, int(shared.max()), max_rest)
    print(f"[case] cascade ranges {name}: B={wl.batch} groups={len(shared)} Hq={hq} Hkv={hkv} D={d}",
          flush=True)
    args = [dev(x) for x in (q, wl.k_pool, wl.v_pool, bt, seq_lens, cu, shared)]
    kw = dict(max_seq_len=bound, max_group_seqs=max_seqs, max_shared_len=int(shared.max()),
              max_rest_len=max_rest, scale=wl.scale)
    need = ops.cs_cascade_decode_workspace_bytes(wl.batch, hq, d, kw["max_shared_len"], max_rest)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")     # NaN everywhere
    outs = []
    for _ in range(2):                                                   # and with its own leftovers
        out = torch.full_like(args[0], float("nan"))
        ops.cs_cascade_decode_attn(*args, out, workspace=ws, **kw)
        torch.cuda.synchronize()
        outs.append(out.view(torch.int16).cpu().numpy().view(np.uint16))
    assert np.array_equal(*outs)
    samples = [(r, h, 0) for r in range(wl.batch) for h in range(hq)]
    ref = oracle.prefill_paged_attn_rows(q, wl.k_pool, wl.v_pool, wl.block_tables, seq_lens - 1,
                                         np.arange(wl.batch + 1, dtype=np.int32), hq, hkv, wl.scale,
                                         samples).reshape(wl.batch, hq, d)
    got = oracle.bf16_bits_to_f64(outs[0])
    assert np.isfinite(got).all()
    err = np.abs(got - ref)
    print(f"    vs oracle max_abs={err.max():.3e} mean_abs={err.mean():.3e}", flush=True)
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS


def test_cascade_ranges_take_a_negative_block_id_as_zeros():
    """Blocks without a slot, shared and own, count as zero K and V and are not
    read, as in the launches in chunks and segments."""
    from paper_2608_14624_amd import ops
    groups, hq, hkv, d, parts = CASES["agents"]
    wl, q, seq_lens, cu, shared = build(groups, hq, hkv, d)
    free = sorted(set(range(wl.num_blocks)) - set(wl.block_tables.flatten().tolist()))[0]
    zeroed = wl.block_tables.copy()
    for r, b in ((r, b) for gr in (1, 3) for r in range(cu[gr], cu[gr + 1])
                 for b in (2, int(shared[gr]) // 16 - 1, int(seq_lens[r] - 1) // 16)):
        wl.block_tables[r, b] = -3
        zeroed[r, b] = free
    rest = max(int(seq_lens[i]) - int(shared[gr]) for gr in range(len(shared)) for i in range(cu[gr], cu[gr + 1]))
    rest = max(rest, (parts - -(-int(shared.max()) // 1024)) * 1024)
    bound = max(int(seq_lens.max()), rest)
    bt = np.concatenate([wl.block_tables, np.full((wl.batch, max(0, -(-bound // 16) - wl.block_tables.shape[1])),
                                                  -1, np.int32)], 1)
    max_seqs = max(len(o) for _, o in groups)
    assert takes_ranges(wl.batch, len(shared), max_seqs, hq, hkv, d, int(shared.max()), rest)
    args = [dev(x) for x in (q, wl.k_pool, wl.v_pool, bt, seq_lens, cu, shared)]
    out = torch.full_like(args[0], float("nan"))
    ops.cs_cascade_decode_attn(*args, out, max_seq_len=bound, max_group_seqs=max_seqs,
                               max_shared_len=int(shared.max()), max_rest_len=rest, scale=wl.scale)
    torch.cuda.synchronize()
    wl.k_pool[free] = wl.v_pool[free] = 0
    samples = [(r, h, 0) for r in range(wl.batch) for h in range(hq)]
    ref = oracle.prefill_paged_attn_rows(q, wl.k_pool, wl.v_pool, zeroed, seq_lens - 1,
                                         np.arange(wl.batch + 1, dtype=np.int32), hq, hkv, wl.scale,
                                         samples).reshape(wl.batch, hq, d)
    got = oracle.bf16_bits_to_f64(out.view(torch.int16).cpu().numpy().view(np.uint16))
    assert np.abs(got - ref).max() <= MAX_ABS


@pytest.mark.parametrize("d", [64, 128])
def test_cascade_ranges_are_as_close_as_the_chunks(d):
    """Long ranges lose no precision against segments of 1024 keys, which the same
    batch takes with tight bounds.  The 2-norm of about 100,000 independent roundings
    repeats to about 0.2%, so 1% is five times that."""
    from paper_2608_14624_amd import ops
    batch, hq, hkv, shared_len = 48, 32, 8, 1008
    rng = np.random.default_rng(23)
    own = rng.integers(2000, 2500, size=batch)
    seq_lens = (own + shared_len).astype(np.int32)
    bound = 20 * 1024
    bt = rng.integers(0, 600, size=(batch, bound // 16), dtype=np.int32)   # any blocks
    for r in range(batch):
        bt[r, :shared_len // 16] = bt[r - r % 16, :shared_len // 16]
    pools = [rng.standard_normal((600, hkv, 16, d), dtype=np.float32) for _ in range(2)]
    q = torch.from_numpy(rng.standard_normal((batch, hq, d), dtype=np.float32)).to("cuda", torch.bfloat16)
    k, v = (torch.from_numpy(x).to("cuda", torch.bfloat16) for x in pools)
    args = (q, k, v, dev(bt), dev(seq_lens), dev(np.arange(0, 49, 16, dtype=np.int32)),
            dev(np.full(3, shared_len, np.int32)))
    kd, vd = k.double(), v.double()
    ref = torch.empty(batch, hq, d, dtype=torch.float64, device="cuda")
    for r in range(batch):
        n = int(seq_lens[r])
        ids = args[3][r, :-(-n // 16)].long()
        kr, vr = (x[ids].transpose(0, 1).reshape(hkv, -1, d)[:, :n] for x in (kd, vd))
        p = torch.softmax((q[r].double().view(hkv, -1, d) @ kr.transpose(1, 2).contiguous()) * d ** -0.5, dim=-1)
        ref[r] = (p @ vr.contiguous()).reshape(hq, d)
    errs = []
    for rest in (2500, bound - shared_len):
        assert takes_ranges(batch, 3, 16, hq, hkv, d, shared_len, rest) == (rest > 2500)
        out = torch.full_like(q, float("nan"))
        ops.cs_cascade_decode_attn(*args, out, max_seq_len=bound, max_group_seqs=16, max_shared_len=shared_len,
                                   max_rest_len=rest, scale=d ** -0.5)
        torch.cuda.synchronize()
        errs.append(((out.double() - ref).norm() / ref.norm()).item())
    print(f"[case] cascade precision D={d}: chunks {errs[0]:.6f}, ranges {errs[1]:.6f}", flush=True)
    assert errs[1] <= 1.01 * errs[0]
