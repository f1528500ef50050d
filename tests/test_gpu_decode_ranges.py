"""GPU parity of the decode launches that deal their keys to one-wave
work-groups in ranges (cs_paged_decode_attn_ws, which ops.cs_paged_decode_attn
calls).

Sizes sit at the edges of the plan: one sequence; lengths around the 32-key
unit and the 16-token block; many more units than ranges and fewer; sequences
cut over many ranges beside whole ones; KV head counts that leave the ranges
uneven; more than 64 sequences (one lane each); a bound far above the lengths;
and the same for sequences that share their first blocks, with sharing that starts
and ends around the probed block.  Launches of enough shared units cut every sequence
at the same positions: batches past one and two lanes' worth of sequences, beside
sequences that share nothing, and on both sides of the rule.  Each
output is compared with the float64 oracle over every element, and with the
one-work-group-per-pair call, whose partial sums differ only in order.
"""

import numpy as np
import pytest

import oracle
from gpu_util import MAX_ABS, MEAN_ABS, poison_tails
from paper_2608_14624_amd.workload import Invocation, build_workload, decode_view

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).cuda()
    return torch.from_numpy(a).cuda()


def workload(lens, hq, hkv, d, anchors=None):
    """Sequences of ``lens`` keys, sequence i the agent i's alone; with
    ``anchors``, agent i % len(anchors)'s, whose anchor of that many tokens it
    shares (its own keys: ``lens``)."""
    n = len(anchors) if anchors else len(lens)
    invs = [Invocation(i % n, x) for i, x in enumerate(lens)]
    blocks = sum(-(-x // 16) + 1 for x in lens) + sum(-(-a // 16) for a in anchors or []) + 2
    return build_workload("ranges", 81, anchors or [0] * n, invs, num_q_heads=hq, num_kv_heads=hkv,
                          head_dim=d, num_blocks=blocks)


def bits(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


# name: lengths, Hq, Hkv, D, bound on the lengths (None: the longest)[, anchors]
CASES = {
    "one_sequence": ([5000], 32, 8, 128, None),
    "one_short_sequence_loose_bound": ([1], 8, 2, 64, 8192),
    "unit_edges": ([127, 128, 129, 31, 32, 33, 255, 256, 257, 15, 16, 17, 500], 32, 8, 128, None),
    "unit_edges_d64": ([127, 128, 129, 31, 32, 33, 255, 256, 257, 15, 16, 17, 500], 8, 2, 64, 600),
    "long_beside_short": ([1, 9000, 3, 700, 1], 16, 4, 128, None),
    "more_units_than_ranges": ([3000 + 311 * i for i in range(17)], 12, 3, 128, None),
    "one_kv_head_group_16": ([600, 2500, 40], 16, 1, 128, None),
    "group_1": ([900, 10, 1300], 6, 6, 64, None),
    "past_one_wave_of_lengths": ([1 + (37 * i) % 600 for i in range(150)], 4, 2, 64, None),
    "loose_bound": ([300, 1200, 77], 32, 8, 128, 131072),
    "shared_two": ([1, 2000], 32, 8, 128, None, [4000]),
    "shared_agents": ([5 + (131 * i) % 900 for i in range(40)], 32, 8, 128, None, [1531, 3000, 64]),
    "shared_past_one_wave": ([1 + (37 * i) % 300 for i in range(130)], 4, 4, 64, None, [700, 512]),
    "shared_at_the_probed_block": ([1, 16, 40], 8, 2, 128, None, [512]),
    "shared_short_of_the_probed_block": ([600, 700, 800], 8, 2, 128, None, [496]),
    "shared_group_16": ([30, 700, 9], 16, 1, 128, 40000, [2100]),
}
# the same, cut at the same positions
ALIGNED = {
    "agents": ([5 + (131 * i) % 900 for i in range(40)], 32, 8, 128, None, [3531, 3000, 4064]),
    "past_two_waves_of_lengths": ([1 + (37 * i) % 300 for i in range(140)], 4, 4, 64, None, [2300, 2516]),
    "two_heads": ([30 + (171 * i) % 700 for i in range(60)], 8, 2, 128, 40000, [7500]),
    "beside_short_ones": ([1 + (131 * i) % 300 for i in range(40)], 16, 8, 128, None, [5600, 5616, 5500, 0]),
}


def plan_and_output(args, bound, scale):
    """(aligned, units of a range or piece) of a call with its workspace, from the
    workspace's end, and the call's output; args as the binding takes them."""
    from paper_2608_14624_amd import ops
    q, k_pool, _, bt, _ = args
    batch, hq, d = q.shape
    num_blocks, hkv = k_pool.shape[:2]
    need = ops.paged_decode_workspace_bytes(batch, bound, hq, hkv, d)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")     # NaN everywhere
    out = torch.full_like(q, float("nan"))
    assert ops.cs_paged_decode_attn_ws_raw(*(t.data_ptr() for t in args), batch, bound, bt.shape[1], num_blocks,
                                           hq, hkv, d, 16, scale, ws.data_ptr(), need, out.data_ptr()) == ops.CS_OK
    torch.cuda.synchronize()
    return ws[-8:].view(torch.int32).tolist(), out


@pytest.mark.parametrize("name", sorted(CASES))
def test_ranges_match_oracle(name):
    check_case(name, CASES[name], False)


@pytest.mark.parametrize("name", sorted(ALIGNED))
def test_aligned_pieces_match_oracle(name):
    check_case(name, ALIGNED[name], True)


def check_case(name, case, aligned):
    from paper_2608_14624_amd import ops
    lens, hq, hkv, d, bound = case[:5]
    wl = workload(lens, hq, hkv, d, *case[5:])
    q, seq_lens = decode_view(wl)
    assert poison_tails(wl) > 0 or all(n % 16 == 0 for n in seq_lens)
    bound = bound or int(seq_lens.max())
    bt = wl.block_tables
    if bound > bt.shape[1] * 16:     # entries past a sequence's last block are not used
        bt = np.concatenate([bt, np.full((len(lens), -(-bound // 16) - bt.shape[1]), -1, np.int32)], 1)
    need = ops.paged_decode_workspace_bytes(len(lens), bound, hq, hkv, d)
    print(f"[case] ranges {name}: B={len(lens)} Hq={hq} Hkv={hkv} D={d} workspace={need}", flush=True)
    assert need > 0
    args = (dev(q), dev(wl.k_pool), dev(wl.v_pool), dev(bt), dev(seq_lens))
    out = torch.full_like(args[0], float("nan"))
    ops.cs_paged_decode_attn(*args, out, max_seq_len=bound, scale=wl.scale)
    plan, again = plan_and_output(args, bound, wl.scale)
    assert plan[0] == aligned
    assert torch.equal(out.view(torch.int16), again.view(torch.int16))
    plain = torch.full_like(out, float("nan"))
    p = [t.data_ptr() for t in args]
    assert ops.cs_paged_decode_attn_raw(*p, len(lens), bound, bt.shape[1], wl.num_blocks, hq, hkv, d,
                                        16, wl.scale, plain.data_ptr()) == ops.CS_OK
    torch.cuda.synchronize()
    samples = [(r, h, 0) for r in range(wl.batch) for h in range(hq)]
    ref = oracle.prefill_paged_attn_rows(q, wl.k_pool, wl.v_pool, wl.block_tables,
                                         seq_lens.astype(np.int32) - 1,
                                         np.arange(wl.batch + 1, dtype=np.int32), hq, hkv, wl.scale,
                                         samples).reshape(wl.batch, hq, d)
    got = oracle.bf16_bits_to_f64(bits(out))
    assert np.isfinite(got).all()
    err = np.abs(got - ref)
    print(f"    vs oracle max_abs={err.max():.3e} mean_abs={err.mean():.3e}", flush=True)
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS
    # the same bf16 products and probabilities up to each one's rounding against
    # another reference maximum: a few bf16 ulps of values of at most about 4
    assert np.abs(got - oracle.bf16_bits_to_f64(bits(plain))).max() <= MAX_ABS


def both_calls(wl, q, seq_lens):
    """Outputs (float64) of the call in ranges and of the one without a workspace."""
    from paper_2608_14624_amd import ops
    hq, hkv, d, bound = wl.num_q_heads, wl.num_kv_heads, wl.head_dim, int(seq_lens.max())
    args = (dev(q), dev(wl.k_pool), dev(wl.v_pool), dev(wl.block_tables), dev(seq_lens))
    assert ops.paged_decode_workspace_bytes(wl.batch, bound, hq, hkv, d) > 0
    out, plain = (torch.full_like(args[0], float("nan")) for _ in range(2))
    ops.cs_paged_decode_attn(*args, out, max_seq_len=bound, scale=wl.scale)
    p = [t.data_ptr() for t in args]
    assert ops.cs_paged_decode_attn_raw(*p, wl.batch, bound, wl.block_tables.shape[1], wl.num_blocks, hq,
                                        hkv, d, 16, wl.scale, plain.data_ptr()) == ops.CS_OK
    torch.cuda.synchronize()
    return [oracle.bf16_bits_to_f64(bits(t)) for t in (out, plain)]


def oracle_rows(wl, q, seq_lens):
    hq, hkv = wl.num_q_heads, wl.num_kv_heads
    samples = [(r, h, 0) for r in range(wl.batch) for h in range(hq)]
    return oracle.prefill_paged_attn_rows(q, wl.k_pool, wl.v_pool, wl.block_tables,
                                          seq_lens.astype(np.int32) - 1,
                                          np.arange(wl.batch + 1, dtype=np.int32), hq, hkv, wl.scale,
                                          samples).reshape(wl.batch, hq, wl.head_dim)


@pytest.mark.parametrize("d,length,sharing,aligned", [
    (64, 2400, 63, True),      # one agent: a little over 36 units per range and sequence that shares
    (64, 2300, 63, False),     # a little under
    (64, 9000, 1, False),      # one pair among sequences of their own
    (64, 9300, 16, True),      # a quarter of the batch
    (64, 12000, 15, False),    # less, and more units
    (128, 1800, 63, True),
    (128, 1700, 63, False),
    (128, 9000, 1, False),
])
def test_pieces_are_aligned_where_enough_is_shared(d, length, sharing, aligned):
    """Aligned pieces are for batches that mostly share: one pair of sequences
    with the same block at the probed index does not move a batch to them.  Block
    ids elsewhere are any: what they hold only has to be the same in both calls."""
    from paper_2608_14624_amd import ops
    batch, hq, hkv = 64, 16, 8
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("lengths are for 256 compute units")
    rng = np.random.default_rng(17)
    bt = rng.integers(0, 256, size=(batch, -(-length // 16)), dtype=np.int32)
    bt[:, 31] = np.maximum(np.arange(batch) - sharing, 0) + 20
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)
               for s in ((batch, hq, d), (256, hkv, 16, d), (256, hkv, 16, d)))
    args = (q, k, v, dev(bt), dev(np.full(batch, length, np.int32)))
    print(f"[case] aligned rule D={d} L={length} sharing={sharing}", flush=True)
    (took, _), out = plan_and_output(args, length, d ** -0.5)
    assert took == aligned
    plain = torch.full_like(out, float("nan"))
    assert ops.cs_paged_decode_attn_raw(*(t.data_ptr() for t in args), batch, length, bt.shape[1], 256, hq, hkv,
                                        d, 16, d ** -0.5, plain.data_ptr()) == ops.CS_OK
    torch.cuda.synchronize()
    assert (out.double() - plain.double()).abs().max().item() <= MAX_ABS


@pytest.mark.parametrize("anchors", [None, [1200]])
@pytest.mark.parametrize("d", [64, 128])
def test_ranges_are_as_close_as_the_call_without_a_workspace(d, anchors):
    """Long ranges lose no precision against the 12 partial sums of a sequence in
    the call without a workspace.  The 2-norm of about 100,000 independent roundings
    repeats to about 0.2%, so 1% is five times that."""
    lens = [2000 + (811 * i) % 3000 for i in range(32)]
    wl = workload(lens, 32, 8, d, anchors)
    q, seq_lens = decode_view(wl)
    ref = oracle_rows(wl, q, seq_lens)
    err, err_plain = (np.linalg.norm(x - ref) / np.linalg.norm(ref) for x in both_calls(wl, q, seq_lens))
    print(f"[case] precision D={d} anchors={anchors}: ranges {err:.6f}, plain {err_plain:.6f}", flush=True)
    assert err <= 1.01 * err_plain


@pytest.mark.parametrize("scale", [None, 1.5])
@pytest.mark.parametrize("d", [64, 128])
def test_ranges_with_logits_of_minus_infinity(d, scale):
    """32 keys whose logits are -inf, at the first unit of a range, inside one
    and at a sequence's start, weigh nothing, also where scale log2(e) is above 1."""
    wl = workload([3000, 700], 4, 4, d)
    wl.scale = scale or wl.scale
    q, seq_lens = decode_view(wl)
    q[:, :, 0] = 0x3F80                                    # 1.0
    ref_pool = wl.k_pool.copy()
    for r, first in ((0, 0), (0, 64), (0, 96), (0, 1024), (1, 160)):
        for b in (first // 16, first // 16 + 1):
            wl.k_pool[wl.block_tables[r, b], :, :, 0] = 0xFF80          # -inf
            ref_pool[wl.block_tables[r, b], :, :, 0] = 0xC8C3           # -399,360: exp of it is 0 as well
    got = both_calls(wl, q, seq_lens)[0]
    wl.k_pool = ref_pool
    assert np.isfinite(got).all()
    assert np.abs(got - oracle_rows(wl, q, seq_lens)).max() <= MAX_ABS


@pytest.mark.parametrize("d", [64, 128])
def test_ranges_take_a_negative_block_id_as_zeros(d):
    """Blocks without a slot (a negative id, the one that is probed for sharing among
    them) count as zero K and V and are not read, as in the call without a
    workspace."""
    wl = workload([1500, 700, 2100, 90], 8, 2, d)
    q, seq_lens = decode_view(wl)
    free = sorted(set(range(wl.num_blocks)) - set(wl.block_tables.flatten().tolist()))[0]
    zeroed = wl.block_tables.copy()
    for r, b in ((0, 0), (0, 31), (0, 93), (1, 31), (1, 32), (2, 64), (3, 5)):
        wl.block_tables[r, b] = -1 - 7 * r
        zeroed[r, b] = free
    got, plain = both_calls(wl, q, seq_lens)
    wl.block_tables = zeroed
    wl.k_pool[free] = wl.v_pool[free] = 0
    ref = oracle_rows(wl, q, seq_lens)
    assert np.isfinite(got).all() and np.isfinite(plain).all()
    assert np.abs(plain - ref).max() <= MAX_ABS
    assert np.abs(got - ref).max() <= MAX_ABS


@pytest.mark.parametrize("lens", [[0], [700, 0, 1, 2500, 0], [0, 0, 90, 4000]])
def test_ranges_write_every_row(lens):
    """A row without keys holds no number, and no other row feels it; nothing of
    what the output held before is left, as in the call without a workspace."""
    wl = workload([max(n, 1) for n in lens], 8, 2, 128)
    q, seq_lens = decode_view(wl)
    lens = np.asarray(lens, np.int32)
    args = (dev(q), dev(wl.k_pool), dev(wl.v_pool), dev(wl.block_tables), dev(lens))
    bound = max(int(seq_lens.max()), 200)
    if bound > wl.block_tables.shape[1] * 16:
        bt = np.zeros((len(lens), -(-bound // 16)), np.int32)
        bt[:, :wl.block_tables.shape[1]] = wl.block_tables
        args = args[:3] + (dev(bt),) + args[4:]
    from paper_2608_14624_amd import ops
    out = torch.full_like(args[0], 3.0)
    ops.cs_paged_decode_attn(*args, out, max_seq_len=bound, scale=wl.scale)
    torch.cuda.synchronize()
    got = oracle.bf16_bits_to_f64(bits(out))
    ref = oracle_rows(wl, q, seq_lens)
    for r, n in enumerate(lens):
        if n == 0:
            assert np.isnan(got[r]).all()
        else:
            assert np.abs(got[r] - ref[r]).max() <= MAX_ABS


def test_ranges_of_a_permuted_batch():
    """A sequence is cut where the whole batch puts its cuts, so another order may
    change low bits of its row, and no more than the roundings of the bf16
    probabilities and output."""
    lens = [300 + (811 * i) % 5000 for i in range(24)]
    wl = workload(lens, 32, 8, 128)
    q, seq_lens = decode_view(wl)
    ref = oracle_rows(wl, q, seq_lens)
    perm = np.random.default_rng(5).permutation(wl.batch)
    kw = dict(bound=int(seq_lens.max()), scale=wl.scale)
    outs = []
    for order in (np.arange(wl.batch), perm):
        args = (dev(q[order]), dev(wl.k_pool), dev(wl.v_pool), dev(wl.block_tables[order]), dev(seq_lens[order]))
        (_, per), out = plan_and_output(args, **kw)
        assert 1 < per < seq_lens.max() // 32
        outs.append(oracle.bf16_bits_to_f64(bits(out)))
        assert np.abs(outs[-1] - ref[order]).max() <= MAX_ABS
    assert np.abs(outs[1] - outs[0][perm]).max() <= MAX_ABS


@pytest.mark.parametrize("anchors", [None, [800]])
def test_ranges_on_another_stream_and_in_a_graph(anchors):
    """The workspace comes from the pool of the launch's stream: calls on two
    streams at once, and replays of a captured call, give the eager bits."""
    from paper_2608_14624_amd import ops
    wl = workload([1500, 4100, 90], 32, 8, 128, anchors)
    q, seq_lens = decode_view(wl)
    args = (dev(q), dev(wl.k_pool), dev(wl.v_pool), dev(wl.block_tables), dev(seq_lens))
    kw = dict(max_seq_len=int(seq_lens.max()), scale=wl.scale)
    want = torch.empty_like(args[0])
    ops.cs_paged_decode_attn(*args, want, **kw)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [torch.full_like(want, float("nan")) for _ in range(8)]
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        s = streams[i % 2]
        ops.cs_paged_decode_attn(*args, o, stream=s if i < 4 else s.cuda_stream, **kw)
    torch.cuda.synchronize()
    assert all(torch.equal(o.view(torch.int16), want.view(torch.int16)) for o in outs)
    graph = torch.cuda.CUDAGraph()
    out = torch.empty_like(want)
    with torch.cuda.graph(graph):
        ops.cs_paged_decode_attn(*args, out, **kw)
    for _ in range(3):
        out.fill_(float("nan"))
        eager = torch.empty_like(want)
        ops.cs_paged_decode_attn(*args, eager, **kw)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16))
        assert torch.equal(eager.view(torch.int16), want.view(torch.int16))
