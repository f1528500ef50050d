"""GPU parity of ping-pong prefill launches of unequal suffixes, whose
work-groups find their tiles from the lengths: empty invocations, lengths around
the tile's tokens, a batch of more than 64 invocations (a lane each) and of more
than 256 (numbered over the longest), tile counts whose last round runs as
halves, is more than half full or is the only one, a KV head count that does
not divide the rounds, and bounds above the lengths.  Every output element is
compared with the float64 oracle.
"""

import numpy as np
import pytest

import oracle
from gpu_util import MAX_ABS, MEAN_ABS, compare_full, poison_slot_zero, poison_tails
from paper_2608_14624_amd.workload import Invocation, build_workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def ragged(seed, n, lo, hi):
    return [int(x) for x in np.random.default_rng(seed).integers(lo, hi, size=n, endpoint=True)]


# name: suffix lengths, prefix, Hq, Hkv, D, multiple of max_q_len passed
# (tiles of 64 tokens with 4 query heads per KV head, 128 with 2, 256 with 1)
CASES = {
    "tile_edges": ([64, 63, 65, 1, 128, 127, 129, 320, 640, 704, 2, 700], 100, 32, 8, 128, 1),
    "tile_edges_d64": ([64, 63, 65, 1, 128, 127, 129, 320, 640, 704, 2, 700], 100, 32, 8, 64, 1),
    "few_real_tiles": ([1300, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1], 40, 32, 8, 128, 1),
    "only_halves": ([700, 3, 9], 300, 16, 4, 128, 6),
    "past_one_wave": (ragged(1, 130, 1, 140), 33, 16, 4, 128, 1),
    "past_one_wave_d64": (ragged(2, 130, 1, 140), 33, 16, 4, 64, 1),
    "past_the_plan": (ragged(3, 270, 1, 90), 20, 8, 2, 64, 1),
    "three_kv_heads": (ragged(4, 20, 1, 600), 50, 12, 3, 128, 1),
    "group_2": (ragged(5, 12, 1, 1500), 17, 8, 4, 128, 2),
    "group_1_many_rounds": (ragged(6, 40, 1, 900), 5, 16, 16, 64, 4),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_ragged_ping_pong_matches_oracle(name):
    from paper_2608_14624_amd import ops, pipeline
    suffixes, prefix, hq, hkv, d, loose = CASES[name]
    invs = [Invocation(i % 2, s, hit=i % 5 != 4) for i, s in enumerate(suffixes)]
    blocks = sum(-(-(s + prefix + 7) // 16) + 1 for s in suffixes) + 2 * (prefix // 16 + 2) + 3
    wl = build_workload("ragged", 95, [prefix, prefix + 7], invs, num_q_heads=hq, num_kv_heads=hkv,
                        head_dim=d, num_blocks=blocks)
    poison_slot_zero(wl)
    poison_tails(wl)
    max_q = loose * wl.max_q_len
    max_kv = max(wl.max_kv_len, max_q)
    kernel, grid, tail = ops.prefill_launch_shape(wl.batch, max_q, hq, hkv)
    print(f"[case] ragged {name}: B={wl.batch} total_q={wl.total_q} grid={grid} tail={tail}", flush=True)
    assert kernel == ops.ATTN_PING_PONG
    dw = pipeline.DeviceWorkload(wl)
    bt = dw.block_tables
    if max_kv > bt.shape[1] * 16:
        pad = torch.full((bt.shape[0], -(-max_kv // 16) - bt.shape[1]), -1, dtype=torch.int32, device="cuda")
        bt = torch.cat([bt, pad], 1).contiguous()
    dw.out.fill_(float("nan"))
    ops.cs_prefill_paged_attn(dw.q, dw.k_pool, dw.v_pool, bt, dw.prefix_lens, dw.cu_q_lens, dw.out,
                              max_q_len=max_q, max_kv_len=max_kv, scale=wl.scale)
    torch.cuda.synchronize()
    ref = oracle.prefill_paged_attn(wl.q, wl.k_pool, wl.v_pool, wl.block_tables, wl.prefix_lens,
                                    wl.cu_q_lens, hq, hkv, wl.scale)
    mx, mean = compare_full(dw.out_bits(), ref)
    print(f"    vs oracle max_abs={mx:.3e} mean_abs={mean:.3e}", flush=True)
    assert mx <= MAX_ABS and mean <= MEAN_ABS


def test_empty_invocations_between_long_ones():
    """Suffix lengths of zero anywhere in the batch take no tile."""
    from paper_2608_14624_amd import ops, pipeline
    suffixes = [900, 1100, 64, 1000]
    invs = [Invocation(0, s) for s in suffixes]
    wl = build_workload("ragged_empty", 96, [160], invs, num_q_heads=32, num_kv_heads=8,
                        head_dim=128, num_blocks=256)
    dw = pipeline.DeviceWorkload(wl)
    want = torch.full_like(dw.out, float("nan"))
    ops.cs_prefill_paged_attn(dw.q, dw.k_pool, dw.v_pool, dw.block_tables, dw.prefix_lens,
                              dw.cu_q_lens, want, max_q_len=1100, max_kv_len=1260, scale=wl.scale)
    order = [None, 0, None, None, 1, 2, 3, None]       # None: an invocation without tokens
    cu, tables, prefix = [0], [], []
    for r in order:
        cu.append(cu[-1] + (suffixes[r] if r is not None else 0))
        tables.append(dw.block_tables[0 if r is None else r])
        prefix.append(160)
    out = torch.full_like(dw.out, float("nan"))
    ops.cs_prefill_paged_attn(dw.q, dw.k_pool, dw.v_pool, torch.stack(tables).contiguous(),
                              torch.tensor(prefix, dtype=torch.int32, device="cuda"),
                              torch.tensor(cu, dtype=torch.int32, device="cuda"), out,
                              max_q_len=1100, max_kv_len=1260, scale=wl.scale)
    torch.cuda.synchronize()
    diff = (out.float() - want.float()).abs().max().item()
    assert diff <= MAX_ABS and torch.isfinite(out.float()).all()
