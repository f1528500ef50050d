"""Host side of cs_paged_decode_attn_ws: which calls take a workspace, its
size, and the arguments it refuses before anything is enqueued."""

import pytest

ops = pytest.importorskip("paper_2608_14624_amd.ops",
                          reason="libcachescout.so not built (run __graft_entry__.build())")


def need(batch, hq, hkv, d, cus=256):
    return (2 * max(1, 8 * cus // hkv) + batch) * hq * (d + 2) * 4 + 8


@pytest.mark.parametrize("args,expect", [
    # batch, longest sequence, Hq, Hkv, D, compute units
    ((1, 129, 32, 8, 128, 256), need(1, 32, 8, 128)),
    ((1, 128, 32, 8, 128, 256), 0),
    ((1024, 5000, 32, 8, 128, 256), need(1024, 32, 8, 128)),
    ((1025, 5000, 32, 8, 128, 256), 0),
    ((32, 512, 32, 8, 64, 256), 0),                       # one round of 256 pairs
    ((33, 512, 32, 8, 64, 256), need(33, 32, 8, 64)),
    ((32, 513, 32, 8, 64, 256), need(32, 32, 8, 64)),
    ((2, 4000, 12, 3, 128, 100), need(2, 12, 3, 128, 100)),
    ((2, 4000, 4096, 4096, 128, 256), need(2, 4096, 4096, 128)),
    ((0, 4000, 32, 8, 128, 256), 0),
    ((-1, 4000, 32, 8, 128, 256), -1),
    ((1, -1, 32, 8, 128, 256), -1),
    ((1, 4000, 32, 5, 128, 256), -1),
    ((1, 4000, 32, 8, 96, 256), -1),
    ((1, 4000, 32, 0, 128, 256), -1),
])
def test_workspace_bytes(args, expect):
    assert ops.paged_decode_workspace_bytes(*args) == expect


FAKE = 1 << 20   # a 16-byte aligned non-null address; never dereferenced here


@pytest.mark.parametrize("kw,status", [
    (dict(batch=-1), ops.CS_ERR_INVALID_ARG),
    (dict(head_dim=96), ops.CS_ERR_UNSUPPORTED),
    (dict(num_q_heads=64, num_kv_heads=2), ops.CS_ERR_UNSUPPORTED),
    (dict(scale=0.0), ops.CS_ERR_UNSUPPORTED),
    (dict(q=None), ops.CS_ERR_INVALID_ARG),
    (dict(workspace_bytes=-1), ops.CS_ERR_INVALID_ARG),
    (dict(batch=0, q=None, workspace=None, workspace_bytes=0), ops.CS_OK),
])
def test_decode_ws_arguments_before_any_gpu_call(kw, status):
    args = dict(q=FAKE, k_pool=FAKE, v_pool=FAKE, block_tables=FAKE, seq_lens=FAKE, batch=2,
                max_seq_len=1000, max_blocks_per_seq=63, num_blocks=64, num_q_heads=8,
                num_kv_heads=2, head_dim=64, block_size=16, scale=0.125, workspace=FAKE,
                workspace_bytes=1 << 30, out=FAKE, stream=0)
    args.update(kw)
    assert ops.cs_paged_decode_attn_ws_raw(**args) == status
