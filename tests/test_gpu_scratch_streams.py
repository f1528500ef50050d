"""The scratch that the binding allocates for a launch belongs to the launch's
stream, the null stream's handle included: the segment that holds it says so, and
the outputs are those of the call on the current (null) stream, bit for bit."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

HQ, HKV, D, LEN = 32, 8, 128, 3000


def i32(*x):
    return torch.tensor(x, dtype=torch.int32, device="cuda")


def inputs(rows):
    gen = torch.Generator(device="cuda").manual_seed(5)
    blocks = -(-LEN // 16)
    k, v = (torch.randn(2 * blocks, HKV, 16, D, generator=gen, device="cuda", dtype=torch.bfloat16)
            for _ in range(2))
    q = torch.randn(rows, HQ, D, generator=gen, device="cuda", dtype=torch.bfloat16)
    order = torch.randperm(2 * blocks, generator=gen, device="cuda").to(torch.int32)
    return q, k, v, order.reshape(2, blocks).contiguous()


def decode(ops, stream):
    q, k, v, tables = inputs(2)
    out = torch.empty_like(q)
    lens = i32(LEN, 77)
    return out, lambda: ops.cs_paged_decode_attn(q, k, v, tables, lens, out, max_seq_len=LEN,
                                                 scale=D ** -0.5, stream=stream)


def prefill(ops, stream):
    q, k, v, tables = inputs(90)
    out = torch.empty_like(q)
    prefix, cu = i32(LEN - 60, 900), i32(0, 60, 90)
    return out, lambda: ops.cs_prefill_paged_attn(q, k, v, tables, prefix, cu, out, max_q_len=60,
                                                  max_kv_len=LEN, scale=D ** -0.5, workspace="auto",
                                                  stream=stream)


def cascade(ops, stream):
    q, k, v, tables = inputs(2)
    tables[1, :100] = tables[0, :100]
    out = torch.empty_like(q)
    lens, cu, shared = i32(LEN, 1700), i32(0, 2), i32(1600)
    return out, lambda: ops.cs_cascade_decode_attn(q, k, v, tables, lens, cu, shared, out, max_seq_len=LEN,
                                                   max_group_seqs=2, max_shared_len=1600,
                                                   max_rest_len=1400, scale=D ** -0.5, stream=stream)


@pytest.mark.parametrize("call", [decode, prefill, cascade])
@pytest.mark.parametrize("name", ["null handle", "null stream", "side handle", "side stream"])
def test_scratch_segment_is_the_launch_streams(call, name, monkeypatch):
    from paper_2608_14624_amd import ops
    side = torch.cuda.Stream()
    stream = {"null handle": 0, "null stream": torch.cuda.default_stream(), "side handle": side.cuda_stream,
              "side stream": side}[name]
    print(f"[case] {call.__name__} scratch on the {name}", flush=True)
    want, run = call(ops, None)
    run()
    torch.cuda.synchronize()
    taken = []
    scratch = ops._scratch
    monkeypatch.setattr(ops, "_scratch", lambda *a: taken.append(scratch(*a)) or taken[-1])
    out, run = call(ops, stream)
    torch.cuda.synchronize()               # the inputs, before another stream reads them
    run()
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))
    assert len(taken) == 1 and taken[0] is not None
    at = taken[0].data_ptr()
    holds = [s for s in torch.cuda.memory_snapshot() if s["address"] <= at < s["address"] + s["total_size"]]
    assert [s["stream"] for s in holds] == [0 if name.startswith("null") else side.cuda_stream]
