"""Calls go to the stream they are given, by default torch's current one. Each call's input is written on that stream behind some
milliseconds of other work: on another stream the call would run before it."""
import numpy as np
import pytest
import torch

import workloads as W
from harness import DeviceCase, align_with_oracle

pytestmark = pytest.mark.gpu


def decode_case():
    return W.decode_structure("streams", 95, B=5, Hq=8, Hkv=2, D=128, P=16, theta=5e5, q_dtype="bf16", kv_dtype="bf16", prefix=48,
                              n_chunks=(1, 4), chunk_tokens=160, pool=4, question=37)


def prefill_case():
    return W.prefill_structure("streams", 96, B=3, Hq=8, Hkv=2, D=128, P=16, theta=5e5, n_chunks=3, chunk_tokens=160, pool=3, q_tokens=30)


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("call,flags", [("attn_decode", 0), ("attn_decode", 2), ("attn_decode_noalloc", 0), ("attn_decode_batched", 0),
                                        ("attn_prefill", 0), ("attn_prefill", 2)])
def test_attention_runs_on_its_stream(mepic, call, flags, given):
    case = W.assemble(st := prefill_case() if call == "attn_prefill" else decode_case(), align_with_oracle(st)[0])
    dc = DeviceCase(mepic, case, flags=flags)
    args = (dc.params,)
    if call == "attn_decode_batched":
        dc.prepare_batched()
        args = (dc.params, dc.plan, dc.plan_info)
    fn = getattr(mepic, call)
    fn(*args)
    torch.cuda.synchronize()
    want, q = dc.out.clone(), dc.q.clone()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for _ in range(2):                                       # (the first call may take longer on the host than the wait on the GPU)
        dc.q.zero_()
        dc.out.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)
            dc.q.copy_(q)
            if not given:
                fn(*args)
        if given:
            fn(*args, stream=side)
        with torch.cuda.stream(side):
            got = dc.out.clone()
        side.synchronize()
        assert torch.equal(got, want)


@pytest.mark.parametrize("given", [False, True])
def test_commit_runs_on_its_stream(mepic, given):
    pages = W.gen_pages(7, 12, 2, 16, 128, "bf16")
    k, v = pages.k.cuda(), pages.v.cuda()
    i32 = lambda a: torch.tensor(np.asarray(a), dtype=torch.int32, device="cuda")
    new = torch.randn(60, 2, 128, device="cuda").to(torch.bfloat16)
    src = torch.zeros_like(new)
    p = mepic.make_commit_params(src, src, k, v, i32([[3, 9, 1, 6]]), i32([0]), i32([2]), i32([0, 60]))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        src.copy_(new)
        if not given:
            mepic.kv_commit(p)
    if given:
        mepic.kv_commit(p, stream=side)
    side.synchronize()
    rows = W.unpack_k(k.cpu())[[3, 9, 1, 6]].permute(0, 2, 1, 3).reshape(64, 2, 128)[2:62]
    assert torch.equal(rows, new.cpu())
