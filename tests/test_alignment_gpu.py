"""q and out at any element of a buffer: the kernels load and store rows in pieces of 8 and 16 bytes, which the memory mode of compute
queues takes at any address."""
import numpy as np
import pytest
import torch

import workloads as W
from harness import DeviceCase, align_with_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_dtype,P,flags,prefill", [("f32", 16, 0, False), ("f32", 16, 0, True), ("bf16", 16, 0, False), ("bf16", 16, 0, True),
                                                      ("bf16", 16, 2, False), ("bf16", 16, 2, True), ("f8e4m3", 32, 0, False),
                                                      ("f8e4m3", 32, 2, False), ("f8e4m3", 32, 0, True)])
def test_rows_at_any_element(mepic, kv_dtype, P, flags, prefill):
    q_dtype = "f32" if kv_dtype == "f32" else "bf16"
    kw = dict(Hq=8, Hkv=2, D=128, P=P, theta=5e5, q_dtype=q_dtype, kv_dtype=kv_dtype, chunk_tokens=160, pool=3)
    st = W.prefill_structure("odd", 98, B=3, n_chunks=3, q_tokens=30, **kw) if prefill else \
        W.decode_structure("odd", 99, B=5, prefix=48, n_chunks=(1, 9), question=37, **kw)
    dc = DeviceCase(mepic, W.assemble(st, align_with_oracle(st)[0]), flags=flags)
    want = dc.run()
    for shift in (1, 3):
        q, out = (torch.full((dc.q.numel() + 8,), 7.0, dtype=dc.q.dtype, device="cuda") for _ in range(2))
        q[shift:shift + dc.q.numel()] = dc.q.flatten()
        dc.params.q, dc.params.out = (t.data_ptr() + shift * t.element_size() for t in (q, out))
        (mepic.attn_prefill if prefill else mepic.attn_decode)(dc.params)
        got = out.double().cpu().numpy()
        assert np.array_equal(got[shift:shift + want.size].reshape(want.shape), want)
        assert (got[:shift] == 7).all() and (got[shift + want.size:] == 7).all()
