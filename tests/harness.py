"""Glue used by the GPU parity tests: run one case through the fp64 oracle (here) and through the library
(paper_2512_16822_amd.device_case)."""
from __future__ import annotations

import numpy as np
import torch

import workloads as W
from oracle import align as OA
from paper_2512_16822_amd.device_case import DeviceCase, align_with_library  # noqa: F401  (re-exported for the tests)


def align_with_oracle(st: W.Structure, num_pages: int = 1 << 20):
    pool = OA.PoolOracle(num_pages, st.P)
    return [pool.align(segs, st.extra_tail) for segs in st.requests], pool


def oracle_out(attn, case: W.Case, rows=None, interleaved=False, sm_scale=0.0) -> np.ndarray:
    st, pg = case.st, case.pages
    return attn.attention(W.raw_numpy(case.q), st.q_dtype, W.raw_numpy(pg.k), W.raw_numpy(pg.v), st.kv_dtype,
                          case.block_tables, case.kv_lens, case.q_positions, Hq=st.Hq, Hkv=st.Hkv, D=st.D, P=st.P,
                          theta=st.theta, cu_q_lens=case.cu_q_lens, k_scales=W.raw_numpy(pg.k_scales),
                          v_scales=W.raw_numpy(pg.v_scales), block_positions=case.block_positions,
                          block_valid_mask=case.block_valid_mask, rows=rows, interleaved=interleaved,
                          sm_scale=sm_scale)


def run_in_long_runs(M, case: W.Case, steps: int, flags: int = 0) -> np.ndarray:
    """The plain decode with at least `steps` steps of 32 slots a wave, however few there are for all the waves: block tables far wider than
    the lengths (and no closer bound on these) make for few partials a request, so for long parts of the work each."""
    st = case.st
    waves = max(2 * torch.cuda.get_device_properties(0).multi_processor_count // st.Hkv, 1) * 4
    pieces = min(4 * -(-waves // st.B), waves)
    width = pieces * steps * 32 // st.P
    assert width >= case.block_tables.shape[1]
    case.block_tables = np.pad(case.block_tables, ((0, 0), (0, width - case.block_tables.shape[1])))
    dc = DeviceCase(M, case, flags=flags)
    dc.params.max_kv_len = 0
    size = M.attn_workspace_size(dc.params, False)
    dc.ws = torch.empty(size, dtype=torch.uint8, device=dc.q.device)
    dc.params.workspace, dc.params.workspace_bytes = dc.ws.data_ptr(), size
    most = (size - 4 * (st.B + 2)) // (4 * st.B * st.Hq * (st.D + 2))  # partials a request: its parts and one for where they begin
    assert (most - 1) * steps <= pieces * steps, "the library means to cut the work finer"
    return dc.run()
