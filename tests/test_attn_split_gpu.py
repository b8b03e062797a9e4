"""The general path's matrix-core kernels (split precision) against the fp64 oracle: every form they take, at the edges of their
tiles, on values of unit variance (large ones: test_split_precision_gpu.py). Their error there is the output's own rounding to bf16
(half an ulp of an 8-bit significand, 2^-8 of the value) plus a remainder of the operands' 2^-18 terms, bounded here by 2^-13 of the
largest output."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
from harness import DeviceCase, align_with_oracle, oracle_out

pytestmark = pytest.mark.gpu


def within_output_rounding(got, want):
    assert np.isfinite(got).all()
    excess = np.abs(got - want) - np.abs(want) * 2.0 ** -8
    assert excess.max() <= np.abs(want).max() * 2.0 ** -13, f"{excess.max():.3e}"


def question_prefill(seed, n_q, kv_dtype="bf16", D=128, P=16, Hq=28, Hkv=4, chunk=150, **kw):
    st = W.prefill_structure("split_prefill", seed, B=len(n_q), Hq=Hq, Hkv=Hkv, D=D, P=P, theta=5e5, n_chunks=3,
                             chunk_tokens=chunk, pool=3, q_tokens=1, max_gap_pages=2, kv_dtype=kv_dtype, **kw)
    st.n_q = list(n_q)
    for b, n in enumerate(n_q):
        st.requests[b][-1] = (0, n + 5 * b, 0)
    return st


def check(M, oracle_attn, st, pads_are_positions=True, interleaved=False, change=None):
    case = W.assemble(st, align_with_oracle(st)[0], pads_are_positions=pads_are_positions)
    if change:
        change(case)
    dc = DeviceCase(M, case, flags=M.FLAG_FORCE_GENERAL | (M.FLAG_ROPE_INTERLEAVED if interleaved else 0))
    got = dc.run()
    within_output_rounding(got, oracle_out(oracle_attn, case, interleaved=interleaved))
    return case, dc


@pytest.mark.parametrize("pads_are_positions", [True, False])
@pytest.mark.parametrize("interleaved", [False, True])
@pytest.mark.parametrize("P", [16, 32])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kv_dtype", ["bf16", "f8e4m3"])
def test_prefill_forms(mepic, oracle_attn, kv_dtype, D, P, interleaved, pads_are_positions):
    """Rows cross token boundaries (G = 7), one request fills more than a row tile, one only part of a wave."""
    check(mepic, oracle_attn, question_prefill(5, [37, 90, 3], kv_dtype, D, P), pads_are_positions, interleaved)


@pytest.mark.parametrize("Hq,Hkv,n_q", [(1, 1, [257]), (16, 1, [16, 17, 1]), (12, 12, [1, 300]), (10, 2, [51, 52])])
@pytest.mark.parametrize("chunk", [5, 64, 700])
def test_prefill_row_tiles_and_contexts(mepic, oracle_attn, Hq, Hkv, n_q, chunk):
    """One row past a tile, exactly a tile, contexts of one tile and of several splits."""
    check(mepic, oracle_attn, question_prefill(9, n_q, "bf16", Hq=Hq, Hkv=Hkv, chunk=chunk), chunk != 64)


@pytest.mark.parametrize("Hkv", [1, 3])
def test_prefill_work_cut_across_requests(mepic, oracle_attn, Hkv):
    """More requests than a wave scans at once, of very different lengths, some without queries or without slots: runs of
    the work sequence begin and end anywhere, row tiles come whole and in pieces."""
    rng = np.random.default_rng(23)
    n_q = [int(x) for x in rng.integers(0, 40, size=70)]
    n_q[3], n_q[50] = 0, 300
    st = question_prefill(23, n_q, "bf16", P=32, Hq=4 * Hkv, Hkv=Hkv, chunk=90)
    st.requests[50].insert(0, (0, 3000, 0))

    def change(case):
        case.kv_lens[[5, 60]] = 0
    check(mepic, oracle_attn, st, change=change)


@pytest.mark.parametrize("kv_dtype,P", [("bf16", 16), ("bf16", 32), ("f8e4m3", 32)])
def test_prefill_non_finite_values_reach_only_the_rows_that_see_them(mepic, oracle_attn, kv_dtype, P):
    """V of a question token that holds Inf (fp8: the NaN code, which the scalar body reads as 480): rows before it stay
    what they were, rows that see it get the Inf."""
    st = question_prefill(13, [40, 9], kv_dtype, P=P)
    case = W.assemble(st, align_with_oracle(st)[0])
    slot = int(case.q_positions[25])
    page = int(case.block_tables[0, slot // P])
    if kv_dtype == "bf16":
        case.pages.v[page, 1, 3, slot % P] = float("inf")
    else:
        case.pages.v.view(torch.uint8)[page, 1, 3, slot % P] = 0x7F
    got = DeviceCase(mepic, case, flags=mepic.FLAG_FORCE_GENERAL).run()
    want = oracle_out(oracle_attn, case)
    hit = np.zeros(got.shape, dtype=bool)
    hit[25:40, 7:14, 3] = True                       # the rows from that token on, the KV head's group, the dim
    if kv_dtype == "bf16":
        assert (got[hit] == np.inf).all() and (want[hit] == np.inf).all()
    within_output_rounding(got[~hit], want[~hit])


def test_prefill_non_finite_in_more_places_than_are_listed(mepic, oracle_attn):
    """Every request has an Inf, and a workgroup gets more row tiles than it can list for the scalar body: all are done again."""
    st = question_prefill(29, [5] * 150, "bf16", D=64, Hq=64, Hkv=64, chunk=20)
    case = W.assemble(st, align_with_oracle(st)[0])
    case.pages.v[:, :, 3, 0] = float("inf")                   # slot 0 of every block, dim 3: visible to every row
    case.pages.v[:, :, 3, 1:] = 0.0
    got, want = DeviceCase(mepic, case, flags=mepic.FLAG_FORCE_GENERAL).run(), oracle_out(oracle_attn, case)
    assert (got[:, :, 3] == np.inf).all() and (want[:, :, 3] == np.inf).all()
    rest = np.arange(64) != 3
    within_output_rounding(got[:, :, rest], want[:, :, rest])


def test_prefill_smaller_workspace_and_refusal(mepic, oracle_attn):
    """The size query reports what the even cut of the work needs; less, down to what the scalar kernel's plan needed, still
    runs, and less than that is refused."""
    st = question_prefill(17, [60, 33], "f8e4m3", P=32, chunk=900)
    case, dc = check(mepic, oracle_attn, st)
    want = oracle_out(oracle_attn, case)
    least = case.n_q * st.Hq * (st.D + 2) * 4
    full = dc.params.workspace_bytes
    assert full >= 4 * least
    rows = case.n_q * st.Hkv
    scalar_splits = min(-(-2048 // rows), -(-int(case.kv_lens.max()) // 256))
    for room in (full - 1, scalar_splits * least):
        dc.params.workspace_bytes = room
        within_output_rounding(dc.run(), want)
    dc.params.workspace_bytes = least - 1
    assert mepic.load().mepic_attn_prefill(ctypes.byref(dc.params), None) == mepic.ERR_CAPACITY


# ------------------------------------------------------------------ decode, and prefill of a few rows
def ragged_decode(seed, kv_dtype="bf16", D=128, P=16, Hq=28, Hkv=4, **kw):
    base = dict(B=5, theta=5e5, q_dtype="bf16", prefix=45, n_chunks=(1, 9), chunk_tokens=150, pool=4, question=37)
    base.update(kw)
    return W.decode_structure("split_decode", seed, Hq=Hq, Hkv=Hkv, D=D, P=P, kv_dtype=kv_dtype, **base)


@pytest.mark.parametrize("pads_are_positions", [True, False])
@pytest.mark.parametrize("interleaved", [False, True])
@pytest.mark.parametrize("P", [16, 32])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kv_dtype", ["bf16", "f8e4m3"])
def test_decode_forms(mepic, oracle_attn, kv_dtype, D, P, interleaved, pads_are_positions):
    check(mepic, oracle_attn, ragged_decode(7, kv_dtype, D, P), pads_are_positions, interleaved)
    few = question_prefill(11, [1, 2, 1], kv_dtype, D, P, Hq=3, Hkv=3)      # below the row tiles' line
    check(mepic, oracle_attn, few, pads_are_positions, interleaved)


@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (28, 4), (32, 2)])
@pytest.mark.parametrize("n_q", [[1], [2, 2, 2], [2, 4, 3], [5, 5]])
def test_prefill_of_few_tokens(mepic, oracle_attn, n_q, Hq, Hkv):
    """Both sides of the line between the two prefill kernels, which goes by tokens, for several group sizes."""
    check(mepic, oracle_attn, question_prefill(31, n_q, "bf16", P=32, Hq=Hq, Hkv=Hkv, chunk=700))


@pytest.mark.parametrize("length", [1, 15, 16, 17, 32, 33, 128, 129, 256, 257, 1025, 5000])
@pytest.mark.parametrize("Hq,Hkv", [(16, 1), (4, 4)])
def test_decode_lengths(mepic, oracle_attn, length, Hq, Hkv):
    """Group, step, table, wave and split edges (one request, the most splits)."""
    st = W.Structure("len", "decode", 2, Hq, Hkv, 128, 16, 5e5, "bf16", "bf16", 51)
    st.requests, st.n_q, st.extra_tail = [[(0, length, 0)], [(0, 1 + length // 2, 0)]], [1, 1], 0
    check(mepic, oracle_attn, st)


@pytest.mark.parametrize("prefill", [False, True])
@pytest.mark.parametrize("P", [16, 32])
def test_block_positions_in_any_order(mepic, oracle_attn, P, prefill):
    """Blocks whose positions jump back and forth by more than the rotation table holds, inside a step and between
    steps, with some blocks wholly masked."""
    def scatter(case):
        rng = np.random.default_rng(5)
        for b in range(case.st.B):
            n = int(case.n_blocks[b])
            case.block_positions[b, :n] = rng.permutation(n) * (P + 3) * rng.choice([1, 7], size=n)
            case.block_valid_mask[b, : n - 1 : 5] = 0
        case.q_positions[:] = case.q_positions + 3000 if not prefill else rng.integers(200, 4000, size=case.n_q)

    st = question_prefill(15, [30, 61], "bf16", P=P) if prefill else ragged_decode(15, "bf16", P=P)
    check(mepic, oracle_attn, st, pads_are_positions=False, change=scatter)


def spread_blocks(case):
    """Of every three requests one whose block positions jump by a step, by less than the whole rotation table and by more, one with 16
    slots left out after every second block, and one without gaps."""
    P, n_all = case.st.P, case.block_positions.shape[1]
    steps = np.array([0, 0, 0, 32, 0, 64, 0, 0, 120, 0, 300, 0])[np.arange(n_all) % 12]
    for b in range(case.st.B):
        n = int(case.n_blocks[b])
        gaps = (np.cumsum(steps), 16 * (np.arange(n_all) // 2), np.zeros(n_all, dtype=np.int64))[(b + n) % 3]
        case.block_positions[b, :n] = (P * np.arange(n_all) + gaps)[:n]
    case.q_positions[:] = case.q_positions + 3000


def one_length_in_seven_short(name, B, Hkv, length, **kw):
    st = W.Structure(name, "decode", B, 2 * Hkv, Hkv, **kw)
    st.requests, st.n_q, st.extra_tail = [[(0, length if b % 7 < 6 else 1 + length // 5, 0)] for b in range(B)], [1] * B, 0
    return st


@pytest.mark.parametrize("B,Hkv,length", [
    (1, 4, 20), (1, 4, 32), (1, 4, 33), (1, 4, 129), (1, 4, 300), (1, 4, 513),  # uncut, 1 1 1 2 3 5 steps a wave
    (1, 4, 900), (1, 4, 4200),                                                  # four parts and seventeen of two steps a wave
    (60, 3, 1000), (60, 3, 1250), (60, 3, 1600), (60, 3, 2000), (60, 3, 2400),  # three parts of 3, 4, 5, 6, 7 steps
    (60, 3, 2800), (60, 5, 4200),      # three of 8, two of 17; more than two workgroups a compute unit, so no turns
    (60, 5, 700), (60, 5, 900), (60, 5, 1100),  # uncut, 300 workgroups: 6 steps, and by turns 8 and 9
    (32, 4, 4000),                     # four parts of 8 steps, 512 workgroups: by turns
])
@pytest.mark.parametrize("D,P,kv_dtype,theta,interleaved", [
    (64, 16, "bf16", 1e4, False), (128, 16, "bf16", 1e4, False), (128, 16, "bf16", 2e5, False), (128, 16, "bf16", 5e5, False),
    (128, 32, "f8e4m3", 1e4, False), (128, 32, "f8e4m3", 5e5, False), (128, 16, "bf16", 5e5, True)])
def test_decode_tables(mepic, oracle_attn, D, P, kv_dtype, theta, interleaved, B, Hkv, length):
    """Rotation tables of every size, of 128 slots and of 256, for runs with and without gaps; with many requests, one in seven so much
    shorter than the others that its last parts are short or empty. The steps of a wave and the workgroups are those of 256 compute units."""
    st = one_length_in_seven_short("tables", B, Hkv, length, D=D, P=P, theta=theta, q_dtype="bf16", kv_dtype=kv_dtype, seed=52)
    check(mepic, oracle_attn, st, pads_are_positions=False, interleaved=interleaved, change=spread_blocks)


@pytest.mark.parametrize("kv_dtype", ["bf16", "f8e4m3"])
def test_decode_non_finite_values(mepic, oracle_attn, kv_dtype):
    """Inf (fp8: the NaN code) in a visible V element reaches its dim of the rows that read it and nothing else."""
    st = ragged_decode(19, kv_dtype, P=32)
    case = W.assemble(st, align_with_oracle(st)[0])
    page = int(case.block_tables[2, 0])              # the private prefix of request 2
    if kv_dtype == "bf16":
        case.pages.v[page, 3, 100, 4] = float("-inf")
    else:
        case.pages.v.view(torch.uint8)[page, 3, 100, 4] = 0xFF
    got = DeviceCase(mepic, case, flags=mepic.FLAG_FORCE_GENERAL).run()
    want = oracle_out(oracle_attn, case)
    hit = np.zeros(got.shape, dtype=bool)
    hit[2, 21:28, 100] = True
    assert kv_dtype != "bf16" or (got[hit] == -np.inf).all()
    within_output_rounding(got[~hit], want[~hit])


# ------------------------------------------------------------------ fp32 pages
@pytest.mark.parametrize("pads_are_positions", [True, False])
@pytest.mark.parametrize("interleaved", [False, True])
@pytest.mark.parametrize("P", [16, 32])
@pytest.mark.parametrize("D", [64, 128])
def test_f32_forms_lengths_and_positions(mepic, oracle_attn, D, P, interleaved, pads_are_positions):
    """Decode of lengths around the group, wave, table and split edges, prefill of a few tokens, and block positions in any
    order. Rounding of sums of a few thousand fp32 terms and of phases good to 2^-24 of a turn: 2^-15 of the largest output
    leaves a factor of ten over what is measured."""
    st = W.Structure("f32", "decode", 14, 10, 2, D, P, 5e5, "f32", "f32", 61)
    for n in (1, 15, 16, 17, 33, 127, 128, 129, 257, 700, 1025, 2049, 3000, 5001):
        st.requests.append([(0, n, 0)] if n < 200 else [(0, 21, 0), (1, n // 2, W.CHUNK_KEY_BASE + n), (0, n - n // 2, 0)])
        st.n_q.append(1)
    pre = W.prefill_structure("f32p", 62, B=3, Hq=10, Hkv=2, D=D, P=P, theta=5e5, n_chunks=2, chunk_tokens=150, pool=3,
                              q_tokens=1, max_gap_pages=2, q_dtype="f32", kv_dtype="f32")
    pre.n_q = [1, 9, 20]
    for b, n in enumerate(pre.n_q):
        pre.requests[b][-1] = (0, n + 5 * b, 0)
    for s in (st, pre):
        case = W.assemble(s, align_with_oracle(s)[0], pads_are_positions=pads_are_positions)
        if not pads_are_positions:
            rng = np.random.default_rng(6)
            for b in range(s.B):
                n = int(case.n_blocks[b])
                case.block_positions[b, :n] = rng.permutation(n) * (P + 3)
            case.q_positions[:] = rng.integers(100, 7000, size=case.n_q)
        got = DeviceCase(mepic, case, flags=mepic.FLAG_ROPE_INTERLEAVED if interleaved else 0).run()
        want = oracle_out(oracle_attn, case, interleaved=interleaved)
        assert np.isfinite(got).all() and np.abs(got - want).max() <= np.abs(want).max() * 2.0 ** -15


@pytest.mark.parametrize("B,Hkv,length", [
    (1, 4, 20), (1, 4, 130), (1, 4, 300), (1, 4, 700), (1, 4, 3000), (20, 4, 1000), (20, 3, 2000),  # up to six groups of slots a wave
    (32, 8, 3600), (32, 4, 7300), (40, 8, 3600)])  # D 128: 29, in 256 workgroups of one part, 256 of two, 320 of one: by turns
@pytest.mark.parametrize("D,interleaved", [(64, False), (128, False), (128, True)])
def test_f32_tables(mepic, oracle_attn, D, interleaved, B, Hkv, length):
    """Parts of the rotation table, for runs of groups with and without gaps, and waves that take turns. Bound as above."""
    st = one_length_in_seven_short("f32tab", B, Hkv, length, D=D, P=16, theta=5e5, q_dtype="f32", kv_dtype="f32", seed=64)
    case = W.assemble(st, align_with_oracle(st)[0], pads_are_positions=False)
    spread_blocks(case)
    got = DeviceCase(mepic, case, flags=mepic.FLAG_ROPE_INTERLEAVED if interleaved else 0).run()
    want = oracle_out(oracle_attn, case, interleaved=interleaved)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= np.abs(want).max() * 2.0 ** -15


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_parts", [63, 64, 65, 130])
def test_many_partials_of_a_row(mepic, oracle_attn, n_parts, dtype, D):
    """One request on one KV head, cut into parts of 256 slots: rows of fewer partials than a turn of the merge takes (64), of as many,
    one more and over two turns, with 256 threads (8 rows)."""
    st = W.Structure("parts", "decode", 1, 8, 1, D, 16, 5e5, dtype, dtype, 65)
    st.requests, st.n_q, st.extra_tail = [[(0, 256 * n_parts - 5, 0)]], [1], 0
    case = W.assemble(st, align_with_oracle(st)[0])
    dc = DeviceCase(mepic, case, flags=mepic.FLAG_FORCE_GENERAL)
    assert dc.params.workspace_bytes >= n_parts * st.Hq * (D + 2) * 4
    got, want = dc.run(), oracle_out(oracle_attn, case)
    if dtype == "bf16":
        within_output_rounding(got, want)
    else:
        assert np.abs(got - want).max() <= np.abs(want).max() * 2.0 ** -15


def test_f32_non_finite_values(mepic, oracle_attn):
    st = W.Structure("f32inf", "decode", 2, 8, 2, 128, 16, 5e5, "f32", "f32", 63)
    st.requests, st.n_q = [[(0, 300, 0)], [(0, 50, 0)]], [1, 1]
    case = W.assemble(st, align_with_oracle(st)[0])
    case.pages.v[int(case.block_tables[0, 2]), 1, 77, 3] = float("inf")
    got, want = DeviceCase(mepic, case).run(), oracle_out(oracle_attn, case)
    hit = np.zeros(got.shape, dtype=bool)
    hit[0, 4:8, 77] = True
    assert (got[hit] == np.inf).all() and np.abs(got[~hit] - want[~hit]).max() <= 1e-4
