"""General path: runs so long that the kernels' windows of page ids, positions, masks and scales turn (64 groups of 16 slots a
window), ending at a turn, one before and one after it; and more prefill requests than the prefill kernel's prefix sums hold."""
import numpy as np
import pytest

import workloads as W
from harness import DeviceCase, align_with_oracle, oracle_out

pytestmark = pytest.mark.gpu


def assembled(st, masks):
    """With masks: some slots of some blocks dropped, some blocks wholly, and positions that leave gaps and jump back."""
    case = W.assemble(st, align_with_oracle(st)[0], pads_are_positions=not masks)
    if masks:
        rng = np.random.default_rng(3)
        for b in range(st.B):
            n = int(case.n_blocks[b])
            case.block_positions[b, :n] = np.arange(n) * (st.P + 2) + rng.choice([0, 1, 300], size=n)
            case.block_valid_mask[b, :n] &= rng.integers(0, 1 << 32, size=n, dtype=np.uint32) | rng.choice([0, 0xFFFFFFFF], size=n).astype(np.uint32)
            case.block_valid_mask[b, 1:n:7] = 0
        case.q_positions[:] = case.q_positions + 20000
    return case


def check(M, oracle_attn, case, rows):
    got, want = DeviceCase(M, case, flags=M.FLAG_FORCE_GENERAL).run(), oracle_out(oracle_attn, case, rows=rows)
    assert np.isfinite(got).all()
    sel = np.stack([got[t, h] for t, h in rows])
    # bf16 results: their own rounding and the split operands' remainder, as in the tests of the forms; fp32: sums of 16 K terms
    rel, rest = (0.0, 2.0 ** -15) if case.st.kv_dtype == "f32" else (2.0 ** -8, 2.0 ** -13)
    for i, (t, h) in enumerate(rows):
        assert (np.abs(sel[i] - want[i]) - np.abs(want[i]) * rel).max() <= np.abs(want).max() * rest, (t, h)


LONG = (4064, 4096, 4097, 8192, 8193, 12300)


@pytest.mark.parametrize("masks", [False, True])
@pytest.mark.parametrize("kv_dtype,P,D,theta,lengths", [(t, P, D, theta, LONG) for t, P in (("bf16", 16), ("f8e4m3", 32))
                                                        for D, theta in ((64, 5e5), (128, 5e5), (128, 1.5e5))]
                         + [("f32", 16, 64, 5e5, (8176, 8192, 8193, 16384, 16400))])
def test_decode_windows(mepic, oracle_attn, kv_dtype, P, D, theta, lengths, masks):
    """512 (token, KV head) pairs, so that one workgroup takes a context whole: four waves with runs of 32, 33, 64, 65 and 97
    steps of 32 slots (fp32: eight waves, 64, 65, 128 and 129 groups of 16). D 128: half the pairs by terms, tables of 256 and of 128 slots."""
    st = W.Structure("windows", "decode", 64, 8, 8, D, P, theta, "f32" if kv_dtype == "f32" else "bf16", kv_dtype, 91)
    st.requests, st.n_q, st.extra_tail = [[(0, n, 0)] for n in lengths] + [[(0, 5, 0)]] * (64 - len(lengths)), [1] * 64, 0
    case = assembled(st, masks)
    rows = [(b, (b + i) % 8) for b in range(len(lengths)) for i in range(3)] + [(63, 7)]
    check(mepic, oracle_attn, case, rows)


@pytest.mark.parametrize("masks", [False, True])
@pytest.mark.parametrize("kv_dtype,P", [("bf16", 16), ("f8e4m3", 32)])
@pytest.mark.parametrize("length", [1024, 1025, 2048, 2049, 2112, 3137])
def test_prefill_windows(mepic, oracle_attn, length, kv_dtype, P, masks):
    """Four workgroups a KV head and four requests of the same length: each takes one of them whole, 16 to 50 tiles of 64 slots
    (16 a window)."""
    st = W.Structure("windows", "prefill", 4, 64, 64, 64, P, 5e5, "bf16", kv_dtype, 92)
    shared = length // 32 * 32 - 32
    st.requests, st.n_q, st.extra_tail = [[(1, shared, W.CHUNK_KEY_BASE + 1), (0, length - shared, 0)]] * 4, [6, 5, 5, 7], 0
    case = assembled(st, masks)
    assert (case.kv_lens == length).all()
    rng = np.random.default_rng(4)
    rows = [(t, int(h)) for t in range(0, case.n_q, 2) for h in rng.integers(0, 64, size=3)]
    check(mepic, oracle_attn, case, rows)


@pytest.mark.parametrize("B", [2048, 2049])
def test_more_prefill_requests_than_the_row_tiles_kernel_takes(mepic, oracle_attn, B):
    st = W.Structure("many", "prefill", B, 2, 2, 64, 16, 5e5, "bf16", "bf16", 93)
    st.requests, st.n_q, st.extra_tail = [[(0, 6 + b % 30, 0)] for b in range(B)], [3 + b % 3 for b in range(B)], 0
    case = assembled(st, False)
    rng = np.random.default_rng(5)
    rows = [(int(t), int(t) % 2) for t in rng.integers(0, case.n_q, size=400)] + [(case.n_q - 1, 1)]
    check(mepic, oracle_attn, case, rows)
