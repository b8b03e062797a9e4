"""NaN, Inf and very large values on every attention path: a row is zeros only where no slot takes part; a NaN or Inf that a row
reads is in the row, wherever the context is cut; and what a row does not read is not."""
import numpy as np
import pytest
import torch

import workloads as W
from harness import DeviceCase, align_with_oracle, oracle_out, run_in_long_runs

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2, "f8e4m3": 2e-2}

# kv_dtype, P, general path, prefill, planned
PATHS = [("bf16", 16, False, False, False), ("f8e4m3", 32, False, False, False), ("bf16", 16, False, False, True),
         ("f8e4m3", 32, False, False, True), ("bf16", 16, True, False, False), ("f32", 16, True, False, False),
         ("bf16", 16, True, True, False), ("f32", 16, True, True, False)]


def structure(kv_dtype, P, prefill, lengths):
    st = W.Structure("nonfinite", "prefill" if prefill else "decode", len(lengths), 8, 2, 128, P, 5e5,
                     "f32" if kv_dtype == "f32" else "bf16", kv_dtype, 81)
    st.requests, st.extra_tail = [[(0, n, 0)] for n in lengths], 0
    st.n_q = [min(n, 40) if prefill else 1 for n in lengths]
    return st


def run(M, case, general, planned):
    dc = DeviceCase(M, case, flags=M.FLAG_FORCE_GENERAL if general else 0)
    return dc.run_batched() if planned else dc.run()


def set_k(pages, page, slot, dim, value):
    X = pages.k.shape[-1]
    if pages.kv_dtype == "f8e4m3":
        assert value != value
        pages.k.view(torch.uint8)[page, :, dim // X, slot, dim % X] = 0x7F
    else:
        pages.k[page, :, dim // X, slot, dim % X] = value


@pytest.mark.parametrize("kv_dtype,P,general,prefill,planned", PATHS)
def test_a_nan_key_reaches_the_rows_that_see_it(mepic, oracle_attn, kv_dtype, P, general, prefill, planned):
    """One element of one key in a long context (many partials), in a short one (written directly), and the only key there is."""
    case = W.assemble(s := structure(kv_dtype, P, prefill, [6000, 200, 1, 700]), align_with_oracle(s)[0])
    for b, n in ((0, 5995), (1, 170), (2, 0)):  # (in prefill some of the query tokens come before it)
        set_k(case.pages, int(case.block_tables[b, n // P]), n % P, 17, float("nan"))
    got, want = run(mepic, case, general, planned), oracle_out(oracle_attn, case)
    hit = np.isnan(want)
    assert hit[-1].any() == False and hit.any() and (np.isnan(got) == hit).all()
    assert np.abs(got[~hit] - want[~hit]).max() <= TOL[kv_dtype]


@pytest.mark.parametrize("value", ["nan", "inf"])
@pytest.mark.parametrize("kv_dtype,P,general,prefill,planned", PATHS)
def test_a_non_finite_value_under_a_vanishing_weight(mepic, oracle_attn, kv_dtype, P, general, prefill, planned, value):
    """Scores some 400 log2 units higher at the end of the context than before: V at its beginning has no weight in fp32, but
    0 x Inf is not 0, whether the two meet inside one partial or when partials are merged."""
    case = W.assemble(s := structure(kv_dtype, P, prefill, [6000, 100]), align_with_oracle(s)[0])
    k, n = W.unpack_k(case.pages.k.float()), 5900          # a key along the pair of dims that hardly turns, and q with it
    high = 40.0 if kv_dtype == "f8e4m3" else 60.0
    if kv_dtype == "f8e4m3":
        k = k * case.pages.k_scales[:, None, None, None]
    k[int(case.block_tables[0, n // P]), :, n % P, 63] = high
    stored, scales = W.store_round(k.nan_to_num(0.0), kv_dtype)
    case.pages.k, case.pages.k_scales = W.pack_k(stored, kv_dtype), scales
    case.q[:, :, 63] = 60.0 if kv_dtype != "f8e4m3" else 120.0
    clean = run(mepic, case, general, planned)
    assert np.isfinite(clean).all()
    hit = np.zeros(clean.shape, dtype=bool)
    for n, dim in ((3, 100), (4803, 101)):                 # before the high score's run of partials, and near it
        page = int(case.block_tables[0, n // P])
        if kv_dtype == "f8e4m3":
            case.pages.v.view(torch.uint8)[page, 1, dim, n % P] = 0x7F
        else:
            case.pages.v[page, 1, dim, n % P] = float(value)
        hit[:int(case.cu_q_lens[1]) if prefill else 1, 4:8, dim] = True
    got = run(mepic, case, general, planned)
    assert not np.isfinite(got[hit]).any()
    assert np.array_equal(got[~hit], clean[~hit]) or np.abs(got[~hit] - clean[~hit]).max() <= TOL[kv_dtype]


@pytest.mark.parametrize("kv_dtype,prefill,rise,power", [("bf16", True, 35.0, 100), ("bf16", False, 5.5, 117), ("f32", False, 5.5, 117)])
def test_values_near_the_largest_float(mepic, oracle_attn, kv_dtype, prefill, rise, power):
    """General path: V of 2^power in one dim, and scores that rise by less than moves the reference maximum, so that probabilities
    are up to 2^rise. Sums of probability x value pass 2^128, the result does not, nor do the sums where the largest probability
    is 1."""
    case = W.assemble(s := structure(kv_dtype, 16, prefill, [700, 90]), align_with_oracle(s)[0])
    case.q[:] = 0.0
    case.q[:, :, 63] = 60.0                                  # one pair of dims, which hardly turns: score = k[63] x 7.65 log2 units
    for n in range(700):                                     # (608: inside a tile and inside a wave's run, behind slots of score 0)
        set_k(case.pages, int(case.block_tables[0, n // 16]), n % 16, 63, rise / 7.65 if n >= 608 else 0.0)
        set_k(case.pages, int(case.block_tables[0, n // 16]), n % 16, 127, 0.0)
    case.pages.v[:, :, 100, :] = torch.where(case.pages.v[:, :, 100, :].isnan(), float("nan"), 2.0 ** power)
    got, want = run(mepic, case, True, False), oracle_out(oracle_attn, case)
    big = np.arange(128) == 100
    assert np.abs(got[:, :, big] / want[:, :, big] - 1.0).max() <= 2.0 ** -7
    assert np.abs(got[:, :, ~big] - want[:, :, ~big]).max() <= TOL[kv_dtype]


def plain_case(kv_dtype, P, lengths, G, theta):
    st = structure(kv_dtype, P, False, lengths)
    st.Hq, st.theta = G * st.Hkv, theta
    return W.assemble(st, align_with_oracle(st)[0])


@pytest.mark.parametrize("value", [float("inf"), -float("inf")])
@pytest.mark.parametrize("dim", [63, 126])
@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("G,theta", [(4, 5e5), (8, 5e5), (3, 1e4), (5, 1e4), (6, 1e4), (8, 1.5e5)])
def test_an_infinite_key(mepic, oracle_attn, G, theta, general, dim, value):
    """bf16 keys, an Inf in the pair of dims that hardly turns: whether a row is NaN or the key has no weight in it depends on the signs
    of its rotated query alone, wherever the rotation is taken from (but at multiples of the tables' span a sine is 0, and 0 x Inf)."""
    case = plain_case("bf16", 16, [700, 90, 300], G, theta)
    for b, n in ((0, 100), (0, 333), (1, 40), (0, 5)):
        set_k(case.pages, int(case.block_tables[b, n // 16]), n % 16, dim, value)
    got, want = run(mepic, case, general, False), oracle_out(oracle_attn, case)
    hit = np.isnan(want)
    assert hit.any() and not hit[:2].all() and (np.isnan(got) == hit).all()
    assert np.abs(got[~hit] - want[~hit]).max() <= TOL["bf16"]


@pytest.mark.parametrize("dim", [32, 40, 63])
@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("G,theta", [(4, 5e5), (8, 5e5), (4, 1e4), (5, 1e4), (6, 1e4)])
def test_scores_below_the_lowest_float(mepic, oracle_attn, G, theta, general, dim):
    """bf16 keys: products of finite numbers that pass -2^128. Such a key has no weight."""
    case = plain_case("bf16", 16, [700, 90], G, theta)
    case.q[:, :, dim], case.q[:, :, dim + 64] = 1e20, 0.0
    case.pages.k.view(torch.int16)[:, :, dim // 8, :, dim % 8] = 0
    case.pages.k.view(torch.int16)[:, :, (dim + 64) // 8, :, dim % 8] = 0
    for b, n in ((0, 600), (0, 699), (0, 650), (1, 80), (1, 70)):
        set_k(case.pages, int(case.block_tables[b, n // 16]), n % 16, dim, -1e21)
    got, want = run(mepic, case, general, False), oracle_out(oracle_attn, case)
    assert np.isfinite(want).all() and np.abs(got - want).max() <= TOL["bf16"]


@pytest.mark.parametrize("G,theta", [(4, 5e5), (8, 5e5), (5, 1e4)])
@pytest.mark.parametrize("B", [7, 70])
def test_infinite_keys_in_some_runs_of_a_wave(mepic, oracle_attn, G, theta, B):
    """Requests in one long run each (7), or parts of the work that go through several requests and cut some (70): what has an infinite key is
    computed again, with a result as before, and the requests around it are not touched."""
    lengths = [(173 * b) % 331 + 1 + (600 if b % 5 == 3 else 0) for b in range(B)]
    case = plain_case("bf16", 16, lengths, G, theta)
    clean = run_in_long_runs(mepic, plain_case("bf16", 16, lengths, G, theta), 45)
    some = [b for b in range(B) if b % 3 == 1]
    for b in some:
        n = lengths[b] - 1 - (lengths[b] % 128 == 1)
        set_k(case.pages, int(case.block_tables[b, n // 16]), n % 16, 63, float("inf"))
    want = oracle_out(oracle_attn, case)
    got = run_in_long_runs(mepic, case, 45)
    hit, others = np.isnan(want), np.setdiff1d(np.arange(B), some)
    assert hit[some].any() and not hit[some].all() and (np.isnan(got) == hit).all()
    assert np.abs(got[~hit] - want[~hit]).max() <= TOL["bf16"]
    assert np.array_equal(got[others], clean[others])


@pytest.mark.parametrize("nothing", [1, 32, 64, 96, 320])
@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("kv_dtype,P,G,theta", [("bf16", 16, 4, 5e5), ("bf16", 16, 8, 5e5), ("bf16", 16, 5, 1e4), ("bf16", 16, 9, 5e5),
                                               ("f8e4m3", 32, 4, 5e5), ("f8e4m3", 32, 9, 5e5)])
def test_no_weight_before_the_first_finite_score(mepic, oracle_attn, kv_dtype, P, G, theta, general, nothing):
    """All scores of a request's first slots (fp8: pages) are -Inf, in part of a turn, a whole one or several: the reference maximum is that of the
    first score that is not."""
    lengths = [700, 90, 333]
    case = plain_case(kv_dtype, P, lengths, G, theta)
    X = case.pages.k.shape[-1]
    if kv_dtype == "f8e4m3":
        case.q[:] = 0.0
    case.q[:, :, 63], case.q[:, :, 127] = 8.0 if kv_dtype == "f8e4m3" else 1e20, 0.0
    raw = case.pages.k.view(torch.uint8 if kv_dtype == "f8e4m3" else torch.int16)
    raw[:, :, 63 // X, :, 63 % X] = raw[:, :, 127 // X, :, 127 % X] = 0
    for b, n in enumerate(lengths):
        for slot in range(min(nothing, n - 5)):
            page = int(case.block_tables[b, slot // P])
            if kv_dtype != "f8e4m3":
                set_k(case.pages, page, slot % P, 63, -1e21)
            elif (slot // P + 1) * P <= min(nothing, n - 5):
                raw[page, :, 63 // X, slot % P, 63 % X] = 0xF0
                case.pages.k_scales[page] = 1e37
    want = oracle_out(oracle_attn, case)
    assert np.isfinite(want).all()
    for got in [run(mepic, case, general, False)] + ([] if general else [run_in_long_runs(mepic, case, 22)]):
        assert np.abs(got - want).max() <= TOL[kv_dtype]
