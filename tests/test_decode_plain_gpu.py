"""Plain decode: the forms its kernel takes (query heads a KV head, speed of the rotary frequencies, page type) at lengths around
its turns, table spans and windows of page ids."""
import numpy as np
import pytest
import torch

import workloads as W
from harness import DeviceCase, align_with_oracle, oracle_out, run_in_long_runs

pytestmark = pytest.mark.gpu

# around one and two steps, the 64-, 128- and 256-slot spans between two advances of Q', a window of 64 page ids (1024, 2048 slots)
LENGTHS = [1, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 96, 127, 128, 129, 160, 255, 256, 257, 300, 511, 513, 1023, 1025, 2049, 2100]


def structure(G, Hkv, kv_dtype, theta, lengths, seed):
    st = W.Structure("plain", "decode", len(lengths), G * Hkv, Hkv, 128, 16 if kv_dtype == "bf16" else 32, theta, "bf16", kv_dtype, seed)
    st.requests, st.extra_tail, st.n_q = [[(0, n, 0)] for n in lengths], 0, [1] * len(lengths)
    return st


def build(G, Hkv, kv_dtype, theta, lengths, seed, edit=None):
    """A case whose real K and V [page, head, slot, dim] `edit(case, k, v)` has changed before they are stored."""
    case = W.assemble(s := structure(G, Hkv, kv_dtype, theta, lengths, seed), align_with_oracle(s)[0], poison=False)
    pg = case.pages
    if edit:
        scale = lambda x, f: x if f is None else x * f[:, None, None, None]
        k, v = scale(W.unpack_k(pg.k.float()), pg.k_scales), scale(W.unpack_v(pg.v.float()), pg.v_scales)
        edit(case, k, v)
        pg.k, pg.k_scales = W.store_round(k, kv_dtype)
        pg.v, pg.v_scales = W.store_round(v, kv_dtype)
        pg.k, pg.v = W.pack_k(pg.k, kv_dtype), W.pack_v(pg.v)
    W.poison_tail(pg, case.block_tables, case.kv_lens)
    return case


def edges_count(case, k, v):
    """Values twice as large in the first and last slot of every 16, eight times in a request's last: one of them lost or taken twice is
    2 % and more of a row of some head, also among thousands of slots."""
    for b, n in enumerate(case.kv_lens):
        v[int(case.block_tables[b, (n - 1) // case.st.P]), :, (n - 1) % case.st.P] *= 4.0 if n % 16 < 2 else 8.0
    v[:, :, 0::16] *= 2.0
    v[:, :, 15::16] *= 2.0


def worst_row(got, want):
    """Largest relative error of a row (request, query head): a long request's rows are small, and count as much as a short one's."""
    return float((np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)).max())


# Q', keys (or their constants), probabilities and results are rounded to 16 bits or better: at most 2^-9 of each, 2^-7 together
BOUND = 2.0 ** -7
# A row in which one key outweighs the others takes that key's error whole: a score of unit variance is off by 2e-3 in the root mean square (three
# roundings of 2^-9 / sqrt 3), by 1e-2 in the worst of some thousand rows, and two roundings of 2^-9 come to it.
ROW_BOUND = 2.0 ** -6


@pytest.mark.parametrize("kv_dtype", ["bf16", "f8e4m3"])
@pytest.mark.parametrize("theta", [3e2, 1e4, 5e5])
@pytest.mark.parametrize("G", [1, 4, 5, 6, 8, 9, 16])
def test_groups_and_frequencies(mepic, oracle_attn, G, theta, kv_dtype):
    """Runs of a step or two, and whole requests in a run each: every count of turns around the spans and the windows."""
    case = build(G, 2, kv_dtype, theta, LENGTHS + ([4097, 4200] if kv_dtype == "f8e4m3" else []), 90 + G, edges_count)
    got, want = DeviceCase(mepic, case).run(), oracle_out(oracle_attn, case)
    assert mepic.last_kernel().startswith("decode_mfma")
    assert worst_row(got, want) <= ROW_BOUND
    assert np.array_equal(DeviceCase(mepic, case, flags=mepic.FLAG_KV_READ_ONCE).run(), got)
    steps = max(-(-n // 32) for n in case.kv_lens)
    got = run_in_long_runs(mepic, case, steps)
    assert worst_row(got, want) <= ROW_BOUND
    assert np.array_equal(run_in_long_runs(mepic, case, steps, mepic.FLAG_KV_READ_ONCE), got)


@pytest.mark.parametrize("kv_dtype", ["bf16", "f8e4m3"])
@pytest.mark.parametrize("Hkv,G,B,most", [(8, 4, 1, 9000), (3, 8, 3, 700), (8, 7, 66, 700), (12, 1, 130, 700), (8, 4, 64, 1300),
                                          (8, 5, 40, 3000), (2, 4, 20, 900), (4, 8, 64, 2000)])
def test_waves_runs_and_requests(mepic, oracle_attn, Hkv, G, B, most, kv_dtype):
    """One request over all waves, several runs a wave, requests cut into pieces of their own (even and mixed lengths)
    or not, lengths in the lanes of a wave and (more than 64 requests) in LDS."""
    lengths = [(97 * b * b + 41) % most + 1 if B != 64 or b % 3 else most for b in range(B)] if B > 1 else [most]
    case = build(G, Hkv, kv_dtype, 1e6, lengths, 7, edges_count)
    got, want = DeviceCase(mepic, case).run(), oracle_out(oracle_attn, case)
    assert worst_row(got, want) <= ROW_BOUND
    assert worst_row(run_in_long_runs(mepic, case, 300 if B == 1 else 34 if B == 3 else 8), want) <= ROW_BOUND  # (fp8: two steps a turn)


@pytest.mark.parametrize("kv_dtype,G,theta", [("bf16", 4, 5e5), ("bf16", 8, 5e5), ("bf16", 5, 1e4), ("bf16", 4, 3e2), ("bf16", 9, 1e4),
                                              ("f8e4m3", 7, 1e6), ("f8e4m3", 9, 1e6)])
@pytest.mark.parametrize("steps", [2, 3, 8, 37])
def test_parts_of_several_requests(mepic, oracle_attn, steps, kv_dtype, G, theta):
    """More requests than lanes: parts of `steps` steps go from one request into the next and cut long ones, at any step."""
    lengths = [(131 * b * b + 17) % 500 + 1 + (1800 if b % 23 == 5 else 0) for b in range(70)]
    case = build(G, 2, kv_dtype, theta, lengths, 8, edges_count)
    want = oracle_out(oracle_attn, case)
    assert worst_row(run_in_long_runs(mepic, case, steps), want) <= ROW_BOUND


@pytest.mark.parametrize("order", ["rising", "falling", "random"])
@pytest.mark.parametrize("G", [4, 8, 9])
def test_page_scales_over_many_turns(mepic, oracle_attn, G, order):
    """V scales over four decades (K scales over one) along runs of up to 132 pages: the reference scale is raised at almost every turn, or at the
    first, and a scale taken from a neighbouring page is wrong by far."""
    def edit(case, k, v):
        rng = np.random.default_rng(3)
        for b, n in enumerate(case.kv_lens):
            pages = case.block_tables[b, :-(-int(n) // 32)].astype(np.int64)
            f = 10.0 ** rng.uniform(-4, 0, size=len(pages))
            f = {"rising": np.sort(f), "falling": np.sort(f)[::-1].copy(), "random": f}[order]
            v[pages] *= torch.from_numpy(f.astype(np.float32))[:, None, None, None]
            k[pages] *= torch.from_numpy(10.0 ** rng.uniform(-1, 0, size=len(pages)).astype(np.float32))[:, None, None, None]
    case = build(G, 2, "f8e4m3", 1e6, [4200, 2100, 65, 33, 2049, 4097, 96], 29, edit)
    got, want = run_in_long_runs(mepic, case, 132), oracle_out(oracle_attn, case)
    assert worst_row(got, want) <= ROW_BOUND


@pytest.mark.parametrize("G,theta", [(4, 4.04e5), (8, 4.04e5), (4, 8.2e3), (5, 8.2e3), (4, 7.9e3), (6, 4.0e5)])
def test_pair_with_the_largest_remainder(mepic, oracle_attn, G, theta):
    """rope_theta on either side of the lines between two terms, three and a rotation; all of q and K in the pair that the terms left out
    concern most. Scores of up to S nats are then off by S (2.5e-3 + 3 x 2^-9) at most; probabilities change by a factor of at most e to
    twice that, and a row by that share of the sum of p |v|, next to the rounding of p and of itself to bf16."""
    pair = np.isin(np.arange(128), (32, 96))
    def edit(case, k, v):
        k[..., ~pair] = 0.0
    case = build(G, 2, "bf16", theta, [700, 129, 40, 1500], 12, edit)
    case.q[:, :, ~pair] = 0.0
    case.q *= 5.0
    want = oracle_out(oracle_attn, case)
    k = W.unpack_k(case.pages.k.float().nan_to_num(0.0)).numpy()
    v, case.pages.v = case.pages.v, case.pages.v.abs()
    size = oracle_out(oracle_attn, case)                                            # sum of p |v|
    case.pages.v = v
    S = np.zeros(want.shape[:2])
    for b, n in enumerate(case.kv_lens):
        keys = np.sqrt((k[case.block_tables[b, :-(-int(n) // 16)]] ** 2).sum(-1)).max(axis=(0, 2))  # largest of each KV head
        S[b] = np.sqrt((case.q[b].float().numpy() ** 2).sum(-1)) * np.repeat(keys, G) / np.sqrt(128.0)
    bound = (np.expm1(2.0 * S * (2.5e-3 + 3 * 2.0 ** -9)) + 2.0 ** -9)[..., None] * size + 2.0 ** -8 * np.abs(want)
    for got in (DeviceCase(mepic, case).run(), run_in_long_runs(mepic, case, 47)):
        print(f"error / bound {(np.abs(got - want) / bound).max():.3f}")
        assert (np.abs(got - want) <= bound).all()


@pytest.mark.parametrize("G", [4, 8, 12])
def test_a_page_keeps_its_precision_beside_one_of_a_large_scale(mepic, oracle_attn, G):
    """Two steps of a request that go through the kernel as one: the second page's V scale is a thousand times the first's, for a value in
    another KV head. The first page's values are all that counts in a row of this one, and they come first. (In short runs the kernel takes the
    steps one by one.)"""
    def edit(case, k, v):
        for b in range(len(case.kv_lens)):
            v[int(case.block_tables[b, 1]), 1, 3, 0] = 4000.0
    case = build(G, 2, "f8e4m3", 1e6, [64, 61, 40, 64], 31, edit)
    want = oracle_out(oracle_attn, case)
    for got in (DeviceCase(mepic, case).run(), run_in_long_runs(mepic, case, 16)):
        assert worst_row(got[:, :G], want[:, :G]) <= BOUND


@pytest.mark.parametrize("G", [4, 8, 12])
def test_a_page_keeps_its_precision_beside_one_of_large_scores(mepic, oracle_attn, G):
    """The second step's scores lie nine log2 units above the first's, and its values are zero in half of the dims, where the first step's
    are the whole result."""
    def edit(case, k, v):
        case.q[:, :, 63], case.q[:, :, 127] = 8.0, 0.0
        k[..., 63], k[..., 127] = 0.0, 0.0
        for b in range(len(case.kv_lens)):
            k[int(case.block_tables[b, 1]), :, :, 63] = 9.0 / (8.0 * np.log2(np.e) / np.sqrt(128.0))
            v[int(case.block_tables[b, 1]), :, :, :64] = 0.0
    case = build(G, 2, "f8e4m3", 1e6, [64, 61, 40, 64], 31, edit)
    want = oracle_out(oracle_attn, case)
    for got in (DeviceCase(mepic, case).run(), run_in_long_runs(mepic, case, 16)):
        assert worst_row(got[..., :64], want[..., :64]) <= BOUND and worst_row(got, want) <= BOUND


@pytest.mark.parametrize("B", [1, 40])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 16, 17, 56, 57, 63, 64, 65, 72, 120, 129])
def test_partials_of_a_row(mepic, oracle_attn, n, B):
    """Rows of 1 to 129 partials (a step of 32 slots each where there are as many waves; else the most that 40 requests come to), merged
    with 256 threads (8 rows) and, where there are more than 1024 rows, 128."""
    Hkv = 8 if B == 1 else 4
    case = build(1 if B == 1 else 7, Hkv, "bf16", 5e5, [32 * n - 5] * B, 300 + n, edges_count)
    got, want = DeviceCase(mepic, case).run(), oracle_out(oracle_attn, case)
    assert worst_row(got, want) <= ROW_BOUND
