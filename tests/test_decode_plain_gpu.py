"""Plain decode: the forms its kernel takes (query heads a KV head, speed of the rotary frequencies, page type) at lengths around
its turns, table spans and windows of page ids."""
import numpy as np
import pytest

import workloads as W
from harness import DeviceCase, align_with_oracle, oracle_out

pytestmark = pytest.mark.gpu

# around one and two steps, the 64-, 128- and 256-slot spans between two advances of Q', a window of 64 page ids (1024, 2048 slots)
LENGTHS = [1, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 96, 127, 128, 129, 160, 255, 256, 257, 300, 511, 513, 1023, 1025, 2049, 2100]


def structure(G, Hkv, kv_dtype, theta, lengths, seed):
    st = W.Structure("plain", "decode", len(lengths), G * Hkv, Hkv, 128, 16 if kv_dtype == "bf16" else 32, theta, "bf16", kv_dtype, seed)
    st.requests, st.extra_tail, st.n_q = [[(0, n, 0)] for n in lengths], 0, [1] * len(lengths)
    return st


def rel(got, want):
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


# Q', keys (or their constants), probabilities and results are rounded to 16 bits or better: at most 2^-9 of each, 2^-7 together
BOUND = 2.0 ** -7


@pytest.mark.parametrize("kv_dtype", ["bf16", "f8e4m3"])
@pytest.mark.parametrize("theta", [3e2, 1e4, 5e5])
@pytest.mark.parametrize("G", [1, 4, 5, 6, 8, 9, 16])
def test_groups_and_frequencies(mepic, oracle_attn, G, theta, kv_dtype):
    case = W.assemble(s := structure(G, 2, kv_dtype, theta, LENGTHS, 90 + G), align_with_oracle(s)[0])
    dc = DeviceCase(mepic, case)
    got, want = dc.run(), oracle_out(oracle_attn, case)
    assert mepic.last_kernel().startswith("decode_mfma")
    assert np.isfinite(got).all() and rel(got, want) <= BOUND
    assert np.array_equal(DeviceCase(mepic, case, flags=mepic.FLAG_KV_READ_ONCE).run(), got)


@pytest.mark.parametrize("kv_dtype", ["bf16", "f8e4m3"])
@pytest.mark.parametrize("Hkv,G,B,most", [(8, 4, 1, 9000), (3, 8, 3, 700), (8, 7, 66, 700), (12, 1, 130, 700), (8, 4, 64, 1300),
                                          (8, 5, 40, 3000), (2, 4, 20, 900), (4, 8, 64, 2000)])
def test_waves_runs_and_requests(mepic, oracle_attn, Hkv, G, B, most, kv_dtype):
    """One request over all waves, several runs a wave, requests cut into pieces of their own (even and mixed lengths)
    or not, lengths in the lanes of a wave and (more than 64 requests) in LDS."""
    lengths = [(97 * b * b + 41) % most + 1 if B != 64 or b % 3 else most for b in range(B)] if B > 1 else [most]
    case = W.assemble(s := structure(G, Hkv, kv_dtype, 1e6, lengths, 7), align_with_oracle(s)[0])
    got, want = DeviceCase(mepic, case).run(), oracle_out(oracle_attn, case)
    assert np.isfinite(got).all() and rel(got, want) <= BOUND


@pytest.mark.parametrize("G,theta", [(4, 4.04e5), (8, 4.04e5), (4, 8.2e3), (5, 8.2e3), (4, 7.9e3), (6, 4.0e5)])
def test_pair_with_the_largest_remainder(mepic, oracle_attn, G, theta):
    """rope_theta on either side of the lines between two terms, three and a rotation; all of q and K in the pair that the terms left out
    concern most. Scores of up to S nats are then off by S (2.5e-3 + 3 x 2^-9) at most, and the result by e to that."""
    case = W.assemble(s := structure(G, 2, "bf16", theta, [700, 129, 40, 1500], 12), align_with_oracle(s)[0])
    keep = np.isin(np.arange(128), (32, 96))
    case.q[:, :, ~keep] = 0.0
    k = W.unpack_k(case.pages.k.float().nan_to_num(0.0))
    k[..., ~keep] = 0.0
    case.pages.k = W.pack_k(W.store_round(k, "bf16")[0], "bf16")
    case.q *= 5.0
    k, q = k.numpy(), np.asarray(case.q.float() if hasattr(case.q, "float") else case.q)
    largest = np.sqrt((q ** 2).sum(-1).max()) * np.sqrt((k ** 2).sum(-1).max()) / np.sqrt(128.0)
    got, want = DeviceCase(mepic, case).run(), oracle_out(oracle_attn, case)
    v = float(case.pages.v.float().nan_to_num(0.0).abs().max())
    bound = (np.exp(2 * largest * (2.5e-3 + 3 * 2.0 ** -9)) - 1) * v + 2.0 ** -8 * v
    assert np.abs(got - want).max() <= bound and rel(got, want) <= 2.0 * BOUND


def fp8_case(G, lengths, edit):
    """fp8 pages whose real K and V [page, head, slot, dim] `edit(case, k, v)` has changed before they are stored."""
    case = W.assemble(s := structure(G, 2, "f8e4m3", 1e6, lengths, 31), align_with_oracle(s)[0], poison=False)
    pg = case.pages
    k = W.unpack_k(pg.k.float()) * pg.k_scales[:, None, None, None]
    v = W.unpack_v(pg.v.float()) * pg.v_scales[:, None, None, None]
    edit(case, k, v)
    for name, x, pack in (("k", k, lambda x: W.pack_k(x, "f8e4m3")), ("v", v, W.pack_v)):
        stored, scales = W.store_round(x, "f8e4m3")
        setattr(pg, name, pack(stored))
        setattr(pg, name + "_scales", scales)
    W.poison_tail(pg, case.block_tables, case.kv_lens)
    return case


def worst_row(got, want):
    """Largest relative error of a row (request, query head)."""
    return float((np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)).max())


@pytest.mark.parametrize("G", [4, 8, 12])
def test_a_page_keeps_its_precision_beside_one_of_a_large_scale(mepic, oracle_attn, G):
    """Two steps of a request that go through the kernel as one: the second page's V scale is a thousand times the first's, for a value in
    another KV head. The first page's values are all that counts in a row of this one, and they come first."""
    def edit(case, k, v):
        for b in range(len(case.kv_lens)):
            v[int(case.block_tables[b, 1]), 1, 3, 0] = 4000.0
    case = fp8_case(G, [64, 61, 40, 64], edit)
    got, want = DeviceCase(mepic, case).run(), oracle_out(oracle_attn, case)
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
    case = fp8_case(G, [64, 61, 40, 64], edit)
    got, want = DeviceCase(mepic, case).run(), oracle_out(oracle_attn, case)
    assert worst_row(got[..., :64], want[..., :64]) <= BOUND and worst_row(got, want) <= BOUND
