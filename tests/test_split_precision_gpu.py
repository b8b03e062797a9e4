"""General path, bf16 and fp8 pages: operands of 16 significant bits. The error of a score grows with the size of its terms, however
much of them cancels, so these keys share a large offset per dim (as real ones do) and scores reach tens and hundreds."""
import numpy as np
import pytest
import torch

import workloads as W
from harness import DeviceCase, align_with_oracle, oracle_out

pytestmark = pytest.mark.gpu


def large_case(kv_dtype, P, prefill, q_scale, theta=5e5, G=4):
    st = W.Structure("large", "prefill" if prefill else "decode", 3, 2 * G, 2, 128, P, theta, "bf16", kv_dtype, 97)
    st.requests, st.n_q, st.extra_tail = [[(0, 3000, 0)], [(0, 500, 0)], [(0, 40, 0)]], [40, 30, 9] if prefill else [1, 1, 1], 0
    case = W.assemble(st, align_with_oracle(st)[0])
    rng = np.random.default_rng(6)
    offset = torch.from_numpy(8.0 * rng.standard_normal((1, st.Hkv, 1, st.D)).astype(np.float32))
    k = torch.from_numpy(rng.standard_normal((case.pages.num_pages, st.Hkv, P, st.D)).astype(np.float32)) + offset
    stored, case.pages.k_scales = W.store_round(k, kv_dtype)
    case.pages.k = W.pack_k(stored, kv_dtype)
    case.q = (case.q.float() * q_scale).to(case.q.dtype)
    return case


def score_terms(case):
    """Per (token, head): the largest sum over rotary pairs of |q||k| over the request's slots, which bounds sum |q_i k_i| at any
    positions, times the score scale."""
    st = case.st
    k = W.unpack_k(case.pages.k.float()).numpy()
    if case.pages.k_scales is not None:
        k = k * case.pages.k_scales.numpy()[:, None, None, None]
    pairs = lambda x: np.hypot(x[..., : st.D // 2], x[..., st.D // 2:])
    q, k = pairs(case.q.float().numpy()), pairs(k)
    cu = np.arange(st.B + 1) if case.cu_q_lens is None else case.cu_q_lens
    out = np.zeros((case.n_q, st.Hq))
    for b in range(st.B):
        n = np.arange(case.kv_lens[b])
        kb = k[case.block_tables[b][n // st.P], :, n % st.P]                        # [slots, Hkv, pairs]
        for h in range(st.Hq):
            out[cu[b]:cu[b + 1], h] = (q[cu[b]:cu[b + 1], h] @ kb[:, h * st.Hkv // st.Hq].T).max(1)
    return out / np.sqrt(st.D)


@pytest.mark.parametrize("q_scale", [1.0, 8.0])
@pytest.mark.parametrize("prefill", [False, True])
@pytest.mark.parametrize("kv_dtype,P", [("bf16", 16), ("f8e4m3", 32)])
def test_error_is_bounded_by_the_terms_of_the_scores(mepic, oracle_attn, kv_dtype, P, prefill, q_scale):
    """With A = sum |q_i k_i| x scale, a score is off by at most A 2^-15: 2^-18 for each operand's two bf16 terms and for the
    remainder product left out, 2^-17 for a chain of 128 fp32 sums, 2^-19 for the phases' sines on both sides make
    A 2^-15.7. Probabilities then change by a factor of at most e^(2 A 2^-15), and a row by that share of the sum of p |v|, next
    to its own rounding to bf16."""
    check_bound(mepic, oracle_attn, large_case(kv_dtype, P, prefill, q_scale))


def check_bound(mepic, oracle_attn, case):
    got = DeviceCase(mepic, case, flags=mepic.FLAG_FORCE_GENERAL).run()
    want = oracle_out(oracle_attn, case)
    v = case.pages.v
    case.pages.v = v.float().abs().to(v.dtype)
    size = oracle_out(oracle_attn, case)                                            # sum of p |v|
    off = np.expm1(2.0 * score_terms(case) * 2.0 ** -15)[..., None]
    bound = np.abs(want) * 2.0 ** -8 + off * size + 2.0 ** -13 * np.abs(want).max()
    print(f"\n{case.st.kv_dtype} theta {case.st.theta:g}: terms {score_terms(case).max():.0f}, error / bound {(np.abs(got - want) / bound).max():.3f}, "
          f"relative {np.linalg.norm(got - want) / np.linalg.norm(want):.2e}")
    assert (np.abs(got - want) <= bound).all()


@pytest.mark.parametrize("kv_dtype,P", [("bf16", 16), ("bf16", 32), ("f8e4m3", 32)])
@pytest.mark.parametrize("G,theta", [(4, 4.07e5), (4, 1.01e5), (8, 4.07e5), (1, 1.01e5), (9, 4.07e5), (4, 9.9e4), (4, float("inf"))])
def test_error_where_terms_take_the_place_of_rotations(mepic, oracle_attn, kv_dtype, P, G, theta):
    """Decode, at the slowest rope_theta of either table span (9 heads a KV head and 9.9e4: rotations; infinite: only the first pair turns): everything in the pair that the terms left out
    concern most. They add 2 J4(0.2) = 2^-16.9 of a score: with the 2^-15.7 above still below 2^-15."""
    case = large_case(kv_dtype, P, False, 4.0, theta, G)
    other = ~np.isin(np.arange(128), (32, 96))
    case.q[:, :, other] = 0.0
    check_bound(mepic, oracle_attn, case)
