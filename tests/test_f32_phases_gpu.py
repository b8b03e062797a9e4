"""fp32 pages at positions of some twenty thousand, where an error of the rotation's phases shows: with the rounding error of
position x frequency in the phase (1e-4 of a turn there) results are 1e-4 of their norm off."""
import numpy as np
import pytest

import workloads as W
from harness import DeviceCase, align_with_oracle, oracle_out

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefill", [False, True])
@pytest.mark.parametrize("D", [64, 128])
def test_phases_of_fp32_pages_at_far_positions(mepic, oracle_attn, D, prefill):
    """A long context, and a short one whose blocks lie anywhere up to position 24 000. 4e-6 of each token's norm: phases good to
    2^-24 of a turn and the hardware sine's 2^-20 give scores good to about 2e-6, the sums of fp32 terms less."""
    st = W.Structure("far", "prefill" if prefill else "decode", 2, 4, 2, D, 16, 5e5, "f32", "f32", 71)
    st.requests, st.n_q, st.extra_tail = [[(0, 20011, 0)], [(0, 700, 0)]], [3, 2] if prefill else [1, 1], 0
    case = W.assemble(st, align_with_oracle(st)[0], pads_are_positions=False)
    case.block_positions[1, :44] = np.random.default_rng(8).integers(0, 24000, size=44)
    case.q_positions[case.q_positions < 1000] = 24007
    got, want = DeviceCase(mepic, case).run(), oracle_out(oracle_attn, case)
    for t in range(case.n_q):
        assert np.linalg.norm(got[t] - want[t]) <= 4e-6 * np.linalg.norm(want[t]), t
