"""Lists of more than 12288 entries, finished in batches, and short bf16 rows of small batches, cut into chunks of one
tile so that a long history finds room."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [True, False])
def test_lists_beyond_any_register_variant(bf16):
    """A prompt of 15000 distinct tokens: the list has more entries than 24 a thread, its segments have room."""
    B, V = 6, 150003
    rng = np.random.default_rng(4)
    z = (rng.standard_normal((B, V)) * 2.5).astype(np.float32)
    hist = [rng.permutation(V)[:15000].tolist() for _ in range(B)]
    params = dict(temperature=[0.8, 0.0, 1.0, 0.7, 1.1, 1.0], top_k=[50, 0, 0, 400, 0, 0], top_p=[0.9, 1, 1, 0.95, 1, 1],
                  min_p=[0, 0, 0.05, 0, 0.1, 0], repetition_penalty=[1.1, 1.3, 1.2, 1.1, 1.05, 1.1])
    w = H.custom("long_lists", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=4)
    d = H.to_device(w)
    for step in (0, 1):
        H.compare(w, H.run_gpu(d, 2, step), 2, step)
        assert (H.last_row_why == 1).all(), H.last_row_why


@pytest.mark.parametrize("B,V", [(6, 40000), (60, 36000), (129, 41001)])
def test_long_histories_of_short_rows(B, V):
    rng = np.random.default_rng(B)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    n = 6000 if B < 100 else 2500
    hist = [rng.integers(0, V, n).tolist() for _ in range(B)]
    params = dict(temperature=rng.uniform(0.6, 1.2, B), min_p=rng.choice([0.02, 0.1], B), top_k=rng.choice([0, 50], B),
                  repetition_penalty=np.full(B, 1.1), frequency_penalty=rng.choice([0.0, 0.3], B))
    w = H.custom(f"short_{V}", workloads.f32_to_bf16_bits(z), params, hist, k_logprobs=2)
    st = H.compare(w, H.run_gpu(H.to_device(w), 8, 0), 8, 0)
    assert st.rows == B and (H.last_row_why == 1).mean() > 0.9, H.last_row_why
