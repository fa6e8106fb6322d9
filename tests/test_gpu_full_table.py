"""The table of multiplicities at its limit, with tokens that do not spread by chance, and far beyond it."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16", [(6, 131072, False), (300, 131072, True)])
def test_distinct_tokens_up_to_the_limit_and_beyond(B, V, bf16):
    rng = np.random.default_rng(B)
    n = 6144                                                    # distinct tokens that the table takes
    z = (rng.standard_normal((B, V)) * 2.5).astype(np.float32)
    runs = (rng.permutation(V // 16)[:n // 16, None] * 16 + np.arange(16)).ravel()
    sets = [rng.permutation(V)[:n], rng.permutation(runs), 5 + 20 * np.arange(n), 21 * np.arange(n)[::-1],
            rng.permutation(V)[:8400], rng.permutation(V)[:n + 1]]
    hist = [np.concatenate((sets[b % 6], sets[b % 6][:500])).tolist() for b in range(B)]
    params = dict(temperature=np.full(B, 0.8), top_k=np.full(B, 40), repetition_penalty=np.full(B, 1.1),
                  frequency_penalty=np.full(B, 0.2))
    w = H.custom(f"table_{B}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=2)
    out = H.run_gpu(H.to_device(w), 3, 0)
    H.compare(w, out, 3, 0, rows=range(min(B, 24)))
    assert np.array_equal(H.last_row_why, np.array([1, 1, 1, 1, 4, 4])[np.arange(B) % 6]), H.last_row_why
