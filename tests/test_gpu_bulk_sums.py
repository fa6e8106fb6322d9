"""The mass outside the list is summed without the list's own entries: thousands of history tokens around the
threshold that their penalty then takes away leave nothing behind in the total."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16", [(4, 70001, False), (4, 70001, True), (224, 75001, False), (240, 60005, True),
                                      (300, 75003, True), (300, 40001, False)])
def test_penalised_tokens_leave_the_total(B, V, bf16):
    rng = np.random.default_rng(V + B)
    z = np.full((B, V), -1000.0, np.float32)                # no mass at all
    hist = []
    for b in range(B):
        at = rng.permutation(V)[:6001]
        z[b, at] = rng.uniform(-0.5, 0.5, 6001)
        z[b, at[0]] = 0.75                                  # the one token that is left, and with it all of the mass
        hist.append(at[1:].tolist())
    params = dict(temperature=np.choose(np.arange(B) % 4, [0.0, 0.5, 1.0, 2.0]), presence_penalty=np.full(B, 200.0))
    w = H.custom(f"bulk_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=1)
    d = H.to_device(w)
    ids, lp_ids, lp = H.run_gpu(d, 5, 0)
    assert (H.last_row_why == 1).all(), H.last_row_why
    assert np.array_equal(ids, np.argmax(z == 0.75, axis=1)) and np.array_equal(lp_ids[:, 1], ids)
    # ln of a total of exactly 1; the hardware logarithm and exponential are good for an ulp each
    assert np.abs(lp).max() <= 2.0 ** -22, np.abs(lp).max()
