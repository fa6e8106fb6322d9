"""The bin of the nucleus cut: at the very top, at the lowest bin of the list, below what min-p or top-k reach, between
values with hundreds of empty bins around them, and thousands of history tokens below the list in one bin."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16", [(24, 40001, True), (24, 36003, False), (260, 40009, True)])
def test_cut_anywhere_in_the_bins(B, V, bf16):
    rng = np.random.default_rng(V)
    kind = np.arange(B) % 12
    z = (rng.standard_normal((B, V)) * 3.0).astype(np.float32)
    hist = [[] for _ in range(B)]
    for b, k in enumerate(kind):
        if k in (3, 4, 5):
            z[b] = -40.0
            z[b, rng.permutation(V)[:600]] = rng.integers(0, 6, 600) * 3.0      # six values, 60 to 100 tokens each
        elif k in (6, 7):
            hist[b] = rng.integers(0, V, 5000).tolist()                          # far more below the list than in it
        elif k == 8:
            z[b, rng.integers(0, V)] = 60.0                                      # one token and nothing beside it
    params = dict(temperature=np.choose(kind, [1.0, 0.7, 0.5, 1.0, 2.0, 0.8, 0.6, 0.5, 1.0, 0.4, 0.7, 0.6]),
                  top_p=np.choose(kind, [1e-7, 0.1, 0.97, 0.2, 0.9, 0.999, 0.9, 0.6, 0.99, 0.999, 0.95, 0.5]),
                  top_k=np.choose(kind, [0, 0, 0, 0, 0, 0, 0, 30, 0, 300, 2, 900]),
                  min_p=np.choose(kind, [0, 0, 0.2, 0, 0.5, 0.01, 0, 0, 0.9, 0.05, 0, 0]),
                  repetition_penalty=np.choose(kind, [1, 1, 1, 1, 1, 1, 1.3, 1.1, 1, 1, 1, 1]),
                  frequency_penalty=np.choose(kind, [0, 0, 0, 0, 0, 0, 0, 0.2, 0, 0, 0, 0]))
    w = H.custom(f"cut_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=3)
    d = H.to_device(w)
    for step in range(5 if B < 30 else 1):
        H.compare(w, H.run_gpu(d, 31, step), 31, step)
