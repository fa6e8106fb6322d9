"""Nuclei of tens of thousands of tokens, cut and drawn over the whole row: thousands of equal values at the cut, more
members of its bin than are listed (a second and third interval), penalties and a min-p in the kept set, a list too
long for its segment on the way.  (Rows in coarse steps are settled on the first interval, the narrow ones on the others; cuts
on the rounded end of an interval: test_gpu_nucleus_edges.py.)"""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16", [(9, 70001, True), (9, 50003, False), (270, 33003, True)])
def test_cut_over_the_whole_row(B, V, bf16):
    rng = np.random.default_rng(V)
    z = rng.standard_normal((B, V)).astype(np.float32)
    kind = np.arange(B) % 9
    for b, k in enumerate(kind):
        if k in (0, 1, 2):
            z[b] = np.round(z[b] * (2, 8, 16)[k]) / (2, 8, 16)[k]       # a cut among hundreds to ten thousands of equal values
        elif k in (3, 4, 5):
            z[b] = 4.0 + z[b] * (2e-3, 1e-5, 3e-7)[k - 3]               # the whole row in one bin of the first interval
        elif k == 8:
            z[b] *= 2.0
    params = dict(temperature=np.choose(kind, [1.0, 0.8, 1.2, 1.0, 1.0, 1.0, 1.0, 0.9, 1.5]),
                  top_p=np.choose(kind, [0.9, 0.6, 0.97, 0.5, 0.9, 0.7, 0.8, 0.95, 0.9]),
                  min_p=np.choose(kind, [0, 0, 0, 0, 0, 0, 0, 1e-3, 0]),
                  repetition_penalty=np.choose(kind, [1.2, 1, 1, 1, 1, 1, 1.3, 1.1, 1]),
                  frequency_penalty=np.choose(kind, [0.2, 0, 0, 0, 0, 0, 0.3, 0, 0]))
    hist = [rng.integers(0, V, 900).tolist() if params["repetition_penalty"][b] != 1 else [] for b in range(B)]
    w = H.custom(f"wide_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=0)
    d = H.to_device(w)
    for step in range(4 if B < 10 else 1):
        H.compare(w, H.run_gpu(d, 13, step), 13, step)
        assert (H.last_row_path[np.isin(kind, (6, 8))] == 16).all(), H.last_row_path[:9]
        if B < 10:                                                  # (one chunk's queues do not take a level of equal values)
            assert np.isin(H.last_row_path[kind < 3], (1, 3, 15, 16)).all(), H.last_row_path
