"""Thresholds wherever the logits lie: with an offset to either side, beyond the sample histogram's range, all of them small,
of very different sizes, masked with -inf or with a large negative number.  The list settles the rows all the same."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16", [(8, 60001, True), (8, 65536, False), (24, 128256, False), (272, 40003, True), (260, 36001, False)])
def test_thresholds_anywhere(B, V, bf16):
    rng = np.random.default_rng(V + B)
    kind = (np.arange(B) + np.arange(B) // 8) % 8
    z = rng.standard_normal((B, V)).astype(np.float32) * 2.0
    for b, k in enumerate(kind):
        if k in (0, 1):
            z[b] += (100.0, -100.0)[k]
        elif k == 2:
            z[b] = z[b] * 4.0 - 600.0
        elif k == 3:
            z[b] *= 1e-4
        elif k == 4:
            z[b, rng.permutation(V)[300:]] = -np.inf
        elif k == 5:
            z[b, rng.random(V) < 0.5] = -1e9
            z[b] -= 90.0
        elif k == 6:
            z[b, rng.random(V) < 0.5] = -1e30
            z[b] += np.where(rng.random(V) < 0.002, 150.0, 0.0).astype(np.float32)
        else:
            z[b] -= 5.2                                            # the threshold about 0
    mode = np.arange(B) // 3 % 4
    params = dict(temperature=np.choose(mode, [0.0, 0.8, 1.0, 0.7]), top_k=np.choose(mode, [0, 50, 0, 0]),
                  top_p=np.choose(mode, [1.0, 0.9, 1.0, 1.0]), min_p=np.choose(mode, [0.0, 0.0, 0.1, 0.0]))
    hist = [rng.integers(0, V, 200).tolist() if b % 5 == 0 else [] for b in range(B)]
    params["repetition_penalty"] = np.full(B, 1.1)
    w = H.custom(f"bins_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=2)
    d = H.to_device(w)
    rows = list(range(0, B, max(1, B // 24)))
    coarse = (kind == 2) & bf16                                    # (a few dozen values at 600)
    settled = ~coarse & ~(np.isin(kind, (2, 3)) & (mode == 2))     # (flat rows under min-p)
    for step in range(2):
        H.compare(w, H.run_gpu(d, 59, step), 59, step, rows=rows)
        why = H.last_row_why[settled]
        assert (why == 1).all(), (kind[settled][why != 1], mode[settled][why != 1], why[why != 1])


@pytest.mark.parametrize("B,V,bf16", [(8, 38144, False), (8, 65936, True), (24, 50001, True)])
def test_largest_in_one_part_of_the_ids(B, V, bf16):
    """A sixth of the ids holds all that is likely, as where ids follow frequency: some of the sample's threads have
    far more than their share of the largest values."""
    rng = np.random.default_rng(V)
    z = rng.standard_normal((B, V)).astype(np.float32)
    z[:, :V // 3] -= 8.0
    z[:, V // 2:] -= 8.0
    params = dict(temperature=np.full(B, 0.5), top_p=np.full(B, 0.5), repetition_penalty=np.full(B, 1.1))
    hist = [rng.integers(0, V, 300).tolist() for _ in range(B)]
    w = H.custom(f"part_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=1)
    H.compare(w, H.run_gpu(H.to_device(w), 59, 0), 59, 0)
    assert (H.last_row_why == 1).all(), H.last_row_why
