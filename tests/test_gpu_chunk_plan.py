"""Chunks as a compute unit's share asks for them: one, two and three to a compute unit, on a few rows with far longer
histories than the others (all of them settled from their lists), both sides of the lines between chunks and a row to a
workgroup, and the longer queues that come with fewer chunks."""
import numpy as np
import pytest

import paper_2506_22033_amd as sip
import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16,long_row", [(64, 128256, False, 11000), (64, 128256, True, 7000), (128, 131072, False, 11000),
                                               (130, 128003, True, 6000), (48, 70001, False, 9000), (193, 66001, True, 300),
                                               (192, 100001, False, 5000), (367, 51201, False, 300), (368, 51203, False, 300)])
def test_shares_of_a_compute_unit(B, V, bf16, long_row):
    rng = np.random.default_rng(V + B)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    kind = np.arange(B) % 4
    params = dict(temperature=np.choose(kind, [0.0, 0.7, 1.0, 0.8]), top_k=np.choose(kind, [0, 40, 0, 0]),
                  min_p=np.choose(kind, [0, 0, 0.05, 0]), repetition_penalty=np.full(B, 1.2))
    hist = [rng.integers(0, V, long_row if b in (1, B // 2, B - 1) else 200).tolist() for b in range(B)]
    w = H.custom(f"plan_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=2)
    d = H.to_device(w)
    rows = sorted(set(range(0, B, max(1, B // 40))) | {1, B // 2, B - 1})
    H.compare(w, H.run_gpu(d, 29, 1), 29, 1, rows=rows)
    assert sip.binding.load().sip_plan_chunks(B, V, sip.SIP_BF16 if bf16 else sip.SIP_F32, 0) * B <= 1024
    assert (H.last_row_why == 1).all(), H.last_row_why


@pytest.mark.parametrize("B,V,bf16,S,n", [(64, 128256, False, 4, 11000), (64, 128256, True, 4, 6000), (128, 131072, False, 4, 6500),
                                          (48, 70001, False, 5, 6000)])
def test_history_in_one_chunk(B, V, bf16, S, n):
    """Three rows' histories lie in the first of the row's S chunks: more of them for each of its eight queues than the 480
    entries that a queue has where four workgroups share a compute unit."""
    assert sip.binding.load().sip_plan_chunks(B, V, sip.SIP_BF16 if bf16 else sip.SIP_F32, 0) == S
    assert sip.sip_call_route(B, V, sip.SIP_BF16 if bf16 else sip.SIP_F32, 0, False, ("top_k", "min_p"), 3 * n, 2) == (5, S)
    assert n > 1.5 * 8 * 480
    rng = np.random.default_rng(V + B)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    kind = np.arange(B) % 3
    params = dict(temperature=np.choose(kind, [0.0, 0.7, 1.0]), top_k=np.choose(kind, [0, 40, 0]),
                  min_p=np.choose(kind, [0, 0, 0.05]), repetition_penalty=np.full(B, 1.2))
    rows = [1, B // 2, B - 1]
    hist = [rng.choice(V // S - 2048, n, replace=False).tolist() if b in rows else [] for b in range(B)]
    w = H.custom(f"plan1_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=2)
    H.compare(w, H.run_gpu(H.to_device(w), 29, 1), 29, 1, rows=rows)
    assert (H.last_row_why == 1).all(), H.last_row_why
