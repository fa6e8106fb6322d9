"""Long histories of rows that one workgroup streams: the queues go out in time, however evenly they fill up."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H
from tests.test_gpu_sharded import _run_sharded

pytestmark = pytest.mark.gpu


def _batch(B, V, bf16, n):
    rng = np.random.default_rng(B + n)
    z = (rng.standard_normal((B, V)) * 2.5).astype(np.float32)
    hist = [rng.permutation(V)[:n].tolist() for _ in range(B)]
    params = dict(temperature=np.full(B, 0.8), top_k=np.full(B, 50), repetition_penalty=np.full(B, 1.1))
    return H.custom(f"queues_{V}_{n}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=1)


@pytest.mark.parametrize("B,V,bf16,n", [(224, 50001, False, 7500), (224, 50001, False, 9000), (224, 50001, False, 13000),
                                        (300, 40000, False, 6500), (240, 60005, True, 10500), (240, 60005, True, 13000)])
def test_history_tokens_by_the_thousand(B, V, bf16, n):
    w = _batch(B, V, bf16, n)
    out = H.run_gpu(H.to_device(w), 4, 0)
    assert (H.last_row_why == 1).all(), H.last_row_why
    H.compare(w, out, 4, 0, rows=range(0, B, 7))


def test_history_tokens_by_the_thousand_in_pieces():
    B, t, V_shard = 224, 4, 12504
    w = _batch(B, t * V_shard, False, 9000)
    out, path = _run_sharded(w, t, 4, 0, w.k_logprobs, pad=8)
    assert (path == 1).all(), path
    H.compare(w, out, 4, 0, rows=range(0, B, 7))
