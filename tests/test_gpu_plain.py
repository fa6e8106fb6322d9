"""Rows without any filter, drawn through the block masses that the streaming kernel leaves: chunk and
block edges, the smallest and largest vocabulary, both kinds of finishing kernel, lists of several
batches and chunks whose list leaves no room for the masses (those rows are drawn the longer way)."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16", [(5, 32769, False), (5, 32769, True), (2, 262144, False), (3, 262144, True),
                                      (7, 66049, False), (300, 33280, True), (300, 33281, False), (530, 40000, False)])
def test_chunk_and_block_edges(B, V, bf16):
    rng = np.random.default_rng(V + B)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    z[0] = -8.0
    z[0, [0, 511, 512, V - 2, V - 1]] = 1.0                  # the mass of a row at the ends of its blocks
    z[1, : V - 700] = -np.inf                                # only the last blocks have any
    params = dict(temperature=rng.uniform(0.5, 1.5, B), repetition_penalty=rng.choice([1.0, 1.2], B),
                  frequency_penalty=rng.choice([0.0, 0.3], B))
    hist = [rng.integers(0, V, int(rng.choice([0, 300, 2000]))).tolist() for _ in range(B)]
    if B < 10:
        hist[1] = list(range(3000, 8500))                    # a list of several batches, one chunk's worth of it
    w = H.custom(f"plain_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=2)
    d = H.to_device(w)
    for step in (0, 1, 2) if B < 10 else (0,):
        H.compare(w, H.run_gpu(d, 11, step), 11, step)
    assert (H.last_row_path == 16).mean() > 0.9 or B < 10, np.unique(H.last_row_path)
