"""Rows without any filter, drawn through the block masses that the streaming kernel leaves: chunk and
block edges, the smallest and largest vocabulary, both kinds of finishing kernel, lists of several
batches and chunks whose list leaves no room for the masses (those rows are drawn the longer way)."""
import numpy as np
import pytest
import torch

import paper_2506_22033_amd as sip
import workloads
from oracle import sip_oracle as O
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16", [(5, 32769, False), (5, 32769, True), (2, 262144, False), (3, 262144, True),
                                      (7, 66049, False), (300, 33280, True), (300, 33281, False), (530, 40000, False)])
def test_chunk_and_block_edges(B, V, bf16):
    rng = np.random.default_rng(V + B)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    z[0] = z[0] * 0.25 - 8.0
    z[0, [0, 1023, 1024, V - 2, V - 1]] = 1.0                  # the mass of a row at the ends of its blocks
    z[1, : V - 150] -= 20.0                                    # only the last blocks have any
    params = dict(temperature=rng.uniform(0.5, 1.5, B), repetition_penalty=rng.choice([1.0, 1.2], B),
                  frequency_penalty=rng.choice([0.0, 0.3], B))
    hist = [rng.integers(0, V, int(rng.choice([0, 300, 2000]))).tolist() for _ in range(B)]
    if B < 10:
        params["repetition_penalty"][[1, -1]] = 1.2
        hist[1] = list(range(3000, 8500))                      # more than a chunk's segment takes
        hist[-1] = hist[-1] if B == 2 else list(range(100, 8100, 3))   # a list of several batches
    w = H.custom(f"plain_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=2)
    d = H.to_device(w)
    for step in (0, 1, 2) if B < 10 else (0,):
        H.compare(w, H.run_gpu(d, 11, step), 11, step)
    # every row through its block masses, but for the one whose list leaves no room for them
    by_blocks = (H.last_row_path == 16) & (H.last_row_why == 1)
    rest = np.flatnonzero(~by_blocks)
    assert np.array_equal(rest, [1] if B < 10 else []), (rest, H.last_row_path[rest], H.last_row_why[rest])


def test_draws_of_flat_rows_against_float64():
    """51200 draws from 512 flat rows of 40000 entries, with an edge of the cumulative distribution every 2.5e-5.
    A cumulative mass that is off by eps moves a draw with probability 2 eps / 2.5e-5.  With integer sums what
    is off are the fp32 sums of the 16-byte loads, 2^-25 of themselves each: 10000 independent ones come to
    3e-10 of the total, to half of that at an edge on the way, so that less than one draw in 51200 is expected to
    move (none does); with block sums in fp32 four of these did."""
    V, B = 40000, 512
    rng = np.random.default_rng(V)
    z = torch.from_numpy((rng.standard_normal((B, V)) * 0.3).astype(np.float32)).to(H.DEV)
    tau = torch.from_numpy(rng.uniform(0.6, 1.4, B).astype(np.float32)).to(H.DEV)
    s = z / tau[:, None]
    cdf = (s.double() - s.max(dim=1, keepdim=True).values.double()).exp_().cumsum_(1)
    cdf /= cdf[:, -1:].clone()
    moved = 0
    for step in range(100):
        u = torch.tensor([O.row_uniform(5, b, step) for b in range(B)], dtype=torch.float64, device=H.DEV)
        want = torch.searchsorted(cdf, u[:, None], right=True)[:, 0]
        moved += int((sip.sip_sample(z, dict(temperature=tau), None, None, 5, step, -1, V=V)[0] != want).sum())
    assert moved <= 1, moved
