"""The threshold of rows that top-p or min-p alone bounds, raised as far as the row's sample allows: peaked rows, rows on
both sides of the line, rows whose largest tokens a penalty takes away (the list then ends too high, and a second one
settles the row), logits far from 0 on either side, where a bin of the sample is wide or the outermost one, and samples with few or equal values."""
import numpy as np
import pytest
import torch

import paper_2506_22033_amd as sip
import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16", [(12, 100003, True), (12, 131072, False), (24, 45001, False), (12, 33001, True),
                                      (240, 70001, True), (300, 36003, True)])
def test_raised_threshold(B, V, bf16):
    rng = np.random.default_rng(V + B)
    kind = np.arange(B) % 12
    z = rng.standard_normal((B, V)).astype(np.float32) * 2.5
    hist = [[] for _ in range(B)]
    for b, k in enumerate(kind):
        if k in (0, 1, 7):
            z[b] = rng.standard_t(3, V) * 2.0
        elif k in (2, 3):
            z[b, rng.integers(0, V, 8)] += 9.0
        elif k == 4:
            z[b] = z[b] * 4.0 + (300.0 if b < 12 else 700.0)       # a group of bins is several powers of e wide; the outermost bin
        elif k == 5:
            z[b] = z[b] * 4.0 - 300.0
        elif k == 6:
            z[b] = np.where(rng.random(V) < 0.02, np.round(z[b]) + 12.0, -np.inf)   # masked, and many equal values
        elif k == 8:
            z[b] = np.round(z[b]) * 2.0                            # a few dozen values
        elif k == 11:
            z[b] *= 1e-3                                           # the bins around 0
        elif k == 9:
            z[b, :V // 2] = -1e30
        if k == 7:
            hist[b] = np.argsort(-z[b])[:V // 100].tolist()        # every token that could be kept is penalised
        elif k in (1, 3, 10):
            hist[b] = rng.integers(0, V, 700).tolist()
    params = dict(temperature=np.choose(kind, [1.0, 0.8, 0.7, 0.6, 0.9, 0.9, 0.5, 1.0, 0.5, 1.0, 0.4, 1.5]),
                  top_p=np.choose(kind, [0.9, 0.95, 0.95, 1.0, 0.9, 0.8, 0.9, 0.9, 0.5, 0.99, 0.9, 0.3]),
                  min_p=np.choose(kind, [0, 0, 0, 0.05, 0, 0.01, 0, 0, 0, 0.02, 0.05, 0]),
                  repetition_penalty=np.choose(kind, [1, 1.2, 1, 1.1, 1, 1, 1, 1.5, 1, 1, 1, 1]),
                  presence_penalty=np.choose(kind, [0, 0, 0, 0, 0, 0, 0, 30.0, 0, 0, 0.5, 0]))
    w = H.custom(f"raised_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=4)
    d = H.to_device(w)
    for step in range(4 if B < 30 else 1):
        H.compare(w, H.run_gpu(d, 23, step), 23, step)
        # what the raised list must not lose: peaked rows are settled from it
        assert (H.last_row_why[np.isin(kind, (0, 1, 3))] == 1).all(), H.last_row_why[:12]


@pytest.mark.parametrize("B,V,bf16", [(12, 65536, True), (12, 65537, False), (66, 40001, True), (300, 36003, False)])
def test_largest_values_around_zero(B, V, bf16):
    """The row's largest in [0, 1/4), on both sides of 0 or just below it, everything else far below: the list reaches
    down to where they begin, so that it settles the rows."""
    rng = np.random.default_rng(V)
    kind = np.arange(B) % 4
    z = -1.05 - np.abs(rng.standard_normal((B, V)).astype(np.float32)) * 4.0
    hist = [[] for _ in range(B)]
    for b, k in enumerate(kind):
        top = rng.permutation(V)[:V // 100]
        z[b, top] = (0.24, 0.1, 0.3, -0.2)[k] + (-0.24, 0.1, -0.5, 0.19)[k] * rng.random(top.size)
        if k == 1:
            hist[b] = rng.integers(0, V, 300).tolist()
    params = dict(temperature=np.choose(kind, [0.1, 0.2, 0.15, 0.1]), top_p=np.choose(kind, [0.9, 0.9, 1, 0.9]),
                  min_p=np.choose(kind, [0, 0, 0.02, 0]), repetition_penalty=np.full(B, 1.1))
    w = H.custom(f"around0_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=2)
    d = H.to_device(w)
    rows = list(range(B)) if B < 30 else list(range(0, B, B // 24))
    for step in range(3 if B < 30 else 1):
        H.compare(w, H.run_gpu(d, 47, step), 47, step, rows=rows)
        assert (H.last_row_why == 1).all(), H.last_row_why[:12]


@pytest.mark.parametrize("B,V,bf16", [(60, 50000, True), (60, 65537, False), (300, 40003, True), (600, 50021, False)])
def test_coarse_values(B, V, bf16):
    """Whole numbers, halves and ties at 0: a raised threshold lies on a value that many tokens have, which the nucleus
    may end with, or which may be the largest there is.  The list settles all of them."""
    rng = np.random.default_rng(V + B)
    kind = np.arange(B) % 6
    z = rng.standard_normal((B, V)).astype(np.float32)
    for b, k in enumerate(kind):
        if k < 4:
            z[b] = np.round(z[b] * (2.0, 2.0, 4.0, 3.0)[k]) / (1.0, 1.0, 2.0, 1.0)[k]
        else:
            z[b] = -1.05 - np.abs(z[b]) * 4.0
            top = rng.permutation(V)[:V // 75]
            z[b, top] = 0.0
            if k == 5:
                z[b, top[::2]] = -0.0
    params = dict(temperature=np.choose(kind, [0.5, 0.3, 0.5, 0.9, 0.1, 0.1]), top_p=np.choose(kind, [0.9, 0.99, 0.9, 1.0, 0.9, 0.9]),
                  min_p=np.choose(kind, [0, 0, 0, 0.05, 0, 0]))
    w = H.custom(f"coarse_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, [[] for _ in range(B)], k_logprobs=0)
    d = H.to_device(w)
    rows = list(range(0, B, max(1, B // 30)))
    for step in range(2):
        H.compare(w, H.run_gpu(d, 53, step), 53, step, rows=rows)
        assert (H.last_row_why == 1).all(), (H.last_row_why[:12], np.bincount(kind[H.last_row_why != 1]))


@pytest.mark.parametrize("B,V", [(12, 131072), (40, 131072)])
def test_which_lists_are_short(B, V):
    """A row's list lies in the workspace, a logit's bits with its index above them.  Peaked rows have the 512 tokens that
    every list holds, give or take three standard deviations of the sample's 32 and a group of bins, which a Student-t
    tail puts a fifth more into; normal logits of standard deviation 3.8, of which 95 % of the mass are some 2000
    tokens, half of what is left out being the least that may lie below a list, have more than twice that many."""
    rng = np.random.default_rng(V + B)
    z = (rng.standard_normal((B, V)) * 3.8).astype(np.float32)
    z[::2] = rng.standard_t(3, (B // 2, V)) * 2.0
    z[::2, 17] = 40.0 + np.arange(B // 2)
    w = H.custom("lists", z, dict(temperature=np.ones(B), top_p=np.full(B, 0.9)), k_logprobs=0)
    d = H.to_device(w)
    ws = torch.zeros(sip.sip_workspace_bytes(B, V, sip.SIP_F32, 0, 0), dtype=torch.uint8, device=H.DEV)
    sip.sip_sample(d.logits, d.params, None, None, 23, 0, 0, V=V, workspace=ws)
    torch.cuda.synchronize()
    assert (ws[:8 * B].view(torch.int32) == 1).all()
    words = ws[:ws.numel() // 8 * 8].view(torch.int64)
    place = torch.arange(V, device=H.DEV) << 32
    for b in range(B):
        bits = d.logits[b, :V].view(torch.int32).to(torch.int64) & 0xFFFFFFFF
        n = int(torch.isin(bits | place, words).sum())
        assert (240 < n < 1000) if b % 2 == 0 else (1100 < n < 4096), (b, n)
