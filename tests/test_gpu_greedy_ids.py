"""Greedy rows of calls that ask for token ids only: the arg max without a list, in chunks, a row to a workgroup and in pieces,
beside rows that take the general way."""
import numpy as np
import pytest
import torch

import paper_2506_22033_amd as sip
import workloads
from tests import sip_harness as H
from tests.test_gpu_state import DeviceState

pytestmark = pytest.mark.gpu


def _rows(B, V, bf16, seed):
    """Rows whose maximum is found at edges: the first and last element, the ends of loads and tiles, several equal ones (the first
    counts), zeros of both signs, all negative, one finite value, none."""
    rng = np.random.default_rng(seed)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    for b in range(B):
        k = b % 12
        if k == 1: z[b, 0] = 50.0
        if k == 2: z[b, V - 1] = 50.0
        if k == 3: z[b, [V - 1, 77, 4096, 16383, 16384, 9]] = 50.0
        if k == 4: z[b] = 0.25
        if k == 5: z[b] = -np.abs(z[b]) - 1.0; z[b, [V // 2, V - 2]] = 0.0; z[b, V // 3] = -0.0
        if k == 6: z[b] -= 1e4
        if k == 7: z[b] = -np.inf; z[b, V - 3] = -1e30
        if k == 8: z[b] = np.round(z[b])
        if k == 9: z[b, [V // 2, V // 2 + 1]] = 50.0
    return workloads.f32_to_bf16_bits(z) if bf16 else z


# one row in many chunks; odd numbers of rows and elements; chunks that the finishing kernels compare, with the heavier logic in the
# same kernel and behind it; a row to a workgroup, one round and several; pieces
@pytest.mark.parametrize("B,V,bf16,t", [(1, 152064, True, 0), (13, 33001, False, 0), (37, 40003, True, 0), (86, 150001, True, 0),
                                        (128, 262144, False, 0), (128, 262142, True, 0), (140, 100000, True, 0), (230, 33333, False, 0),
                                        (300, 40001, True, 0), (260, 52003, False, 0), (24, 8192 * 8, False, 8), (100, 40000, True, 2), (230, 32768, True, 4),
                                        (260, 52000, False, 4)])
def test_arg_max(B, V, bf16, t):
    z = _rows(B, V, bf16, V + B)
    kind = np.arange(B) % 12
    some = kind == 10                       # sampled rows, and greedy ones with a penalty, in between
    params = dict(temperature=np.where(some, 0.8, np.where(kind == 11, 0.7, 0.0)), top_k=np.where(some, 40, np.where(kind == 11, 1, 0)),
                  repetition_penalty=np.where(kind == 0, 1.3, 1.0))
    rng = np.random.default_rng(B)
    hist = [rng.integers(0, V, 40).tolist() for _ in range(B)]
    w = H.custom(f"greedy_{B}_{V}", z, params, hist, k_logprobs=-1)
    d = H.to_device(w)
    rows = [b for b in range(B) if b < 26 or b % 7 == 0]
    if t:
        n = V // t
        pieces = [d.logits[:, i * n:(i + 1) * n].contiguous() for i in range(t)]
        ids, _, _ = sip.sip_sample_sharded(pieces, d.params, d.indptr, d.tokens, 3, 1, -1)
        torch.cuda.synchronize()
        out = (ids.cpu().numpy(), None, None)
    else:
        out = H.run_gpu(d, 3, 1, k_logprobs=-1)
    H.compare(w, out, 3, 1, rows=rows, k_logprobs=-1)


@pytest.mark.parametrize("B,V", [(3, 50001), (200, 40001), (300, 60001), (1100, 33001)])
def test_nothing_above_minus_infinity(B, V):
    """The general path's, beside rows that have something: no list is there for it.  And a state gets the ids."""
    z = torch.randn(B, (V + 3) // 4 * 4, device=H.DEV)
    z[1] = float("-inf")
    params = {"temperature": torch.zeros(B, device=H.DEV)}
    ids, _, _ = sip.sip_sample(z, params, None, None, 3, 1, -1, V=V)
    one, lp_ids, _ = sip.sip_sample(z, params, None, None, 3, 1, 0, V=V)       # the same with log-probabilities: by way of a list
    torch.cuda.synchronize()
    assert torch.equal(ids, one)
    st = DeviceState(B, 4)
    slot = torch.arange(B, dtype=torch.int32, device=H.DEV)
    for _ in range(2):
        got, _, _ = sip.sip_sample_state(z, params, st.buf, B, 4, slot, 3, 1, -1, V=V)
    tick, ovf, length, tokens = st.read()
    assert tick == 2 and (length == 2).all() and np.array_equal(tokens[:, 0], ids.cpu().numpy()) and np.array_equal(tokens[:, 1], ids.cpu().numpy())
