"""Batches whose chunks have a compute unit each: one kernel, the last of a row's workgroups finishing it."""
import numpy as np
import pytest
import torch

import paper_2506_22033_amd as sip
import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


def _inputs(B, V, bf16, n_hist, seed, k):
    rng = np.random.default_rng(seed)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    kind = np.arange(B) % 5
    params = dict(temperature=np.choose(kind, [0.0, 0.7, 1.0, 0.8, 0.9]), top_k=np.choose(kind, [0, 40, 0, 0, 9000]),
                  min_p=np.choose(kind, [0, 0, 0.05, 0, 0]), top_p=np.choose(kind, [1, 0.9, 1, 1, 1]),
                  repetition_penalty=np.full(B, 1.2), frequency_penalty=np.choose(kind, [0, 0.2, 0, 0.1, 0]))
    hist = [rng.integers(0, V, n_hist if b % 3 else 0).tolist() for b in range(B)]
    return H.custom(f"alone_{B}_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=k)


# one row; rows in odd numbers, a grid that is no multiple of the XCDs; the smallest rows of several chunks; batches beyond 32
# rows, which two kernels serve, or a row to a workgroup; ids only
@pytest.mark.parametrize("B,V,bf16,n_hist,k", [(1, 40001, False, 50, 3), (1, 262144, True, 3000, 0), (7, 33000, True, 700, 5), (37, 50003, False, 300, 20),
                                               (85, 66001, False, 200, 1), (86, 66001, True, 200, -1), (127, 34567, True, 2500, 2),
                                               (128, 131073, True, 300, 1), (129, 40000, False, 100, 1)])
def test_against_the_oracle(B, V, bf16, n_hist, k):
    w = _inputs(B, V, bf16, n_hist, V + B, k)
    d = H.to_device(w)
    rows = sorted(set(range(0, B, max(1, B // 25))) | {B - 1})
    for step in range(2):
        H.compare(w, H.run_gpu(d, 5, step), 5, step, rows=rows)


@pytest.mark.parametrize("fill", [0x00, 0xFF, None])
def test_whatever_the_workspace_holds(fill):
    """Nothing in the workspace has to be cleared; None: what other calls of the same and of other shapes have left."""
    w = _inputs(24, 60001, False, 500, 11, 4)
    d = H.to_device(w)
    want = H.run_gpu(d, 9, 0)
    H.compare(w, want, 9, 0, rows=range(0, 24, 5))
    need = sip.sip_workspace_bytes(24, d.V, sip.SIP_F32, d.tokens.numel(), 4)
    ws = torch.empty(need, dtype=torch.uint8, device=H.DEV)
    for rep in range(3):
        if fill is None:
            z = torch.randn(3 + rep, 40000, device=H.DEV)
            sip.sip_sample(z, None, None, None, 1, rep, 0, workspace=ws)
        else:
            ws.fill_(fill)
        ids, lp_ids, lp = sip.sip_sample(d.logits, d.params, d.indptr, d.tokens, 9, 0, 4, V=d.V, workspace=ws)
        for got, ref in zip((ids, lp_ids, lp), want):
            assert np.array_equal(got.cpu().numpy(), ref)


def test_recorded_call_replayed():
    """The words that count a row's workgroups are as a replay needs them, whatever ran in between on the workspace."""
    w = _inputs(12, 70001, True, 400, 3, 2)
    d = H.to_device(w)
    ids = torch.empty(12, dtype=torch.int32, device=H.DEV)
    lp_ids = torch.empty(12, 3, dtype=torch.int32, device=H.DEV)
    lp = torch.empty(12, 3, dtype=torch.float32, device=H.DEV)
    ws = torch.empty(sip.sip_workspace_bytes(12, d.V, sip.SIP_BF16, d.tokens.numel(), 2), dtype=torch.uint8, device=H.DEV)
    call = lambda: sip.sip_sample(d.logits, d.params, d.indptr, d.tokens, 7, 0, 2, V=d.V, out_ids=ids, out_lp_ids=lp_ids,    # noqa: E731
                                  out_lp=lp, workspace=ws)
    call()
    torch.cuda.synchronize()
    want = [x.cpu().numpy().copy() for x in (ids, lp_ids, lp)]
    H.compare(w, want, 7, 0)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for rep in range(4):
        ids.zero_()
        lp.zero_()
        if rep == 2:
            call()
            ids.zero_()
        g.replay()
        torch.cuda.synchronize()
        for got, ref in zip((ids, lp_ids, lp), want):
            assert np.array_equal(got.cpu().numpy(), ref)


def test_pieces():
    """As many chunks as there are pieces, and several of a piece."""
    rng = np.random.default_rng(4)
    for t, B in ((2, 3), (4, 60), (8, 20)):
        V = 16384 * t
        z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
        w = H.custom(f"alone_pieces_{t}", z, dict(temperature=0.8, top_p=0.9, top_k=50), None, k_logprobs=3)
        pieces = [torch.from_numpy(np.ascontiguousarray(z[:, i * 16384:(i + 1) * 16384])).to(H.DEV) for i in range(t)]
        p = {k: None if v is None else torch.from_numpy(v).to(H.DEV) for k, v in w.params.items()}
        out = sip.sip_sample_sharded(pieces, p, None, None, 3, 1, 3)
        H.compare(w, [x.cpu().numpy() for x in out], 3, 1, rows=range(0, B, 4))


# the most rows and, in 36 units of 1024 elements, the longest chunks that go this way; eleven and sixteen chunks; the second to
# last and the last element of every chunk in a history
@pytest.mark.parametrize("B,V,bf16,k", [(32, 184320, True, 5), (32, 184317, False, 0), (22, 262142, True, 0), (16, 262144, False, 5), (11, 70003, True, 3)])
def test_longest_chunks(B, V, bf16, k):
    rng = np.random.default_rng(V + B)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    kind = np.arange(B) % 5                  # no filter, top-p, min-p, top-k, greedy
    params = dict(temperature=np.choose(kind, [0.8, 0.7, 1.0, 0.9, 0.0]), top_p=np.choose(kind, [1, 0.3, 1, 1, 1]),
                  min_p=np.choose(kind, [0, 0, 0.05, 0, 0]), top_k=np.choose(kind, [0, 0, 0, 60, 0]), repetition_penalty=np.full(B, 1.3))
    w = H.custom(f"longest_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, None, k_logprobs=k)
    route, S = sip.sip_call_route(B, V, sip.SIP_BF16 if bf16 else sip.SIP_F32, 0, False, w.params, 0, k)
    assert route == 2 and 1 < S and B * S <= 176
    n = -(-V // 1024)
    ends = sorted({min((c + 1) * n // S * 1024, V) - i for c in range(S) for i in (1, 2)})
    w = H.custom(f"longest_{V}", w.logits, params, [ends + rng.integers(0, V, 100).tolist() for _ in range(B)], k_logprobs=k)
    H.compare(w, H.run_gpu(H.to_device(w), 5, 1), 5, 1, rows=range(0, B, 2))
    assert (H.last_row_why == 1).all(), H.last_row_why


# ids only and no filter: chunks of up to 131072 elements (128 blocks), and of several whole pieces (three of 43000 elements have
# load numbers of six bits)
@pytest.mark.parametrize("B,V,bf16,t,S", [(128, 262144, False, 0, 2), (128, 262142, True, 0, 2), (86, 200001, True, 0, 2), (37, 262143, False, 0, 6),
                                          (128, 258000, True, 6, 2), (66, 258000, False, 6, 3), (100, 131072, True, 8, 2), (100, 100000, False, 4, 2)])
def test_ids_of_rows_without_a_filter(B, V, bf16, t, S):
    rng = np.random.default_rng(V + B)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    z[0, V - 1] = z[3, V // 2 - 1] = z[4, V // 2] = 30.0
    kind = np.arange(B) % 3
    params = dict(temperature=np.choose(kind, [0.0, 0.8, 0.0]), repetition_penalty=np.choose(kind, [1.0, 1.2, 1.2]))
    hist = [np.concatenate(([V - 1, V // S - 1, 0], rng.integers(0, V, 50))).tolist() for _ in range(B)]
    w = H.custom(f"no_filter_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=-1)
    assert sip.sip_call_route(B, V, sip.SIP_BF16 if bf16 else sip.SIP_F32, t, False, w.params, 53 * B, -1) == (2, S)
    d = H.to_device(w)
    rows = sorted(set(range(0, B, max(1, B // 24))) | {3, 4, B - 1})
    if t:
        n = V // t
        ids, _, _ = sip.sip_sample_sharded([d.logits[:, i * n:(i + 1) * n].contiguous() for i in range(t)], d.params, d.indptr, d.tokens, 3, 1, -1)
        out = (ids.cpu().numpy(), None, None)
    else:
        out = H.run_gpu(d, 3, 1, k_logprobs=-1)
        assert (H.last_row_why == 1).all(), H.last_row_why
    H.compare(w, out, 3, 1, rows=rows, k_logprobs=-1)
