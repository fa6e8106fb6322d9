"""Rows streamed and finished by one workgroup: both sides of the rule that chooses it, both of its kernels, rows
that it passes on, queues that go out early or overflow, pieces, and a state (whose call number is taken ahead)."""
import numpy as np
import pytest
import torch

import paper_2506_22033_amd as sip
import workloads
from tests import sip_harness as H
from tests.test_gpu_sharded import _run_sharded
from tests.test_gpu_state import DeviceState

pytestmark = pytest.mark.gpu


def _batch(B, V, bf16, seed):
    """Rows of eight kinds: everything on, a long list and history (queues go out early), a history of thousands of
    neighbours (queues overflow), plain, greedy, a wide nucleus, masked almost everywhere, coarse values."""
    rng = np.random.default_rng(seed)
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    kind = np.arange(B) % 8
    hist = []
    for b, k in enumerate(kind):
        if k == 5:
            z[b] *= 0.2
        elif k == 6:
            keep = rng.choice(V, 300, replace=False)
            row = np.full(V, -np.inf, np.float32)
            row[keep] = z[b, keep]
            z[b] = row
        elif k == 7:
            z[b] = np.round(z[b] * 8) / 8
        n = [700, 9000, 12000, 40, 0, 300, 300, 2000][k]
        hist.append((np.arange(n) + b if k == 2 else rng.integers(0, V, n)).tolist())
    params = dict(temperature=np.choose(kind, [0.8, 1.0, 0.9, 1.1, 0.0, 1.2, 1.0, 0.7]),
                  top_k=np.choose(kind, [50, 2500, 60, 0, 0, 0, 100, 40]),
                  top_p=np.choose(kind, [0.9, 0.99, 1.0, 1.0, 1.0, 0.9, 0.95, 0.9]),
                  min_p=np.choose(kind, [0.02, 0, 0, 0, 0, 0, 0, 0.01]),
                  repetition_penalty=np.choose(kind, [1.2, 1.1, 1.1, 1.0, 1.0, 1.0, 1.3, 1.1]),
                  frequency_penalty=np.choose(kind, [0.3, 0, 0, 0, 0, 0, 0.2, 0.1]))
    return H.custom(f"row_{B}_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=3)


@pytest.mark.parametrize("B,V,bf16", [(224, 33001, False), (226, 36005, True), (130, 40000, True), (261, 34000, True),
                                      (515, 33000, False)])
def test_rows_of_every_kind(B, V, bf16):
    w = _batch(B, V, bf16, B)
    d = H.to_device(w)
    st = H.compare(w, H.run_gpu(d, 5, 0), 5, 0)
    assert st.rows == B
    path, why, kind = H.last_row_path, H.last_row_why, np.arange(B) % 8
    assert (why[np.isin(kind, (0, 3, 4))] == 1).all() and (path[kind == 3] == 16).all()
    assert (why[kind == 2] == 3).all(), why[kind == 2]               # the overflow is seen and the row taken over


@pytest.mark.parametrize("B,t,V_shard,bf16", [(224, 4, 8200, True), (300, 5, 8192, False)])
def test_pieces(B, t, V_shard, bf16):
    w = _batch(B, t * V_shard, bf16, B)
    out, path = _run_sharded(w, t, 9, 1, w.k_logprobs, pad=8)
    H.compare(w, out, 9, 1)
    assert (path[np.arange(B) % 8 == 0] == 1).all()


def test_state_calls_take_their_number_and_append():
    """1030 rows: the same bits as a call without a state on the same histories, twice, the second time with the
    first call's ids appended and the next number."""
    B, V, L = 1030, 33000, 64
    rng = np.random.default_rng(3)
    z = torch.from_numpy((rng.standard_normal((B, V)) * 2.0).astype(np.float32)).to(H.DEV)
    hist = [rng.integers(0, V, int(n)).tolist() for n in rng.integers(0, L - 4, B)]
    f = lambda x: torch.full((B,), x, device=H.DEV)                                     # noqa: E731
    params = dict(temperature=f(0.9), top_p=f(0.95), top_k=torch.full((B,), 60, dtype=torch.int32, device=H.DEV),
                  frequency_penalty=f(0.4), repetition_penalty=f(1.1))
    st = DeviceState(B, L)
    slots = rng.permutation(B).astype(np.int32)
    st.assign(slots.tolist(), hist)
    slot_of_row = torch.from_numpy(slots).to(H.DEV)
    for call in (0, 1):
        got = sip.sip_sample_state(z, params, st.buf, B, L, slot_of_row, 21, 7, 2)
        indptr = torch.from_numpy(np.concatenate(([0], np.cumsum([len(h) for h in hist]))).astype(np.int64)).to(H.DEV)
        tokens = torch.tensor([t for h in hist for t in h], dtype=torch.int32, device=H.DEV)
        want = sip.sip_sample(z, params, indptr, tokens, 21, 7 + call, 2, V=V)
        torch.cuda.synchronize()
        for g, x in zip(got, want):
            assert torch.equal(g, x)
        for h, i in zip(hist, want[0].tolist()):
            h.append(i)
    tick, overflow, length, _ = st.read()
    assert tick == 2 and overflow == 0 and [int(length[s]) for s in slots] == [len(h) for h in hist]
