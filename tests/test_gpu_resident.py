"""Rows that one workgroup holds in registers (vocabularies up to 32768): sizes at the edges of the
kernel's variants and of its loads, every kind of row, pieces, a separate prompt, a state."""
import numpy as np
import pytest
import torch

import paper_2506_22033_amd as sip
import workloads
from oracle import sip_oracle as O
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


def _rows(rng, B, V):
    kind = np.arange(B) % 10
    params = dict(temperature=np.choose(kind, [0.0, 1.0, 0.7, 1.3, 0.9, 1.0, 0.3, 0.0, 1.0, 1e-3]),
                  top_k=np.choose(kind, [0, 0, 40, min(V, 4096), 0, 1, 1000, 0, 3, 0]),
                  top_p=np.choose(kind, [1.0, 1.0, 0.95, 0.9, 0.999, 1.0, 0.8, 1.0, 1.0, 0.5]),
                  min_p=np.choose(kind, [0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.05, 0.0, 0.02, 0.0]),
                  repetition_penalty=rng.choice([1.0, 1.3, 0.8], B),
                  frequency_penalty=rng.choice([0.0, 0.4], B),
                  presence_penalty=rng.choice([0.0, 0.3, -0.2], B))
    hist = [rng.integers(-1, V + 1, int(rng.choice([0, 3, 700]))).tolist() for _ in range(B)]
    return params, hist


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("V", [1, 7, 511, 4096, 4097, 8192, 8193, 16384, 16385, 20011, 32767, 32768])
def test_vocabularies_at_the_edges_of_the_variants(V, bf16):
    rng = np.random.default_rng(V + bf16)
    B = 21
    z = (rng.standard_normal((B, V)) * 2.5).astype(np.float32)
    z[4, : V // 2] = -np.inf
    z[11] = np.round(z[11], 1)                                # many equal values
    z[15] = 0.25                                              # all of them equal
    if V > 100:
        z[13, 3:] = -np.inf                                   # fewer finite entries than logprobs asked for
        z[16, 17] = 60.0
    params, hist = _rows(rng, B, V)
    w = H.custom(f"resident_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=5)
    d = H.to_device(w)
    for step in (0, 1):
        H.compare(w, H.run_gpu(d, 3, step), 3, step)
    if V >= 4096:
        assert (H.last_row_why == 1).mean() > 0.8, H.last_row_why


@pytest.mark.parametrize("V,bf16", [(1000, False), (4097, True), (16383, False)])
def test_a_state(V, bf16):
    """Below 16384 entries a state's rows are held in registers too: tick taken ahead, ids appended."""
    rng = np.random.default_rng(V)
    B, L_max, k = 6, 40, 2
    prompts = [rng.integers(0, V, n).tolist() for n in (0, 1, 5, 30, 38, 12)]
    ost = O.DecodeState(B, L_max, V)
    state = torch.zeros(sip.sip_state_bytes(B, L_max), dtype=torch.uint8, device=H.DEV)
    sip.sip_state_init(state, B, L_max)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=H.DEV)                       # noqa: E731
    for s, p in enumerate(prompts):
        ost.assign(s, p)
    indptr = torch.tensor(np.concatenate(([0], np.cumsum([len(p) for p in prompts]))), dtype=torch.int64, device=H.DEV)
    sip.sip_state_assign(state, B, L_max, i32(list(range(B))), indptr, i32([t for p in prompts for t in p]))
    params = dict(temperature=np.float32([0.0, 0.8, 1.0, 1.2, 0.7, 1.0]), top_k=np.int32([0, 20, 0, 0, 5, 300]),
                  top_p=np.float32([1, 1, 0.9, 1, 0.8, 1]), frequency_penalty=np.full(B, 0.4, np.float32),
                  repetition_penalty=np.full(B, 1.2, np.float32))
    full = {n: params.get(n) for n in ("temperature", "top_k", "top_p", "min_p", "repetition_penalty",
                                       "frequency_penalty", "presence_penalty")}
    dev = {n: torch.from_numpy(v).to(H.DEV) for n, v in params.items()}
    ws = torch.empty(sip.sip_workspace_bytes(B, V, sip.SIP_BF16 if bf16 else sip.SIP_F32, B * L_max, k),
                     dtype=torch.uint8, device=H.DEV)
    order = [3, 0, 5, 1, 4, 2]
    for t in range(4):                                        # (slot 4 is full after two of them)
        z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
        zz = workloads.f32_to_bf16_bits(z) if bf16 else z
        out = sip.sip_sample_call(logits=H.logits_to_device(zz), V=V, state=state, slots=B, L_max=L_max, params=dev,
                                  slot_of_row=i32(order), seed=4, step=0, k_logprobs=k, workspace=ws)
        torch.cuda.synchronize()
        assert (ws[4 * B:8 * B].view(torch.int32) == 1).all()
        ref = O.sample_state(zz, full, ost, order, 4, 0, k)
        H.check_rows(f"state step {t}", range(B), ref, tuple(x.cpu().numpy() for x in out), k)


@pytest.mark.parametrize("t,V_shard,bf16", [(2, 4, False), (3, 5000, True), (8, 4096, False), (1, 9000, True)])
def test_pieces(t, V_shard, bf16):
    rng = np.random.default_rng(t)
    B, V = 11, t * V_shard
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    params, hist = _rows(rng, B, V)
    zz = workloads.f32_to_bf16_bits(z) if bf16 else z
    w = H.custom("pieces", zz, params, hist, k_logprobs=2)
    d = H.to_device(w)
    shards = [H.logits_to_device(np.ascontiguousarray(zz[:, i * V_shard:(i + 1) * V_shard])) for i in range(t)]
    out = sip.sip_sample_sharded(sip.ShardTable(shards, V_shard), d.params, d.indptr, d.tokens, 5, 1, 2)
    torch.cuda.synchronize()
    H.compare(w, tuple(x.cpu().numpy() for x in out), 5, 1)
    whole = H.run_gpu(d, 5, 1)
    for x, y in zip(out, whole):
        assert np.array_equal(x.cpu().numpy(), y)


def test_counts_beyond_the_counters_and_a_separate_prompt():
    """Histories that repeat tokens more often than a 15-bit counter holds, one just within, and
    prompt tokens, which only the repetition penalty looks at."""
    rng = np.random.default_rng(9)
    B, V = 4, 6000
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    params = dict(temperature=1.0, top_k=50, frequency_penalty=[1e-4, 1e-4, 0.0, 0.3],
                  presence_penalty=[0.0, 0.1, 0.2, 0.3], repetition_penalty=1.2)
    hist = [rng.permutation([7] * 50000 + [V - 1] * 16385 + [0] * 16384).tolist(), [7] * 32767, [7] * 40000, [1, 2, 2]]
    w = H.custom("long", z, params, hist, k_logprobs=3)
    d = H.to_device(w)
    H.compare(w, H.run_gpu(d, 1, 0), 1, 0)
    assert (H.last_row_why == 1).all(), H.last_row_why
    prompts = [rng.integers(0, V, 3000).tolist() for _ in range(B)]
    p_ind = torch.from_numpy(np.concatenate(([0], np.cumsum([len(p) for p in prompts]))).astype(np.int64)).to(H.DEV)
    p_tok = torch.from_numpy(np.concatenate(prompts).astype(np.int32)).to(H.DEV)
    out = sip.sip_sample_call(logits=d.logits, V=V, params=d.params, hist_indptr=d.indptr, hist_tokens=d.tokens,
                              prompt_indptr=p_ind, prompt_tokens=p_tok, seed=1, step=0, k_logprobs=3)
    torch.cuda.synchronize()
    ref = O.sample_batch(w.logits, w.params, w.hist_indptr, w.hist_tokens, 1, 0, 3,
                         prompt_indptr=p_ind.cpu().numpy(), prompt_tokens=p_tok.cpu().numpy())
    H.check_rows("prompt", range(B), ref, tuple(x.cpu().numpy() for x in out), 3)


def test_masses_are_as_accurate_as_a_float_exponential():
    """Two tokens x apart: the better one's log-probability is -log(1 + e^-x), which gives the mass of the
    other back.  What it is off by, rms: expf's error against float64, 2.62e-8, and the rounding of the
    log-probability to fp32, 2.69e-8 as worked out here."""
    x = np.linspace(0.0, 8.0, 1 << 17, dtype=np.float32)
    z = torch.zeros(len(x), 8, dtype=torch.float32, device=H.DEV)
    z[:, 1] = -torch.from_numpy(x).to(H.DEV)
    _, ids, lp = sip.sip_sample(z, dict(temperature=torch.ones(len(x), device=H.DEV)), None, None, 0, 0, 1, V=2)
    assert int(ids[:, 1].max()) == 0
    got, want = np.expm1(-lp[:, 1].double().cpu().numpy()), np.exp(-x.astype(np.float64))
    rms = float(np.sqrt(np.mean((got / want - 1.0) ** 2)))
    rounded = np.expm1(np.log1p(want).astype(np.float32).astype(np.float64)) / want - 1.0
    assert rms < 1.03 * np.hypot(2.62e-8, np.sqrt(np.mean(rounded ** 2))), rms


@pytest.mark.parametrize("params,k,rounds,in_registers", [
    (dict(top_k=12000, top_p=0.9), 0, 1, True), (dict(top_k=12000, top_p=0.9), 0, 2, False),
    (dict(top_k=12000), 5, 1, True), (dict(top_k=12000), 0, 2, False),
    ({}, 0, 1, True), ({}, 0, 5, True), ({}, 1, 1, False), (dict(min_p=0.0), 0, 3, True), (dict(min_p=0.0), 0, 4, False)])
@pytest.mark.parametrize("bf16", [False, True])
def test_which_way_a_batch_goes(params, k, rounds, in_registers, bf16):
    """Vocabularies that both ways serve: one row more than fills a round of workgroups changes over, where a
    call's parameters say so.  A k that no candidate list holds (code 2), or no filter (path 16), tells which."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(rounds)
    B, V = (rounds - 1) * cus + (1 if rounds > 1 else cus), 20000
    z = np.tile((rng.standard_normal((8, V)) * 2.0).astype(np.float32), ((B + 7) // 8, 1))[:B]
    w = H.custom("ways", workloads.f32_to_bf16_bits(z) if bf16 else z, dict(temperature=0.9, **params), None, k_logprobs=k)
    out = H.run_gpu(H.to_device(w), 2, 0)
    if params.get("top_k"):
        assert (H.last_row_why == (1 if in_registers else 2)).all(), np.unique(H.last_row_why)
    else:
        assert (H.last_row_path == (1 if in_registers else 16)).all(), np.unique(H.last_row_path)
    H.compare(w, out, 2, 0, rows=range(0, B, max(1, B // 16)))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("V", [16500, 32768])
def test_more_equal_values_than_can_be_compared(V, bf16):
    """Cuts through more than 1024 entries of one bin: all of one value (a row of equal values, 3000 equal
    largest, logits in steps of one half), which is settled from the registers, or two values (general path)."""
    rng = np.random.default_rng(V)
    B = 12
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    z[:3] = 0.25
    for b in range(3, 6):
        z[b, rng.permutation(V)[:3000]] = 11.0
    z[6:9] = np.round(z[6:9] * 2) / 2
    for b in range(9, 12):                                     # two values in one of 2047 bins over 30 and more
        z[b, 0], z[b, 1] = -25.0, 12.0
        z[b, rng.permutation(V)[:3000]] = rng.choice(np.float32([11.0, 10.9999]), 3000)
    params = dict(temperature=1.0, top_k=[50, 0, 50] * 4, top_p=[1.0, 0.8, 0.8] * 4)
    hist = [rng.integers(0, V, 50).tolist() for _ in range(B)]
    w = H.custom("ties", workloads.f32_to_bf16_bits(z) if bf16 else z, dict(params, presence_penalty=0.3), hist, k_logprobs=0)
    d = H.to_device(w)
    for step in (0, 1):
        H.compare(w, H.run_gpu(d, 8, step), 8, step)
    assert (H.last_row_why[:9] == 1).all(), H.last_row_why
    if not bf16:
        assert (H.last_row_why[9:] == 9).all(), H.last_row_why
