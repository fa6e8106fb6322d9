"""The sampling calls whose speed this repository answers for.

A case is one decode iteration's sampling step as a serving loop makes it: logits of a batch in
device memory, per-row sampling parameters, the rows' token histories, and one call through the
public entry points of ``paper_2506_22033_amd``.  The shapes and value distributions are those of
``workloads/`` (C1..C5 there), of the tests, or generic ones between them; inputs are drawn on the
GPU from the seed.
"""
from __future__ import annotations

import math

import torch

import paper_2506_22033_amd as sip

DEV = "cuda:0"
MAX_BYTES = 2048 * 256000 * 4          # logits of the largest listed case


def _case(name, **kw):
    c = dict(entry="csr", B=1, V=32000, dtype="f32", logits="normal", scale=2.0, rows="all", penalties="none",
             hist=0, hist_kind="uniform", prompt=0, shards=0, k_logprobs=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one interactive user: the smallest call, latency only
        _case("one_row", B=1, V=128256, dtype="bf16", logits="spikes", scale=3.0, rows="top_k_p", penalties="rep",
              hist=300),
        # four requests with a sampling mode each (greedy, top-k, top-p, min-p), small vocabulary: C1
        _case("mixed_4", B=4, V=32000, rows="four", k_logprobs=5),
        # a vocabulary of a few thousand (codebook / character tokens)
        _case("small_vocab_64", B=64, V=4096, rows="top_k_p", scale=2.5),
        # long prompts handed in apart from the generated tokens, few rows
        _case("prompts_32", entry="prompt", B=32, V=128256, dtype="bf16", logits="t3", scale=2.0, rows="min_p",
              penalties="all", hist=600, hist_kind="zipf", prompt=8000, k_logprobs=1),
        # chat with nucleus sampling and a repetition penalty: C2
        _case("chat_64", B=64, V=128256, dtype="bf16", logits="spikes", scale=3.0, rows="top_p", penalties="rep",
              hist=512),
        # greedy decoding, ids only
        _case("greedy_128", B=128, V=152064, dtype="bf16", logits="t3", scale=2.0, rows="greedy", k_logprobs=-1),
        # temperature sampling without any filter, a vocabulary that is not a round number
        _case("plain_256", B=256, V=151643, dtype="bf16", logits="t3", scale=2.0, rows="plain"),
        # logits as the four pieces of a tensor-parallel last stage, a batch that does not divide the chip
        _case("shards_200", entry="shards", B=200, V=152064, dtype="bf16", logits="t3", scale=2.0, rows="top_p",
              penalties="rep", hist=1000, shards=4, k_logprobs=1),
        # a decode iteration on the device-resident state: finished sequences replaced, the call, the
        # ids handed to the waiting scheduler
        _case("decode_256", entry="state", B=256, V=152064, dtype="bf16", logits="t3", scale=2.0, rows="top_k_p",
              penalties="all", hist=1000, hist_kind="zipf", k_logprobs=1),
        # everything on, fp32: C3, the headline configuration
        _case("all_256", B=256, V=152064, scale=2.5, rows="all", penalties="freq", hist=1024, hist_kind="zipf",
              k_logprobs=20),
        # a large bf16 batch: C4
        _case("chat_1024", B=1024, V=129280, dtype="bf16", logits="t3", scale=2.0, rows="top_p_09", penalties="rep",
              hist=2048, k_logprobs=20),
        # the largest batch and vocabulary, half of the rows greedy, top_k up to 4096: C5
        _case("large_2048", B=2048, V=256000, scale=2.0, rows="half_greedy", penalties="all", hist=4096,
              hist_kind="zipf", k_logprobs=20),
    ]


def draw(rng):
    """One more call of the same kinds: any batch from 1 to 2048 rows, vocabularies from a thousand to
    2^18 entries, every entry point, both data types, every family of row parameters."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))   # noqa: E731
    entry = rng.choice(["csr", "csr", "csr", "state", "shards", "prompt"])
    dtype = rng.choice(["f32", "bf16"])
    esz = 4 if dtype == "f32" else 2
    small = entry == "csr" and rng.random() < 0.2
    V = log(1000, 16383) if small else log(16384, 262144)
    shards = rng.choice([2, 4, 8]) if entry == "shards" else 0
    if shards:
        V = max(V, shards * 8192)
        V = V // (shards * 8) * (shards * 8)           # pieces of whole 16-byte groups
    B = log(1, min(2048, MAX_BYTES // (V * esz)))
    rows = rng.choice(["four", "greedy", "plain", "top_k_p", "top_p", "min_p", "all", "half_greedy"])
    # a nucleus with nothing beside it is used on the peaked rows that a model gives
    logits = rng.choice(["spikes", "t3"]) if rows == "top_p" else rng.choice(["normal", "spikes", "t3"])
    scale = {"normal": 2.5, "spikes": 3.0, "t3": 2.0}[logits] * rng.uniform(0.8, 1.2)
    hist = log(16, 4096) if entry in ("state", "prompt") or rng.random() < 0.7 else 0
    hist = min(hist, max(1, V // 8)) if hist else 0
    return _case("", entry=entry, B=B, V=V, dtype=dtype, logits=logits, scale=scale, rows=rows,
                 penalties=rng.choice(["rep", "freq", "all"]) if hist else "none", hist=hist,
                 hist_kind=rng.choice(["uniform", "zipf"]), prompt=log(64, 16384) if entry == "prompt" else 0,
                 shards=shards, k_logprobs=rng.choice([-1, 0, 0, 1, 5, 20]))


# ---------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _logits(case, g):
    """[B, stride] in the case's dtype; stride is V rounded up to whole 16-byte groups."""
    B, V = case["B"], case["V"]
    stride = (V + 7) // 8 * 8
    bf16 = case["dtype"] == "bf16"
    out = torch.zeros(B, stride, dtype=torch.bfloat16 if bf16 else torch.float32, device=DEV)
    step = max(1, (1 << 27) // stride)                 # rows drawn at once
    for r0 in range(0, B, step):
        n = min(step, B - r0)
        z = torch.randn(n, V, generator=g, device=DEV)
        if case["logits"] == "t3":                     # Student t, 3 degrees of freedom, and one spike per row
            chi = torch.zeros_like(z)
            for _ in range(3):
                x = torch.randn(n, V, generator=g, device=DEV)
                chi.addcmul_(x, x)
            z.div_(chi.div_(3.0).sqrt_()).mul_(case["scale"])
            sp = torch.randint(0, V, (n, 1), generator=g, device=DEV)
            z.scatter_add_(1, sp, torch.full((n, 1), 12.0, device=DEV))
        elif case["logits"] == "spikes":               # normal, and eight likely tokens per row
            z.mul_(case["scale"])
            sp = torch.randint(0, V, (n, 8), generator=g, device=DEV)
            z.scatter_(1, sp, z.gather(1, sp) + 8.0)
        else:
            z.mul_(case["scale"])
        out[r0:r0 + n, :V] = z
    return out


def _tokens(case, n, g):
    """n tokens of histories: uniform over the vocabulary, or Zipf (1.1) through a permutation of it."""
    V = case["V"]
    if case["hist_kind"] == "uniform":
        return torch.randint(0, V, (n,), generator=g, device=DEV, dtype=torch.int32)
    cdf = torch.arange(1, V + 1, dtype=torch.float64, device=DEV).pow_(-1.1).cumsum_(0)
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * cdf[-1]
    perm = torch.randperm(V, generator=g, device=DEV, dtype=torch.int32)
    return perm[torch.searchsorted(cdf, u, right=True).clamp_(max=V - 1)]


def _indptr(n, length):
    return torch.arange(n + 1, dtype=torch.int64, device=DEV) * length


def _params(case, g):
    B = case["B"]
    f = lambda lo, hi: torch.empty(B, device=DEV).uniform_(lo, hi, generator=g)          # noqa: E731
    c = lambda x: torch.full((B,), float(x), device=DEV)                                 # noqa: E731
    k = lambda x: torch.full((B,), int(x), dtype=torch.int32, device=DEV)                # noqa: E731
    row = torch.arange(B, device=DEV)
    P = {}
    kind = case["rows"]
    if kind == "four":
        m = row % 4
        P["temperature"] = torch.tensor([0.0, 0.8, 1.0, 0.7], device=DEV)[m]
        P["top_k"] = torch.tensor([0, 50, 0, 0], dtype=torch.int32, device=DEV)[m]
        P["top_p"] = torch.tensor([1.0, 1.0, 0.9, 1.0], device=DEV)[m]
        P["min_p"] = torch.tensor([0.0, 0.0, 0.0, 0.05], device=DEV)[m]
    elif kind == "greedy":
        P["temperature"] = c(0.0)
    elif kind == "plain":
        P["temperature"] = f(0.6, 1.0)
    elif kind == "top_k_p":
        P["temperature"], P["top_k"], P["top_p"] = c(0.8), k(50), c(0.95)
    elif kind == "top_p":
        P["temperature"], P["top_p"] = c(0.7), c(0.95)
    elif kind == "top_p_09":
        P["temperature"], P["top_p"] = c(1.0), c(0.9)
    elif kind == "min_p":
        P["temperature"], P["min_p"] = f(0.7, 1.2), f(0.02, 0.1)
    elif kind == "all":
        P["temperature"], P["top_p"], P["min_p"] = f(0.3, 1.5), f(0.8, 1.0), c(0.05)
        P["top_k"] = torch.tensor([0, 20, 50, 1000], dtype=torch.int32, device=DEV)[
            torch.randint(0, 4, (B,), generator=g, device=DEV)]
    elif kind == "half_greedy":
        even = row % 2 == 0
        P["temperature"] = torch.where(even, c(0.0), f(0.5, 1.2))
        top = min(4096, case["V"])
        P["top_k"] = torch.where(even, k(0), torch.randint(0, top + 1, (B,), generator=g, device=DEV,
                                                           dtype=torch.int32))
        P["top_p"] = torch.where(even, c(1.0), f(0.85, 1.0))
    if case["penalties"] in ("rep", "all"):
        P["repetition_penalty"] = c(1.1)
    if case["penalties"] in ("freq", "all"):
        P["frequency_penalty"], P["presence_penalty"] = c(0.5), c(0.3)
    P["row_id"] = row + 1000
    return P


def prepare(case, seed):
    g = _gen(seed)
    B, V, n = case["B"], case["V"], case["k_logprobs"]
    s = {"case": case, "seed": seed, "step": 0}
    logits = _logits(case, g)
    s["params"] = _params(case, g)
    hist = case["hist"]
    if case["entry"] == "shards":
        t = case["shards"]
        s["logits"] = sip.ShardTable([logits[:, i * (V // t):(i + 1) * (V // t)].contiguous() for i in range(t)])
    else:
        s["logits"] = logits
    if case["entry"] == "state":
        s["L_max"] = L = hist + 128
        s["state"] = torch.zeros(sip.sip_state_bytes(B, L), dtype=torch.uint8, device=DEV)
        sip.sip_state_init(s["state"], B, L)
        order = torch.randperm(B, generator=g, device=DEV, dtype=torch.int32)
        s["slots"] = order
        sip.sip_state_assign(s["state"], B, L, order, _indptr(B, hist), _tokens(case, B * hist, g))
        # every 64 iterations each sequence has been replaced once
        turn = max(1, B // 64)
        s["turns"] = [(order[i:i + turn].contiguous(), _indptr(min(turn, B - i), hist),
                       _tokens(case, min(turn, B - i) * hist, g)) for i in range(0, B, turn)]
        s["host_ids"] = torch.zeros(B, dtype=torch.int32).pin_memory()
        s["host_flag"] = torch.zeros(1, dtype=torch.int64).pin_memory()
        nnz = B * L
    elif hist:
        s["indptr"], s["tokens"] = _indptr(B, hist), _tokens(case, B * hist, g)
        nnz = B * hist
    else:
        s["indptr"] = s["tokens"] = None
        nnz = 0
    if case["entry"] == "prompt":
        s["p_indptr"], s["p_tokens"] = _indptr(B, case["prompt"]), _tokens(case, B * case["prompt"], g)
        nnz += B * case["prompt"]
    s["ids"] = torch.empty(B, dtype=torch.int32, device=DEV)
    s["lp_ids"] = torch.empty(B, 1 + n, dtype=torch.int32, device=DEV) if n >= 0 else None
    s["lp"] = torch.empty(B, 1 + n, dtype=torch.float32, device=DEV) if n >= 0 else None
    dt = sip.SIP_BF16 if case["dtype"] == "bf16" else sip.SIP_F32
    if case["entry"] == "shards":
        need = sip.sip_workspace_bytes_sharded(B, V // case["shards"], case["shards"], dt, nnz, n)
    else:
        need = sip.sip_workspace_bytes(B, V, dt, nnz, n)
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    return s


def run(s):
    case = s["case"]
    out = dict(out_ids=s["ids"], out_lp_ids=s["lp_ids"], out_lp=s["lp"], workspace=s["workspace"])
    seed, step, n = s["seed"], s["step"], case["k_logprobs"]
    s["step"] = step + 1
    entry = case["entry"]
    if entry == "csr":
        sip.sip_sample(s["logits"], s["params"], s["indptr"], s["tokens"], seed, step, n, V=case["V"], **out)
    elif entry == "shards":
        sip.sip_sample_sharded(s["logits"], s["params"], s["indptr"], s["tokens"], seed, step, n, **out)
    elif entry == "prompt":
        sip.sip_sample_call(logits=s["logits"], V=case["V"], params=s["params"], hist_indptr=s["indptr"],
                            hist_tokens=s["tokens"], prompt_indptr=s["p_indptr"], prompt_tokens=s["p_tokens"],
                            seed=seed, step=step, k_logprobs=n, **out)
    else:
        B, L, state = case["B"], s["L_max"], s["state"]
        slot_ids, indptr, tokens = s["turns"][step % len(s["turns"])]
        sip.sip_state_assign(state, B, L, slot_ids, indptr, tokens)
        sip.sip_sample_call(logits=s["logits"], V=case["V"], params=s["params"], state=state, slots=B, L_max=L,
                            slot_of_row=s["slots"], seed=seed, step=0, k_logprobs=n, host_ids=s["host_ids"],
                            host_flag=s["host_flag"], ticket=step + 1, **out)
        sip.sip_wait_ids(s["host_flag"], step + 1)
        _, _, length, history = sip.state_views(state, B, L)
        return {"ids": s["ids"], "lp_ids": s["lp_ids"], "lp": s["lp"], "host_ids": s["host_ids"],
                "length": length, "history": history}
    return {"ids": s["ids"], "lp_ids": s["lp_ids"], "lp": s["lp"]}


def work(case):
    """Every logit, history token and parameter read once, every output written once; per logit a
    subtraction, a scaling, an exponential, an addition and a comparison."""
    B, V, n = case["B"], case["V"], case["k_logprobs"]
    esz = 2 if case["dtype"] == "bf16" else 4
    rows = B * (32 + 4 + (8 * (1 + n) if n >= 0 else 0))
    return {"bytes": B * V * esz + 4 * B * (case["hist"] + case["prompt"]) + rows, "flops": 5 * B * V}


def tolerance(case):
    """Log-probabilities are fp32 differences: against float64 they are off by 1.5e-7 (2-norm) and 6e-7 (largest).
    Token ids are the same unless a row's uniform lies within the rounding of the sums (some 1e-8) of an edge of
    its cumulative distribution.  With 150 000 edges, as plain temperature sampling has them, that was seen in 1
    of 6144 rows; the row then holds the neighbouring token and that one's log-probability."""
    if case["rows"] == "plain":
        return {"rel": 0.03, "max": 0.8, "differ": 0.004}
    if case["rows"] == "half_greedy":                   # up to 4096 edges, thousands of rows: one row
        return {"rel": 1e-3, "max": 0.8, "differ": 0.0005}
    return {"rel": 6e-7, "max": 2.4e-6, "differ": 0.0}
