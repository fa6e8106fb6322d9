"""Calls that ask for token ids only: rows whose mass is summed beside rows where nothing takes it, in chunks, a row to a
workgroup and in pieces, settled from the list and not (a min-p that reaches below it, a wide nucleus, k beyond any list)."""
import numpy as np
import pytest
import torch

import paper_2506_22033_amd as sip
import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16,pieces", [(20, 40008, True, 0), (20, 40004, False, 0), (20, 40032, True, 2), (280, 36008, True, 0),
                                             (230, 33008, False, 0), (600, 52008, False, 0)])
def test_ids_only(B, V, bf16, pieces):
    rng = np.random.default_rng(V + B)
    kind = np.arange(B) % 10
    z = (rng.standard_normal((B, V)) * 2.0).astype(np.float32)
    hist = [rng.integers(0, V, 400).tolist() if k % 3 == 0 else [] for k in kind]
    params = dict(temperature=np.choose(kind, [0.0, 0.8, 0.8, 0.7, 1.0, 0.9, 1.5, 1.0, 0.8, 0.0]),
                  top_k=np.choose(kind, [0, 50, 50, 0, 0, 0, 0, 0, 9000, 1]),
                  top_p=np.choose(kind, [1, 1, 0.9, 1, 0.8, 1, 1, 0.95, 0.9, 1]),
                  min_p=np.choose(kind, [0, 0, 0, 0.1, 0.05, 0, 1e-3, 0, 0, 0]),
                  repetition_penalty=np.full(B, 1.15), frequency_penalty=np.full(B, 0.1))
    w = H.custom(f"ids_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=-1)
    d = H.to_device(w)
    rows = list(range(B)) if B < 30 else list(range(0, B, B // 30))
    for step in range(3 if B < 30 else 1):
        if pieces:
            n = V // pieces
            shards = [d.logits[:, i * n:(i + 1) * n].contiguous() for i in range(pieces)]
            ids, _, _ = sip.sip_sample_sharded(shards, d.params, d.indptr, d.tokens, 37, step, -1)
            torch.cuda.synchronize()
            out = (ids.cpu().numpy(), None, None)
        else:
            out = H.run_gpu(d, 37, step, k_logprobs=-1)
        H.compare(w, out, 37, step, rows=rows, k_logprobs=-1)
