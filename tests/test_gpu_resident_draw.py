"""Rows held in registers: draws that fall anywhere in the row, so that every block of a load and a wave has its turn, for
every number of loads a thread may have; whole rows, min-p, and cuts whose members few loads have."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("V", [4095, 8192, 8200, 12001, 16384, 16390, 32768])
def test_draws_from_every_block(V, bf16):
    rng = np.random.default_rng(V + bf16)
    B = 40
    kind = np.arange(B) % 5
    z = (rng.standard_normal((B, V)) * 0.5).astype(np.float32)
    z[5:10, V // 3:] = -np.inf                                # nothing in most of the loads
    params = dict(temperature=np.choose(kind, [1.0, 1.0, 1.3, 0.9, 1.0]), top_k=np.choose(kind, [0, 0, 0, 100, 0]),
                  top_p=np.choose(kind, [1.0, 1.0, 0.97, 1.0, 0.3]), min_p=np.choose(kind, [0.0, 0.1, 0.0, 0.0, 0.05]))
    w = H.custom(f"draw_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, [[] for _ in range(B)], k_logprobs=3)
    d = H.to_device(w)
    for step, k in enumerate((3, 0, -1, 3)):                  # best three, the sampled token's alone, ids only
        H.compare(w, H.run_gpu(d, 71, step, k_logprobs=k), 71, step, k_logprobs=k)
