"""The streaming loop's one multiply-add per element: which side of the threshold an element is on at extreme
temperatures and among equal values, history tokens at every place of a load, and sums that list entries are
taken out of again (blocks that begin with nothing but list entries)."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,bf16", [(8, 33003, True), (8, 40002, False), (300, 36001, True)])
def test_threshold_side_and_sums(B, V, bf16):
    rng = np.random.default_rng(V)
    z = (rng.standard_normal((B, V)) * 1.5).astype(np.float32)
    kind = np.arange(B) % 8
    heads = np.concatenate([np.arange(b, min(b + 11, V)) for b in range(0, V, 1024)])
    for b in range(B):
        if kind[b] in (0, 1):
            z[b, heads] = 3.5 + 0.5 * rng.random(len(heads))      # each block begins with list entries only
        elif kind[b] == 4:
            z[b] = np.round(z[b] * 4) / 4                        # a few dozen values, hundreds of elements each
        elif kind[b] == 5:
            z[b] = -np.abs(z[b]) - 1e-3
        elif kind[b] == 6:
            z[b] *= 1e-20
    tau = np.choose(kind, [1.0, 0.7, 1e20, 1e-20, 0.9, 0.5, 1e-20, 0.8])
    params = dict(temperature=tau, top_k=np.choose(kind, [0, 0, 40, 40, 40, 0, 40, 60]),
                  top_p=np.choose(kind, [1, 1, 1, 1, 1, 0.7, 1, 0.9]),
                  repetition_penalty=np.choose(kind, [1, 1.3, 1, 1, 1.2, 1.1, 1, 1.4]))
    near = [list(range(g, g + 17)) for g in (0, 1019, 4091, V - 17)]          # every place of a load, chunk ends
    hist = [sum(near, []) if k in (1, 4, 7) else rng.integers(0, V, 50).tolist() for k in kind]
    w = H.custom(f"stream_{V}", workloads.f32_to_bf16_bits(z) if bf16 else z, params, hist, k_logprobs=3)
    d = H.to_device(w)
    for step in range(6 if B < 10 else 1):
        H.compare(w, H.run_gpu(d, 3, step), 3, step)
