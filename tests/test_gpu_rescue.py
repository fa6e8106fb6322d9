"""Rows passed on to the rescue kernel: every one of them is found, whatever its place in the batch, and no other."""
import numpy as np
import pytest

from tests import sip_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [257, 1025, 2300])
def test_unsettled_rows_anywhere_in_the_batch(B):
    V = 16421
    rng = np.random.default_rng(B)
    z = (rng.standard_normal((B, V)) * 3.0).astype(np.float32)
    z[np.arange(B), rng.integers(0, V, B)] += 25.0                       # peaked: settled from the list
    flat = (np.arange(B) % 5 == 3) | (np.abs(np.arange(B) - 1024) < 70) | (np.arange(B) >= B - 3)
    z[flat] *= 0.02                                                      # a nucleus below any list
    w = H.custom(f"rescue_{B}", z, dict(temperature=np.full(B, 1.0), top_p=np.full(B, 0.9)), k_logprobs=1)
    st = H.compare(w, H.run_gpu(H.to_device(w), 6, 0), 6, 0)
    assert st.rows == B and np.array_equal(H.last_row_path == 16, flat), (H.last_row_path, H.last_row_why)
