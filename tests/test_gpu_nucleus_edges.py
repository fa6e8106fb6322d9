"""Wide nuclei whose cut lies on a value at the lower edge of its bin, as rounding puts it there: the bin holds the
value, the next interval's computed lower end lies an ulp or so above it."""
import numpy as np
import pytest

import workloads
from tests import sip_harness as H

pytestmark = pytest.mark.gpu
f32 = np.float32
BINS, SPAN = 2048, 28.0


def _bins_and_ends(s, m, level):
    """Bins of the values ``s`` on every interval down to ``level`` (rows) and the lower end of the interval below
    each, every operation rounded to fp32 as on the device."""
    lo, w = np.full(s.shape, m - f32(SPAN), f32), f32(SPAN)
    bins = []
    for _ in range(level):
        b = np.clip(((s - lo) * (f32(BINS) / w)).astype(np.int64), 0, BINS - 1)
        w = f32(w * f32(1 / BINS))
        lo = lo + b.astype(f32) * w
        bins.append(b)
    return np.stack(bins), lo


def _edge_values(rng, bf16, tau, level):
    """(largest logit, cut value, next larger value of the same bin), all representable: the cut value lies below
    the end of the interval its bin becomes, the other above it."""
    for _ in range(20000):
        top = f32(rng.integers(144, 256) / 32)
        if level == 1:
            z = np.arange(512, 1024) / f32(256)
            z = (z[::4] if bf16 else z).astype(f32)                            # (steps of 1/64: bf16 from 2 to 4)
        else:
            # on the two sides of a step of the list's threshold (18-bit keys), which leaves the cut value below it
            z = f32(2 + rng.integers(1, 512) / 256) + np.arange(-1, 1, dtype=f32) * f32(2.0 ** -22)
        s, m = (z / f32(tau)).astype(f32), top / f32(tau)
        bins, lo = _bins_and_ends(s, m, level)
        at = np.flatnonzero((s[:-1] < lo[:-1]) & (bins[:, :-1] == bins[:, 1:]).all(axis=0) & (s[1:] > lo[1:]))
        if len(at):
            i = int(rng.choice(at))
            return top, z[i], z[i + 1]
    return None


@pytest.mark.parametrize("tau,bf16,level", [(1.5, True, 1), (1.2, True, 1), (0.9, False, 1), (0.7, False, 1),
                                            (1.1, False, 1), (1.3, False, 2), (1.7, False, 2)])
def test_cut_on_a_value_below_the_computed_end_of_its_interval(tau, bf16, level):
    B, V = 6, 70001
    rng = np.random.default_rng(int(tau * 100) + level)
    z = (rng.standard_normal((B, V)) * 0.2 - 2.0).astype(np.float32)
    top_p = np.ones(B)
    for b in range(B):
        found = _edge_values(rng, bf16, tau, level)
        assert found is not None
        top, cut, above = found
        at = rng.permutation(V)
        z[b, at[0]], z[b, at[1:6001]], z[b, at[6001:26001]] = top, above, cut
        # the limit half way through the mass of the cut value (20000 elements, all of them kept)
        e = np.exp(np.float64(z[b]) / tau)
        top_p[b] = (e[z[b] > cut].sum() + 0.5 * e[z[b] == cut].sum()) / e.sum()
    logits = workloads.f32_to_bf16_bits(z) if bf16 else z
    w = H.custom(f"edge_{tau}_{level}", logits, dict(temperature=np.full(B, tau), top_p=top_p), k_logprobs=0)
    d = H.to_device(w)
    for step in range(3):
        out = H.run_gpu(d, 3, step)
        assert (H.last_row_path == 16).all(), H.last_row_path
        H.compare(w, out, 3, step)
