"""The views of a state buffer are the same whichever way they are made: from 32-bit words, or slice by slice where the
buffer does not allow that (its size, its place in the storage, a buffer that is too small)."""
import pytest
import torch

import paper_2506_22033_amd as sip


@pytest.mark.parametrize("slots,L_max", [(1, 1), (7, 33), (256, 130)])
@pytest.mark.parametrize("lead,tail", [(0, 0), (0, 3), (8, 0), (8, 5), (256, 64)])
def test_views_of_a_state(slots, L_max, lead, tail):
    size = sip.sip_state_bytes(slots, L_max)
    store = torch.zeros(lead + size + tail, dtype=torch.uint8)
    state = store[lead:]
    len_bytes = (4 * slots + 255) // 256 * 256
    base = 256 + 2 * len_bytes
    views = sip.state_views(state, slots, L_max)
    for v, off, shape, dtype in zip(views, (0, 8, 256, base), ((1,), (1,), (slots,), (slots, L_max)),
                                    (torch.int64, torch.int32, torch.int32, torch.int32)):
        assert v.dtype == dtype and tuple(v.shape) == shape and v.is_contiguous() and v.data_ptr() == state.data_ptr() + off
    views[3].fill_(5)
    views[2].fill_(6)
    assert int(state.sum()) == 5 * slots * L_max + 6 * slots
    with pytest.raises(RuntimeError):
        sip.state_views(state[:base + 4 * slots * L_max - 4], slots, L_max)
