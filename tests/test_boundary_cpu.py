"""Host-side checks of the C boundary that need no GPU: the library loads, exports every
symbol the headers under include/ declare, sizes its workspace sensibly and rejects bad arguments on
the host before anything is enqueued."""
import ctypes
import os
import re

import pytest

import paper_2506_22033_amd as sip
from paper_2506_22033_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    inc = os.path.join(ROOT, "include")
    names = set()
    for h in sorted(os.listdir(inc)):
        if h.endswith(".h"):
            text = re.sub(r"/\*.*?\*/", "", open(os.path.join(inc, h)).read(), flags=re.S)
            names |= set(re.findall(r"\b(sip_[a-z_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    lib = sip.load()
    names = declared_functions()
    assert {"sip_sample", "sip_workspace_bytes", "sip_status_string", "sip_version"} <= set(names)
    for n in names:
        assert getattr(lib, n) is not None
    assert sip.sip_version() >= 100


def test_status_strings():
    seen = {sip.sip_status_string(s) for s in range(7)}
    assert len(seen) == 7 and "ok" in seen
    assert sip.sip_status_string(99) == "unknown status"


def test_workspace_query():
    small = sip.sip_workspace_bytes(4, 32000, sip.SIP_F32, 0, 5)
    big = sip.sip_workspace_bytes(256, 152064, sip.SIP_F32, 256 * 1024, 20)
    assert small > 0 and small % 256 == 0 and big % 256 == 0
    assert big >= 256 * 1024 * 8
    assert sip.sip_workspace_bytes(0, 10, sip.SIP_F32, 0, 0) == 0
    assert sip.sip_workspace_bytes(1, 0, sip.SIP_F32, 0, 0) == 0
    assert sip.sip_workspace_bytes(1, sip.SIP_MAX_V + 1, sip.SIP_F32, 0, 0) == 0
    assert sip.sip_workspace_bytes(1, 10, 7, 0, 0) == 0
    assert sip.sip_workspace_bytes(1, 10, sip.SIP_F32, -1, 0) == 0
    assert sip.sip_workspace_bytes(1, 10, sip.SIP_F32, 0, sip.SIP_MAX_K_LOGPROBS + 1) == 0


def _call(**over):
    """sip_sample with fake but well-formed device addresses; every case below must be
    rejected on the host, so nothing is ever dereferenced or launched."""
    lib = sip.load()
    a = dict(logits=0x10000, B=4, V=1000, stride=1000, dtype=sip.SIP_F32, params=None, indptr=None, tokens=None,
             nnz=0, seed=0, step=0, out_ids=0x20000, out_lp_ids=0x30000, out_lp=0x40000, k=5,
             ws=0x50000, ws_bytes=1 << 20, stream=None)
    a.update(over)
    p = a["params"]
    return lib.sip_sample(a["logits"], a["B"], a["V"], a["stride"], a["dtype"],
                          ctypes.byref(p) if p is not None else None, a["indptr"], a["tokens"], a["nnz"],
                          a["seed"], a["step"], a["out_ids"], a["out_lp_ids"], a["out_lp"], a["k"],
                          a["ws"], a["ws_bytes"], a["stream"])


@pytest.mark.parametrize("over,want", [
    (dict(B=0), binding.SIP_ERR_INVALID_ARG),
    (dict(B=-3), binding.SIP_ERR_INVALID_ARG),
    (dict(V=0), binding.SIP_ERR_INVALID_ARG),
    (dict(logits=None), binding.SIP_ERR_INVALID_ARG),
    (dict(out_ids=None), binding.SIP_ERR_INVALID_ARG),
    (dict(dtype=5), binding.SIP_ERR_INVALID_ARG),
    (dict(stride=999), binding.SIP_ERR_INVALID_ARG),                 # stride < V
    (dict(stride=1001), binding.SIP_ERR_INVALID_ARG),                # rows not 16-byte aligned
    (dict(logits=0x10004), binding.SIP_ERR_INVALID_ARG),             # base not 16-byte aligned
    (dict(dtype=binding.SIP_BF16, stride=1004), binding.SIP_ERR_INVALID_ARG),
    (dict(k=-1), binding.SIP_ERR_INVALID_ARG),                       # logprob buffers given but k < 0
    (dict(out_lp=None), binding.SIP_ERR_INVALID_ARG),                # k >= 0 needs both buffers
    (dict(k=-2, out_lp=None, out_lp_ids=None), binding.SIP_ERR_INVALID_ARG),
    (dict(nnz=10), binding.SIP_ERR_INVALID_ARG),                     # history size without arrays
    (dict(nnz=-1), binding.SIP_ERR_INVALID_ARG),
    (dict(V=binding.SIP_MAX_V + 8, stride=binding.SIP_MAX_V + 8), binding.SIP_ERR_UNSUPPORTED),
    (dict(k=binding.SIP_MAX_K_LOGPROBS + 1), binding.SIP_ERR_UNSUPPORTED),
    (dict(ws=None), binding.SIP_ERR_WORKSPACE),
    (dict(ws=0x50010), binding.SIP_ERR_WORKSPACE),                   # not 256-byte aligned
    (dict(ws_bytes=16), binding.SIP_ERR_WORKSPACE),
    (dict(nnz=1 << 20, indptr=0x60000, tokens=0x70000, ws_bytes=1 << 20), binding.SIP_ERR_WORKSPACE),
])
def test_bad_arguments_are_rejected_on_the_host(over, want):
    assert _call(**over) == want


def test_state_size_query():
    table = 2 * 4096 * 4                                  # per slot: 4096 keys and 4096 multiplicities
    assert sip.sip_state_bytes(256, 4096) == 256 + 2 * 1024 + 256 * 4096 * 4 + 256 * table
    assert sip.sip_state_bytes(3, 5) == 256 + 2 * 256 + 256 + 3 * table
    for slots, L in [(0, 5), (-1, 5), (4, 0), (sip.SIP_MAX_SLOTS + 1, 4), (4, sip.SIP_MAX_L + 1)]:
        assert sip.sip_state_bytes(slots, L) == 0


def _call_state(**over):
    """sip_sample_state / sip_state_init / sip_state_assign with fake addresses; every case is
    rejected on the host."""
    lib = sip.load()
    a = dict(logits=0x10000, B=4, V=1000, stride=1000, dtype=sip.SIP_F32, state=0x80000, state_bytes=1 << 20,
             slots=8, L_max=64, slot_of_row=0x90000, out_ids=0x20000, out_lp_ids=0x30000, out_lp=0x40000, k=5,
             ws=0x50000, ws_bytes=1 << 22)
    a.update(over)
    return lib.sip_sample_state(a["logits"], a["B"], a["V"], a["stride"], a["dtype"], None, a["state"],
                                a["state_bytes"], a["slots"], a["L_max"], a["slot_of_row"], 0, 0, a["out_ids"],
                                a["out_lp_ids"], a["out_lp"], a["k"], a["ws"], a["ws_bytes"], None)


@pytest.mark.parametrize("over,want", [
    (dict(slots=0), binding.SIP_ERR_INVALID_ARG),
    (dict(L_max=0), binding.SIP_ERR_INVALID_ARG),
    (dict(L_max=binding.SIP_MAX_L + 1), binding.SIP_ERR_INVALID_ARG),
    (dict(slot_of_row=None), binding.SIP_ERR_INVALID_ARG),
    (dict(B=0), binding.SIP_ERR_INVALID_ARG),
    (dict(state=None), binding.SIP_ERR_WORKSPACE),
    (dict(state=0x80010), binding.SIP_ERR_WORKSPACE),                # not 256-byte aligned
    (dict(state_bytes=256 + 2 * 256 + 8 * 64 * 4 + 8 * 2 * 4096 * 4 - 1), binding.SIP_ERR_WORKSPACE),
    (dict(logits=None), binding.SIP_ERR_INVALID_ARG),                # the checks of sip_sample apply too
    (dict(stride=1001), binding.SIP_ERR_INVALID_ARG),
    (dict(ws_bytes=4 * 64 * 8 - 1), binding.SIP_ERR_WORKSPACE),      # side tables of B * L_max entries
])
def test_bad_state_arguments_are_rejected_on_the_host(over, want):
    assert _call_state(**over) == want


def test_state_init_and_assign_reject_bad_arguments_on_the_host():
    lib = sip.load()
    assert lib.sip_state_init(None, 1 << 20, 8, 64, None) == binding.SIP_ERR_WORKSPACE
    assert lib.sip_state_init(0x80000, 100, 8, 64, None) == binding.SIP_ERR_WORKSPACE
    assert lib.sip_state_init(0x80000, 1 << 20, 0, 64, None) == binding.SIP_ERR_INVALID_ARG
    assert lib.sip_state_assign(0x80000, 1 << 20, 8, 64, 2, None, None, None, 0, None) == binding.SIP_ERR_INVALID_ARG
    assert lib.sip_state_assign(0x80000, 1 << 20, 8, 64, 2, 0x90000, None, None, 5, None) == binding.SIP_ERR_INVALID_ARG
    assert lib.sip_state_assign(0x80000, 1 << 20, 8, 64, -1, 0x90000, None, None, 0, None) == binding.SIP_ERR_INVALID_ARG
    assert lib.sip_state_assign(0x80000, 100, 8, 64, 2, 0x90000, None, None, 0, None) == binding.SIP_ERR_WORKSPACE
    assert lib.sip_state_assign(0x80000, 1 << 20, 8, 64, 0, None, None, None, 0, None) == binding.SIP_OK   # nothing to do


def _call_sharded(**over):
    lib = sip.load()
    a = dict(ptrs=[0x10000, 0x20000], t=2, B=4, V_shard=20000, stride=20000, dtype=sip.SIP_F32, nnz=0,
             out_ids=0x30000, out_lp_ids=0x40000, out_lp=0x50000, k=5, ws=0x60000, ws_bytes=1 << 30)
    a.update(over)
    table = None if a["ptrs"] is None else (ctypes.c_void_p * len(a["ptrs"]))(*a["ptrs"])
    return lib.sip_sample_sharded(table, a["t"], a["B"], a["V_shard"], a["stride"], a["dtype"], None, None, None,
                                  a["nnz"], 0, 0, a["out_ids"], a["out_lp_ids"], a["out_lp"], a["k"], a["ws"],
                                  a["ws_bytes"], None)


@pytest.mark.parametrize("over,want", [
    (dict(t=0), binding.SIP_ERR_INVALID_ARG),
    (dict(t=binding.SIP_MAX_SHARDS + 1, ptrs=[0x10000] * 9), binding.SIP_ERR_INVALID_ARG),
    (dict(ptrs=None), binding.SIP_ERR_INVALID_ARG),
    (dict(ptrs=[0x10000, None]), binding.SIP_ERR_INVALID_ARG),
    (dict(ptrs=[0x10000, 0x20004]), binding.SIP_ERR_INVALID_ARG),          # piece not 16-byte aligned
    (dict(V_shard=20001, stride=20004), binding.SIP_ERR_INVALID_ARG),       # pieces must be whole 16-byte groups
    (dict(stride=19996), binding.SIP_ERR_INVALID_ARG),                      # stride < V_shard
    (dict(stride=20002), binding.SIP_ERR_INVALID_ARG),
    (dict(V_shard=0), binding.SIP_ERR_INVALID_ARG),
    (dict(B=0), binding.SIP_ERR_INVALID_ARG),
    (dict(V_shard=binding.SIP_MAX_V // 2 + 8, stride=binding.SIP_MAX_V // 2 + 8), binding.SIP_ERR_UNSUPPORTED),
    (dict(ws_bytes=4 * 40000 * 4 - 1), binding.SIP_ERR_WORKSPACE),          # room for B whole rows
    (dict(nnz=3), binding.SIP_ERR_INVALID_ARG),
])
def test_bad_sharded_arguments_are_rejected_on_the_host(over, want):
    assert _call_sharded(**over) == want


def test_sharded_workspace_query():
    two = sip.sip_workspace_bytes_sharded(4, 20000, 2, sip.SIP_F32, 0, 5)
    assert two > 4 * 40000 * 4 and two % 256 == 0                   # holds B whole rows, and more
    assert sip.sip_workspace_bytes_sharded(4, 20000, 0, sip.SIP_F32, 0, 5) == 0
    assert sip.sip_workspace_bytes_sharded(4, 20000, 9, sip.SIP_F32, 0, 5) == 0
    assert sip.sip_workspace_bytes_sharded(4, sip.SIP_MAX_V, 2, sip.SIP_F32, 0, 5) == 0


def test_wait_for_a_ticket_on_the_host():
    """sip_wait_ids is plain host code: flag already there, flag that never comes (time-out), flag
    set by another thread while the call spins."""
    import threading
    import time
    import numpy as np
    lib = sip.load()
    flag = np.zeros(1, dtype=np.uint64)
    addr = flag.ctypes.data
    flag[0] = 7
    assert lib.sip_wait_ids(addr, 7, 0) == binding.SIP_OK
    assert lib.sip_wait_ids(addr, 3, 0) == binding.SIP_OK                      # tickets only grow: a later one serves
    t0 = time.perf_counter()
    assert lib.sip_wait_ids(addr, 8, 2_000_000) == binding.SIP_ERR_TIMEOUT      # 2 ms
    assert 0.001 < time.perf_counter() - t0 < 0.5
    threading.Timer(0.01, lambda: flag.__setitem__(0, 8)).start()
    assert lib.sip_wait_ids(addr, 8, 5_000_000_000) == binding.SIP_OK
    assert lib.sip_wait_ids(None, 1, 0) == binding.SIP_ERR_INVALID_ARG
    assert lib.sip_wait_ids(addr + 4, 1, 0) == binding.SIP_ERR_INVALID_ARG       # not 8-byte aligned
    assert sip.sip_status_string(binding.SIP_ERR_TIMEOUT) == "timed out"


def test_publish_rejects_bad_arguments_on_the_host():
    lib = sip.load()
    ok = dict(ids=0x10000, B=4, host_ids=0x20000, flag=0x30000)
    for over in (dict(ids=None), dict(host_ids=None), dict(flag=None), dict(B=0), dict(flag=0x30004),
                 dict(host_ids=0x20002)):
        a = dict(ok, **over)
        assert lib.sip_publish_ids(a["ids"], a["B"], a["host_ids"], a["flag"], 1, None) == binding.SIP_ERR_INVALID_ARG


def test_probe_read_rejects_bad_arguments_on_the_host():
    lib = sip.load()
    ok = dict(src=0x10000, nbytes=1 << 20, wgs=64, ws=0x20000, ws_bytes=4096)
    for over, want in ((dict(src=None), binding.SIP_ERR_INVALID_ARG), (dict(src=0x10008), binding.SIP_ERR_INVALID_ARG),
                       (dict(nbytes=8), binding.SIP_ERR_INVALID_ARG), (dict(wgs=0), binding.SIP_ERR_INVALID_ARG),
                       (dict(ws=None), binding.SIP_ERR_WORKSPACE), (dict(ws_bytes=255), binding.SIP_ERR_WORKSPACE)):
        a = dict(ok, **over)
        assert lib.sip_probe_read(a["src"], a["nbytes"], a["wgs"], a["ws"], a["ws_bytes"], None, None, None) == want


def _a_call(**over):
    c = binding.SipCall()
    c.logits, c.row_stride, c.V, c.B, c.dtype = 0x10000, 20000, 20000, 4, sip.SIP_F32
    c.out_ids, c.out_lp_ids, c.out_lp, c.k_logprobs = 0x20000, 0x30000, 0x40000, 5
    c.workspace, c.workspace_bytes = 0x50000, 1 << 30
    for k, v in over.items():
        setattr(c, k, v)
    return c


def test_call_description_is_checked_on_the_host():
    lib = sip.load()
    two = (ctypes.c_void_p * 2)(0x60000, 0x70000)
    pieces = dict(logits=None, shard_logits=ctypes.cast(two, ctypes.POINTER(ctypes.c_void_p)), t_shards=2,
                  V_shard=20000, shard_stride=20000)
    state = dict(state=0x80000, state_bytes=1 << 20, slots=8, L_max=64, slot_of_row=0x90000)
    cases = [
        (dict(B=0), binding.SIP_ERR_INVALID_ARG),
        (dict(t_shards=9), binding.SIP_ERR_INVALID_ARG),
        (dict(t_shards=2, V_shard=20000), binding.SIP_ERR_INVALID_ARG),                    # pieces announced, no table
        (dict(pieces, V_shard=binding.SIP_MAX_V), binding.SIP_ERR_UNSUPPORTED),
        (dict(state, hist_nnz=4), binding.SIP_ERR_INVALID_ARG),                            # two sources of history
        (dict(state, slot_of_row=None), binding.SIP_ERR_INVALID_ARG),
        (dict(state, state_bytes=100), binding.SIP_ERR_WORKSPACE),
        (dict(hist_nnz=4), binding.SIP_ERR_INVALID_ARG),
        (dict(host_ids=0xA0000), binding.SIP_ERR_INVALID_ARG),                             # hand-off needs both
        (dict(host_ids=0xA0000, host_flag=0xB0004), binding.SIP_ERR_INVALID_ARG),
        (dict(logits=None), binding.SIP_ERR_INVALID_ARG),
        (dict(workspace_bytes=16), binding.SIP_ERR_WORKSPACE),
        (dict(pieces, **state, workspace_bytes=4 * 40000 * 4), binding.SIP_ERR_WORKSPACE),  # rows to gather + side tables
    ]
    for over, want in cases:
        assert lib.sip_sample_call(ctypes.byref(_a_call(**over))) == want, over
    assert lib.sip_sample_call(None) == binding.SIP_ERR_INVALID_ARG
    # the workspace query follows the description
    plain = lib.sip_call_workspace_bytes(ctypes.byref(_a_call()))
    assert plain == sip.sip_workspace_bytes(4, 20000, sip.SIP_F32, 0, 5)
    both = lib.sip_call_workspace_bytes(ctypes.byref(_a_call(**dict(pieces, **state))))
    assert both == sip.sip_workspace_bytes_sharded(4, 20000, 2, sip.SIP_F32, 4 * 64, 5)
    assert lib.sip_call_workspace_bytes(ctypes.byref(_a_call(B=0))) == 0


def _chunk_begin(ch, V, S, unit):
    """A row is cut into S chunks of whole units, sizes differing by at most one unit (the rule
    the header states for sip_plan_chunks)."""
    n = (V + unit - 1) // unit
    return min(ch * n // S * unit, V)


def test_every_chunk_of_every_plan_is_non_empty():
    """The streaming kernel's workgroups each need something to stream (an empty chunk would leave
    its summary unwritten): sweep batch sizes, vocabularies, dtypes and piece counts."""
    lib = sip.load()
    seen_fast = 0
    unit = 1024
    for dtype in (sip.SIP_F32, sip.SIP_BF16):
        for t in (0, 1, 2, 3, 4, 5, 6, 7, 8):
            for V_piece in (8192, 8200, 9000, 16032, 16384, 19008, 32768, 65536, 100000 // 8 * 8, 262144):
                V = V_piece * max(t, 1)
                for B in (1, 2, 3, 4, 7, 16, 63, 64, 100, 128, 129, 255, 256, 257, 300, 512, 513, 1024, 2048, 5000):
                    S = lib.sip_plan_chunks(B, V, dtype, t)
                    assert S >= 0, (B, V, dtype, t)
                    if S == 0:
                        assert V < 16384 or V > 262144 or V_piece < 8192
                        continue
                    seen_fast += 1
                    assert 1 <= S <= 16
                    pieces = max(t, 1)
                    if S >= pieces:
                        assert S % pieces == 0
                        per = S // pieces
                        for lc in range(per):                  # chunks inside one piece
                            assert _chunk_begin(lc, V_piece, per, unit) < _chunk_begin(lc + 1, V_piece, per, unit)
                        assert _chunk_begin(per, V_piece, per, unit) == V_piece
                    else:
                        assert pieces % S == 0                 # a chunk is whole pieces
    assert seen_fast > 1000
    assert lib.sip_plan_chunks(0, 20000, sip.SIP_F32, 0) == -1
    assert lib.sip_plan_chunks(4, 20001, sip.SIP_F32, 2) == -1
    assert lib.sip_plan_chunks(4, 20000, sip.SIP_F32, 9) == -1


ROUTE_RESIDENT, ROUTE_CHUNKS_ALONE, ROUTE_CHUNKS_FUSED, ROUTE_CHUNKS = 1, 2, 5, 6


@pytest.mark.parametrize("on_state,params,k", [(False, ("temperature", "top_p"), 0), (False, ("temperature",), -1), (True, (), 1)])
def test_no_call_cuts_a_row_into_empty_chunks(on_state, params, k):
    """As above, over the cuts that calls take: with a compute unit to each chunk, and on a state."""
    seen = dict.fromkeys((ROUTE_CHUNKS_ALONE, ROUTE_CHUNKS_FUSED, ROUTE_CHUNKS), 0)
    for dtype in (sip.SIP_F32, sip.SIP_BF16):
        for t in range(9):
            for V_piece in (8192, 8200, 9000, 16032, 19008, 32768, 43000, 66560, 131072, 262144):
                V = V_piece * max(t, 1)
                if V > 262144:
                    continue
                for B in (1, 2, 3, 5, 8, 13, 16, 21, 29, 32, 37, 43, 64, 65, 85, 86, 100, 127, 128, 129, 200, 300):
                    route, S = sip.sip_call_route(B, V, dtype, t, on_state, params, 0, k)
                    if route not in seen:
                        assert S == 1
                        continue
                    seen[route] += 1
                    if route != ROUTE_CHUNKS_ALONE:
                        assert S == sip.load().sip_plan_chunks(B, V, dtype, t)
                    pieces = max(t, 1)
                    most = 131072 if route == ROUTE_CHUNKS_ALONE else 73728       # elements that a chunk's bitmap holds
                    if S >= pieces:
                        assert S % pieces == 0
                        edges = [_chunk_begin(i, V_piece, S // pieces, 1024) for i in range(S // pieces + 1)]
                        assert edges[-1] == V_piece and all(0 < b - a <= most for a, b in zip(edges, edges[1:])), (B, V, dtype, t, S)
                    else:
                        assert pieces % S == 0 and pieces // S * V_piece <= most
                    if route == ROUTE_CHUNKS_ALONE:
                        assert S >= 2 and B * S <= 256 and not on_state
    assert seen[ROUTE_CHUNKS_FUSED] > 50 and seen[ROUTE_CHUNKS] > 50 and (seen[ROUTE_CHUNKS_ALONE] > 50) == (not on_state)


@pytest.mark.parametrize("B,V,dtype,state,k,route", [
    (1, 128256, sip.SIP_BF16, False, 0, 2), (64, 4096, sip.SIP_F32, False, 0, 1), (64, 32768, sip.SIP_F32, False, 0, 1),
    (64, 300000, sip.SIP_F32, False, 0, 0), (150, 128256, sip.SIP_BF16, False, 1, 5), (200, 152064, sip.SIP_F32, False, 1, 3),
    (256, 152064, sip.SIP_F32, False, 20, 3), (64, 128256, sip.SIP_BF16, True, 0, 5), (300, 152064, sip.SIP_F32, False, 0, 6),
    (1024, 129280, sip.SIP_BF16, False, 20, 4), (600, 152064, sip.SIP_BF16, True, 0, 6)])
def test_kernels_of_a_call(B, V, dtype, state, k, route):
    assert sip.sip_call_route(B, V, dtype, 0, state, ("temperature", "top_p"), 0, k)[0] == route


@pytest.mark.parametrize("B,V,dtype,route", [(128, 152064, sip.SIP_BF16, 2), (128, 40000, sip.SIP_BF16, 3), (128, 40000, sip.SIP_F32, 3),
                                             (64, 40000, sip.SIP_BF16, 2), (100, 262144, sip.SIP_F32, 2), (129, 152064, sip.SIP_BF16, 5)])
def test_kernels_of_a_call_that_greedy_rows_make(B, V, dtype, route):
    assert sip.sip_call_route(B, V, dtype, 0, False, ("temperature",), 0, -1)[0] == route


def test_route_of_no_call():
    for bad in (dict(B=0), dict(V=0), dict(dtype=3), dict(t_shards=9), dict(V=20001, t_shards=2), dict(k_logprobs=-2), dict(hist_nnz=-1)):
        with pytest.raises(ValueError):
            sip.sip_call_route(**{**dict(B=4, V=20000, dtype=sip.SIP_F32), **bad})


def test_binding_refuses_host_tensors():
    import torch
    with pytest.raises(TypeError):
        sip.sip_sample(torch.zeros(2, 8), None, None, None, 0, 0, 0)


@pytest.mark.parametrize("B,V,dtype", [(61, 24275, sip.SIP_BF16), (1, 16384, sip.SIP_BF16), (128, 16384, sip.SIP_F32),
                                       (85, 40000, sip.SIP_BF16)])
def test_small_chunks_do_not_push_a_call_out_of_the_built_in_scratch(B, V, dtype):
    """Cut into chunks of one tile a small batch takes more workspace than in chunks of two: histories that fit the
    built-in scratch with the latter (whose segments take 30 KB a chunk) still do."""
    scratch, tile = sip.sip_noalloc_scratch_bytes(), 4096 if dtype == sip.SIP_F32 else 8192
    coarse = max(1, -(-V // tile) // 2)
    fixed = B * (coarse * (3840 * 8 + 32) + 64 + 8) + 8192           # segments, summaries, rows' records, alignment
    nnz = (scratch - fixed) // 8
    assert sip.sip_workspace_bytes(B, V, dtype, 0, 0) > fixed - 8192
    assert scratch - 16384 < sip.sip_workspace_bytes(B, V, dtype, nnz, 0) <= scratch
    assert sip.sip_workspace_bytes(B, V, dtype, nnz + 2048, 0) > scratch


@pytest.mark.parametrize("dtype", [sip.SIP_F32, sip.SIP_BF16])
@pytest.mark.parametrize("V", [16384, 24280, 40000, 65536])
def test_a_workspace_sized_for_the_longest_histories_and_largest_batch_serves_smaller_calls(V, dtype):
    """The size neither falls as the history grows, across the place where a call's chunks of one tile give way, nor
    with the rows of a batch of short rows."""
    scratch = sip.sip_noalloc_scratch_bytes()
    pieces = lambda B, nnz: sip.sip_workspace_bytes_sharded(B, V // 2, 2, dtype, nnz, 0)              # noqa: E731
    whole = lambda B, nnz: sip.sip_workspace_bytes(B, V, dtype, nnz, 0)                               # noqa: E731
    for need in (whole, pieces):
        for B in (1, 2, 7, 61, 85, 128, 200, 256):
            sizes = [need(B, nnz) for nnz in range(0, scratch // 8 + (1 << 19), 5003)]
            assert sizes == sorted(sizes), (B, [i for i in range(1, len(sizes)) if sizes[i] < sizes[i - 1]])
        if V * (2 if dtype == sip.SIP_BF16 else 4) <= 128 * 1024:
            for nnz in (0, 100_000, 4_000_000, 4_540_000, 5_000_000):
                sizes = [need(B, nnz) for B in range(1, 257)]
                assert sizes == sorted(sizes), (nnz, [i + 1 for i in range(1, 256) if sizes[i] < sizes[i - 1]])


def test_stream_handle_without_the_private_torch_function(monkeypatch):
    """The current stream's handle is the one that torch's public interface names where torch has no function
    that gives it without a Stream object."""
    class Stream:
        def __init__(self, handle):
            self.cuda_stream = handle
    asked = []
    monkeypatch.setattr(binding.torch.cuda, "current_stream", lambda dev: asked.append(dev) or Stream(77))
    monkeypatch.setattr(binding, "_current_raw_stream", None)
    dev = binding.torch.device("cuda", 3)
    assert binding._stream_handle(dev, None) == 77 and asked == [dev]
    assert binding._stream_handle(dev, Stream(5)) == 5 and len(asked) == 1
    monkeypatch.setattr(binding, "_current_raw_stream", lambda index: 100 + index)
    assert binding._stream_handle(dev, None) == 103 and len(asked) == 1


@pytest.mark.parametrize("k,params", [(0, ("temperature", "top_p")), (5, ()), (-1, ("temperature", "top_k"))])
def test_chunks_with_a_compute_unit_each_leave_room_for_another_batch(k, params):
    """A workgroup of such a chunk fills its compute unit: with more of them than this, two batches in flight took turns
    instead of running side by side (64 rows of V = 128256 bf16 17.7 us a call for 13.2).  Calls that look like greedy rows of which
    only ids are wanted may take all of the chip."""
    seen = 0
    for dtype in (sip.SIP_F32, sip.SIP_BF16):
        for t in (0, 2, 4, 8):
            for V in (33000, 40000, 65536, 100000, 128256, 200000, 262144):
                for B in range(1, 129):
                    route, S = sip.sip_call_route(B, V // 64 * 64 if t else V, dtype, t, False, params, 1000 * B, k)
                    if route == ROUTE_CHUNKS_ALONE:
                        seen += 1
                        assert B * S <= 176 and B <= 32, (B, V, dtype, t, S)
    assert seen > 500
    assert sip.sip_call_route(128, 152064, sip.SIP_BF16, 0, False, ("temperature",), 0, -1) == (ROUTE_CHUNKS_ALONE, 2)
