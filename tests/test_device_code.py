"""What the built device code looks like where its speed depends on it: the functions that are not inlined into the
kernels reach LDS by LDS instructions, and the kernels that hardly ever call them keep small frames."""
import collections
import os
import re
import subprocess

import pytest

from paper_2506_22033_amd import build as sip_build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    if not os.path.exists(f"{LLVM}/llvm-objdump"):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(sip_build.LIB):
        sip_build.build()
    d = tmp_path_factory.mktemp("code")
    os.symlink(sip_build.LIB, d / "libsip.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "libsip.so"], cwd=d, check=True, capture_output=True)
    return next(d / f for f in os.listdir(d) if "gfx950" in f)


def test_functions_reach_lds_by_lds_instructions(code_object):
    kinds, name = collections.defaultdict(collections.Counter), None
    out = subprocess.Popen([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", code_object], stdout=subprocess.PIPE, text=True)
    for line in out.stdout:
        m = re.match(r"[0-9a-f]+ <_ZN3sip\d+(\w+?)ILi", line)
        if m or line.endswith(">:\n"):
            name = m and m.group(1)
        elif name:
            op = line.split(None, 1)
            for kind in ("ds_", "flat_"):
                if op and op[0].startswith(kind):
                    kinds[name][kind] += 1
    assert out.wait() == 0
    for f in ("exact_row", "restream_row", "whole_row_window", "whole_row_nucleus", "whole_row_draw", "rescue_apart"):
        # (flat ones are left where the arguments or a row are read by a plain pointer; with LDS among them there were 1.7
        # times as many as LDS instructions in exact_row, the fewest)
        assert kinds[f]["ds_"] > 0 and kinds[f]["flat_"] <= 1.2 * kinds[f]["ds_"], (f, kinds[f])


def test_frames_are_small(code_object):
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", code_object], capture_output=True, text=True, check=True).stdout
    frames = {}
    for block in notes.split("- .agpr_count")[1:]:
        frames[re.search(r"\.name:\s+(_ZN3sip\S+)", block).group(1)] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block).group(1))
    fused = {n: f for n, f in frames.items() if "_rescue_kernel" in n or "13rescue_kernel" in n}
    assert len(fused) >= 20
    # 432 bytes a lane are the registers that a function which may be a tail call saves
    assert max(fused.values()) <= 160, fused
