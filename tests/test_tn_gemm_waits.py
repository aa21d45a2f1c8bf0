"""The K-minor tiles keep several stages of LDS-direct loads in flight and count them by hand: every wait of a kernel's
loop must leave whole stages in flight, i.e. a multiple of the loads that one pass of the loop issues.  Reads the
compiled kernels.  CPU only (hipcc cross-compiles)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2210_05064_amd import build as b

CSRC = os.path.join(os.path.dirname(os.path.abspath(b.__file__)), "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_waits_leave_whole_stages_in_flight(tmp_path):
    src, asm = tmp_path / "tn.hip", tmp_path / "tn.s"
    src.write_text('#include "gemm.h"\n')
    subprocess.check_call(["hipcc", *b.FLAGS, f"-I{CSRC}", "--offload-device-only", "-S", str(src), "-o", str(asm)], stderr=subprocess.DEVNULL)
    loops = 0
    for name, body in re.findall(r"^(_ZN\S*gemm_tn_dma\S*):[^\n]*\n(.*?)^\.Lfunc_end", asm.read_text(), re.S | re.M):
        loads, waits, header = {}, {}, None
        for line in body.splitlines():   # every block's label says which loop it belongs to
            if re.match(r"\.LBB\d+_\d+:|; %bb\.\d+:", line):
                at = re.search(r"Header=(BB\d+_\d+)", line)
                header = at.group(1) if at else (line[2:line.index(":")] if "Loop Header" in line else None)
            elif "offen lds" in line:
                loads[header] = loads.get(header, 0) + 1
            elif m := re.match(r"\s*s_waitcnt vmcnt\((\d+)\)$", line):
                waits.setdefault(header, set()).add(int(m.group(1)))
        for header, n in loads.items():
            if header in waits:   # (the loop that fills the first stages has no wait)
                assert waits[header] in ({0, n}, {0, n, 2 * n}), (name, header, n, waits[header])
                loops += 1
    assert loops == 6, loops   # two kernels of one loop each, two grouped kernels of two
