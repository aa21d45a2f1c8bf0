"""The time loops of up to four alive pieces are bound by the instructions of one wave, and every scalar that the compiler keeps in a spill
lane is a v_readlane per use there: before the loops took turns in one kernel with those of many pieces they had 24 to 33 per timestep in the
consumer layer, with them in place 54 to 89.  Reads the compiled kernels.  CPU only (hipcc cross-compiles)."""
import re
import shutil

import pytest

from tests.test_many_loop_waits import assembly

MOST = 33


def loops(body):
    """The instructions of every outermost loop."""
    lines, top, cur, found = body.splitlines(), {}, None, {}
    for i, line in enumerate(lines):
        if re.match(r"\.LBB\d+_\d+:|; %bb\.\d+:", line):
            about = line
            for more in lines[i + 1:]:   # the nest is told in the comments behind a label
                if not re.match(r"\s+;", more) or "ASM" in more:
                    break
                about += "\n" + more
            label = line[2:line.index(":")] if line.startswith(".L") else None
            outer = re.search(r"Parent Loop (BB\d+_\d+) Depth=1\b", about) or re.search(r"Header=(BB\d+_\d+) Depth=1\b", about)
            inner = re.search(r"in Loop: Header=(BB\d+_\d+) ", about)
            cur = outer.group(1) if outer else label if re.search(r"Loop Header: Depth=1\b", about) else top.get(inner.group(1)) if inner else None
            if label and cur:
                top[label] = cur
        elif cur and re.match(r"\t[a-z]", line):
            found.setdefault(cur, []).append(line)
    return found.values()


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_scalars_of_the_loops_of_few_pieces(tmp_path):
    kernels = ["lstm_pipe_bwd_kernel<MODE_F32, 1, 8, 16>(PipeBwdArgs)", "lstm_pipe_bwd_kernel<MODE_BF16, 2, 4, 32>(PipeBwdArgs)"]
    for kernel, asm in assembly(kernels, tmp_path).items():
        body = re.search(r"^_ZN3ver\d+lstm_pipe_bwd_kernel\w*:[^\n]*\n(.*?)^\.Lfunc_end", asm, re.S | re.M).group(1)
        count = lambda loop, what: sum(bool(re.search(what, line)) for line in loop)
        # up to four pieces: a product, no LDS-direct loads, one timestep of four stores per pass
        reads = [count(l, r"v_readlane") for l in loops(body) if count(l, r"v_mfma|v_fmac\w*_dpp") and not count(l, r"offen lds") and count(l, r"buffer_store") == 4]
        assert len(reads) == 4 and max(reads) <= MOST, (kernel, reads)   # producer and consumer, two sizes each


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_scalars_of_the_consumers_loop_of_five_to_sixteen_pieces(tmp_path):
    """Forward, two timesteps per pass: 15 to 24 before, 32 to 40 with the loops of many pieces in place."""
    for kernel, asm in assembly(["lstm_pipe_fwd_kernel<MODE_BF16, 2, 4, 4, true>(PipeFwdArgs)", "lstm_pipe_fwd_kernel<MODE_BF16, 2, 2, 16, true>(PipeFwdArgs)"], tmp_path).items():
        body = re.search(r"^_ZN3ver\d+lstm_pipe_fwd_kernel\w*:[^\n]*\n(.*?)^\.Lfunc_end", asm, re.S | re.M).group(1)
        count = lambda loop, what: sum(bool(re.search(what, line)) for line in loop)
        # four barriers per timestep: of the wait for a chunk, of that for the flags, behind the partial sums and behind their last read
        reads = [count(l, r"v_readlane") for l in loops(body) if count(l, r"v_mfma") and not count(l, r"offen lds") and count(l, r"s_barrier") == 8]
        assert len(reads) == 1 and reads[0] <= 24, (kernel, reads)
