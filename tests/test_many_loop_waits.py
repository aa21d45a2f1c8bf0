"""The time loops beyond 16 alive pieces (lstm_many.h) request a unit's rows and saved values in the unit before, in front of that
unit's stores, and wait with a count of those stores written by hand.  On every path of the compiled kernels at least that
many stores must have been issued since the last of the loads, or a wave may read what the unit before last left there.
CPU only (hipcc cross-compiles)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2210_05064_amd import build as b

CSRC = os.path.join(os.path.dirname(os.path.abspath(b.__file__)), "csrc")
VMEM = re.compile(r"\t(buffer|global|flat|scratch)_(load|store|atomic)")
NONE = 1 << 20   # no load in flight


# Kernels of every role, direction and arithmetic: the widest ones and the general form of the narrow bf16 layers.
KERNELS = {
    "fwd": ["lstm_rec_fwd_kernel<MODE_F32, 2, 4, 8, true>(RecFwdArgs)", "lstm_pipe_fwd_kernel<MODE_F32, 2, 4, 8, true>(PipeFwdArgs)",
            "lstm_pipe_fwd_kernel<MODE_BF16, 2, 2, 16, true>(PipeFwdArgs)", "lstm_triple_fwd_kernel<MODE_BF16, 2, 4, 4, false>(TripleFwdArgs)"],
    "bwd": ["lstm_rec_bwd_kernel<MODE_F32, 1, 8, 16>(RecBwdArgs)", "lstm_pipe_bwd_kernel<MODE_F32, 1, 8, 0>(PipeBwdArgs)",
            "lstm_pipe_bwd_kernel<MODE_BF16, 2, 4, 32>(PipeBwdArgs)", "lstm_triple_bwd_kernel<MODE_BF16, 1, 8, 0>(TripleBwdArgs)"]}


def assembly(kernels, out):
    """Device assembly of the named instantiations, compiled side by side."""
    runs = []
    for i, k in enumerate(kernels):
        (out / f"{i}.hip").write_text(f'#include "lstm_pipe.h"\nnamespace ver {{ template __global__ void {k}; }}\n')
        runs.append(subprocess.Popen(["hipcc", *b.FLAGS, f"-I{CSRC}", "--offload-device-only", "-S", str(out / f"{i}.hip"), "-o", str(out / f"{i}.s")],
                                     stderr=subprocess.DEVNULL))
    assert not any([r.wait() for r in runs])
    return {k: (out / f"{i}.s").read_text() for i, k in enumerate(kernels)}


def blocks_of(body):
    """Basic blocks of a function as lists of events, and the blocks that may follow each.  An event: "load" (of a unit's rows or saved
    values), "op" (any other memory operation), ("wait", n), ("hand", n): the same, written by hand."""
    events, after, at, hand, falls = [[]], [[]], {}, False, True

    def begin(falls):
        events.append([])
        after.append([])
        if falls:
            after[-2].append(len(events) - 1)
    for line in body.splitlines():
        label = re.match(r"(\.L\w+):", line)
        if label:
            begin(falls)
            falls = True
            at[label.group(1)] = len(events) - 1
        elif "#ASMSTART" in line:
            hand = True
        elif "#ASMEND" in line:
            hand = False
        elif VMEM.match(line):
            events[-1].append("load" if line.startswith("\tbuffer_load") else "op")
        elif line.startswith("\ts_waitcnt"):
            count = re.search(r"vmcnt\((\d+)\)", line)
            if count:
                events[-1].append(("hand" if hand else "wait", int(count.group(1))))
        elif branch := re.match(r"\ts_(c?)branch\w*\s+(\.L\w+)", line):
            after[-1].append(branch.group(2))
            falls = bool(branch.group(1))
            begin(falls)
        elif line.startswith("\ts_endpgm") or line.startswith("\ts_setpc"):
            falls = False
            begin(False)
    return events, [[at[s] if isinstance(s, str) else s for s in out] for out in after]


def short_waits(body, stores):
    """(operations since the last load, at the fewest) of every wait for all but `stores` operations that is reached with fewer."""
    events, after = blocks_of(body)
    state, todo, short, seen = {0: NONE}, [0], [], 0
    while todo:
        k = todo.pop()
        n = state[k]
        for e in events[k]:
            if e == "load":
                n = 0
            elif e == "op":
                n = min(n + 1, NONE)
            elif n >= e[1]:
                n = NONE
        for s in after[k]:
            if n < state.get(s, NONE + 1):
                state[s] = n
                todo.append(s)
    for k, n in state.items():
        for e in events[k]:
            if e == ("hand", stores):
                seen += 1
                if n < stores:
                    short.append(n)
            if e == "load":
                n = 0
            elif e == "op":
                n = min(n + 1, NONE)
            elif n >= e[1]:
                n = NONE
    return short, seen


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_no_load_is_left_in_flight(tmp_path):
    stores = {"fwd": 6, "bwd": 4}   # STORES of many_fwd and many_bwd
    text = open(os.path.join(CSRC, "lstm_many.h")).read()
    assert [int(n) for n in re.findall(r"constexpr int STORES = (\d+);", text)] == list(stores.values())
    for kernel, asm in assembly(KERNELS["fwd"] + KERNELS["bwd"], tmp_path).items():
        name = re.match(r"\w+", kernel).group(0)
        body = re.search(rf"^_ZN3ver\d+{name}\w*:[^\n]*\n(.*?)^\.Lfunc_end", asm, re.S | re.M).group(1)
        short, seen = short_waits(body, stores[kernel.split("_")[2]])
        assert seen and not short, (kernel, seen, short)


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_only_kernels_that_run_the_form_have_it(tmp_path):
    """fp32 backward up to 256 units never runs it (many_pays_bwd): the kernels of 128 and 256 units, which have loops of their own, leave it out."""
    for kernel, asm in assembly([f"lstm_rec_bwd_kernel<MODE_F32, 1, 8, {ni}>(RecBwdArgs)" for ni in (4, 8)], tmp_path).items():
        assert short_waits(re.search(r"^_ZN3ver\d+lstm_rec_bwd\w*:[^\n]*\n(.*?)^\.Lfunc_end", asm, re.S | re.M).group(1), 4) == ([], 0), kernel
