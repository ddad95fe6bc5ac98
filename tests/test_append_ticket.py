"""The window-parallel append lets the work-group with the last ticket advance the sequence lengths, so a
work-group may take its ticket only after every one of its waves has read them: a wave that read them later
would see the advanced lengths and code a window that is not there. Each wave marks the point from which its
copy is in registers; checked here on the generated gfx950 code, for every key metadata format: on each path
from the mark to the counter's atomic the work-group passes a barrier (a work-group without a window, as a
shorter sequence of a ragged batch leaves it, takes another path than one with a window)."""

import os
import re
import subprocess

import pytest

from paper_2609_11582_amd import _build

SRC = "append_window.hip"


def _kernels(asm):
    """Name -> lines (labels and instructions) of each window-append kernel in the assembly."""
    out, name = {}, None
    for line in asm.splitlines():
        line = line.strip()
        m = re.match(r"(_Z\w*k_append_window\w*):", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and line:
            out[name].append(line)
    return out


def _blocks(lines):
    """Basic blocks (lists of lines) and their successors."""
    blocks, label = [[]], {}
    for line in lines:
        m = re.match(r"(\.LBB\w+):", line)
        if m:
            blocks.append([])
            label[m.group(1)] = len(blocks) - 1
            continue
        blocks[-1].append(line)
        if re.match(r"s_c?branch|s_endpgm", line):
            blocks.append([])
    succ = []
    for i, b in enumerate(blocks):
        last = b[-1].split() if b else [""]
        if last[0] == "s_endpgm":
            succ.append([])
        elif last[0] == "s_branch":
            succ.append([label[last[1]]])
        else:
            succ.append(([label[last[1]]] if last[0].startswith("s_cbranch") else []) + [i + 1][: i + 1 < len(blocks)])
    return blocks, succ


def _step(block, ok, at_ticket=None):
    for line in block:
        if "okvq: lengths read" in line:
            ok = False
        elif line.startswith("s_barrier"):
            ok = True
        elif re.match(r"(flat|global)_atomic_add", line) and at_ticket is not None:
            at_ticket.append(ok)
    return ok


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "append_window.s")
    cmd = [_build.hipcc(), *_build.FLAGS, *_build.EXTRA.get(SRC, []), "-I", _build.INCLUDE, "-I", _build.CSRC,
           "--cuda-device-only", "-S", os.path.join(_build.CSRC, SRC), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    with open(out) as f:
        return f.read()


def test_no_ticket_before_every_wave_has_read_the_lengths(asm):
    kernels = _kernels(asm)
    assert len(kernels) == 3
    for name, lines in kernels.items():
        assert sum("okvq: lengths read" in x for x in lines) == 1, name
        blocks, succ = _blocks(lines)
        # on entry to a block: True where every path to it has passed a barrier since the mark
        enter = [None] * len(blocks)
        enter[0] = False
        work = [0]
        while work:
            i = work.pop()
            ok = _step(blocks[i], enter[i])
            for j in succ[i]:
                new = ok if enter[j] is None else (enter[j] and ok)
                if new != enter[j]:
                    enter[j] = new
                    work.append(j)
        tickets = []
        for b, ok in zip(blocks, enter):
            if ok is not None:
                _step(b, ok, tickets)
        assert tickets and all(tickets), f"{name}: tickets taken after a barrier: {tickets}"
