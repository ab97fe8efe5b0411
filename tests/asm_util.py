"""Kernels' assembly for tests that read it (hipcc, no GPU): instructions, control flow, registers."""
import functools
import os
import re
import subprocess
import tempfile

import pytest

from paper_2504_08966_amd import build as B


@functools.lru_cache(maxsize=None)
def _assembly(source):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "out.s")
        cmd = [B._hipcc(), *B.FLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, source), "-o", out]
        try:
            r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
        except FileNotFoundError:
            pytest.skip("no hipcc")
        assert r.returncode == 0, r.stderr
        with open(out) as f:
            return f.read()


def kernels(source):
    """[(name, body)] of the kernels that `source` (a file of csrc/) compiles to."""
    return re.findall(r"^(_ZN4pact\w+):(.*?)^\.Lfunc_end", _assembly(source), re.S | re.M)


def spills(source):
    """{name: (vector registers spilled, bytes of scratch, scalar registers spilled)} of its kernels."""
    out = {}
    for m in re.finditer(r"- \.agpr_count:.*?\.wavefront_size", _assembly(source), re.S):
        of = lambda field: int(re.search(r"\." + field + r":\s+(\d+)", m.group(0)).group(1))
        out[re.search(r"\.name:\s+(\w+)", m.group(0)).group(1)] = (of("vgpr_spill_count"), of("private_segment_fixed_size"), of("sgpr_spill_count"))
    return out


def registers(text):
    """Vector, accumulation and scalar registers named in `text`: {"v3", "a0", "s12", ..}."""
    out = set()
    for m in re.finditer(r"\b([vas])(?:(\d+)|\[(\d+):(\d+)\])(?![\w:])", text):
        out |= {m.group(1) + str(i) for i in range(int(m.group(2) or m.group(3)), int(m.group(2) or m.group(4)) + 1)}
    return out


class Program:
    """Instructions of one kernel, the instructions that may follow each, and the vector registers that are left undefined ahead of it."""

    def __init__(self, body):
        self.ins, self.undefined, labels = [], {}, {}
        for line in body.splitlines():
            m = re.search(r"; implicit-def: \$(\S+)", line)
            if m and "spill" not in line:
                self.undefined.setdefault(len(self.ins), set()).update("v" + r for r in re.findall(r"vgpr(\d+)", m.group(1)))
            text = line.split(";")[0].strip()
            label = re.match(r"^(\.LBB\w+):", text)
            if label:
                labels[label.group(1)] = len(self.ins)
            elif text and not text.startswith("."):
                self.ins.append(text)
        self.after = []
        for i, text in enumerate(self.ins):
            op = text.split()[0]
            if op == "s_branch":
                self.after.append([labels[text.split()[1]]])
            elif op.startswith("s_cbranch"):
                self.after.append([i + 1, labels[text.split()[1]]])
            else:
                self.after.append([i + 1] if op != "s_endpgm" and i + 1 < len(self.ins) else [])
