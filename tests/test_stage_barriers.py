"""The built GEMM kernels, read back from the library: no workgroup barrier is reached with LDS reads of the same wave
in flight.  Behind such a barrier the other waves copy new data over the stage the reads come from, and a copy is not
ordered against a read.  Host only: the library's own code objects are disassembled, nothing is run."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2310_09259_amd", "libquik.so")
OBJDUMP = "/opt/rocm/lib/llvm/bin/llvm-objdump"


def _kernels(tmp):
    """{kernel: [(address, mnemonic, operands, branch target or None)]} of every kernel that copies global -> LDS."""
    if not os.path.exists(LIB):
        from paper_2310_09259_amd import build
        build.build()
    shutil.copy(LIB, tmp)
    subprocess.run([OBJDUMP, "--offloading", "libquik.so"], cwd=tmp, check=True, stdout=subprocess.DEVNULL)
    out = {}
    for obj in sorted(glob.glob(os.path.join(tmp, "*gfx950"))):
        text = subprocess.run([OBJDUMP, "-d", obj], check=True, stdout=subprocess.PIPE, text=True).stdout
        name, start = None, 0
        for line in text.splitlines():
            head = re.match(r"^([0-9a-f]+) <(\w+)>:$", line)
            if head:
                name, start = head[2], int(head[1], 16)
                out[name] = []
                continue
            ins = re.match(r"^\t(\S+) ?(.*?)\s*// ([0-9A-F]+):(.*)$", line)
            if not ins or name is None:
                continue
            target = None
            if ins[1].startswith(("s_cbranch", "s_branch")):
                at = re.search(r"<\w+?(?:\+0x([0-9a-f]+))?>$", ins[4])
                target = start + int(at[1] or "0", 16)
            out[name].append((int(ins[3], 16), ins[1], ins[2], target))
    # (the measurement probes run a K loop's instructions on data that nobody looks at)
    return {k: v for k, v in out.items()
            if "probe" not in k and any(m.startswith("buffer_load") and o.endswith(" lds") for _, m, o, _ in v)}


def _barriers_with_reads_in_flight(code):
    """Largest number of outstanding LDS reads over all paths, by instruction, to a fixed point."""
    index = {a: i for i, (a, _, _, _) in enumerate(code)}
    before = [-1] * len(code)
    before[0], work, bad = 0, [0], set()
    while work:
        i = work.pop()
        n = before[i]
        _, op, args, target = code[i]
        if op.startswith("ds_read") or (op.startswith(("ds_", "s_load", "s_buffer_load")) and n):
            n = min(n + 1, 15)
        elif op == "s_waitcnt":
            lgkm = re.search(r"lgkmcnt\((\d+)\)", args)
            if lgkm:
                n = min(n, int(lgkm[1]))
        elif op == "s_barrier" and n:
            bad.add(code[i][0])
        follow = [] if op in ("s_endpgm", "s_branch") else [i + 1]
        if target is not None:
            follow.append(index[target])
        for j in follow:
            if j < len(code) and n > before[j]:
                before[j] = n
                work.append(j)
    return bad


def test_no_barrier_is_reached_with_lds_reads_in_flight(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    kernels = _kernels(str(tmp_path))
    assert len(kernels) > 100
    barriers = sum(op == "s_barrier" for code in kernels.values() for _, op, _, _ in code)
    assert barriers > 300
    bad = {k: sorted(hex(a) for a in b) for k, code in kernels.items() for b in [_barriers_with_reads_in_flight(code)] if b}
    assert not bad, bad
