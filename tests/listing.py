"""The kernels of the built library as the disassembler lists them."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

from paper_2508_00441_amd import binding

LLVM = "/opt/rocm/llvm/bin/"
AVAILABLE = os.path.exists(LLVM + "llvm-objdump")


class Instruction:
    __slots__ = ("text", "at", "target")             # target: of a branch, else None

    def __init__(self, text, at, target):
        self.text, self.at, self.target = text, at, target


@functools.lru_cache(maxsize=None)
def texts():
    """{symbol: the lines of its listing}"""
    out = {}
    with tempfile.TemporaryDirectory() as d:
        lib = shutil.copy(binding.LIB_PATH, os.path.join(d, "lib.so"))
        subprocess.check_call([LLVM + "llvm-objdump", "--offloading", lib], cwd=d, stdout=subprocess.DEVNULL)
        for name in sorted(os.listdir(d)):
            if "gfx950" not in name:
                continue
            text = subprocess.check_output([LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", os.path.join(d, name)], text=True)
            for part in re.split(r"^<(?=_Z)", text, flags=re.M)[1:]:
                head, _, body = part.partition(">:\n")
                out[head] = body
    return out


def instructions(symbol):
    found = []
    for line in texts()[symbol].splitlines():
        m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+): [0-9A-F ]+(?:<\S+?\+0x([0-9a-f]+)>)?$", line)
        if m:
            found.append((m.group(1), int(m.group(2), 16), m.group(3)))
    start = found[0][1]
    return [Instruction(t, at - start, int(to, 16) if to is not None and "branch" in t else None) for t, at, to in found]


def vector_registers(text):
    used = {int(r) for r in re.findall(r"\bv(\d+)\b", text)}
    for lo, hi in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        used |= set(range(int(lo), int(hi) + 1))
    return used
