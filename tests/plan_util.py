"""The forward's plan for a shape, from the library's own rules compiled for the host."""
import functools
import os
import shutil
import subprocess
import tempfile
from typing import NamedTuple

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = os.environ.get("CXX", "g++")


class Plan(NamedTuple):
    kernel: str          # row, short, ring or chunk
    nseg: int            # time segments (1: none)
    seg_len: int
    pieces: int          # pre-pass pieces per segment
    waves: int           # per chain
    workgroups: int
    threads: int         # per workgroup
    carry: int           # bytes


def have_compiler() -> bool:
    return shutil.which(CXX) is not None


@functools.lru_cache(maxsize=None)
def _exe() -> str:
    exe = os.path.join(tempfile.mkdtemp(prefix="plan_"), "plan")
    subprocess.run([CXX, "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2401_13660_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "plan_main.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    return exe


def plans(shapes, *, dstate=16, dtype="bf16", out_bytes=4, gate=True, aligned=True, ckpt=False,
          npos=0, h0=False, cus=256):
    lines = "".join(f"{b} {d} {L} {dstate} {2 if dtype == 'bf16' else 4} {out_bytes} {int(gate)} {int(aligned)} "
                    f"{int(ckpt)} {npos} {int(h0)} {cus}\n" for b, d, L in shapes)
    out = subprocess.run([_exe()], input=lines, check=True, capture_output=True, text=True).stdout
    return [Plan(w[0], *map(int, w[1:])) for w in (line.split() for line in out.splitlines())]


def plan(shape, **kw) -> Plan:
    return plans([shape], **kw)[0]
