"""Helper of the CPU tests of the library's host-side launch plans: a small C++
program over the internal headers, linked with the built library."""
from __future__ import annotations

import os
import subprocess

from paper_2511_13508_amd import build as B


def run(tmp_path, source: str) -> list[list[str]]:
    """Compile `source` as a program, run it, and return its output lines as words."""
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(source)
    subprocess.run(["g++", *B.CXX_FLAGS, f"-I{B.CSRC}", str(src), "-o", str(exe), B.OUT, f"-L{B.ROCM}/lib", "-lamdhip64",
                    f"-Wl,-rpath,{B.ROCM}/lib", f"-Wl,-rpath,{os.path.dirname(B.OUT)}"], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120).stdout
    return [line.split() for line in out.splitlines()]
