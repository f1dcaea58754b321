"""Compiles tests/host/probe.hip for the host and runs it (no GPU needed)."""
import functools
import os
import subprocess
import tempfile

import paper_2606_09862_amd as bla
from paper_2606_09862_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
_dir = tempfile.TemporaryDirectory()


@functools.lru_cache(maxsize=1)
def probe():
    if not os.path.exists(bla.LIB_PATH):
        build.build()
    exe = os.path.join(_dir.name, "probe")
    subprocess.run([build.HIPCC, "-std=c++17", "-O1", "--cuda-host-only", "-x", "hip", f"-I{build.INCLUDE}",
                    f"-I{build.CSRC}", "-Wno-unused-result", os.path.join(HERE, "host", "probe.hip"), "-o", exe + ".o",
                    "-c", "-fPIE"], check=True, capture_output=True)
    subprocess.run([build.HIPCC, "-fPIE", exe + ".o", bla.LIB_PATH, f"-Wl,-rpath,{os.path.dirname(bla.LIB_PATH)}",
                    "-o", exe], check=True, capture_output=True)
    return exe


def run(command, lines=()):
    res = subprocess.run([probe(), command], input="\n".join(lines), capture_output=True, text=True, check=True)
    return res.stdout.splitlines()


def plans(cases):
    """cases: (form, B, H, L, d, M, S, bf16, chunk, anchor).  A dict per case, None where unsupported."""
    out = []
    for line in run("plan", [" ".join(map(str, c)) for c in cases]):
        if line == "unsupported":
            out.append(None)
            continue
        w = line.split()
        i = w.index("tables")
        d = {k: int(v) for k, v in zip(w[:i:2], w[1:i:2])}
        d["tables"] = tuple(map(int, w[i + 1:]))
        out.append(d)
    return out
