"""The library's launches, read on the host: tests/c/launch_rule.cpp compiled with
the library's source and the product's or the checking build's constants."""
from __future__ import annotations

import dataclasses
import os
import subprocess
from typing import List

from paper_2607_18020_amd.csrc import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "c", "launch_rule.cpp")


@dataclasses.dataclass
class Launch:
    kernel: str        # "fwd_kernel<OpHeat, 256, 4, false, false, 8>"
    blocks: int
    threads: int
    chunk: int = 0     # marching kernels: planes (rows, time levels) per chunk
    tiles: tuple = ()  # and tiles across and down

    @property
    def name(self):
        return self.kernel.split("<")[0]

    @property
    def args(self):
        """Template arguments after the operator."""
        inner = self.kernel[self.kernel.index("<") + 1:self.kernel.rindex(">")]
        depth = 0
        for i, ch in enumerate(inner):
            depth += (ch == "<") - (ch == ">")
            if ch == "," and depth == 0:
                return tuple(x.strip() for x in inner[i + 1:].split(","))
        return ()


def compile_rule(out_dir, extra=()) -> str:
    """The program, for the product's constants or (extra = CHECK_FLAGS) the
    checking build's."""
    obj, exe = os.path.join(str(out_dir), "launch_rule.o"), os.path.join(str(out_dir), "launch_rule")
    defines = [f for f in B.FLAGS if f.startswith(("-std", "-W"))]
    subprocess.run([B.HIPCC, "--cuda-host-only", "-O1", *defines, *extra, "-I",
                    os.path.join(ROOT, "include"), "-I", B.HERE, "-c", SRC, "-o", obj], check=True)
    # (the device code object that the registration names does not exist)
    subprocess.run(["g++", "-no-pie", obj, "-Wl,--unresolved-symbols=ignore-in-object-files",
                    "-o", exe], check=True)
    return exe


def _plain(names):
    r = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True,
                       check=True)
    return {m: d.replace("fpde::", "").split("(")[0].replace("void ", "")
            for m, d in zip(names, r.stdout.splitlines())}


def kernels(exe: str) -> set:
    """Every kernel of the library."""
    names = subprocess.run([exe, "kernels"], capture_output=True, text=True, check=True).stdout
    return set(_plain(names.split()).values())


def residency(exe: str):
    """(kind, op, tile width, tile height, workgroups per CU, the same on a periodic grid)
    for every tile of the rule."""
    out = subprocess.run([exe, "residency"], capture_output=True, text=True, check=True).stdout
    return sorted({(w[0], *map(int, w[1:])) for w in map(str.split, out.splitlines())})


def launches(exe: str, requests) -> List[List[Launch]]:
    """For each (call, op, shape, bc_mode): its launches.  Every call must succeed."""
    text = "".join(f"{call} {op} {bc} {len(shape)} {' '.join(map(str, shape))}\n"
                   for call, op, shape, bc in requests)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
    names = sorted({ln.split()[0] for ln in out.splitlines() if ln.startswith("_Z")})
    plain = _plain(names)
    res, cur = [], []
    for ln in out.splitlines():
        w = ln.split()
        if w[0] == "=":
            assert w[1] == "0", requests[len(res)]
            res.append(cur)
            cur = []
        else:
            v = [int(x) for x in w[1:]]
            cur.append(Launch(plain[w[0]], v[0], v[1], *(v[2:3]), tuple(v[3:5])))
    assert len(res) == len(requests)
    return res
