"""Builds the library and main.cpp for the CPU, with an address sanitizer, against the HIP names in
hip/hip_runtime.h.  The sources are those of csrc/ but for the two forms that plain C++ does
not have: kernel<<<...>>>(...) becomes a call of lanes::Launch, and the empty asm statements that
hide an index from the GPU's compiler are left out."""

import concurrent.futures as cf
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CLANG = "/opt/rocm/llvm/bin/clang++"
FLAGS = ["-std=c++20", "-O1", "-g1", "-mfma", "-ffp-contract=off", "-w", "-fsanitize=address"]


def plain(text: str) -> str:
    text = re.sub(r'asm volatile\("" : "\+v"\((\w+)\)\);', "", text)
    while (i := text.find("<<<")) >= 0:
        b = i
        if text[b - 1] == ">":                      # template arguments of the kernel
            depth = 0
            while True:
                b -= 1
                depth += {">": 1, "<": -1}.get(text[b], 0)
                if depth == 0:
                    break
        while re.match(r"\w", text[b - 1]):
            b -= 1
        e = text.index(">>>", i)
        p = text.index("(", e)
        text = (text[:b] + f"lanes::Launch({text[i + 3:e]})([](auto... a_) {{ {text[b:i]}(a_...); }}, "
                + text[p + 1:])
    return text


def build(out: str) -> str:
    """Compiles into the directory out; returns the program's path."""
    from paper_0907_3261_amd import build as lib
    csrc = os.path.join(out, "paper", "csrc")
    os.makedirs(csrc, exist_ok=True)
    inc = ["-I", HERE, "-I", os.path.join(ROOT, "include")]
    srcs = []
    for name in lib.SOURCES + ["wd_internal.h"]:
        with open(os.path.join(lib.CSRC, name)) as f:
            text = plain(f.read()).replace('"../../include/wdsolve.h"', '"wdsolve.h"')
        path = os.path.join(csrc, name.replace(".hip", ".cpp"))
        with open(path, "w") as f:
            f.write(text)
        if path.endswith(".cpp"):
            srcs.append(path)
    srcs.append(os.path.join(HERE, "main.cpp"))
    objs = [os.path.join(out, os.path.basename(s) + ".o") for s in srcs]

    def run(cmd):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, " ".join(cmd) + "\n" + r.stderr[-4000:]

    with cf.ThreadPoolExecutor(len(srcs)) as ex:
        list(ex.map(run, [[CLANG, *FLAGS, *inc, "-c", s, "-o", o] for s, o in zip(srcs, objs)]))
    exe = os.path.join(out, "main")
    run([CLANG, "-fsanitize=address", "-o", exe, *objs])
    return exe
