"""Builds the library's own sources for the CPU (host_model/), for the tests that
run its kernels with no GPU (not collected: no test_ prefix).

The sources are taken as they are but for four rewrites of the text: a launch
``k<<<g, b, 0, s>>>(...)`` becomes a call of the CPU runtime's launcher, a
``__shared__`` array a block of its LDS, address spaces and unroll hints go, and
the lists of FFT lengths are cut to those that hold every first radix and one,
two and three stages (LENGTHS), which keeps the build short."""

import hashlib
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2107_06729_amd")
MODEL = os.path.join(HERE, "host_model")
CLANG = "/opt/rocm/llvm/bin/clang++"
# first radices 2 4 8 (16) 3 4 5 6 10 12 20; three stages from 128 on
LENGTHS = (2, 4, 8, 16, 24, 32, 40, 48, 64, 80, 96, 128, 160)


def _launches(text):
    """k<..><<<cfg>>>( -> host::launcher("k", &k<..>, cfg)("""
    out, pos = [], 0
    for m in re.finditer(r"<<<(.*?)>>>", text, re.S):
        i = m.start()
        if text[i - 1] == ">":
            depth, i = 0, i - 1
            while True:
                depth += (text[i] == ">") - (text[i] == "<")
                if depth == 0:
                    break
                i -= 1
        while re.match(r"\w", text[i - 1]):
            i -= 1
        kernel = text[i:m.start()]
        out += [text[pos:i], f'host::launcher("{kernel.split("<")[0]}", &{kernel}, {m.group(1)})']
        pos = m.end()
    return "".join(out) + text[pos:]


def rewrite(name, text):
    text = _launches(text)
    text, shared = re.subn(r"__shared__ ([^;]*?) (\w+)((?:\[[^\]]*\])*);",
                           r"using \2_lds = std::remove_cv_t<\1>\3; \2_lds& \2 = host::lds<\2_lds>([] {});", text)
    text = re.sub(r"__attribute__\(\(address_space\(\d\)\)\)", "", text)
    text = re.sub(r"#pragma unroll.*", "", text)
    keep = {str(v) for v in LENGTHS}
    if name == "fft_lds.hpp":
        def cut(m):
            names = re.findall(r"M\((\d+)\)", m.group(0))
            return m.group(1) + " " + " ".join(f"M({v})" for v in names if v in keep)
        text = re.sub(r"(#define LLGX_(?:POW2|MIXED)_LENGTHS(?:_LONG)?\(M\)).*", cut, text)
    if name == "batch.hip":
        text = re.sub(r"\bC_\((\d+)\)", lambda m: m.group(0) if m.group(1) in keep | {"0", "1"} else "", text)
    assert "<<<" not in text and "__shared__" not in text, name
    return "#include <type_traits>\n" * bool(shared) + text


def build():
    """Path of the CPU library of the present sources (built once for them)."""
    import importlib.util
    spec = importlib.util.spec_from_file_location("llgx_build_lib", os.path.join(PKG, "build_lib.py"))
    lib = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(lib)
    files = {n: open(os.path.join(lib.CSRC, n)).read() for n in sorted(os.listdir(lib.CSRC))}
    model = [os.path.join(MODEL, "runtime.cpp"), os.path.join(MODEL, "hip", "hip_runtime.h")]
    key = hashlib.sha256("".join([open(os.path.abspath(__file__)).read(), *(open(f).read() for f in model),
                                  open(os.path.join(ROOT, "include", "llgx.h")).read(),
                                  *files.values()]).encode()).hexdigest()[:16]
    top = os.path.join(lib.BUILD, "host")
    out = os.path.join(top, key, "libllgx_host.so")
    if os.path.exists(out):
        return out
    shutil.rmtree(top, ignore_errors=True)  # those of other sources
    work = os.path.join(top, f"{key}.{os.getpid()}")
    os.makedirs(work)
    for n, text in files.items():
        with open(os.path.join(work, n), "w") as f:
            f.write(rewrite(n, text))
    base = [CLANG, "-x", "c++", "-std=c++17", "-O2", "-fno-unroll-loops", "-fno-vectorize", "-fno-slp-vectorize", "-fPIC", "-w", "-ffp-contract=off", "-fno-strict-aliasing",
            "-I", MODEL, "-I", work, "-I", os.path.join(ROOT, "include")]
    cmds = [base + [f"-DLLGX_INST={k}"] * (k is not None) + ["-c", os.path.join(work, s), "-o",
                                                             os.path.join(work, f"{s}_{k}.o")] for s, k in lib.SOURCES]
    cmds.append(base + ["-c", model[0], "-o", os.path.join(work, "runtime.o")])

    def run(c):
        r = subprocess.run(c, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode:
            raise RuntimeError(f"{' '.join(c)}\n{r.stdout[-4000:]}")
    with ThreadPoolExecutor(min(len(cmds), os.cpu_count() or 1)) as ex:
        list(ex.map(run, cmds))
    objs = [c[-1] for c in cmds]
    tmp = os.path.join(work, "libllgx_host.so")
    run([CLANG, "-shared", "-fPIC", "-o", tmp] + objs)
    os.makedirs(os.path.dirname(out), exist_ok=True)
    os.replace(tmp, out)
    shutil.rmtree(work)
    return out


if __name__ == "__main__":
    print(build())
