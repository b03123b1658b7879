"""Builds libfs.so (the C-ABI library) and _launch.so (the launch path of runner.py) in-tree with hipcc for gfx950.

    python -m paper_1811_05213_amd.build

The device building blocks (csrc/fs_device.h) are compiled ahead of time once (probe
kernels + a self-test instantiation) and embedded as text for the run-time compiler.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libfs.so")
LAUNCH = os.path.join(HERE, "_launch.so")
SOURCES = ["fs_graph.cpp", "fs_group.cpp", "fs_codegen.cpp", "fs_runtime.cpp", "fs_perflib.cpp", "fs_probe.hip", "fs_device_src.cpp"]
HIP_FLAGS = ["--offload-arch=gfx950", "-O2", "-std=c++17", "-fPIC", "-ffp-contract=off",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def _embed_device_header() -> str:
    """Writes csrc/fs_device_src.cpp: the text of fs_device.h, without its comment lines, as a string constant."""
    with open(os.path.join(CSRC, "fs_device.h"), "r") as f:
        # (comment lines stay out: plan creation hashes this text for every plan, and the run-time compiler reads it)
        text = "".join(ln for ln in f if not ln.lstrip().startswith("//"))
    out = os.path.join(CSRC, "fs_device_src.cpp")
    chunks = [text[i:i + 8000] for i in range(0, len(text), 8000)]
    body = "\n".join('R"FSDEV(' + c + ')FSDEV"' for c in chunks)
    new = ("// generated by paper_1811_05213_amd/build.py from fs_device.h - do not edit\n"
           "namespace fs {\nconst char* device_header_source() {\n  static const char* text =\n" + body +
           ";\n  return text;\n}\n}  // namespace fs\n")
    old = open(out).read() if os.path.exists(out) else None
    if old != new:
        with open(out, "w") as f:
            f.write(new)
    return out


def build(verbose: bool = False) -> str:
    _embed_device_header()
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    procs = []
    for src in SOURCES:
        obj = os.path.join(bdir, src + ".o")
        objs.append(obj)
        cmd = [hipcc] + HIP_FLAGS + ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-c", os.path.join(CSRC, src), "-o", obj]
        if src.endswith(".cpp"):
            cmd.insert(1, "-xhip")
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        lines = [ln for ln in out.splitlines() if "packed-fp32-ops" not in ln]
        if p.returncode != 0 or (verbose and lines):
            print(f"--- {src}\n" + "\n".join(lines), file=sys.stderr)
        failed |= p.returncode != 0
    if failed:
        raise RuntimeError("hipcc failed")
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs + ["-lhiprtc", "-ldl"]
    subprocess.run(cmd, check=True)
    # the Python module of the launch path: host code only
    subprocess.run([hipcc, "-xc++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "fs_pylaunch.cpp"), "-o", LAUNCH], check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
