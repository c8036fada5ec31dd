"""Build the HIP library ``_lisaresp.so`` for gfx950 in the package directory.

Run ``python -m paper_2204_06633_amd.csrc.build`` (or call ``build()``).  Every
call recompiles.  Flags: -O3, C++17, no fast-math (IEEE division and square
root), FMA contraction allowed, packed-FP32 instructions disabled.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.dirname(HERE)
ROOT = os.path.dirname(PKG)
TARGET = os.path.join(PKG, "_lisaresp.so")
# The fused batched forward has 8 (group, tile) variants per tap count and
# TDI generation; its explicit instantiations are generated per (generation,
# tap count) into the build directory, 32 small translation units that
# spread evenly over the compile jobs.
FUSED_UNITS = [(g, nt) for nt in range(2, 33, 2) for g in (1, 2)]
SOURCES = (["forward_%s.hip" % k for k in "abcd"] + ["adjoint_%s.hip" % k for k in "abcd"] +
           ["tdifir_%s.hip" % k for k in "abcd"] + ["farrow_%s.hip" % k for k in "abcd"] +
           ["batchfwd%d_n%d.hip" % u for u in FUSED_UNITS] +
           ["batchadj_%s.hip" % k for k in "abcd"] +
           ["util.hip", "fd_kernels.hip", "gb_kernels.hip", "dispatch.cpp", "api.cpp", "api_batch.cpp",
            "api_fd.cpp", "api_gb.cpp", "api_noalloc.hip", "build_config.hip"])
ARCH = os.environ.get("LR_OFFLOAD_ARCH", "gfx950")


def _weight(src):
    """Rough compile cost of a unit (for the job order)."""
    if src.startswith("batchfwd"):
        return 10 + int(src.split("_n")[1][:-4])
    return 30 if src.startswith(("adjoint", "batchadj", "forward", "tdifir", "farrow")) else 1


def hipcc():
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def flags():
    return ["-O3", "-std=c++17", "--offload-arch=" + ARCH, "-fPIC",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-munsafe-fp-atomics", "-fno-fast-math", "-Wall", "-Wno-unused-variable",
            "-I" + os.path.join(ROOT, "include")]


def link_flags():
    """The roctx library of the call ranges (trace.hpp)."""
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc())))
    return ["-L" + os.path.join(rocm, "lib"), "-lrocprofiler-sdk-roctx"]


def _fused_unit(out_dir, name):
    """Write the generated instantiation unit ``name`` (batchfwd<g>_n<NT>.hip)
    into out_dir and return its path."""
    g, nt = name[len("batchfwd"):-len(".hip")].split("_n")
    path = os.path.join(out_dir, name)
    text = ('// Generated by build.py: fused batched forward, TDI generation %s, %s taps.\n'
            '#include "%s"\n\nnamespace lr {\nLR_INSTANTIATE_BATCH_FWD(%s, %s)\n}  // namespace lr\n'
            % (g, nt, os.path.join(HERE, "batch_kernels.hpp"), nt, g))
    if not os.path.exists(path) or open(path).read() != text:
        with open(path, "w") as f:
            f.write(text)
    return path


def farrow_header(out_dir):
    """Write farrow_tables.hpp into out_dir: for every tap count N the Lagrange
    weights as polynomials in u = eps - 1/2 on [-1/2, 1/2], exact rationals
    rounded once, of degree N - 1 or economised (Chebyshev) to kFarrowDegree.
    Dropping the higher terms changes an interpolant by at most 2.5e-17 of the
    largest sample (N = 32; 9e-18 at N = 26)."""
    from fractions import Fraction as F
    degree = 15
    cheb = [[F(1)], [F(0), F(1)]]                     # T_n(x), powers of x
    for n in range(2, 32):
        t = [F(0)] + [2 * c for c in cheb[-1]]
        for i, c in enumerate(cheb[-2]):
            t[i] -= c
        cheb.append(t)

    def polynomial(N, i):
        """Weight of the tap at u = i + 1/2, powers of x = 2 u."""
        nodes = [F(2 * (k - N // 2) + 1) for k in range(N)]
        x0, p = F(2 * i + 1), [F(1)]
        for x in nodes:
            if x != x0:
                q = [F(0)] * (len(p) + 1)
                for k, c in enumerate(p):
                    q[k + 1] += c / (x0 - x)
                    q[k] -= c * x / (x0 - x)
                p = q
        for n in range(N - 1, degree, -1):            # drop T_n, highest first
            lead = p[n] / cheb[n][n]
            p = [c - lead * t for c, t in zip(p, cheb[n])]
            p.pop(n) if len(p) > n else None
        return p

    out = ["// Generated by build.py (farrow_header).", "#pragma once", "namespace lr {",
           "constexpr int kFarrowDegree = %d;" % degree, "template <int N>", "struct FarrowTable;"]
    for N in range(2, 33, 2):
        D = min(N - 1, degree)
        rows = [polynomial(N, i) for i in range(N // 2)]
        out += ["template <>", "struct FarrowTable<%d> {" % N, "  static constexpr int D = %d;" % D]
        for name, first in (("e", 0), ("o", 1)):
            js = range(first, D + 1, 2)
            out.append("  static constexpr double %s[%d][%d] = {" % (name, len(js), N // 2))
            for j in js:
                out.append("      {%s}," % ", ".join(float(r[j] * 2 ** j).hex() for r in rows))
            out.append("  };")
        out.append("};")
    text = "\n".join(out + ["}  // namespace lr", ""])
    path = os.path.join(out_dir, "farrow_tables.hpp")
    if not os.path.exists(path) or open(path).read() != text:
        with open(path, "w") as f:
            f.write(text)


def source_path(src, out_dir):
    if src.startswith("batchfwd"):
        return _fused_unit(out_dir, src)
    return os.path.join(HERE, src)


def build(verbose=True, jobs=None, target=TARGET, defines=(), out_dir=None):
    """Compile every source to an object in parallel, then link the library.
    ``defines``: extra -D options (tuning macros such as LR_PROJ_MIN_WAVES),
    for variant libraries built to ``target`` with objects in ``out_dir``."""
    out_dir = out_dir or os.path.join(HERE, "_build")
    os.makedirs(out_dir, exist_ok=True)
    farrow_header(out_dir)
    cc = hipcc()
    t0 = time.time()
    jobs = jobs or min(os.cpu_count() or 4, int(os.environ.get("MAX_JOBS", "8")), 16)
    objs = [os.path.join(out_dir, src.rsplit(".", 1)[0] + ".o") for src in SOURCES]
    # the largest units first, so the long compiles do not start last
    pending = sorted(zip(SOURCES, objs), key=lambda so: -_weight(so[0]))
    running = []
    while pending or running:
        while pending and len(running) < jobs:
            src, obj = pending.pop(0)
            cmd = [cc, *flags(), "-I" + out_dir, *["-D" + d for d in defines], "-c", source_path(src, out_dir),
                   "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            running.append((src, subprocess.Popen(cmd)))
        # wait for whichever job ends first
        done = None
        while done is None:
            for k, (src, p) in enumerate(running):
                if p.poll() is not None:
                    done = k
                    break
            else:
                time.sleep(0.2)
        src, p = running.pop(done)
        if p.returncode != 0:
            for _, q in running:
                q.wait()
            raise RuntimeError("compilation of %s failed" % src)
    tmp = target + ".tmp%d" % os.getpid()
    cmd = [cc, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp, *objs, *link_flags()]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, target)
    if verbose:
        print("built %s in %.1f s" % (target, time.time() - t0), flush=True)
    return target


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
