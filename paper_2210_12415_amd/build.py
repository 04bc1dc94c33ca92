"""Builds libalt.so (HIP, gfx950 only) and the binding's call module (C) next to this file.

    python -m paper_2210_12415_amd.build [-j N] [--force]

Every .hip/.cpp under csrc/ is one translation unit; objects go to
csrc/_build/ and are rebuilt when the source or any header is newer."""
import argparse
import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libalt.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Wall", "-Wno-unused-function", "-Wno-unused-command-line-argument",
         # packed-fp32 VALU forms are switched off for all device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def _newest_header():
    hs = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    return max(os.path.getmtime(h) for h in hs)


def _compile(src, force, hdr_time):
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    if (not force and os.path.exists(obj) and os.path.getmtime(obj) >= os.path.getmtime(src)
            and os.path.getmtime(obj) >= hdr_time):
        return obj, False, ""
    cmd = [HIPCC] + FLAGS + ["-x", "hip", "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), r.stderr[-6000:]))
    warn = "\n".join(l for l in r.stderr.splitlines()
                     if "packed-fp32-ops" not in l and l.strip())
    return obj, True, warn


def build_calls(force=False, verbose=True):
    """The marshalling of repeated calls (native/altcall.c), which nothing needs: without Python's headers or a C compiler that takes it
    there is none, and the binding goes through ctypes alone.  Returns the module's path or None."""
    src = os.path.join(HERE, "native", "altcall.c")
    out = os.path.join(HERE, "_altcall" + sysconfig.get_config_var("EXT_SUFFIX"))
    if not force and os.path.exists(out) and os.path.getmtime(out) >= os.path.getmtime(src):
        return out
    include = sysconfig.get_paths()["include"]
    tmp = out + ".tmp%d" % os.getpid()
    try:
        if not os.path.exists(os.path.join(include, "Python.h")):
            raise RuntimeError("no Python.h")
        r = subprocess.run([os.environ.get("CC", "gcc"), "-O2", "-shared", "-fPIC", "-Wall", "-I" + include, src, "-o", tmp], capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("compile failed: %s\n%s" % (src, r.stderr[-4000:]))
    except (OSError, RuntimeError) as e:
        for stale in (tmp, out):              # (an older module would be loaded still)
            if os.path.exists(stale):
                os.remove(stale)
        if verbose:
            print("[build] calls go through ctypes: %s" % e, flush=True)
        return None
    os.replace(tmp, out)
    if verbose:
        print("[build] %s" % os.path.basename(out), flush=True)
    return out


def build(jobs=8, force=False, verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    build_calls(force, verbose)
    hdr = _newest_header()
    objs, rebuilt = [], False
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as ex:
        futs = {ex.submit(_compile, s, force, hdr): s for s in sources()}
        for f in concurrent.futures.as_completed(futs):
            obj, did, warn = f.result()
            objs.append(obj)
            rebuilt |= did
            if verbose and did:
                print("[build] %s" % os.path.basename(futs[f]), flush=True)
            if verbose and warn and "warning" in warn:
                print(warn, flush=True)
    if rebuilt or not os.path.exists(LIB):
        tmp = LIB + ".tmp%d" % os.getpid()
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + sorted(objs)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n" + r.stderr[-4000:])
        os.replace(tmp, LIB)
        if verbose:
            print("[build] linked %s" % LIB, flush=True)
    return LIB


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    ap.add_argument("-j", type=int, default=8)
    ap.add_argument("--force", action="store_true")
    a = ap.parse_args()
    build(a.j, a.force)
