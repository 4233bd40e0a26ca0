"""Build libhidet_mi355x.so: every (tile configuration, input type) instance object plus the C ABI; and _host_calls.so, the
extension module through which the binding reaches it.

    python -m paper_2210_09603_amd.build            # incremental
    python -m paper_2210_09603_amd.build --force    # recompile everything
    HIDET_CONFIGS=0,3,14 python -m paper_2210_09603_amd.build   # development subset of the schedule space

hipcc cross-compiles for gfx950 without a GPU.  Objects live in _build/ (not committed); the shared
library is written next to this file so that it travels with the source tree.
"""
import concurrent.futures
import hashlib
import os
import re
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libhidet_mi355x.so")
HOST_CALLS = os.path.join(HERE, "_host_calls.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# (loops begin on a line of the instruction cache: a main loop that an unrelated change had moved across one ran 3 % longer, 14
# images of 512x10x10, 5x5, on the 128x64 K-splitting tile 99.6 and 102.5 us; over 1019 random GEMMs and convolutions 0.3 %
# shorter together, between 4 % shorter and 5 % longer; longer as a kind only the packed weights on the 32x32 tile of a K tile
# of 64 in registers, 20 calls by 1.2 %)
FLAGS = ["--offload-arch=gfx950", "-O3", "-falign-loops=64", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def schedule_space():
    """[(index, is_f32)] parsed from configs.def."""
    out = []
    with open(os.path.join(CSRC, "configs.def")) as fh:
        for line in fh:
            m = re.match(r"\s*X(16|32)\((\d+),", line)
            if m:
                out.append((int(m.group(2)), m.group(1) == "32"))
    return out


def _sources_digest():
    h = hashlib.sha256()
    for name in sorted(n for n in os.listdir(CSRC) if not n.endswith(".cpp")):
        with open(os.path.join(CSRC, name), "rb") as fh:
            h.update(name.encode())
            h.update(fh.read())
    with open(os.path.join(HERE, "..", "include", "hidet_mi355x.h"), "rb") as fh:
        h.update(fh.read())
    h.update(" ".join(FLAGS).encode())
    return h.hexdigest()


def _host_commands(obj, out):
    """The g++ commands that compile and link the extension module, which reads torch tensors (against the libraries that
    `import torch` has loaded before it)."""
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    from paper_2210_09603_amd.binding import built_for

    cxx = os.environ.get("CXX", "g++")
    flags = ["-O2", "-std=c++17", "-fPIC", "-Wall", "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
             '-DHIDET_BUILT_FOR="%s"' % built_for(), "-I" + sysconfig.get_paths()["include"]] + ["-isystem" + d for d in include_paths()]
    libraries = ["-L" + d for d in library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    return ([cxx] + flags + ["-c", os.path.join(CSRC, "host_calls.cpp"), "-o", obj], [cxx, "-shared", "-fPIC", "-o", out, obj] + libraries)


def _host_digest():
    """Of the module's sources, of what it is compiled against and of how."""
    h = hashlib.sha256()
    for path in (os.path.join(CSRC, "host_calls.cpp"), os.path.join(HERE, "..", "include", "hidet_mi355x.h")):
        with open(path, "rb") as fh:
            h.update(fh.read())
    h.update(repr(_host_commands("", "")).encode())
    return h.hexdigest()


def _up_to_date(stamp, digest):
    return os.path.exists(stamp) and open(stamp).read() == digest


def _write(path, text):
    with open(path, "w") as fh:
        fh.write(text)


def _build_host_calls(force):
    obj, stamp = os.path.join(BUILD, "host_calls.o"), os.path.join(BUILD, "host_digest.txt")
    digest = _host_digest()
    if not force and os.path.exists(HOST_CALLS) and _up_to_date(stamp, digest):
        return
    tmp = HOST_CALLS + ".tmp.%d" % os.getpid()
    for cmd in _host_commands(obj, tmp):
        if subprocess.run(cmd).returncode != 0:
            raise RuntimeError("%s failed on %s (%s is built)" % (cmd[0], os.path.basename(HOST_CALLS), os.path.basename(LIB)))
    os.replace(tmp, HOST_CALLS)
    _write(stamp, digest)


def _compile(args):
    src, obj, defines = args
    cmd = [HIPCC] + FLAGS + defines + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass does not know the packed-fp32 feature and says so on every file; drop that line
    log = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    return r.returncode, obj, log


def build(force=False, jobs=None, verbose=True):
    os.makedirs(BUILD, exist_ok=True)
    digest = _sources_digest()
    subset = os.environ.get("HIDET_CONFIGS")
    chosen = None if not subset else {int(x) for x in subset.split(",") if x.strip()}
    stamp = os.path.join(BUILD, "digest.txt")
    if force or not _up_to_date(stamp, digest):
        for f in os.listdir(BUILD):
            if f.endswith(".o") and f != "host_calls.o":
                os.remove(os.path.join(BUILD, f))
    tasks, objs = [], []
    for idx, is_f32 in schedule_space():
        if chosen is not None and idx not in chosen:
            continue
        for t in ([0] if is_f32 else [1, 2]):
            obj = os.path.join(BUILD, "inst_%d_%d.o" % (idx, t))
            objs.append(obj)
            if not os.path.exists(obj):
                tasks.append((os.path.join(CSRC, "instances.hip"), obj, ["-DHIDET_TU=%d" % idx, "-DHIDET_TYPE=%d" % t]))
    for name in ("api", "conv_patch", "probe", "reduce"):
        obj = os.path.join(BUILD, name + ".o")
        objs.append(obj)
        if not os.path.exists(obj):
            tasks.append((os.path.join(CSRC, name + ".hip"), obj, []))
    jobs = jobs or min(8, os.cpu_count() or 1)
    failed = False
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as ex:
        for rc, obj, log in ex.map(_compile, tasks):
            if verbose:
                print("[build] %s rc=%d" % (os.path.basename(obj), rc), flush=True)
            if log.strip() and (rc != 0 or verbose):
                print(log)
            if rc != 0:
                failed = True
                if os.path.exists(obj):
                    os.remove(obj)
    if failed:
        raise RuntimeError("hipcc failed")
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, check=True)
    os.replace(tmp, LIB)
    _write(stamp, digest)
    _build_host_calls(force)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
