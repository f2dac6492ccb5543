"""Builds libkvlinc.so (the C-ABI library), libkvlinc_probe.so (the benchmark's read-only probe kernel) and libkvlinc_nolooks.so (the
library with a decode in which every wait runs out at once, for the tests) in-tree with hipcc for gfx950."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libkvlinc.so")
PROBE_PATH = os.path.join(HERE, "libkvlinc_probe.so")
NOLOOKS_PATH = os.path.join(HERE, "libkvlinc_nolooks.so")

COMMON = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first 14 words of a kernel's arguments come with the launch, in scalar registers
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]
# object: source and extra flags; the append path holds the bit-exact contracts, no contraction of a*b+c there
OBJECTS = {
    "kvlinc_api": ("kvlinc_api.hip", []),
    "kvlinc_append": ("kvlinc_append.hip", ["-ffp-contract=off"]),
    "kvlinc_decode": ("kvlinc_decode.hip", []),
    "kvlinc_decode_nolooks": ("kvlinc_decode.hip", ["-DKVLINC_LOOKS=0"]),
}
LIBRARIES = {
    LIB_PATH: ["kvlinc_api", "kvlinc_append", "kvlinc_decode"],
    NOLOOKS_PATH: ["kvlinc_api", "kvlinc_append", "kvlinc_decode_nolooks"],
}
PROBE_SOURCE = "kvlinc_readprobe.hip"


def build(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    obj_path = lambda name: os.path.join(CSRC, name + ".o")
    procs = []
    for name, (src, extra) in OBJECTS.items():
        cmd = [hipcc] + COMMON + extra + ["-c", os.path.join(CSRC, src), "-o", obj_path(name)]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((name, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    probe_cmd = [hipcc] + COMMON + ["-shared", os.path.join(CSRC, PROBE_SOURCE), "-o", PROBE_PATH]
    procs.append((PROBE_SOURCE, subprocess.Popen(probe_cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
        if verbose and out.strip():
            print(out)
    for path, names in LIBRARIES.items():
        r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", path] + [obj_path(n) for n in names],
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n" + r.stdout)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
