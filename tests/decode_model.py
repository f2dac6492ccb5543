"""Host build of the decode kernel's headers of integer arithmetic, with the model of its workgroups in decode_model.cpp."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build_model(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("model") / "model.so")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--cuda-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2510_05373_amd", "csrc"),
                    os.path.join(ROOT, "tests", "decode_model.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)
