"""Builds _build/libhzp_dispatch.so (test infrastructure): libhzp's host code without the device's, linked with a stand-in for the HIP runtime
that records launches (recording_runtime.cpp).  Nothing of it can reach a GPU.  A scheduler, which needs streams, cannot be made with it."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
OUT = os.path.join(ROOT, "_build")


def build():
    os.makedirs(OUT, exist_ok=True)
    csrc = os.path.join(ROOT, "paper_2510_20111_amd", "csrc")
    include = ["-I" + os.path.join(ROOT, "include"), "-I" + csrc]
    kernels, lib = os.path.join(OUT, "dispatch_kernels.o"), os.path.join(OUT, "libhzp_dispatch.so")
    subprocess.run(["hipcc", "--offload-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-c"] + include +
                   [os.path.join(csrc, "kernels.hip"), "-o", kernels], check=True)
    names = subprocess.run(["nm", "--undefined-only", "--format=posix", kernels], check=True, capture_output=True, text=True).stdout.split()
    device_code = [n for n in names if n.startswith("__hip_fatbin")]        # (there is none here; only its address is taken)
    # (symbolic: a process that has PyTorch loaded has the real runtime's functions under the same names)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wall", "-pthread", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__"] + include +
                   ["-I/opt/rocm/include"] + ["-Wl,--defsym=%s=0x1000" % n for n in device_code] +
                   [os.path.join(csrc, f) for f in ("planner.cpp", "api.cpp", "scheduler.cpp")] +
                   [os.path.join(HERE, "recording_runtime.cpp"), kernels, "-o", lib], check=True)
    return lib


if __name__ == "__main__":
    print(build())
