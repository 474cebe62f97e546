"""Compiles a host program of tests/host against the built library (no GPU needed)."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2311_13177_amd")


def run_host(tmp_path, name, text=""):
    """Builds tests/host/<name>.cpp and runs it with `text` as input: (exit code, output)."""
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                    os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", exe, "-rdynamic", "-pthread",
                    os.path.join(PKG, "libvp.so"), "-Wl,-rpath," + PKG], check=True)
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=120)
    return r.returncode, r.stdout + r.stderr
