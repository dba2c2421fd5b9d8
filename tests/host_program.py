"""Builds and runs a small host program against the library's internal headers,
for rules that are decided on the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2204_07816_amd")


def run(tmp_path, source):
    """(exit status, output) of `source` compiled with nqs_internal.h on its path."""
    lib = os.path.join(PKG, "libnqs.so")
    assert os.path.exists(lib), "libnqs.so is not built: run __graft_entry__.build()"
    src, exe = tmp_path / "prog.hip", tmp_path / "prog"
    src.write_text(source)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    r = subprocess.run([hipcc, "--offload-host-only", "-std=c++17", "-O1", "-I",
                        os.path.join(PKG, "csrc"), str(src), "-o", str(exe), "-L" + PKG,
                        "-l:libnqs.so", "-Wl,-rpath," + PKG], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    return r.returncode, r.stdout
