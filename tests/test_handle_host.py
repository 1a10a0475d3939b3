"""The handle's states on the CPU (handle_host.cpp): every device allocation
of every setup call made to fail in turn, failed factorisations, variants
chosen at any time and during a capture; a kernel must find its buffers, of
the present factorisation, or the call must refuse."""

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_handle_states(tmp_path):
    exe = str(tmp_path / "handle_host")
    subprocess.check_call(["g++", "-std=c++17", "-g", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", "-w", "-x", "c++", os.path.join(HERE, "handle_host.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
