"""The memory pool's rules (csrc/pool.hip) on the CPU, with the driver's
calls and the clock stood in for (pool_host.cpp), and the public call that
empties it."""

import os
import subprocess

from paper_2508_04917_amd import ddilu

HERE = os.path.dirname(os.path.abspath(__file__))


def test_pool_rules(tmp_path):
    exe = str(tmp_path / "pool_host")
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w", "-x", "c++",
                           os.path.join(HERE, "pool_host.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_public_call_reaches_the_pool(monkeypatch):
    class Lib:
        calls = []

        def dd_destroy(self, p):
            self.calls.append(p)

    monkeypatch.setattr(ddilu, "lib", lambda: Lib())
    ddilu.dd_destroy(None)
    h = ddilu.Handle(17)
    ddilu.dd_destroy(h)
    ddilu.dd_destroy(h)  # already closed
    assert Lib.calls[0] is None and [c.value for c in Lib.calls[1:]] == [17]
