"""The workspace header's protocol on the CPU: csrc/header_tag.h compiled for
the host, with workgroups as calls and threads. Whatever the header holds when
a call starts and whichever workgroup runs first (workgroup 0 last, say, when
another stream holds the compute units that it needs), exactly one workgroup
clears it, nobody folds into it before that, and nobody waits for a workgroup
that has not started."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_header_protocol_in_any_order(tmp_path):
    exe = str(tmp_path / "header_tag")
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-Wall", "-Werror",
                    os.path.join(HERE, "host_header_tag.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
