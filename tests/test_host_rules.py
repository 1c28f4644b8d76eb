"""Launch rules of the library's host code (tests/host_rules_main.cpp), compiled for the CPU from the library's headers."""
import os
import subprocess

from paper_2411_08461_amd import build as hipbuild

HERE = os.path.dirname(os.path.abspath(__file__))


def test_host_rules(tmp_path):
    obj, out = tmp_path / "main.o", tmp_path / "main"
    flags = [f for f in hipbuild.CFLAGS if not f.startswith("--offload-arch") and f != "-O3"]
    subprocess.run([hipbuild.HIPCC, "-x", "hip", "--offload-host-only", "-O1", *flags, "-c",
                    os.path.join(HERE, "host_rules_main.cpp"), "-o", str(obj)], check=True, capture_output=True)
    subprocess.run(["g++", str(obj), "-o", str(out)], check=True, capture_output=True)
    r = subprocess.run([str(out)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stderr
