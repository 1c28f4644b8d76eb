"""Device buffers and the block cache on the CPU: tests/block_cache_main.cpp compiles the library's own host code
against a device runtime of fixed capacity that it answers itself (no GPU, no HIP library)."""
import os
import subprocess

import pytest

from paper_2411_08461_amd import build as hipbuild

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("block_cache")
    obj, out = d / "main.o", d / "main"
    flags = [f for f in hipbuild.CFLAGS if not f.startswith("--offload-arch") and f != "-O3"]
    subprocess.run([hipbuild.HIPCC, "-x", "hip", "--offload-host-only", "-O1", *flags, "-c",
                    os.path.join(HERE, "block_cache_main.cpp"), "-o", str(obj)], check=True, capture_output=True)
    subprocess.run(["g++", str(obj), "-o", str(out), "-pthread"], check=True, capture_output=True)
    return str(out)


@pytest.mark.parametrize("scenario", ["out_of_memory", "full_cache", "error_left_behind"])
def test_block_cache(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stderr
