"""Rules that the device code shares with the host, compiled alone and checked
over their whole range (tests/host/).  Runs without a GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")
CXX = shutil.which("g++") or "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CXX), reason="no host compiler")
@pytest.mark.parametrize("name", sorted(f[:-4] for f in os.listdir(HERE) if f.endswith(".cpp")))
def test_host_rules(name, tmp_path):
    exe = str(tmp_path / name)
    subprocess.run([CXX, "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, name + ".cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
