"""Host parts of the library that need no GPU, compiled on their own: the
device work lists around a failed allocation, and the staged read-back around
threads or copies that fail."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name", ["item_list_test", "widen_test"])
def test_host_part(name, tmp_path):
    exe = tmp_path / name
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread",
                    "-I", os.path.join(ROOT, "paper_1310_6143_amd", "csrc"),
                    os.path.join(ROOT, "tests", "helpers", name + ".cpp"), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr
