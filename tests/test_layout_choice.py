"""The layout that cl_create chooses without a cap goes by the bytes that it would
allocate, with a cap by cl_query_workspace (tests/layout_checks.c, no GPU needed)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_layout_by_free_memory_and_by_cap(tmp_path):
    from paper_2209_08189_amd import claire
    if shutil.which("gcc") is None:
        pytest.skip("gcc not found")
    lib = os.path.dirname(os.path.abspath(claire.LIB_PATH))
    exe = str(tmp_path / "layout_checks")
    subprocess.run(["gcc", "-O1", "-Wall", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "layout_checks.c"), "-L", lib, "-lclairehip", "-Wl,-rpath," + lib,
                    "-Wl,--unresolved-symbols=ignore-in-shared-libs", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120, env=dict(os.environ, HIP_VISIBLE_DEVICES=""))
    print(r.stdout, r.stderr)
    assert r.returncode == 0, r.stderr
    assert "0 failure(s)" in r.stdout
