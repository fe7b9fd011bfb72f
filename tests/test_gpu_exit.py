"""A simulation that outlives the program's main function."""
import os
import shutil
import subprocess

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")
def test_simulation_closed_at_exit(tmp_path):
    """Closed by a handler that was registered before the library's first
    call, so that it runs after the library's own objects have ended."""
    import paper_1512_03126_amd as P

    print("[gpu-case] exit: a C program closes its simulation in an exit handler", flush=True)
    exe = str(tmp_path / "exit_driver")
    subprocess.run(["gcc", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "helpers", "exit_driver.c"), P.LIB_PATH, "-o", exe,
                    f"-Wl,-rpath,{os.path.dirname(P.LIB_PATH)}"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.endswith("closed\n"), (r.returncode, r.stdout, r.stderr)
