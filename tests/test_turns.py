"""The books that let one owner at a time launch kernels whose blocks wait for
each other: who is refused, until when, and who counts as one owner (CPU)."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1512_03126_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_turns_and_owners(tmp_path):
    exe = str(tmp_path / "turns")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-fsanitize=address,undefined", "-I", CSRC,
                    os.path.join(HERE, "helpers", "turn_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_no_stream_or_event_is_asked_whose_turn_it_is():
    """A launch in turn looks at its own books and at a word of host memory:
    the stream of the last launch may be gone, or be captured by its owner."""
    src = open(os.path.join(CSRC, "rdos_api.cpp")).read()
    assert "hipEventQuery" not in src and "hipEventSynchronize" not in src


def test_every_launch_that_waits_for_its_blocks_takes_a_turn():
    """Each kernel launched cooperatively says when it has ended, and its
    launcher is called with a turn's number, or out of turn where its blocks
    do not wait for each other or a graph will launch it."""
    launchers = []
    for f in sorted(os.listdir(CSRC)):
        if not f.endswith(".hip"):
            continue
        src = open(os.path.join(CSRC, f)).read()
        for at in (m.start() for m in re.finditer("hipLaunchCooperativeKernel", src)):
            launchers.append(re.findall(r"\nhipError_t (\w+)\(([^{]*)\)\n\{", src[:at])[-1])
        if launchers and launchers[-1][0] in src:
            assert "end_block(" in src, f
    assert sorted(name for name, _ in launchers) == ["launch_persist", "launch_resident"]
    assert all("LaunchEnd" in args for _, args in launchers)
    calls = [f for f in ("rdos_api.cpp", "rdos_engine.cpp")
             if re.search(r"\blaunch_(persist|resident)\(", open(os.path.join(CSRC, f)).read())]
    assert calls == ["rdos_api.cpp"]
