"""The mailbox words that the workgroups of a batch of SOR iterations exchange
(sor_mail.h), in a model whose stores land late and in any order: every value
arrives, none twice, also after a launch that was abandoned.  Slots that their
reader empties lose values there."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1710_09421_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("sor_mail") / "model")
    cxx = shutil.which("g++") or shutil.which("c++")
    assert cxx, "no host compiler"
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, os.path.join(HERE, "sor_mail_model.cpp"),
                    "-o", exe], check=True)
    return lambda *a: subprocess.run([exe] + [str(v) for v in a], capture_output=True, text=True,
                                     timeout=120)


@pytest.mark.parametrize("gy,gz", [(1, 1), (1, 2), (2, 2), (3, 2), (4, 4)])
@pytest.mark.parametrize("seed", range(4))
def test_every_value_arrives(model, gy, gz, seed):
    r = model("words", gy, gz, 60, seed)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout


def test_slots_with_two_writers_lose_values(model):
    """What the words replace: the reader's emptying store lands after the
    next value."""
    lost = [model("emptied", 4, 4, 60, seed) for seed in range(4)]
    assert all(r.returncode == 1 and "lost" in r.stdout for r in lost), [r.stdout for r in lost]
