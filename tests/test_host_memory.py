"""A host allocation that fails inside the library ends the call with
SC_ENOMEM: tests/c/host_memory_check.cpp (built by __graft_entry__.build() into
paper_2311_14941_amd/_build/) fails one allocation of a call after the other
until the call succeeds.  Loading a mechanism on
the CPU; a plan and its mapping, with nothing left on the device, on the GPU."""
import os
import subprocess

import pytest

from synth.mechgen import standard_mechanism

EXE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_14941_amd", "_build",
                   "host_memory_check")


def check(tmp_path, what):
    assert os.path.exists(EXE), "host_memory_check is built by __graft_entry__.build()"
    path = tmp_path / "mech.txt"
    path.write_text(standard_mechanism("h2_9").to_text())
    r = subprocess.run([EXE, str(path), what], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-2000:])
    print(r.stdout)
    words = r.stdout.split()
    return {k: int(v) for k, v in zip(words, words[1:]) if v.lstrip("-").isdigit()}


def test_mechanism(tmp_path):
    assert check(tmp_path, "load")["load"] > 50


@pytest.mark.gpu
def test_plan_and_mapping(tmp_path):
    n = check(tmp_path, "plan")
    assert n["plan"] > 20 and n["mapping"] >= 1
    assert n["kept"] <= 8 << 20, n
