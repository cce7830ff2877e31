"""What the host runtime promises about its calls, without a GPU: mhd_runtime.cpp compiled against an
emulation of the HIP calls on host memory (tests/emu/runtime_emu.cpp), which records them."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
EMU = os.path.join(HERE, "emu")
CSRC = os.path.join(os.path.dirname(HERE), "paper_2211_09370_amd", "csrc")


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("emu") / "runtime_emu")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-w", "-I" + EMU, os.path.join(EMU, "runtime_emu.cpp"),
                    os.path.join(CSRC, "mhd_resident_plan.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("scenario", [
    "step",          # the first steps after new markers or parameters wait for nothing and allocate nothing
    "step_noalloc",  # nor do the allocation-free ones
    "other_gpu",     # a call held up on one GPU does not hold up steps on another
    "long_call",     # nor, for more than a bounded number of steps, on the same one
    "odd_counts",    # the control block is read to an address it can stand at
    "copy_error",    # a failing call in the middle of a field copy leaves no copy under way
    "stall",         # a stalled step is not reported as an unstable state
    "given_up",      # a roll call given up sends the next steps to the launch sequence
    "batch_forms",   # tile forms of a batch share a launch where that is the faster way
    "device",        # calls made while another GPU is the current one
])
def test_scenario(emu, scenario):
    r = subprocess.run([emu, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr)
