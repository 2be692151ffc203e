"""Kernels whose lanes exchange data, built from their source files for the CPU and run lane by
lane (tests/cpu_wave/hip/hip_runtime.h): missing waits, entries nobody wrote and indices out
of range show there every time, and cannot fault a GPU."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2606_15622_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.fixture(scope="module")
def build(tmp_path_factory):
    """build(name): tests/cpu_wave/<name>.cpp as a program, once per module.  The sources are taken
    without their inline assembly (empty statements that only bind the device compiler)."""
    out, done = tmp_path_factory.mktemp("cpu_wave"), {}
    for f in os.listdir(CSRC):
        with open(os.path.join(CSRC, f)) as src:
            (out / f).write_text(re.sub(r'__asm__ volatile\("".*?\);', ";", src.read(), flags=re.S))

    def make(name):
        if name not in done:
            done[name] = str(out / name)
            subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O2", "-ftrapv", "-ffp-contract=off", "-w",
                            "--rtlib=compiler-rt", "--unwindlib=libgcc",
                            "-I", os.path.join(HERE, "cpu_wave"), "-I", str(out), "-I", CSRC,
                            os.path.join(HERE, "cpu_wave", name + ".cpp"), "-o", done[name]], check=True)
        return done[name]
    return make


def run(program, *args):
    r = subprocess.run([program, *map(str, args)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr)


# offsets as the contract has them; some decreasing; some beyond the particles; some negative; some
# at the ends of the 32-bit range (signed overflows trap; so do those of invalid keys)
@pytest.mark.parametrize("kind", [0, 1, 2, 3, 4])
def test_source_indices_of_the_resort(build, kind):
    run(build("rebin_count"), kind)


def test_chain_of_the_lite_training(build):
    run(build("lite_train"))


def test_training_of_the_network(build):
    run(build("nn_train"))
