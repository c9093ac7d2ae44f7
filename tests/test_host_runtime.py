"""Host code of the library against a HIP runtime of two devices in tests/host: what no test
on one GPU reaches (streams of another device than the current one, resources that run out)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_2002_09217_amd", "csrc")


@pytest.fixture(scope="session")
def program(tmp_path_factory):
    """Builds tests/host/<name>.cpp, with library sources, once; returns its path."""
    built = {}

    def build(name, *sources):
        if name not in built:
            exe = str(tmp_path_factory.mktemp("host") / name)
            subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", HOST, "-I", CSRC,
                            "-I", os.path.join(ROOT, "include"), "-x", "c++", os.path.join(HOST, name + ".cpp"),
                            *(os.path.join(CSRC, s) for s in sources), "-o", exe], check=True)
            built[name] = exe
        return built[name]
    return build


def run(*cmd, **kw):
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=120, **kw)
    assert r.returncode == 0, f"{cmd[1:]}: {r.returncode} {r.stdout}{r.stderr}"


@pytest.mark.parametrize("what", ["device", "events", "locked", "on_device", "small"])
def test_read_back(program, what):
    run(program("readback"), what)


def test_read_back_on_one_core(program):
    run(program("readback"), "one_core", preexec_fn=lambda: os.sched_setaffinity(0, sorted(os.sched_getaffinity(0))[:1]))


@pytest.mark.parametrize("what", ["device", "shortage", "memory"])
def test_batch(program, what):
    run(program("batch", "pond_batch.hip"), what)
