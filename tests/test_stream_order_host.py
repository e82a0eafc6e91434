"""Which work of the library is still queued when a call returns, and which
buffers that work uses: the host code against a model of a HIP stream
(tests/emu/stream_model.cpp).  No GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_14697_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("model") / "stream_model")
    srcs = [os.path.join(ROOT, "tests", "emu", "stream_model.cpp")] + [
        os.path.join(CSRC, f) for f in ("sv_api.cpp", "sv_batch.cpp", "sv_exec.cpp", "sv_gates.cpp", "sv_plan.cpp",
                                        "sv_passplan.cpp")]
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}"] + srcs + ["-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.mark.parametrize("scenario", ["program", "batcher", "staging", "launches"])
def test_queued_work(model, scenario):
    r = subprocess.run([model, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
