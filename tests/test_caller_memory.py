"""Where a caller's state lies decides how it is reached: only memory of the stream's own
GPU, at a double's alignment, is read or written by a kernel; memory of another GPU, host
and managed memory, pointers the runtime does not know and bytes off that alignment go
through one copy of the whole state, as hipMemcpyAsync takes them all.  Run against a
recording stand-in for the HIP runtime (caller_memory_main.cpp): host only, no device."""
import os
import shutil
import subprocess

import pytest

from paper_2608_14048_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
STATE = 16 * 4 * 4 * 8 * 8  # bytes of the grid's MHD state; the dust state has as many fields

pytestmark = [pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libmhd950.so not built"),
              pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")]


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("caller") / "caller_memory")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-o", exe, os.path.join(HERE, "caller_memory_main.cpp"),
                    "-ldl"], check=True)

    def run(kind, offset=0):
        r = subprocess.run([exe, B.LIB_PATH, kind, str(offset)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        out = {}
        for line in r.stdout.splitlines():
            words = line.split(" ", 3)
            out[" ".join(words[:3])] = words[3]
        return out

    return run


SETS = ["fp64 mhd set", "fp64 dust set", "fp64 batch set", "fp32 batch set", "fp64 block set", "fp32 block set",
        "fp64 closure coarse"]
GETS = ["fp64 mhd get", "fp64 dust get", "fp64 batch get", "fp32 batch get", "fp64 block get", "fp32 block get"]
KINDS = ["other", "host", "managed", "unknown"]


def _bytes(name):
    return STATE * (2 if "batch" in name else 1)


@pytest.mark.parametrize("kind,offset", [("own", 4)] + [(k, 0) for k in KINDS])
def test_fp32_states_of_one_grid_go_through_the_staging_area(calls, kind, offset):
    """Nor do the FP32 forms' kernels follow such a pointer, or one off a double's alignment."""
    got = calls(kind, offset)
    for who in ("fp32 mhd ", "fp32 dust "):
        assert got[who + "set"].startswith(f"[in {STATE}]k"), got[who + "set"]
        assert got[who + "get"] == f"k[out {STATE}]", got[who + "get"]


@pytest.mark.parametrize("kind", KINDS)
def test_foreign_memory_goes_through_one_copy(calls, kind):
    got = calls(kind)
    for name in SETS:
        assert got[name].count("[") == 1 and f"[in {_bytes(name)}]" in got[name], (name, got[name])
        assert got[name].endswith("k"), (name, got[name])  # read by a kernel after the copy
    for name in GETS:
        assert got[name].endswith(f"[out {_bytes(name)}]") and got[name].count("[") == 1, (name, got[name])


def test_own_memory_is_read_in_place(calls):
    got = calls("own")
    # (a single FP64 block leaves by a copy wherever it goes)
    assert got["fp64 block get"] == f"[out {STATE}]"
    for name in SETS:
        assert "[" not in got[name] and "k" in got[name], (name, got[name])
    for name in ("fp64 batch get", "fp32 batch get", "fp32 block get", "fp32 mhd get", "fp32 dust get"):
        assert got[name] == "k", (name, got[name])
