"""What attention calls lay out in their workspace and launch, on contexts without a device: a C++ program in the place
of the kernels' launchers sees every descriptor (tests/host_sanitize/plans_host.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_20878_amd", "csrc")
HOST_SOURCES = ["ha_rag_api.hip", "ha_rag_pool.hip", "ha_rag_load.hip", "ha_rag_attend.hip", "ha_rag_io.hip"]
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")

OK, ENOSPC = 0, -3


@pytest.fixture(scope="module")
def plans_host(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plans") / "plans_host")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17",
           "-Xarch_host", "-fsanitize=address,undefined", "-Xarch_host", "-fno-omit-frame-pointer",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
           "-x", "hip", os.path.join(ROOT, "tests", "host_sanitize", "plans_host.cpp"),
           *[os.path.join(CSRC, f) for f in HOST_SOURCES], "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def run(exe, args, text=None):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0", UBSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([exe, *args], input=text, capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    return r.stdout


def calls(exe, lines):
    """Per line: return code, workspace bytes, end of the last record, scoring waves, pieces, runs, longest run."""
    return [[int(x) for x in l.split()] for l in run(exe, ["calls"], "\n".join(lines) + "\n").splitlines()]


# Documents enough for a run to end because it may hold no more of them, next to ones long enough for runs to be long:
# the requests then have more runs than blocks / run length says.
MANY_DOCUMENTS = [
    "8 32" + " / 12 128*256 / 64 16*130" * 4,
    "16 64" + " / 32 1580*29 8*298" * 11,
    "8 64 / 16 944*106 / 256 16*176 / 16 96*134 / 16 / 16 / 16",
]


@pytest.mark.parametrize("how,codes", [("workspace", [OK, OK, OK]), ("static", [ENOSPC, ENOSPC, OK])])
def test_records_lie_in_the_workspace_when_runs_end_at_the_most_documents(plans_host, how, codes):
    seen = calls(plans_host, [how + " " + c for c in MANY_DOCUMENTS])
    assert [s[0] for s in seen] == codes
    for rc, need, end, *_ in seen:
        assert end <= (need if how == "workspace" else 32 << 20)


def test_random_calls_lay_every_record_out_once_and_inside(plans_host):
    assert "plans_host ok" in run(plans_host, ["random", "7", "2500"])
