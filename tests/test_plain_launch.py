"""The rule by which a single-pass launch is plain or cooperative, run on the
CPU (tests/host/plain_launch.cpp): the launches that may be in flight together
leave a workgroup's room on the chip beside their unfinished teams, and a
stream that has not the whole chip, or cannot be asked, is launched
cooperatively with no error left behind."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
NULL, LEGACY, PER_THREAD, OWN = range(4)


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("plain") / "plain_launch")
    r = subprocess.run([HIPCC, "-std=c++17", "-O1", "--offload-host-only", "-I",
                        os.path.join(ROOT, "paper_2607_14530_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host", "plain_launch.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(G=32, cus=256, per_cu=1, stream=OWN, prio_status=0, prio=0, mask_status=0, bits=None, **env):
        base = {k: v for k, v in os.environ.items()
                if k not in ("GPU_MAX_HW_QUEUES", "HSA_CU_MASK", "ROC_GLOBAL_CU_MASK")}
        line = " ".join(map(str, (G, cus, per_cu, stream, prio_status, prio, mask_status,
                                  cus if bits is None else bits)))
        out = subprocess.run([exe], input=line, capture_output=True, text=True, env={**base, **env})
        assert out.returncode == 0, out.stderr
        plain, calls, errors = map(int, out.stdout.split())
        return bool(plain), calls, errors
    return run


def test_ordinary_streams_are_launched_plainly(rule):
    for G in (1, 2, 17, 32):
        assert rule(G=G)[0]
        for stream in (NULL, LEGACY, PER_THREAD):
            assert rule(G=G, stream=stream) == (True, 0, 0)   # (never asked: not every call knows these handles)


def test_a_masked_or_prioritised_stream_is_not(rule):
    for bits in (1, 31, 64, 255):
        assert rule(bits=bits) == (False, 2, 0)
    assert not rule(G=1, bits=64)[0]
    assert not rule(prio=-1)[0]


def test_a_masked_process_is_not(rule):
    assert not rule(HSA_CU_MASK="0:0-63")[0]
    assert not rule(ROC_GLOBAL_CU_MASK="0xffff")[0]


def test_a_stream_that_cannot_be_asked_leaves_no_error(rule):
    assert rule(prio_status=1) == (False, 1, 0)
    assert rule(mask_status=1) == (False, 2, 0)


def test_unfinished_teams_leave_room(rule):
    """One launch per hardware queue and a cooperative one: whatever of them is in flight, their
    unfinished teams (G - 1 workgroups) do not fill the chip."""
    for queues in range(1, 40):
        for G in range(1, 33):
            for slots in (64, 128, 248, 249, 256):
                if queues in (1, 4, 7, 8, 39) and G in (1, 9, 17, 32) or (queues == 4 and slots == 256):
                    plain = rule(G=G, cus=slots, GPU_MAX_HW_QUEUES=str(queues))[0]
                    assert not plain or (queues + 1) * (G - 1) < slots, (queues, G, slots)
                    if queues <= 7 and G == 1:
                        assert plain
