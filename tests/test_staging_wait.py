"""The host's wait for a staging slot that a kernel reads (csrc/staging.h), built with the host compiler: it lasts as long as the
kernel's stream is busy, and ends in an error when that stream has failed or has run dry without the kernel's flags."""
import ctypes as C
import os
import shutil
import subprocess
import threading
import time

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
BUSY, DRAINED, FAILED = 0, 1, 2
SEQ, N = 7, 5


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    lib = tmp_path_factory.mktemp("staging") / "staging_wait.so"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", os.path.join(HERE, "staging_wait_shim.cpp"), "-o", str(lib)], check=True)
    return C.CDLL(str(lib))


def wait(shim, flags, answers, set_after=None, grace_ms=50):
    """Waits in a thread of its own; answers(k) is the stream's state when asked the k-th time.  Returns (result, questions)."""
    asked = []

    def ask():
        asked.append(time.monotonic())
        return answers(len(asked) - 1)

    cb = C.CFUNCTYPE(C.c_int)(ask)
    result = []
    t = threading.Thread(target=lambda: result.append(shim.wait_flags(flags.ctypes.data_as(C.c_void_p), N, SEQ, grace_ms, cb)), daemon=True)
    t.start()
    if set_after is not None:
        time.sleep(set_after)
        assert not result, "the wait ended before the flags were set"
        flags[:] = SEQ
    t.join(10)
    assert result, "the wait did not end"
    return result[0], len(asked)


def test_flags_that_are_set_need_no_question(shim):
    assert wait(shim, np.full(N, SEQ, np.uint32), lambda k: FAILED) == (1, 0)


def test_a_busy_stream_is_waited_for(shim):
    got, asked = wait(shim, np.full(N, SEQ - 1, np.uint32), lambda k: BUSY, set_after=0.3)
    assert got == 1 and asked >= 2


@pytest.mark.parametrize("missing", [0, N - 1])
def test_a_failed_stream_ends_the_wait(shim, missing):
    flags = np.full(N, SEQ, np.uint32)
    flags[missing] = SEQ - 1
    assert wait(shim, flags, lambda k: FAILED if k >= 3 else BUSY) == (0, 4)


def test_a_stream_that_ran_dry_without_the_flags_ends_the_wait(shim):
    t0 = time.monotonic()
    got, _ = wait(shim, np.zeros(N, np.uint32), lambda k: DRAINED, grace_ms=100)
    assert got == 0 and time.monotonic() - t0 >= 0.1


def test_flags_set_within_the_grace_count(shim):
    assert wait(shim, np.zeros(N, np.uint32), lambda k: DRAINED, set_after=0.1, grace_ms=5000)[0] == 1


def test_the_grace_starts_anew_when_the_stream_is_busy_again(shim):
    assert wait(shim, np.zeros(N, np.uint32), lambda k: BUSY if k % 4 == 3 else DRAINED, set_after=0.4, grace_ms=60)[0] == 1
