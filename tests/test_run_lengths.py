"""The rule that decides how many iterations of a solve or batch are queued between two
looks at its flags, and whether such a run ends with the true-residual update
(paper_1701_00426_amd/csrc/runs.hpp), compiled for the host.  No GPU is used.

A caller's short runs (poll_every below 8) leave the update to the host: five launches
after every one to seven iterations cost more than they save."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1701_00426_amd", "csrc")
SRC = """
#include "runs.hpp"
extern "C" {
int queued(int poll, int mixed, unsigned long long n) { return stg::queued_update(poll, mixed, n); }
int run(int poll, int upd, int mixed, unsigned vh, int live) {
    return stg::run_iterations(poll, upd, mixed, vh, live);
}
int bqueued(int run, int small) { return stg::batch_queued_update(run, small); }
int brun(int poll, int small) { return stg::batch_run(poll, small); }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("runs")
    (d / "r.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "r.cpp"),
                    "-o", str(d / "r.so")], check=True)
    lib = ctypes.CDLL(str(d / "r.so"))
    lib.queued.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_ulonglong]
    return lib


@pytest.mark.parametrize("poll,small,large", [(1, 0, 0), (2, 0, 0), (7, 0, 0), (8, 1, 0),
                                              (64, 1, 0), (0, 1, 0)])
def test_update_at_the_end_of_a_run(rule, poll, small, large):
    assert rule.queued(poll, 1, 128) == small
    assert rule.queued(poll, 1, 1 << 17) == small
    assert rule.queued(poll, 1, (1 << 17) + 1) == large
    assert rule.queued(poll, 0, 128) == 0  # FP64: no update until the end
    run = rule.brun(poll, 1)
    assert rule.bqueued(run, 1) == small
    assert rule.bqueued(rule.brun(poll, 0), 0) == 0
    assert run == (poll if poll else 8)


@pytest.mark.parametrize("vh,live", [(128, 1), (2048, 4), (32768, 3), (32768, 12), (524288, 1),
                                     (524288, 32)])
@pytest.mark.parametrize("mixed", [0, 1])
def test_run_lengths(rule, mixed, vh, live):
    for poll in (1, 3, 100):
        assert rule.run(poll, rule.queued(poll, mixed, vh * live), mixed, vh, live) == poll
    n = rule.run(0, rule.queued(0, mixed, vh * live), mixed, vh, live)
    if mixed and vh * live <= 1 << 17:
        assert n == 12
    else:
        assert (2 if live > 1 else 8) <= n <= (8 if mixed else 16)
