"""How calls are cut into launches (csrc/schedule.hpp, host code), compiled on its own."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1511_00242_amd", "csrc")


@pytest.fixture(scope="module")
def sched(tmp_path_factory):
    d = tmp_path_factory.mktemp("schedule")
    src, so = d / "s.cpp", d / "s.so"
    src.write_text("""#include "schedule.hpp"
extern "C" {
int tail(int n, int per, int exact) { return lbfv::tail_launches(n, per, exact); }
int steps(int left, int launches, int per, int exact) { return lbfv::launch_steps(left, launches, per, exact); }
int trial(int per, int n) { return lbfv::trial_length(per, n); }
}
""")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    return C.CDLL(str(so))


def cut(sched, n, per, exact):
    out, launches = [], sched.tail(n, per, exact)
    for left in range(launches, 0, -1):
        k = sched.steps(n, left, per, exact)
        out.append(k)
        n -= k
    assert n == 0
    return out


@pytest.mark.parametrize("per", range(1, 9))
def test_calls_are_cut_into_launches(sched, per):
    for n in range(0, 300):
        even = cut(sched, n, per, 1)
        assert all(1 <= k <= per for k in even) and (len(even) - n) % 2 == 0
        assert len(even) <= -(-n // per) + 1 and (not even or max(even) - min(even) <= 1)
        plain = cut(sched, n, per, 0)
        assert len(plain) == -(-n // per) and all(k == per for k in plain[:-1])


@pytest.mark.parametrize("per", range(1, 9))
def test_trials_of_the_autotuner_run_whole_launches(sched, per):
    for asked in list(range(1, 100)) + [1000, 2 ** 31 - 1]:
        n = sched.trial(per, asked)
        assert n >= asked
        if n < 10 ** 6:
            assert n < asked + 2 * per and set(cut(sched, n, per, 1)) == {per}
