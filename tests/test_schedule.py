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
int cut(int n, int per, int exact, int no_twos, int *out) {
    lbfv::Cut c(n, per, exact, no_twos);
    int count = 0;
    while (const int k = c.next()) out[count++] = k;
    return count;
}
int trial(int per, int n) { return lbfv::trial_length(per, n); }
}
""")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    return C.CDLL(str(so))


def cut(sched, n, per, exact, no_twos=0):
    out = (C.c_int * (n + 8))()
    out = list(out[:sched.cut(n, per, exact, no_twos, out)])
    assert sum(out) == n
    return out


@pytest.mark.parametrize("per", range(1, 9))
def test_calls_are_cut_into_launches(sched, per):
    for n in range(0, 300):
        even = cut(sched, n, per, 1)
        assert all(1 <= k <= per for k in even) and (len(even) - n) % 2 == 0
        assert len(even) <= -(-n // per) + 1 and (not even or max(even) - min(even) <= 1)
        mixed = cut(sched, n, per, 1, 1)
        assert all(1 <= k <= per for k in mixed) and (len(mixed) - n) % 2 == 0 and len(mixed) <= len(even)
        assert mixed == even if per < 3 else 2 not in mixed
        plain = cut(sched, n, per, 0)
        assert len(plain) == -(-n // per) and all(k == per for k in plain[:-1])


@pytest.mark.parametrize("per", range(1, 9))
def test_trials_of_the_autotuner_run_whole_launches(sched, per):
    for asked in list(range(1, 100)) + [1000, 2 ** 31 - 1]:
        n = sched.trial(per, asked)
        assert n >= asked
        if n < 10 ** 6:
            assert n < asked + 2 * per and set(cut(sched, n, per, 1)) == {per}
