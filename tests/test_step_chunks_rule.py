"""How swe_step cuts a call into graphs (csrc/swe_internal.h), compiled on the
host: a call that the short graph serves does not build the long one for a
single replay, whatever graph another step mode left behind."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2307_16758_amd", "csrc")

MAIN = """
#include <cstdio>
#include <cstdlib>
#include "swe_internal.h"
int main(int, char **v)
{
    long long at = atoll(v[1]);
    int n = atoi(v[2]), left = n;
    while (left > 0) {
        const int k = swe::steps_next(at, left, n, 0.25, atof(v[3]) >= 0.0, atof(v[3]));
        printf("%d ", k);
        at += k;
        left -= k;
    }
}
"""


@pytest.fixture(scope="module")
def chunks(tmp_path_factory):
    d = tmp_path_factory.mktemp("chunks")
    (d / "m.cpp").write_text(MAIN)
    exe = str(d / "m")
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(d / "m.cpp"), "-o", exe])
    return lambda at, n, long_dt: [int(x) for x in subprocess.check_output([exe, str(at), str(n), str(long_dt)]).split()]


NONE, CFL, OWN, OTHER = -1, 0, 0.25, 0.5


@pytest.mark.parametrize("at", [0, 1, 5, 6, 47])
@pytest.mark.parametrize("n", [1, 5, 6, 23, 24, 30, 47, 48, 53, 200])
@pytest.mark.parametrize("long_dt", [NONE, CFL, OWN, OTHER])
def test_pieces(chunks, at, n, long_dt):
    """Calls of n steps of 0.25 s, with a long graph of long_dt at hand."""
    got = chunks(at, n, long_dt)
    assert sum(got) == n and set(got) <= {1, 6, 24}
    for k in got:
        assert k == 1 or at % 6 == 0
        at += k
    if long_dt != OWN and n < 48:
        assert 24 not in got            # not built for one replay
    if long_dt == OWN and n >= 24 + 5:
        assert 24 in got                # used where it is there
