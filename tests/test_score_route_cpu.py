"""Which forward a scoring call takes and what it launches, on the host: a small
C++ program with the library's own header asks the rules themselves."""
import os
import subprocess

import pytest

from paper_2606_00946_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "ls_internal.h"

// argv: what to ask, then its numbers
int main(int, char** a) {
    if (!strcmp(a[1], "groups")) printf("%u\n", ls::chain_groups(atoll(a[2]), atoi(a[3]), atoi(a[4])));
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("route")
    src, exe = str(d / "route.cpp"), str(d / "route")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.check_call([build.HIPCC, "-std=c++17", "-O1", "-I", build.CSRC, "-I", build.INCLUDE, src, "-o", exe,
                           "-L", build.PKG, "-l:liblodestar.so", f"-Wl,-rpath,{build.PKG}"])
    return lambda *args: [int(v) for v in subprocess.check_output([exe, *map(str, args)], text=True).split()]


# a launch takes fewer than 2^32 threads: with 256 for 64 pairs that is 2^30
# pairs, half of what 64 threads for 32 pairs take
@pytest.mark.parametrize("per_group,threads", [(64, 256), (32, 256), (64, 128), (32, 64), (64, 64)])
@pytest.mark.parametrize("pairs", [1, 31, 64, 65, 1 << 20, (1 << 29) - 1, 1 << 29, 1 << 30, (1 << 30) + 33, 1 << 31,
                                   (1 << 40) + 1])
def test_chain_launch_fits(ask, pairs, per_group, threads):
    (groups,) = ask("groups", pairs, per_group, threads)
    whole = -(-pairs // per_group)
    assert groups * threads < 1 << 32
    assert groups == whole if whole * threads < 1 << 32 else groups >= (1 << 32) // threads - 1
