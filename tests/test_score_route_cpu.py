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
    if (!strcmp(a[1], "route")) {              // chain kernels on?, instances, then the hidden widths
        ls_model_config cfg{};
        cfg.d = 32;
        const int N = atoi(a[3]);
        for (char** w = a + 4; *w; ++w) cfg.hidden[cfg.n_hidden++] = atoi(*w);
        cfg.dtype = LS_FP32;
        cfg.block_tokens = 16;
        ls::ModelDims m = ls::make_dims(cfg);
        m.mfma_chains = atoi(a[2]) != 0;
        printf("%d %d\n", ls::chain_scores(m, N) ? 1 : 0, ls::scores_by_layer(m, N) ? 1 : 0);
    }
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


# (hidden widths, fused chain kernel, layer by layer); with the chain kernels off
# two layers keep the vector-ALU scorer and the rest go layer by layer
@pytest.mark.parametrize("hidden,chain,by_layer",
                         [((64,), 1, 0), ((128, 128), 1, 0), ((256, 256, 256), 1, 0), ((96,), 0, 1), ((96, 96), 0, 0),
                          ((128, 64), 0, 0), ((128, 64, 128), 0, 1), ((512, 512, 512), 0, 1)])
def test_one_route_for_sizing_and_launching(ask, hidden, chain, by_layer):
    assert ask("route", 1, 64, *hidden) == [chain, by_layer]
    assert ask("route", 0, 64, *hidden) == [0, int(len(hidden) != 2)]


# the chain kernels index the instance partials, h x N, in 32 bits; more goes to
# the scorers that index in 64
@pytest.mark.parametrize("hidden", [(64,), (256,), (256, 256), (128, 128, 128)])
def test_instances_within_the_index(ask, hidden):
    most = (1 << 32) // hidden[0]
    assert ask("route", 1, most, *hidden) == [1, 0]
    assert ask("route", 1, most + 1, *hidden) == [0, int(len(hidden) != 2)]
