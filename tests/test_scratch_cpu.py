"""Scratch sizes of the data path's calls, on the host: a small C++ program with
the library's own layout header prints where every array of a call's scratch
begins and how many bytes the call allocates."""
import os
import subprocess

import pytest

from paper_2606_00946_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2606_00946_amd")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "ls_scratch.h"

// argv: kind, then its numbers.  One line: bytes allocated, then each array's offset.
int main(int argc, char** argv) {
    std::vector<long long> a;
    for (int i = 2; i < argc; ++i) a.push_back(atoll(argv[i]));
    ls::WsCarve size;
    char* base = reinterpret_cast<char*>(1 << 20);
    ls::WsCarve w{base};
    std::vector<const void*> at;
    if (argv[1][0] == 'p') {
        auto carve = [&](ls::WsCarve& c) {
            return ls::carve_push(c, (int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)a[4], a[5], a[6]);
        };
        (void)carve(size);
        w.cap = size.off;
        const ls::PushScratch s = carve(w);
        at = {s.codes, s.cx, s.cy, s.ax, s.ay, s.forward, s.cemb, s.admitted, s.admission};
    } else {
        auto carve = [&](ls::WsCarve& c) { return ls::carve_train(c, (int)a[0], (int)a[1], (int)a[2], (int)a[3], a[4]); };
        (void)carve(size);
        w.cap = size.off;
        const ls::TrainScratch s = carve(w);
        at = {s.codes, s.bx, s.by, s.step_loss, s.loss_sum, s.update};
    }
    printf("%d %lld", w.ok() ? 1 : 0, (long long)size.off);
    for (const void* p : at) printf(" %lld", (long long)(reinterpret_cast<const char*>(p) - base));
    printf("\n");
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("scratch")
    src, exe = str(d / "scratch.cpp"), str(d / "scratch")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(PKG, "csrc"), src, "-o", exe])
    return lambda *args: [int(v) for v in subprocess.check_output([exe, *map(str, args)], text=True).split()]


def _fits(out, sizes):
    """Every array of `sizes` bytes lies in the allocation, aligned, and none reaches into another."""
    ok, total, *at = out
    assert ok and len(at) == len(sizes)
    ends = [o + n for o, n in zip(at, sizes)]
    assert all(o % 256 == 0 for o in at)
    assert all(e <= o for e, o in zip(ends, at[1:] + [total])), (out, sizes)


# d = 16, 64-64 units, 729 rows a minibatch: rows and targets rounded up together
# once came to 256 bytes less than rounded up each, and the total to whole MiB
@pytest.mark.parametrize("epochs,n,batch,d,update", [(5, 9936, 729, 16, 4 * (11712 + 2 * 768 + 4 * 46656)),
                                                     (1, 1, 1, 6, 1), (3, 1000, 77, 37, 12345), (2, 2007, 2007, 32, 4096)])
def test_train_scratch(program, epochs, n, batch, d, update):
    _fits(program("train", epochs, n, batch, d, update), [4 * epochs * n, 4 * batch * d, 4 * batch, 4, 8, update])


@pytest.mark.parametrize("B,nc,n_all,d,H,forward,admission",
                         [(1, 0, 0, 16, 64, 0, 0), (1, 1, 17, 37, 96, 5000, 777), (1000, 1000, 6000, 64, 256, 3470000, 43 << 20),
                          (729, 729, 729, 16, 64, 60000, 1 << 20), (300, 20, 0, 21, 33, 0, 0)])
def test_push_scratch(program, B, nc, n_all, d, H, forward, admission):
    _fits(program("push", B, nc, n_all, d, H, forward, admission),
          [4 * (nc + B), 4 * nc * d, 4 * nc, 4 * n_all * d, 4 * n_all, 4 * forward, 8 * nc * H, 4, admission])


ROUND_PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "ls_internal.h"

// argv: d, hidden layers, width, bf16, rows, minibatch.  The round's workspace and each of its steps'.
int main(int, char** a) {
    ls_model_config cfg{};
    cfg.d = atoi(a[1]);
    cfg.n_hidden = atoi(a[2]);
    for (int l = 0; l < cfg.n_hidden; ++l) cfg.hidden[l] = atoi(a[3]);
    cfg.dtype = atoi(a[4]) ? LS_BF16 : LS_FP32;
    cfg.block_tokens = 16;
    const ls::ModelDims m = ls::make_dims(cfg);
    const int n = atoi(a[5]), batch = atoi(a[6]);
    printf("%lld", (long long)ls::round_workspace_bytes(m, n, batch));
    for (int b : {batch < n ? batch : n, n % batch})
        if (b > 0) printf(" %lld", (long long)ls::update_workspace_bytes(m, b));
    printf("\n");
}
"""


@pytest.fixture(scope="module")
def round_program(tmp_path_factory):
    d = tmp_path_factory.mktemp("round")
    src, exe = str(d / "round.cpp"), str(d / "round")
    with open(src, "w") as f:
        f.write(ROUND_PROGRAM)
    subprocess.check_call([build.HIPCC, "-std=c++17", "-O1", "-I", build.CSRC, "-I", build.INCLUDE, src, "-o", exe,
                           "-L", PKG, "-l:liblodestar.so", f"-Wl,-rpath,{PKG}"])
    return lambda *args: [int(v) for v in subprocess.check_output([exe, *map(str, args)], text=True).split()]


# a last minibatch one row short of a full one, where a full one's gradients take
# fewer and larger chunks; two-launch steps; a minibatch larger than the round
@pytest.mark.parametrize("d,layers,width,bf16,n,batch",
                         [(64, 2, 256, 0, 32769, 16385), (16, 2, 64, 0, 65537, 32769), (32, 3, 128, 1, 32769, 16385),
                          (64, 2, 512, 0, 16385, 8193), (64, 2, 256, 1, 16385, 8193), (16, 2, 64, 0, 1000, 300),
                          (16, 1, 64, 0, 20, 4096), (37, 2, 300, 0, 16384, 16385)])
def test_round_workspace_holds_every_minibatch(round_program, d, layers, width, bf16, n, batch):
    whole, *steps = round_program(d, layers, width, bf16, n, batch)
    assert steps and whole >= max(steps)
