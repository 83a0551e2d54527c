"""Admission to replay pools of up to 6,144 members (Section 4.3.2) against the
oracle, at the sizes and inputs where its walk can go wrong: pools of one and
two, a pool that fills within a chunk of candidates, chunks of 512 and one
more, more refusals in a row than are looked at ahead, many members with the
same nearest neighbour, members whose whole list of near ones has been
replaced, the largest pool and one slot more, units that do not fill a tile.
Pool rows, slots and counts are the oracle's exactly."""
import dataclasses

import numpy as np
import pytest

import oracle
from gpu_helpers import note, to_dev
from paper_2606_00946_amd import lodestar, synth

pytestmark = pytest.mark.gpu

CASES = [
    # hidden, dtype, FIFO, pool, pushes, rows
    ((64, 64), "fp32", 4, 1, [4, 30], "all"),
    ((64, 64), "fp32", 4, 2, [4, 30, 3], "all"),
    ((40, 33), "fp32", 16, 100, [60, 300, 1], "all"),
    ((64, 64), "bf16", 8, 70, [520, 521, 9], "all"),
    ((64, 64), "fp32", 8, 130, [138, 400], "copies"),      # pool of a few distinct rows, then distinct candidates
    ((64, 64), "fp32", 8, 130, [600, 600], "refused"),     # distinct pool, then copies of its rows
    ((17,), "fp32", 2, 1500, [1400, 700], "all"),
    ((8, 9, 5), "fp32", 2, 6144, [6100, 90], "all"),
    ((8, 9, 5), "fp32", 2, 6145, [6100, 90], "all"),
]


@pytest.mark.parametrize("hidden,dtype,F,P,pushes,rows", CASES)
def test_admission_matches_oracle(hidden, dtype, F, P, pushes, rows):
    import torch
    n = sum(pushes)
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], hidden=hidden, dtype=dtype, update_batch=n, R=33, N=5, seed=P + n)
    w = synth.generate(cfg)
    x, y = w.upd_feats[:n].copy(), w.upd_ttft[:n].copy()
    for k in range(5, n, 5):                               # copies: ties
        x[k], y[k] = x[k // 2], y[k // 2]
    if rows == "copies":
        for k in range(pushes[0]):
            x[k], y[k] = x[k % 3], y[k % 3]
    if rows == "refused":
        x[pushes[0] + 40:], y[pushes[0] + 40:] = x[20], y[20]
    ctx = lodestar.Context(cfg.d, hidden, dtype)
    ctx.ls_set_model(w.params, w.mu, w.inv_sigma)
    ctx.ls_buffer_init(F, P)
    ob = oracle.Buffer(cfg.d, F, P)
    at = 0
    for k in pushes:
        note(f"admission hidden={hidden} pool={P} rows {at}..{at + k} {rows}")
        adm = torch.zeros(1, dtype=torch.int32, device="cuda")
        ctx.ls_buffer_push(to_dev(x[at:at + k]), to_dev(y[at:at + k]), adm)
        want = oracle.buffer_push("bf16" if dtype == "bf16" else "fp32", hidden, w.params, w.mu, w.inv_sigma, ob,
                                  x[at:at + k], y[at:at + k])
        got = [t.cpu().numpy() for t in ctx.ls_buffer_read()]
        for a, b in zip(got, [*ob.fifo_rows(), *ob.replay_rows()]):
            np.testing.assert_array_equal(a, b)
        assert int(adm.item()) == want
        at += k
    ctx.close()
