"""Canonical scores on the matrix cores for one to three equal layers (Section
4.1) against the oracle bit for bit, at the batch sizes where the kernel's
groups can go wrong: one pair, a group's 32 pairs and one more or less, the
smallest batch that takes two groups a workgroup and the largest that takes
one (on eight compute units 1,024 pairs, or listed requests), instances that
do not divide a group, and the band's rescoring over a list."""
import dataclasses

import numpy as np
import pytest

import oracle
from gpu_helpers import GpuRun, note
from paper_2606_00946_amd import lodestar, synth
from test_gpu_depth import mode_of

pytestmark = pytest.mark.gpu

MODELS = [(16, (64,), "fp32"), (16, (64, 64), "fp32"), (32, (128, 128, 128), "fp32"), (37, (128, 128), "fp32"),
          (48, (256, 256), "fp32"), (21, (64, 64, 64), "bf16"), (64, (256, 256, 256), "bf16"), (30, (128,), "bf16")]


@pytest.mark.parametrize("d,hidden,dtype", MODELS)
def test_scores_bit_for_bit(d, hidden, dtype):
    for R, N in ((1, 1), (31, 1), (11, 3), (1023, 1), (1024, 1), (147, 7)):
        note(f"chain scores d={d} hidden={hidden} {dtype} R={R} N={N}")
        cfg = dataclasses.replace(synth.CONFIGS["tiny"], d=d, hidden=hidden, dtype=dtype, R=R, N=N, update_batch=64,
                                  seed=R + N)
        w = synth.generate(cfg)
        run = GpuRun(w)
        run.ctx.ls_set_cu_limit(8)
        got = run.score()
        want = oracle.score(mode_of(w), d, hidden, w.params, w.mu, w.inv_sigma, w.req_off, w.req_hashes, w.prompt_len,
                            w.inst_feat, w.inst_off, w.inst_hashes)
        assert np.array_equal(got["scores"], want["scores"].astype(np.float32)), (R, N)
        assert np.array_equal(got["chosen"], want["chosen"]), (R, N)
        run.ctx.close()


@pytest.mark.parametrize("d,hidden", [(16, (64, 64)), (32, (128, 128)), (64, (256, 256))])
def test_rescored_minima_bit_for_bit(d, hidden):
    for R, N in ((1, 2), (33, 5), (1023, 3), (1024, 3), (1089, 2)):
        note(f"rescored minima d={d} hidden={hidden} R={R} N={N}")
        cfg = dataclasses.replace(synth.CONFIGS["tiny"], d=d, hidden=hidden, dtype="bf16", R=R, N=N, update_batch=64,
                                  seed=R + N)
        w = synth.generate(cfg)
        run = GpuRun(w)
        run.ctx.ls_set_cu_limit(8)
        got = run.score(with_scores=False)
        want = oracle.score("bf16", d, hidden, w.params, w.mu, w.inv_sigma, w.req_off, w.req_hashes, w.prompt_len,
                            w.inst_feat, w.inst_off, w.inst_hashes)
        assert np.array_equal(got["chosen"], want["chosen"]), (R, N)
        assert np.array_equal(got["min_ttft"], want["scores"].astype(np.float32).min(1)), (R, N)
        run.ctx.close()


def test_three_layers_fit_the_allocation_free_call():
    """69,300 pairs of 3 x 128: the chain kernels take no scratch per layer, so
    the batch fits ls_score_batch_noalloc; layer by layer it does not."""
    import torch
    cfg = dataclasses.replace(synth.CONFIGS["homogeneous"], hidden=(128, 128, 128), R=2100, N=33,
                              capacity=tuple(2000 for _ in synth.CONFIGS["homogeneous"].capacity), warmup_requests=0,
                              update_batch=64)
    w = synth.generate(cfg)
    run = GpuRun(w)
    note("three layers, allocation-free scoring of 69,300 pairs")
    want = run.score(with_scores=False)
    chosen = torch.full((cfg.R,), -7, dtype=torch.int32, device="cuda")
    mt = torch.zeros(cfg.R, device="cuda")
    args = (run.req_off, run.req_hashes, run.prompt_len, run.inst_feat, chosen, mt)
    run.ctx.ls_score_batch_noalloc(*args)
    torch.cuda.synchronize()
    assert np.array_equal(chosen.cpu().numpy(), want["chosen"])
    assert np.array_equal(mt.cpu().numpy(), want["min_ttft"])
    run.ctx.ls_set_chain_kernels(1)
    with pytest.raises(lodestar.LodestarError) as e:
        run.ctx.ls_score_batch_noalloc(*args)
    assert e.value.code == lodestar.LS_ERR_INVALID
    run.ctx.close()
