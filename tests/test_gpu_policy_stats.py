"""The batch statistics of the routing policy (Alg. 1 to 4) at the instance
counts where their staging can go wrong: one instance, a full pass of 1,024 and
one more, with bounds that the last instance alone breaks."""
import dataclasses

import numpy as np
import pytest

import oracle
from gpu_helpers import note
from paper_2606_00946_amd import synth
from test_gpu_route import BASE, mode_of, run_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 1024, 1025])
def test_statistics_over_many_instances(N):
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], R=40, N=N, update_batch=64, seed=N)
    w = synth.generate(cfg)
    rnd = np.random.default_rng(3).integers(0, 1 << 32, (cfg.R, 3), dtype=np.uint64).astype(np.uint32)
    lo = np.full(cfg.d, -np.inf, np.float32)
    hi = np.full(cfg.d, np.inf, np.float32)
    hi[2] = np.nextafter(np.float32(w.inst_feat[-1, 2]), np.float32(-np.inf))
    for name, pol in (("kfilter", dict(BASE, kv_col=4, tau_sat=0.3, tau_ben=64.0, k_filter=2, delta=0.01)),
                      ("loads", dict(BASE, n_samples=5)), ("bounds", dict(BASE, lo=lo, hi=hi))):
        note(f"policy statistics N={N} {name}")
        chosen, status, heur, _ = run_route(w, pol, rnd)
        want = oracle.route(mode_of(w), cfg.d, cfg.hidden, w.params, w.mu, w.inv_sigma, w.req_off, w.req_hashes,
                            w.prompt_len, w.inst_feat, w.inst_off, w.inst_hashes, oracle.policy(**pol), rnd)
        np.testing.assert_array_equal(chosen, want[0], err_msg=name)
        np.testing.assert_array_equal(status, want[1], err_msg=name)
        np.testing.assert_array_equal(heur, want[2], err_msg=name)
