"""The drift kernel of the 32- and 40-slot buckets against the FP64 oracle (the narrower ones
are in test_gpu_parity.py; the same bars)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [25, 32, 33, 40])
def test_drift_of_wide_buckets_matches_oracle(gpu_lib, oracle_mod, n):
    ts = workloads.make_structure(n, 0.25, 0.03 + 0.001 * np.arange(n), 2,
                                  workloads.exp_decay_vol(), [1.0])
    o = oracle_mod.Oracle(ts, seed=1)
    rng = np.random.default_rng(5)
    gamma = np.sqrt(ts.alpha ** 2 - ts.beta ** 2)
    with gpu_lib.Plan(ts, max_paths=64) as plan:
        for k in (0, 2 * (n // 2) + 1, ts.n_steps - 1):
            L = ts.L0[None, :] * np.exp(rng.normal(0.0, 0.25, size=(5, n)))
            print(f"drift N={n} step {k}", flush=True)
            b = plan.drift(k, L)
            first, u = k // 2, ts.vol[k]
            sq = np.sqrt(np.maximum(ts.alpha ** 2 - (ts.beta + u) ** 2, 0.0))
            kap_tol = 8 * 2.0 ** -53 * (np.abs(ts.delta_nig * ts.beta / gamma * u)
                                        + ts.delta_nig * (gamma + sq))
            for i in range(len(L)):
                ref = o.drift(k, L[i])
                assert np.all(np.abs(b[i] - ref)[first:]
                              <= 1e-5 * np.abs(ref[first:]) + kap_tol[first:]), (k, i)
                assert np.all(b[i, :first] == 0.0)
