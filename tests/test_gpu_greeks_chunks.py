"""Greeks passes whose states take more than one chunk of paths.

Two rates at 4000 steps per period keep 20,004 floats per path, so 16 GiB hold
214,000 paths and 300,001 take two chunks, the second ending in a ragged
wavefront.  The pass's prices are the FULL pass's bit for bit, and both
derivatives agree with central differences of FULL prices under the same
streams (h = 1e-3: price rounding 1e-7 / h and the payoff's kink, on a fraction
~ h of the paths, stay below 1e-2; a lost or doubled chunk is off by 29% or
more).  The vector-Jacobian product equals weights x Jacobian to the rounding of
its FP32 seeds."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def test_greeks_over_two_chunks(gpu_lib):
    n, h = 300_001, 1e-3
    ts = workloads.make_structure(2, 0.5, 0.04, 4000, workloads.exp_decay_vol(), [1.0])
    with gpu_lib.Plan(ts, max_paths=n) as plan:
        plan.execute(gpu_lib.FULL, n, seed=3)
        price = plan.results()["price"][:, 0]
        plan.greeks(n, seed=3)
        g = plan.greeks_results()
        w = np.array([0.7, -1.3])
        plan.greeks_vjp(n, w, seed=3)
        v = plan.greeks_vjp_results()
    assert np.array_equal(g["price"], price) and np.array_equal(v["price"], price)
    for l in range(2):
        for key in ("dP_dL0", "dP_dvol"):
            out = []
            for sign in (1.0, -1.0):
                L0, vol = ts.L0.copy(), ts.vol.copy()
                if key == "dP_dL0":
                    L0[l] *= 1.0 + sign * h
                else:
                    vol[:4000 * (l + 1), l] += sign * h
                shifted = ts.copy(L0=L0, vol=vol)
                out.append(gpu_lib.price_caplets(shifted, n, gpu_lib.FULL, seed=3)["price"][:, 0])
            step = 2 * h * (ts.L0[l] if key == "dP_dL0" else 1.0)
            fd = (out[0] - out[1]) / step
            scale = np.abs(g[key]).max()
            assert np.all(np.abs(fd - g[key][:, l]) <= 1e-2 * scale), (key, l, fd, g[key][:, l])
    for key, got in (("dP_dL0", v["vjp_L0"]), ("dP_dvol", v["vjp_vol"])):
        ref = w @ g[key]
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(w) @ np.abs(g[key])), (key, got, ref)
