"""Small passes (four lanes a path) against the wide kernel (a lane a path), which the
same plan takes for more paths.

Every path's state sees the same operations in the same order in both kernels, so the
fixed rates of FP32 plans are equal bit for bit; the discount products multiply up to
40 FP64 factors in either order (rtol 40 * 2^-52 < 1e-14).  FP64 fixings are allowed 1e-12
(a few units of 2^-52 a step, 200 steps).  Prices of a pass are the means of the paths' FP64
payoffs summed in another order: three small passes over a path range average
to the wide pass over all of it to 1e-12 of the sum of positive terms."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

WIDE = 66000  # above every bound of the small-pass kernel


def _structure(N, s, product=0, driver=0, S=1, heavy=False):
    if heavy:
        return workloads.kluge_example()
    mults = np.linspace(0.8, 1.2, S)
    kw = dict(driver=workloads.DRIVER_BROWNIAN, c=0.5) if driver else {}
    ts = workloads.make_structure(N, 0.25, 0.04, s, workloads.exp_decay_vol(), mults, **kw)
    ts.product = product
    return ts


@pytest.mark.parametrize("scheme", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("fp64,N,s,P", [
    (0, 1, 1, 1), (0, 4, 3, 63), (0, 8, 9, 64), (0, 9, 1, 65), (0, 16, 4, 200), (0, 17, 5, 31),
    (0, 21, 3, 257), (0, 32, 2, 100), (0, 33, 8, 100), (0, 40, 5, 129),
    (1, 1, 7, 5), (1, 8, 3, 100), (1, 9, 5, 64), (1, 16, 2, 33), (1, 24, 4, 100)])
def test_paths_equal_the_wide_kernel(gpu_lib, scheme, fp64, N, s, P):
    import torch
    ts = _structure(N, s)
    with gpu_lib.Plan(ts, precision=fp64, max_paths=WIDE) as plan:
        small = torch.full((P, N, 2), -1.0, dtype=torch.float64, device="cuda")
        wide = torch.empty((WIDE, N, 2), dtype=torch.float64, device="cuda")
        plan.execute(scheme, WIDE, seed=5, path_fix=wide)
        plan.execute(scheme, P, seed=5, path_fix=small)
        r = plan.results()
    a, b = small.cpu().numpy(), wide.cpu().numpy()[:P]
    if fp64:
        assert np.allclose(a, b, rtol=1e-12, atol=0)
    else:
        assert np.array_equal(a[..., 0], b[..., 0])
        assert np.allclose(a[..., 1], b[..., 1], rtol=1e-14, atol=0)
    pay = b[..., 1] * np.maximum(b[..., 0] - np.asarray(ts.strikes)[:, 0], 0.0)
    bond = np.asarray(r["price"])[:, 0] / np.maximum(pay.mean(axis=0), 1e-300)
    live = pay.mean(axis=0) > 0
    assert np.allclose(bond[live], bond[live][:1], rtol=1e-11) if live.any() else True


@pytest.mark.parametrize("N,s,fp64,kw", [
    (5, 2, 0, dict(S=8)), (20, 3, 0, dict(S=3, product=1)), (40, 2, 0, dict(S=5, product=1)),
    (9, 5, 0, dict(heavy=True)), (12, 4, 0, dict(driver=1, S=2)), (20, 2, 1, dict(S=7, product=1)),
    (9, 5, 1, dict(heavy=True)), (7, 3, 1, dict(driver=1, S=4))])
@pytest.mark.parametrize("scheme", [0, 1, 4])
def test_prices_of_a_split_range(gpu_lib, scheme, N, s, fp64, kw):
    ts = _structure(N, s, **kw)
    third = WIDE // 3
    with gpu_lib.Plan(ts, precision=fp64, max_paths=WIDE) as plan:
        plan.execute(scheme, WIDE, seed=3)
        ref = {k: np.array(v) for k, v in plan.results().items()}
        price, resid, itm = 0.0, 0.0, 0
        for i in range(3):
            plan.execute(scheme, third, seed=3, path_offset=i * third)
            r = plan.results()
            price, itm = price + np.array(r["price"]) / 3, itm + np.array(r["n_itm"])
            resid = resid + np.array(r["mart_resid"]) / 3
    assert np.allclose(price, ref["price"], rtol=1e-12, atol=0)
    assert np.array_equal(itm, ref["n_itm"])
    assert np.allclose(resid, ref["mart_resid"], rtol=0, atol=1e-12)


@pytest.mark.parametrize("scheme", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("N,s,kw", [(6, 3, {}), (13, 2, dict(S=4)), (19, 2, dict(S=2)),
                                    (24, 2, dict(product=1)), (40, 2, dict(S=3)),
                                    (11, 2, dict(product=1, S=3))])
def test_partial_sums_equal_the_wide_kernels(gpu_lib, scheme, N, s, kw):
    """The sums of 64 paths do not depend on the kernel (FP32): shards of a run concatenate."""
    ts = _structure(N, s, **kw)
    with gpu_lib.Plan(ts, precision=0, max_paths=WIDE) as plan:
        plan.execute(scheme, WIDE, seed=11)
        wide = plan.partials()[:3]
        plan.execute(scheme, 192, seed=11)
        assert np.array_equal(plan.partials(), wide)
