"""The Gauss rules the kernels integrate the coupling on against the 64-node
rule they are taken from, on the host in FP64, and the FP64 drift kernel on them.

The coupling sums sum_q W_q E_{i,q} (prod_{l>i} (1 + ell_l E_{l,q}) - 1) of both
rules are formed for states from nearly zero to nearly one.  A period's rule is
accepted at 2^-30 (FP32 plans) or 2^-47 (FP64) of the integrals of
|e^{lambda_i x} - 1| |e^{a x} - 1| at the extreme subset sums a, so the same
holds for the coupling relative to its average over those terms: the coupling
itself with vols of one sign, at most sum W |E_i| (prod (1 + ell |E|) - 1) with
both.  The host
sums of the 64 terms carry a few units of 2^-52 of sum W |E|."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def structures():
    decay = workloads.exp_decay_vol()
    mk = workloads.make_structure
    return {
        "n1": mk(1, 0.5, 0.04, 3, decay, [1.0]),
        "n2": mk(2, 0.25, 0.04, 1, decay, [1.0]),
        "n20": workloads.gpu_scale(),
        "n40_two_decays": mk(40, 0.25, 0.05, 2, workloads.exp_decay_vol(0.05, 0.3, 2.0), [1.0]),
        "heavy": workloads.kluge_example(),
        "skewed": mk(17, 0.5, 0.03, 2, decay, [1.0], alpha=12.0, beta=-5.0, delta_nig=0.5),
        "negative": mk(12, 0.5, 0.03, 2, lambda t, T, r: -0.2, [1.0]),
        "mixed": mk(15, 0.5, 0.03, 2, lambda t, T, r: 0.2 * (-1) ** r, [1.0]),
        "tiny": mk(6, 0.5, 0.03, 2, lambda t, T, r: 1e-6, [1.0]),
        "zero": mk(6, 0.5, 0.03, 2, lambda t, T, r: 0.0, [1.0]),
        "n64": mk(64, 0.25, 0.03, 1, decay, [1.0]),
    }


def product_less_one(t):
    """prod_{l>i} (1 + t_l) - 1 by row, without the cancellation against 1."""
    R = np.zeros_like(t)
    for i in range(len(t) - 2, -1, -1):
        R[i] = R[i + 1] + t[i + 1] * (1.0 + R[i + 1])
    return R


@pytest.mark.parametrize("name", sorted(structures()))
@pytest.mark.parametrize("precision,tol", [(0, 2.0 ** -30), (1, 2.0 ** -47)])
def test_gauss_rule_reproduces_the_64_node_couplings(gpu_lib, name, precision, tol):
    ts = structures()[name]
    if precision == 1 and ts.n_rates > 24:
        pytest.skip("FP64 plans hold up to 24 rates")
    N, s = ts.n_rates, ts.steps_per_period
    with gpu_lib.Plan(ts, precision=precision, max_paths=64) as plan:
        full, rules = plan.tables(), plan.nodes()
    assert np.all((rules["count"] >= 3) & (rules["count"] <= 64))
    worst = 0.0
    for m in range(N):
        n = rules["count"][m]
        for k in {m * s, m * s + s - 1}:
            lam = ts.vol[k, m:]
            sums, sizes = [], []
            for x, w in ((full["x"], full["w"]), (rules["x"][m, :n], rules["w"][m, :n])):
                E = np.expm1(lam[:, None] * x)
                per = []
                for lo, hi in ((1e-4, 1e-3), (0.005, 0.03), (0.3, 0.7), (0.99, 1.0)):
                    ell = np.random.default_rng(m).uniform(lo, hi, N - m)
                    per.append((w * E * product_less_one(ell[:, None] * E)).sum(axis=1))
                    sizes.append((w * np.abs(E) * product_less_one(ell[:, None] * np.abs(E))).sum(axis=1))
                sums.append(np.array(per))
            ref, got = sums
            one_sign = np.all(lam >= 0) or np.all(lam <= 0)
            size = np.abs(ref) if one_sign else np.array(sizes[:len(ref)])
            noise = 2.0 ** -52 * (full["w"] * np.abs(np.expm1(lam[:, None] * full["x"]))).sum(axis=1)
            assert np.all(np.abs(got - ref) <= tol * size + 16 * noise), (m, k, n)
            worst = max(worst, float(n))
    if name in ("n20", "skewed"):
        assert worst <= 10   # the rule is worth having where the tails are light


def test_few_nodes_where_tails_are_light(gpu_lib):
    with gpu_lib.Plan(workloads.gpu_scale(), precision=0, max_paths=64) as plan:
        assert plan.nodes()["count"].max() <= 6
    with gpu_lib.Plan(workloads.learned_drift(), precision=0, max_paths=64) as plan:
        assert plan.nodes()["count"].max() <= 8
