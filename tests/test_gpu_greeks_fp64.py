"""Volatility and forward derivatives of the adjoint kernels against FP64 derivatives on the
same increments, where a node of a period's rule lies next to the origin.

There e^{lambda x} - 1 is far below the FP32 rounding of 1, while the node's weight is that
much larger and it holds most of the coupling integral: the product prod_l (1 + ell_l E_l) - 1
has to be carried without the 1.  The rule's middle node crosses the origin where the driver's
skew balances the live vols, so beta is bisected on the rules the plan reports until the
node of one period is within the stated distance.

The reference differentiates the Euler recursion on the 64-node rule in FP64 by torch's
reverse mode.  Bar 1e-5 of the norm: the FP32 recursion rounds each of the 36 steps at 2^-24 of
terms of one sign (36 * 2^-24 = 2e-6), in the states and in the sweep.

With hundreds of steps a period, a step moves the state adjoint by less than its rounding; the
forward derivatives have sums of their own and stay within 1e-6 of the norm (the payoff's
adjoint and the sum of the moves, each rounded at 2^-24, with a factor of 16 to spare)."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

N, S_STEPS, PATHS, SEED = 12, 3, 300, 5
BAR = 1e-5


def structure(beta, product):
    ts = workloads.make_structure(N, 0.25, 0.03 + 0.001 * np.arange(N), S_STEPS,
                                  workloads.exp_decay_vol(), [0.8], beta=beta)
    return workloads.coterminal_swaptions(ts, [0.8]) if product else ts


def long_structure(n, s):
    return workloads.make_structure(n, 0.25, 0.03 + 0.001 * np.arange(n), s,
                                    workloads.exp_decay_vol(), [0.8])


def middle_node(lib, beta, m):
    with lib.Plan(structure(beta, 0), max_paths=64) as plan:
        r = plan.nodes()
    n = int(r["count"][m])
    return (n, float(np.sort(r["x"][m, :n])[n // 2])) if n % 2 else (n, np.nan)


def beta_with_node_at_origin(lib, distance):
    """(beta, period): an odd rule whose middle node is within distance of the origin."""
    grid = np.linspace(-1.4, -0.1, 27)
    for m in range(N - 1):
        nodes = [middle_node(lib, b, m) for b in grid]
        for (b0, (n0, x0)), (b1, (n1, x1)) in zip(zip(grid, nodes), zip(grid[1:], nodes[1:])):
            if n0 != n1 or not x0 * x1 < 0.0:
                continue
            for _ in range(60):
                b = 0.5 * (b0 + b1)
                n, x = middle_node(lib, b, m)
                if n != n0:
                    break
                if abs(x) <= distance:
                    return b, m
                b0, b1 = (b, b1) if x * x0 > 0.0 else (b0, b)
    raise AssertionError("no period's middle node crosses the origin")


def fp64_jacobian(plan, ts, paths=PATHS):
    """Prices (strike 0) and their derivatives, all in FP64 on the host."""
    N, s = ts.n_rates, ts.steps_per_period
    t = plan.tables()
    x, w = torch.tensor(t["x"]), torch.tensor(t["w"])
    L0 = torch.tensor(ts.L0, requires_grad=True)
    v = torch.zeros(N, dtype=torch.float64, requires_grad=True)
    dl = torch.tensor(ts.delta)
    a, b, dn = ts.alpha, ts.beta, ts.delta_nig
    gamma = np.sqrt(a * a - b * b)
    X = [torch.zeros(paths, dtype=torch.float64) for _ in range(N)]
    price = []
    B0T = ts.B0_T1 / torch.prod(1.0 + dl * L0)
    for k in range(N * s):
        m = k // s
        dt = (ts.tenor[m] - (ts.tenor[m - 1] if m else 0.0)) / s
        dH = torch.tensor(plan.increments(k, 0, paths, seed=SEED)[1])
        R = torch.zeros(paths, len(x), dtype=torch.float64)
        for i in range(N - 1, m - 1, -1):
            lam = ts.vol[k, i] + v[i]
            E = torch.expm1(lam * x)
            kappa = -dn * b / gamma * lam + dn * (gamma - torch.sqrt(a * a - (b + lam) ** 2))
            L = L0[i] * torch.exp(X[i])
            ell = (dl[i] * L / (1.0 + dl[i] * L))[:, None]
            C = (R * (w * E)).sum(1)
            R = R + ell * E * (1.0 + R)
            X[i] = X[i] + (-kappa - C) * dt + lam * dH
        if (k + 1) % s == 0:
            L = [L0[l] * torch.exp(X[l]) for l in range(m, N)]
            Q, A = torch.ones(paths, dtype=torch.float64), 0.0
            for l in range(N - 1, m - 1, -1):
                D = Q
                A = A + dl[l] * Q
                Q = Q * (1.0 + dl[l] * L[l - m])
            K = float(ts.strikes[m, 0])
            pay = (Q - 1.0) - K * A if ts.product else D * (L[0] - K)
            price.append((1.0 if ts.product else dl[m]) * B0T * pay.clamp_min(0.0).mean())
    dL, dV = np.zeros((N, N)), np.zeros((N, N))
    for i, p in enumerate(price):
        gL, gV = torch.autograd.grad(p, (L0, v), retain_graph=True)
        dL[i], dV[i] = gL.numpy(), gV.numpy()
    return dL, dV


@pytest.mark.parametrize("product", [0, 1])
@pytest.mark.parametrize("distance", [1e-5, 1e-9, None])
def test_derivatives_with_a_node_next_to_the_origin(gpu_lib, distance, product):
    beta = -4.0 if distance is None else beta_with_node_at_origin(gpu_lib, distance)[0]
    ts = structure(beta, product)
    g = np.linspace(-0.5, 1.5, N)
    with gpu_lib.Plan(ts, max_paths=PATHS) as plan:
        dL, dV = fp64_jacobian(plan, ts)
        plan.greeks(PATHS, seed=SEED)
        jac = plan.greeks_results()
        plan.greeks_vjp(PATHS, g, seed=SEED)
        vjp = plan.greeks_vjp_results()
    err = {name: np.linalg.norm(got - ref) / np.linalg.norm(ref)
           for name, got, ref in (("dP_dL0", jac["dP_dL0"], dL), ("dP_dvol", jac["dP_dvol"], dV),
                                  ("vjp_L0", vjp["vjp_L0"], g @ dL),
                                  ("vjp_vol", vjp["vjp_vol"], g @ dV))}
    print(f"beta {beta:.9f}", {k: f"{e:.1e}" for k, e in err.items()}, flush=True)
    assert max(err.values()) <= BAR, err


@pytest.mark.parametrize("n,s", [(4, 100), (4, 400), (10, 50)])
def test_forward_derivatives_over_many_steps(gpu_lib, n, s):
    ts, paths = long_structure(n, s), 64
    with gpu_lib.Plan(ts, max_paths=paths) as plan:
        ref, _ = fp64_jacobian(plan, ts, paths)
        plan.greeks(paths, seed=SEED)
        err = [np.linalg.norm(plan.greeks_results()["dP_dL0"] - ref) / np.linalg.norm(ref)]
        for g in (np.ones(n), np.linspace(-0.5, 1.5, n)):
            plan.greeks_vjp(paths, g, seed=SEED)
            got = plan.greeks_vjp_results()["vjp_L0"]
            err.append(np.linalg.norm(got - g @ ref) / np.linalg.norm(g @ ref))
    print(n, s, [f"{e:.1e}" for e in err], flush=True)
    assert max(err) <= 1e-6, err
