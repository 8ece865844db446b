"""The training tile kernel at the edges of its 64-sample tiles, on rows at any
alignment and on the smallest sets a batch is drawn from.

Tolerances: a BF16 rounding boundary crossed by the device's FP32 sums moves one
activation by 2^-8 of itself, so the outputs agree with the FP64 reference (same operand
rounding) to 2e-3 of their scale and the gradients to 1e-2 in norm.  The loss is
compared on labels an order of magnitude above the outputs, where the outputs' 2e-3
is at most 4e-4 of it: bound 1e-3.  The alignment changes no arithmetic: equal bits.
"""
import numpy as np
import pytest

from oracle import mlp as M

pytestmark = pytest.mark.gpu


def _features(rng, n):
    return M.bf16(np.concatenate([rng.uniform(0, 1, (n, 1)), rng.normal(0, 0.3, (n, 40)),
                                  np.eye(40)[rng.integers(0, 40, n)], np.zeros((n, 15))], axis=1))


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129])
def test_tile_edges(gpu_lib, n):
    rng = np.random.default_rng(n)
    X, t = _features(rng, n), rng.normal(0, 1, n).astype(np.float32)
    with gpu_lib.Mlp(seed=7) as net:
        p = net.params().astype(np.float64)
        out = net.eval(X.astype(np.float32), t)
        again = net.eval(X.astype(np.float32))
    y, _ = M.forward(p, X, bf=True)
    loss, g = M.loss_and_grad(p, X, t, bf=True)
    assert np.max(np.abs(out["y"] - y)) <= 2e-3 * np.sqrt(np.mean(y ** 2)) + 1e-6
    assert np.array_equal(out["y"], again["y"])
    offs = [0, 6144, 6208, 10304, 10368, 14464, 14528, 14592, 14593]
    for a, b in zip(offs[:-1], offs[1:]):
        err = np.linalg.norm(out["grad"][a:b] - g[a:b]) / max(np.linalg.norm(g[a:b]), 1e-30)
        assert err < 1e-2, (a, b, err)


@pytest.mark.parametrize("n_pairs,batch", [(1, 64), (2, 100), (3, 65), (1000, 4097)])
def test_drawn_rows(gpu_lib, oracle_mod, n_pairs, batch):
    import torch
    rng = np.random.default_rng(n_pairs)
    X = _features(rng, n_pairs)
    t = (rng.uniform(10, 30, n_pairs) * rng.choice([-1, 1], n_pairs)).astype(np.float32)
    flat = torch.zeros(n_pairs * 96 + 8, dtype=torch.bfloat16, device="cuda")
    got = []
    for shift in (0, 1, 3, 8):
        feat = flat[shift:shift + n_pairs * 96].view(n_pairs, 96)
        feat.copy_(torch.tensor(X.astype(np.float32)))
        loss = torch.zeros(2, device="cuda")
        with gpu_lib.Mlp(seed=7) as net:
            p = net.params().astype(np.float64)
            net.train_dev(feat, torch.tensor(t).cuda(), 1.0, 2, batch=batch, lr=1e-3, seed=9,
                          loss=loss)
            torch.cuda.synchronize()
            got.append((loss.cpu().numpy(), net.params()))
    idx = M.minibatch(oracle_mod.philox4x32_10, 9, 1, batch, n_pairs)
    ref, _ = M.loss_and_grad(p, X[idx], t[idx], bf=True)
    assert abs(got[0][0][0] - ref) <= 1e-3 * ref
    for loss, params in got[1:]:
        assert np.array_equal(loss, got[0][0]) and np.array_equal(params, got[0][1])
