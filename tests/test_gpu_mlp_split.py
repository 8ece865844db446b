"""The surrogate pass carries 64 paths on 4, 2 or 1 wavefronts, by the size of the
pass.  Every path's fixings are the same bits at the three sizes (the network's
outputs do not depend on which wavefront evaluates them), the ragged last
wavefront included, and so are the pass's fallback and rate-step counts on the
paths both sizes run."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("product", [0, 1])
def test_split_passes_give_the_same_paths(gpu_lib, product):
    import torch
    ts = workloads.make_structure(40, 0.25, 0.03 + 0.001 * np.arange(1, 41), 2,
                                  workloads.exp_decay_vol(), [0.9, 1.1])
    if product:
        ts = workloads.coterminal_swaptions(ts, [0.9, 1.1])
    sizes = (64 * 512, 64 * 512 + 7, 64 * 1024, 64 * 1024 + 1, 64 * 3)   # 4, 2, 2, 1, 4
    out = {}
    with gpu_lib.Plan(ts, max_paths=max(sizes)) as plan, gpu_lib.Mlp(seed=2) as net:
        net.generate(plan, 2048, 8, seed=1)
        net.train(50, batch=4096, lr=2e-3, seed=1)
        box = net.info()
        lo, hi = 0.5 * box["lo"], 0.5 * box["hi"]      # some paths leave it
        net.set_box(lo, hi)
        for n in sizes:
            fix = torch.full((n, 80), -1.0, dtype=torch.float64, device="cuda")
            plan.execute_mlp(net, True, n, seed=9, path_fix=None if product else fix)
            out[n] = (plan.results(), plan.sums(), plan.partials(), fix.cpu().numpy(),
                      plan.mlp_stats())
    ref = out[64 * 1024 + 1]
    assert ref[4]["fallbacks"] > 0
    for n in sizes:
        full = n // 64                                  # wavefronts without idle lanes
        assert np.array_equal(out[n][2][:full], ref[2][:full]), n
        if not product:
            assert np.array_equal(out[n][3], ref[3][:n]), n
    assert out[64 * 1024][4]["rate_steps"] == 2 * out[64 * 512][4]["rate_steps"]
    one = out[64 * 512][4]["fallbacks"], out[64 * 1024][4]["fallbacks"]
    assert 0 < one[0] < one[1] < ref[4]["fallbacks"] + 1
