"""The batch autotuner times the untuned plan's own choice beside its candidates:
for dense items of one cap per disk that is the form by lists on bins of at least
the radius (1.4 times as fast as the best ring search), which no table could name
before.  Outputs do not depend on the table: counts and picks equal, depths within
2e-5 relative (each side within 1e-5 of the definition)."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_untuned_choice_is_timed(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    side, r, cap = 256, 6.0, 16
    n = int(cap * (2.0 * side + 2 * r) ** 2 / (math.pi * r * r))
    rng = np.random.default_rng(4)
    keep, items = [], []
    for _ in range(24):
        p = [torch.from_numpy(a).cuda() for a in (rng.uniform(-r, 2.0 * side + r, n),
                                                  rng.uniform(-r, 2.0 * side + r, n),
                                                  rng.normal(-800.0, 3.0, n))]
        out = [torch.empty((side, side), dtype=t, device="cuda")
               for t in (torch.float32, torch.int32, torch.int32)]
        items.append(ag.batch_item(ag.make_desc(0.0, 0.0, 2.0, 2.0, side, side), *p,
                                   ag.idw_params(radius=r, min_pts=1, max_pts=cap), *out))
        keep.append((p, out))
    table = str(tmp_path / "tune.txt")
    plain = ag.Batch(items)
    ag.auv_batch_autotune(items, plain.ws, table)
    tuned = ag.Batch(items, table)
    results = []
    for b in (plain, tuned):
        b.launch()
        torch.cuda.synchronize()
        results.append([[t.clone() for t in out] for _, out in keep])
    plan = tuned.item_plan_full(0)
    plain.close()
    tuned.close()
    assert plan[1] == ag.AUV_ALGO_DENSE and 2 ** plan[0] >= r * 65536
    for (z0, c0, i0), (z1, c1, i1) in zip(*results):
        assert torch.equal(c0, c1) and torch.equal(i0, i1)
        assert torch.equal(torch.isnan(z0), torch.isnan(z1))
        ok = ~torch.isnan(z0)
        assert ((z0[ok] - z1[ok]).abs() / z0[ok].abs()).max().item() <= 2e-5
