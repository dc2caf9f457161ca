"""GPU parity of the budget count and its folded gate backward where a block's layers are looked up 64 at a time: layer
counts at the edges of one, two and three lookup steps, runs of empty layers, layers that end at block edges."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_support import dev_f32, empty_f32, say, sync

pytestmark = pytest.mark.gpu


def _check_dlogits(got, dg, per, y, tau):
    dg, per, y = (a.astype(np.float64) for a in (dg, per, y))
    # six roundings of 2^-24 or fewer: the sum, 1 - y, two products, tau and the quotient
    bound = 6 * 2.0 ** -24 * np.abs(y * (1.0 - y) / tau) * (np.abs(dg) + np.abs(per))
    assert np.all(np.abs(got.astype(np.float64) - oracle.gate_bwd(dg + per, y, tau)) <= bound + 1e-30)


@pytest.mark.parametrize("L,big", [(1, 0), (2, 4096), (64, 4096), (65, 9000), (224, 5000), (4096, 4097), (4097, 8192)])
def test_layer_lookup(L, big):
    import torch
    import paper_2609_33977_amd as gm
    say(f"budget layer lookup: L={L} big={big}")
    r = workloads.gen.rng_for(951, L)
    sizes = r.integers(1, 40, size=L)
    if big:
        sizes[L // 2] = big
        sizes[-1] = 4096 - int(sizes[:-1].sum()) % 4096  # the last layer ends at a block's edge
    n = int(sizes.sum())
    params = sizes * 256
    flat = (r.uniform(size=n) < 0.5).astype(np.float32)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    i64 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int64)).cuda()
    off, par, m = i64(offsets), i64(params), dev_f32(flat)
    kept, loss, coeff = i64(np.full(L, -1)), torch.empty(1, dtype=torch.float64, device="cuda"), empty_f32(L)
    gm.gm_budget_loss(m, off, par, 0.5, 16.0, False, kept, loss, coeff)
    dg, y = r.normal(size=n).astype(np.float32), r.uniform(0.01, 0.99, size=n).astype(np.float32)
    dl, alias = empty_f32(n), dev_f32(dg)
    gm.gm_gate_bwd_budget(dev_f32(dg), dev_f32(y), 0.4, off, coeff, dl)
    gm.gm_gate_bwd_budget(alias, dev_f32(y), 0.4, off, coeff, alias)
    sync()
    assert np.array_equal(kept.cpu().numpy(), np.add.reduceat(flat, offsets[:-1]).astype(np.int64))
    _check_dlogits(dl.cpu().numpy(), dg, np.repeat(coeff.cpu().numpy(), sizes), y, 0.4)
    assert np.array_equal(alias.cpu().numpy(), dl.cpu().numpy())


def test_layer_lookup_empty_layers():
    import torch
    import paper_2609_33977_amd as gm
    say("budget layer lookup: empty layers between, before and after full ones")
    sizes = np.array([0] * 70 + [5000] + [0] * 130 + [4096, 0, 77] + [0] * 3)
    n, L = int(sizes.sum()), len(sizes)
    offsets = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)).cuda()
    r = workloads.gen.rng_for(952)
    dg, c = r.normal(size=n).astype(np.float32), r.normal(size=L).astype(np.float32)
    y = r.uniform(0.01, 0.99, size=n).astype(np.float32)
    dl = empty_f32(n)
    gm.gm_gate_bwd_budget(dev_f32(dg), dev_f32(y), 0.5, offsets, dev_f32(c), dl)
    sync()
    _check_dlogits(dl.cpu().numpy(), dg, np.repeat(c, sizes), y, 0.5)
