"""Neighbour initialisation with a radius past the adjacent tiles, at surfel
counts about the 64 that a wavefront then looks through, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from tests.helpers import random_unit_cap
from tests.parity import oracle_keyframe, oracle_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,grids", [
    (4, [(9, 7), (64, 1), (13, 5), (127, 1), (1, 128), (3, 43), (1, 1)]), (8, [(16, 12)]), (16, [(5, 13), (6, 2)])])
@pytest.mark.parametrize("radius", [2.6, 5.1, 1000.0])          # tile edges; the last reaches every surfel
@pytest.mark.parametrize("share", [0.02, 0.5, 0.95, 1.0])
def test_wide_radius(S, grids, radius, share):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        rng = np.random.default_rng(int(100 * share) + S)
        kfs = []
        for gw, gh in grids:
            m, W, H = gw * gh, gw * S + S // 2, gh * S + 1
            ids = rng.uniform(0.3, 1.5, m).astype(np.float32)
            ns = np.array([random_unit_cap(rng, 20) for _ in range(m)], np.float32)
            flags = np.where(rng.random(m) < 0.1, oracle.UNINIT, 0).astype(np.uint32)
            img, f = torch.zeros((H, W), dtype=torch.float32), 0.9 * max(W, H)
            new = (rng.random(m) < share).astype(np.uint8)
            new[m // 2] = 1
            kfs.append((engine.DeviceKeyframe(ctx, img, img[None], np.eye(3)[None], np.zeros((1, 3)),
                                              (f, f, W / 2, H / 2), S, ids, ns, is_new=new, flags=flags),
                        ids, ns, flags, new))
        print(f"case init radius {radius} S={S} new {share}", flush=True)
        prm = sg.params(iters=0, beta_r=radius * S)
        sg.sgn_optimize_batch(ctx.handle, sg.batch_array([k[0].item() for k in kfs]), len(kfs), prm)
        torch.cuda.synchronize()
        for dk, ids, ns, flags, new in kfs:
            st = oracle_state(ids, ns, flags)
            oracle.init_from_neighbours(oracle_keyframe(dk), st, new, oracle.OracleParams(iters=0, beta_r=radius * S))
            h = dk.state.to_host()
            uninit = (np.asarray(st["flags"]) & oracle.UNINIT) != 0
            assert np.array_equal((h["flags"] & sg.FLAG_UNINIT) != 0, uninit)
            # a mean of at most 192 float terms of up to 2.3, summed in order
            tol = 192 * 2.3 * 6e-8
            assert np.abs(h["inv_depth"] - st["inv_depth"])[~uninit].max(initial=0) < tol
            on = np.stack([st["nx"], st["ny"], st["nz"]], 1)
            assert np.abs(h["n"] - on)[~uninit].max(initial=0) < tol
            old = new == 0
            assert np.array_equal(h["inv_depth"][old], ids[old]) and np.array_equal(h["n"][old], ns[old])
    finally:
        ctx.close()
