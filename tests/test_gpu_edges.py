"""Sizes at the edges of the launches' tiles and scans, against the oracle:
one bucket, a few, and trees whose node and bucket counts lie on either side of
a workgroup's share.  Tolerance: J within 1e-4 of the oracle (FP32 optical
depths, floor 1e-12 of the band's largest J), work counters equal."""
import numpy as np
import pytest

import oracle
from paper_2310_15235_amd import scenes

pytestmark = pytest.mark.gpu


def _check_J(sc, act, order_scene=False):
    import torch
    from paper_2310_15235_amd import api
    if order_scene:   # the scene-by-scene bucket order has its own bin scan
        F = api.Forest([sc, sc.with_()])
        F.set_config(4)
        Jg = F.split(F.compute_J(F.flat_active([act, act])))[1].cpu().numpy()
        cg = F.counters(1)
        F.check()
        F.close()
    else:
        Jg, cg = api.compute_J(sc, active=act)
    Jo, co = oracle.OracleTree(sc).compute_J(act)
    a = act.astype(bool)
    floor = 1e-12 * np.abs(Jo[:, a]).max(axis=1, keepdims=True)
    err = np.abs(Jg[:, a] - Jo[:, a]) / np.maximum(np.abs(Jo[:, a]), floor)
    assert err.max() <= 1e-4
    for k in ("buckets", "segments", "source_entries", "absorber_entries", "near_pairs",
              "near_src_hits"):
        assert cg[k] == co[k], (k, cg[k], co[k])
    torch.cuda.synchronize()


# 4 nodes per thread of 256 in the bucket list (1024 nodes: about 2600 elements
# at 8 per leaf), 16 words per thread of 1024 in the offset scans
@pytest.mark.parametrize("frac", [1.0, 0.05])
@pytest.mark.parametrize("n", [1, 8, 9, 65, 700, 2590, 2700, 5300])
def test_bucket_list_and_offsets(n, frac):
    sc = scenes.uniform_scene(n=n, seed=n, n_src=max(1, n // 16), bands=(1.0, 10.0), nside=2)
    _check_J(sc, scenes.active_subset(sc, frac, 5))


@pytest.mark.parametrize("n", [9, 2700])
def test_scene_order(n):
    sc = scenes.uniform_scene(n=n, seed=n, n_src=max(1, n // 16), bands=(1.0, 10.0), nside=1)
    _check_J(sc, scenes.active_subset(sc, 0.5, 6), order_scene=True)


# leaf size 1: one bucket per element, so the buckets pass the offset scans'
# 16384-word chunks
def test_offsets_past_one_scan_chunk():
    sc = scenes.uniform_scene(n=17000, seed=3, n_src=40, bands=(1.0,), nside=1, leaf_size=1)
    _check_J(sc, sc.active)
