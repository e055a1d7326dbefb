"""Sizes at the edges of the launches' tiles and scans, against the oracle:
one bucket, a few, and trees whose node and bucket counts lie on either side of
a workgroup's share; trees as tests/test_gpu_parity.py compares them (topology
equal, FP64 moments to 1e-12, FP32 tables to 2e-6).  Tolerance: J within 1e-4
of the oracle (FP32 optical depths, floor 1e-12 of the band's largest J), work
counters equal."""
import numpy as np
import pytest

import oracle
from paper_2310_15235_amd import scenes
from tests.test_gpu_parity import compare_tree

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


# one node per thread of 256 in the bucket list (256 nodes: about 650 elements
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


# the LDS sort's last and the radix passes' first size, a tile's edges, the
# switch of the tile size, one subtree's elements
@pytest.mark.parametrize("n,leaf", [(1, 8), (8, 8), (9, 8), (64, 1), (512, 8), (513, 3), (4095, 8),
                                    (4096, 1), (4097, 8), (5120, 12), (5121, 8), (16385, 8),
                                    (524288, 8), (524289, 8)])
def test_tree_sizes(n, leaf):
    compare_tree(scenes.uniform_scene(n=n, seed=n + leaf, n_src=max(1, n // 16), bands=(1.0, 2.0, 5.0),
                                     nside=1, leaf_size=leaf))


# crowded keys: elements within 2^-9 .. 2^-16 of the box (32 bits of the key
# tell few or none of them apart, so the full sort runs), one place for all, a
# deep chain (each half of the elements eight times closer to a corner), equal
# places in runs longer than a bucket
# (the order and the topology, all integers: where boxes are 2^-16 of the
# root's, the log of a transmission near 1 over such a chord has lost its digits
# in the oracle as here, so these trees' averages are no check of the build)
@pytest.mark.parametrize("kind", ["cluster9", "cluster13", "cluster16", "one", "chain", "runs"])
@pytest.mark.parametrize("n", [700, 6000])
def test_tree_crowded(kind, n):
    sc = scenes.uniform_scene(n=n, seed=4, n_src=30, bands=(1.0,), nside=1)
    pos = sc.positions().astype(np.float64)
    if kind.startswith("cluster"):
        pos[2:] = 0.3 + (pos[2:] - 0.5) * 2.0 ** -int(kind[7:])
    elif kind == "one":
        pos[:] = pos[0]
    elif kind == "chain":
        pos *= 8.0 ** -np.minimum(np.arange(n) % 7, 6)[:, None]
    else:
        pos = pos[np.arange(n) // 40 * 40]
    x, y, z = (np.ascontiguousarray(pos[:, a], np.float32) for a in range(3))
    from paper_2310_15235_amd import api
    for box in (sc.box, None):
        moved = sc.with_(x=x, y=y, z=z, box=box)
        T = api.Tree.from_scene(moved)
        g = T.export()
        T.check()
        O = oracle.OracleTree(moved)
        o = O.nodes()
        assert np.array_equal(g["perm"], O.perm()[0])
        for k in ("first", "count", "lown", "split", "child0", "child1", "next"):
            assert np.array_equal(g[k], o[k]), k
        T.close()


# the adjoint's scratch asked for by the forward: the buffer keeps its size and
# the gradients equal those of the growing one (FP32 rounding of atomic sums:
# 1e-5 of a value, 1e-6 of the array's largest).  One scene whose near sets the
# estimate covers, one whose it does not.
@pytest.mark.parametrize("n,nside", [(3000, 1), (1200, 4)])
def test_adjoint_room(n, nside):
    import torch
    from paper_2310_15235_amd import api
    sc = scenes.lognormal_scene(n=n, seed=2, grid=16, bands=(1.0, 10.0), nside=nside)
    gJ = torch.as_tensor(np.random.default_rng(1).normal(size=(2, n)), device="cuda")
    plain = api.compute_J_backward(sc, gJ.cpu().numpy())
    for reserve in (False, True):
        T = api.Tree.from_scene(sc)
        if reserve:
            T.reserve_adjoint()
        else:
            T.tune(api.TUNE_ADJOINT, 1)
        T.compute_J()
        size = T.scratch.numel()
        got = T.compute_J_backward(gJ)
        T.check()
        assert T.scratch.numel() == size
        for a, b in zip(got, plain):
            a = a.cpu().numpy()
            assert np.all(np.abs(a - b) <= 1e-5 * np.abs(b) + 1e-6 * np.abs(b).max())
        T.close()
    T = api.Tree.from_scene(sc)
    with pytest.raises(api.TrevrError):
        T.tune(api.TUNE_ADJOINT, 2)
    T.close()


# the candidate rays of cells and elements in every direction and at every
# angular size: a ray missed would lose segments or optical depth.  Elements
# around an off-centre source at N_side 1 to 16 (one to 48 groups of rays), the
# last group not full at 1, 2 and 8; with a directed ray, which is off its place
# in the table.
@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("nside,n", [(1, 3000), (2, 3000), (4, 2000), (8, 900), (16, 300)])
def test_candidate_rays(nside, n, directed):
    sc = scenes.lognormal_scene(n=n, seed=nside, grid=16, bands=(1.0, 10.0), nside=nside)
    if directed:
        sc = sc.with_(directed=(0.31, 0.72, 0.44))
    _check_J(sc, scenes.active_subset(sc, 0.3 if nside <= 4 else 0.1, 2))


# heavy buckets in parts: few buckets with large near sets and many near sources
# (each with passes of 256 pairs to share out), one and several receiver chunks
# per bucket, in a lone tree and in a forest whose job log the adjoint reads.
# Gradients against the forest without a log (culled again): FP32 rounding of
# atomic sums, 1e-5 of a value + 1e-6 of the array's largest.
@pytest.mark.parametrize("leaf", [8, 20])
def test_parts(leaf):
    import torch
    from paper_2310_15235_amd import api
    scs = [scenes.lognormal_scene(n=n, seed=n, grid=16, bands=(1.0, 10.0, 3.0)[:b], nside=4,
                                  leaf_size=leaf, src_frac=0.4)
           for n, b in ((1500, 2), (700, 1), (1100, 2))]
    _check_J(scs[0], scs[0].active)
    _check_J(scs[0], scenes.active_subset(scs[0], 0.1, 3))
    F = api.Forest(scs)
    gJ = torch.as_tensor(np.random.default_rng(3).normal(size=int(F.boff[-1])), device="cuda")
    J0 = F.compute_J()
    plain = F.compute_J_backward(gJ)
    for room in (2 * F.counters()["pp_log_entries"] + (1 << 26), 1 << 19):
        F.set_job_log(room)
        J1 = F.compute_J()
        logged = F.compute_J_backward(gJ)
        F.check()
        for a, b in zip((J1,) + tuple(logged), (J0,) + tuple(plain)):
            assert bool(((a - b).abs() <= 1e-5 * b.abs() + 1e-6 * b.abs().max()).all())
    F.close()


# far-field windows: cut lists on either side of a listing round (2048 entries),
# more sources on a group of rays than a window holds (448 and more: several
# windows) and fewer.  The adjoint by Euler's identity: J is homogeneous of degree
# one in the luminosities (their centres do not move when all are scaled), so
# sum L dE/dL = sum gJ J for E = sum gJ J; with gJ > 0 every term is positive
# and carries some FP32 roundings: 1e-5.
@pytest.mark.parametrize("n,theta,n_src,windows", [(30000, 0.2, 6000, True), (6000, 0.6, 40, False)])
def test_source_windows(n, theta, n_src, windows):
    from paper_2310_15235_amd import api
    sc = scenes.uniform_scene(n=n, seed=7, n_src=n_src, bands=(1.0, 10.0), nside=1, theta=theta)
    act = scenes.active_subset(sc, 0.005, 4)
    _check_J(sc, act)
    Jg, c = api.compute_J(sc, active=act)
    assert (c["max_cut"] > 2048 and c["source_entries"] > 448 * c["buckets"]) == windows
    a = act.astype(bool)
    gJ = np.zeros((2, n))
    gJ[:, a] = 1.0 / np.maximum(Jg[:, a], 1e-300)
    gL = api.compute_J_backward(sc, gJ, active=act)[0]
    want = float((gJ[:, a] * Jg[:, a]).sum())
    assert abs(float((gL * sc.lum).sum()) - want) <= 1e-5 * want
