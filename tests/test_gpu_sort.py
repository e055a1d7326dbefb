"""The build's sort where keys crowd: runs of elements whose 32 highest varying
key bits agree are ordered in place up to 24 elements, longer ones send the whole
build through the 64-bit passes.  Order and topology equal the oracle's; the
moments agree to 1e-12 (FP64 sums in the same order).  (The transmission averages
of boxes 2^-10 of the root's and smaller have lost their digits in the oracle as
here, and are no check.)"""
import numpy as np
import pytest

import oracle
from paper_2310_15235_amd import scenes

pytestmark = pytest.mark.gpu


def _compare(sc, pos):
    from paper_2310_15235_amd import api
    x, y, z = (np.ascontiguousarray(pos[:, a], np.float32) for a in range(3))
    sc = sc.with_(x=x, y=y, z=z, box=(0.0, 0.0, 0.0, 1.0))
    T = api.Tree.from_scene(sc)
    g = T.export()
    T.check()
    T.close()
    O = oracle.OracleTree(sc)
    o = O.nodes(with_alpha=False)
    perm, keys = O.perm()
    assert np.array_equal(g["perm"], perm)
    for k in ("first", "count", "lown", "split", "child0", "child1", "next"):
        assert np.array_equal(g[k], o[k]), k
    np.testing.assert_allclose(g["cen"], o["cen"], rtol=1e-12, atol=1e-14)
    for k in ("Lb", "Lbol", "kmass"):
        np.testing.assert_allclose(g[k], o[k], rtol=1e-12, atol=0)
    # lengths of the runs of equal leading bits: 63-bit keys, all of them varying
    top = np.asarray(keys, np.uint64) >> np.uint64(31)
    return set(np.unique(np.unique(top, return_counts=True)[1]).tolist())


def _scene(n):
    return scenes.uniform_scene(n=n, seed=4, n_src=max(2, n // 8), bands=(1.0, 3.0), nside=1)


# groups of `sizes` elements inside cells of 2^-11 of the box, each with a few at
# one place, scattered over the input; 4100 and more elements take the passes
# over global memory, 524289 and more their larger tiles
@pytest.mark.parametrize("n", [4200, 9000, 530000])
@pytest.mark.parametrize("sizes", [(2, 3, 23, 24), (3, 24, 25), (200,)])
def test_runs_of_equal_leading_bits(n, sizes):
    sc = _scene(n)
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3))
    free = list(rng.permutation(n))
    for i, k in enumerate(sizes):
        corner = np.array([300 + 200 * i, 700, 900]) / 2048.0
        at = corner + rng.random((k, 3)) * 2.0 ** -11 * 0.98
        at[1::5] = at[0]   # equal keys keep the input order
        pos[free[:k]] = at
        free = free[k:]
    runs = _compare(sc, pos)
    assert set(sizes) <= runs and max(runs) == max(sizes)


# every element within 2^-k of the box, and all but one at one place
@pytest.mark.parametrize("kind,n", [("one", 700), ("one", 6000)] +
                         [(k, n) for k in ("cluster9", "cluster13") for n in (700, 6000, 524400)])
def test_moments_of_crowded_trees(kind, n):
    sc = _scene(n)
    pos = np.random.default_rng(7).random((n, 3))
    if kind == "one":
        pos[1:] = pos[0]
        pos[0] = 0.9
    else:
        pos[2:] = 0.3 + (pos[2:] - 0.5) * 2.0 ** -int(kind[7:])
    runs = _compare(sc, pos)
    if n > 4096:
        assert max(runs) > 24
