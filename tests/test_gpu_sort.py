"""The radix sort behind the tree's particle order at the edges of its paths: one
workgroup up to 4096 keys (1024 and 4096 per launch shape), tiles that add up
each other's counts up to 64 tiles of 2048, a scan kernel beyond; ragged last
wavefronts and tiles.  Keys ascend, equal keys keep their input order, and
every particle appears once."""
import numpy as np
import pytest

import synth
from gpu_helpers import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 65, 1023, 1024, 1025, 4095, 4096, 4097, 6145, 131071, 131072, 131073])
def test_particle_order(n):
    import paper_1312_1128_amd as g

    gen = synth.rng(700 + n)
    x, y = gen.uniform(-1, 1, n), gen.uniform(-1, 1, n)
    dup = gen.integers(0, n, n // 3)  # equal keys, scattered over the input
    x[: dup.size], y[: dup.size] = x[dup], y[dup]
    say(f"[gpu] sort n={n}")
    tree = g.Tree().build(dev(x), dev(y), dev(np.ones(n)), dev(np.full(n, 0.01)), theta=0.3, q=3.0, leaf_size=16, order=4)
    ex = tree.export()
    key, perm = np.asarray(ex["key"]), np.asarray(ex["perm"]).astype(np.int64)
    assert np.all(key[1:] >= key[:-1])
    eq = key[1:] == key[:-1]
    assert n < 1000 or eq.any()
    assert np.all(perm[1:][eq] > perm[:-1][eq])
    np.testing.assert_array_equal(np.sort(perm), np.arange(n))
