"""Density-matrix rows summed in LDS (states with more pairs than subset
records) against the sort-and-join path: subsets shared by a few and by
hundreds of determinants, the widest row (32 orbitals, 15,872 columns), a full
sector with ten pairs per join record, a subset shared by more determinants
than the pass orders (the pairs then go to memory), and one so crowded beside
that that the join is taken."""
import math

import numpy as np
import pytest

from paper_2411_07920_amd.inputs import enumerate_pool, make_integrals

pytestmark = pytest.mark.gpu


def _keys(rng, n, na, nb, count, width):
    key = np.zeros(count, dtype=np.uint64)
    for spin, occ in ((0, na), (1, nb)):
        o = np.argsort(rng.exponential(width, (count, n)) + np.arange(n), axis=1)[:, :occ]
        for c in range(occ):
            key |= np.uint64(1) << (2 * o[:, c] + spin).astype(np.uint64)
    return key


def _state(n, na, nb, count, width, seed):
    rng = np.random.default_rng(seed)
    got = np.zeros(0, dtype=np.uint64)
    while len(got) < count:
        got = np.unique(np.concatenate([got, _keys(rng, n, na, nb, count, width)]))
    return rng.permutation(got)[:count]


def _around(n, na, nb, count):
    """Random determinants, and every one that holds a given na - 2 alphas and
    nb - 1 betas."""
    keys = [sum(1 << (2 * p) for p in range(na - 2)) | sum(1 << (2 * p + 1) for p in range(nb - 1)) |
            1 << (2 * a) | 1 << (2 * b) | 1 << (2 * c + 1)
            for a in range(na - 2, n) for b in range(na - 2, a) for c in range(nb - 1, n)]
    keys = np.union1d(np.array(keys, dtype=np.uint64), _state(n, na, nb, count, 1e6, 4))
    return np.random.default_rng(5).permutation(keys)


@pytest.mark.parametrize("n,na,nb,count,width,taken", [
    (15, 6, 5, 40000, 6.0, True),
    (20, 3, 3, 50000, 1e6, True),
    (32, 3, 3, 30000, 6.0, True),
    (12, 6, 6, 853776, 1e6, True),
    (20, 4, 4, 10000, 0.0, True),
    (32, 2, 2, 100000, 1e6, False),
])
def test_rows_against_join(n, na, nb, count, width, taken):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import swcs
    h, eri = make_integrals(n, n, 50 + n)
    ref = sum(1 << (2 * p) for p in range(na)) | sum(1 << (2 * p + 1) for p in range(nb))
    ctx = swcs.make_context(n, na, nb, h, eri, enumerate_pool(n), ref)
    keys = _state(n, na, nb, count, width, 900 + n) if width else _around(n, na, nb, count)
    rng = np.random.default_rng(6)
    ctx.set_state(keys, rng.standard_normal(len(keys)) * 10.0 ** rng.uniform(-4, 0, len(keys)))
    print(f"[rows] {n} orbitals, {na}+{nb} electrons, {len(keys)} determinants", flush=True)
    g = ctx.pool_gradients()
    auto = ctx.pool_stats()["keys"]
    ctx.set_pool_method("join")
    ref = ctx.pool_gradients()
    assert (auto == len(keys) * math.comb(na + nb, 3)) == taken
    # as between the other paths: sums of the same terms in FP64
    assert np.abs(ref).max() > 1e-6
    assert np.abs(g - ref).max() < 1e-12 * max(1.0, np.abs(ref).max())
    ctx.close()
