"""Density-matrix rows in LDS where the subsets are split into hash classes (more than
2^28 records): a crowded state, and one whose first or second class holds a subset of
more determinants than the pass orders, so that this class goes by pairs and the other
by rows into the same matrix.  Against the external sigma of a few hundred operators."""
import itertools
import math

import numpy as np
import pytest

from paper_2411_07920_amd.inputs import enumerate_pool, make_integrals

pytestmark = pytest.mark.gpu

M64 = (1 << 64) - 1


def _mix64(x):
    x ^= x >> 30
    x = x * 0xbf58476d1ce4e5b9 & M64
    x ^= x >> 27
    x = x * 0x94d049bb133111eb & M64
    return x ^ x >> 31


def _active(core, active, occ, count, seed):
    """`count` determinants of `core` filled orbitals and occ + occ electrons in the
    next `active` ones."""
    strings = np.array([sum(1 << (2 * p) for p in range(core)) | sum(1 << (2 * (core + p)) for p in c)
                        for c in itertools.combinations(range(active), occ)], dtype=np.uint64)
    at = np.random.default_rng(seed).choice(len(strings) ** 2, count, replace=False)
    return strings[at // len(strings)] | strings[at % len(strings)] << np.uint64(1)


def _around(n, na, nb, cls):
    """Every determinant that holds one subset of na - 2 alphas and nb - 1 betas, the
    subset chosen to be in hash class cls of two."""
    for shift in range(n - na):
        al, be = range(shift, shift + na - 2), range(nb - 1)
        S = sum(1 << (2 * p) for p in al) | sum(1 << (2 * p + 1) for p in be)
        if _mix64(S) >> 56 & 1 == cls:
            break
    else:
        raise AssertionError("no subset of this class")
    fa, fb = [p for p in range(n) if p not in al], [p for p in range(n) if p not in be]
    return np.array([S | 1 << (2 * a) | 1 << (2 * b) | 1 << (2 * c + 1)
                     for a, b in itertools.combinations(fa, 2) for c in fb], dtype=np.uint64)


@pytest.mark.parametrize("case", ["crowded", "long bucket in class 0", "long bucket in class 1"])
def test_rows_in_two_classes(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import swcs
    if case == "crowded":
        n, na, nb = 13, 6, 6
        keys = _active(0, 13, 6, 1_400_000, 1)
    else:
        n, na, nb = 24, 8, 8
        more = _around(n, na, nb, int(case[-1]))
        assert len(more) > 2048
        keys = np.random.default_rng(2).permutation(np.union1d(_active(2, 13, 6, 500_000, 3), more))
    total = len(keys) * math.comb(na + nb, 3)
    assert 1 << 28 < total < 1 << 29
    h, eri = make_integrals(n, n, 50 + n)
    pool = enumerate_pool(n)
    ref = sum(1 << (2 * p) for p in range(na)) | sum(1 << (2 * p + 1) for p in range(nb))
    ctx = swcs.make_context(n, na, nb, h, eri, pool, ref)
    rng = np.random.default_rng(6)
    ctx.set_state(keys, rng.standard_normal(len(keys)) * 10.0 ** rng.uniform(-4, 0, len(keys)))
    print(f"[classes] {case}: {len(keys)} determinants, {total} records", flush=True)
    g = ctx.pool_gradients()
    st = ctx.pool_stats()
    assert st["keys"] == total and st["batches"] == 2
    some = np.sort(rng.choice(len(pool), 300, replace=False)).astype(np.int32)
    ctx.set_pool_method("table")
    want = ctx.pool_gradients(some)
    print(f"[classes] {np.abs(g[some] - want).max()} of {np.abs(want).max()}", flush=True)
    # sums of the same terms in FP64, as between the other paths
    assert np.abs(want).max() > 1e-6
    assert np.abs(g[some] - want).max() < 1e-12 * np.abs(want).max()
    ctx.close()
