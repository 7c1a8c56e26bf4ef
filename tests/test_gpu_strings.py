"""sigma_P by spin strings (taken by AUTO for large states) against hole-pair
grouping, which the oracle pins on smaller states: unequal spins, one electron of
a spin or none, all strings of a spin present, 32 orbitals with 256
single excitations, rows in runs shorter and longer than a wavefront's eight,
pruned entries, and a full sector that AUTO leaves to hole pairs."""
import numpy as np
import pytest

from paper_2411_07920_amd.inputs import enumerate_pool, make_integrals

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def swcs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import swcs as mod
    mod.load()
    return mod


def _state(n, na, nb, count, seed):
    """Distinct random determinants, the whole sector if it is no larger."""
    rng = np.random.default_rng(seed)
    got = np.zeros(0, dtype=np.uint64)
    for _ in range(40):
        key = np.zeros(count, dtype=np.uint64)
        for spin, occ in ((0, na), (1, nb)):
            o = np.argsort(rng.random((count, n)), axis=1)[:, :occ]
            for c in range(occ):
                key |= np.uint64(1) << (2 * o[:, c] + spin).astype(np.uint64)
        got = np.unique(np.concatenate([got, key]))
        if len(got) >= count:
            break
    keys = rng.permutation(got)[:count]
    return keys, rng.standard_normal(len(keys)) * 10.0 ** rng.uniform(-4, 0, len(keys))


@pytest.mark.parametrize("n,na,nb,count", [
    (26, 8, 8, 40000), (16, 5, 1, 60000), (15, 6, 5, 40000), (13, 2, 7, 70000), (32, 3, 3, 20000),
    (32, 16, 16, 5000), (32, 5, 4, 20000), (11, 5, 4, 152460), (24, 0, 10, 20000), (12, 6, 6, 853776)])
def test_against_hole_pairs(swcs, n, na, nb, count):
    import torch
    h, eri = make_integrals(n, n, n)
    pool = enumerate_pool(n)
    ref = sum(1 << (2 * p) for p in range(na)) | sum(1 << (2 * p + 1) for p in range(nb))
    c = swcs.Context(n, na, nb)
    try:
        c.use_torch_allocator()
        c.set_integrals(h, eri)
        c.set_reference(ref)
        c.set_pool(pool)
        keys, amps = _state(n, na, nb, count, 7 * n + na)
        c.set_state(keys, amps)
        for dead in (False, True):
            if dead:  # a small rotation moves little; the threshold kills a part of the entries
                c.apply_gates(np.array([len(pool) // 2]), np.array([0.01]), eps=1e-3)
            e = {}
            for m in ("auto", "hole_pairs"):
                c.set_sigma_method(m)
                e[m] = (*c.energy(), *c.sigma_projected())
            (e1, _, _, k1, s1), (e2, _, norm2, k2, s2) = e["auto"], e["hole_pairs"]
            assert np.array_equal(k1, k2)
            # at most some 5,000 terms a sum, each correct to a few 2^-53
            assert np.linalg.norm(s1 - s2) <= 1e-12 * np.linalg.norm(s2)
            assert abs(e1 - e2) <= 1e-12 * np.linalg.norm(s2) / np.sqrt(norm2)
        torch.cuda.synchronize()
    finally:
        c.close()
