"""Pool gradients from the three-body density matrix (taken by AUTO for large
states) against the sort-and-join and accumulation-table paths, which the
oracle pins on smaller states: orbital counts on both sides of the matrix
tiles (16 orbitals per row tile, 4 per k step), unequal and single spins,
pruned entries, hash-class batches, subsets, and a state too crowded for it."""
import math

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


def _state(n, na, nb, count, width, seed):
    """Distinct determinants around the reference: each spin occupies the
    orbitals of smallest orbital number plus exponential noise of mean width."""
    rng = np.random.default_rng(seed)
    got = np.zeros(0, dtype=np.uint64)
    one = np.uint64(1)
    while len(got) < count:
        key = np.zeros(2 * count, dtype=np.uint64)
        for spin, occ in ((0, na), (1, nb)):
            o = np.argsort(rng.exponential(width, (2 * count, n)) + np.arange(n), axis=1)[:, :occ]
            for c in range(occ):
                key |= one << (2 * o[:, c] + spin).astype(np.uint64)
        got = np.unique(np.concatenate([got, key]))
    keys = rng.permutation(got)[:count]
    return keys, rng.standard_normal(count) * 10.0 ** rng.uniform(-4, 0, count)


def _context(swcs, n, na, nb):
    h, eri = make_integrals(n, n, 50 + n)
    pool = enumerate_pool(n)
    ref = sum(1 << (2 * p) for p in range(na)) | sum(1 << (2 * p + 1) for p in range(nb))
    return swcs.make_context(n, na, nb, h, eri, pool, ref), pool


def _triples(ne):
    return math.comb(ne, 3)


# every sum is FP64 over terms of the same sign pattern as the gradient's own:
# the paths may differ by rounding only
REL = 1e-12


@pytest.mark.parametrize("n,na,nb,count,width,batches", [
    (26, 8, 8, 2500, 6.0, 1),     # seven k steps, two row tiles, ragged both ways
    (20, 6, 6, 6000, 6.0, 1),     # five full k steps
    (17, 6, 5, 9000, 6.0, 1),     # one orbital beyond a row tile; odd electron count
    (16, 7, 4, 9000, 6.0, 1),     # exactly one row tile
    (13, 5, 5, 15000, 1e6, 1),    # one row tile, last k step of one orbital
    (30, 8, 0, 25000, 1e6, 1),    # one spin only
    (25, 1, 7, 10000, 1e6, 1),    # a lone alpha: no pair of that spin
    (20, 16, 16, 60000, 1e6, 2),  # 4,960 triples a determinant: two hash classes
])
def test_density_matrix_against_join(swcs, n, na, nb, count, width, batches):
    ctx, pool = _context(swcs, n, na, nb)
    keys, amps = _state(n, na, nb, count, width, 900 + n)
    ctx.set_state(keys, amps)
    print(f"[density] {n} orbitals, {na}+{nb} electrons, {count} determinants", flush=True)
    g = ctx.pool_gradients()
    st = ctx.pool_stats()
    assert st["keys"] == count * _triples(na + nb) and st["table_slots"] == 0 and st["batches"] == batches
    sub = np.sort(np.random.default_rng(2).choice(len(pool), (3 * len(pool)) // 5, replace=False)).astype(np.int32)
    g_sub = ctx.pool_gradients(sub)
    ctx.set_pool_method("join")
    ref = ctx.pool_gradients()
    assert ctx.pool_stats()["keys"] != st["keys"]
    tol = REL * max(1.0, np.abs(ref).max())
    assert np.abs(ref).max() > 1e-6
    assert np.abs(g - ref).max() < tol
    assert np.abs(g_sub - ref[sub]).max() < tol
    ctx.close()


def test_density_matrix_screened_pruned_and_repeated(swcs):
    """A pruned ansatz state (dead entries stored): the screened entry points
    (host and device) and the whole pool agree with the accumulation table, an
    index outside the pool gives NaN, and a second, smaller state on the same
    context is not touched by what the first left in the buffers."""
    import torch
    n, na, nb = 26, 8, 8
    ctx, pool = _context(swcs, n, na, nb)
    rng = np.random.default_rng(5)
    ref = sum(1 << p for p in range(na + nb))
    ann = np.array([sum(1 << int(x) for x in r[2:]) if r[2] >= 0 else 1 << int(r[1]) for r in pool], dtype=object)
    exc = [k for k in range(len(pool)) if (ref & ann[k]) == ann[k] and not any((ref >> int(x)) & 1 for x in (
        pool[k][:2] if pool[k][2] >= 0 else pool[k][:1]))]
    for M in (40, 34):
        ops = rng.choice(exc, M, replace=False).astype(np.int32)
        ctx.apply_ansatz(ops, rng.uniform(-0.2, 0.2, M), 1e-6)
        stored, alive = ctx.state_counts()
        assert stored > alive > 1500
        print(f"[density] {alive} of {stored} entries alive", flush=True)
        ctx.set_pool_method("table")
        want = ctx.pool_gradients()
        ctx.set_pool_method("auto")
        g = ctx.pool_gradients()
        assert ctx.pool_stats()["keys"] == alive * _triples(16)
        tol = REL * max(1.0, np.abs(want).max())
        assert np.abs(g - want).max() < tol
        sub = rng.choice(len(pool), 15000, replace=False).astype(np.int32)
        assert np.abs(ctx.pool_gradients(sub) - want[sub]).max() < tol
        sub[7] = len(pool)
        out = torch.zeros(len(sub), dtype=torch.float64, device="cuda")
        ctx.pool_gradients_device(torch.from_numpy(sub).cuda(), out)
        got = out.cpu().numpy()
        ok = np.arange(len(sub)) != 7
        assert np.isnan(got[7]) and np.abs(got[ok] - want[sub[ok]]).max() < tol
    ctx.close()


def test_crowded_state_stays_on_the_join(swcs):
    """A full sector (63,504 determinants of 10 orbitals, 5 + 5 electrons) has
    more pairs within a triple excitation than connections: AUTO joins."""
    ctx, _ = _context(swcs, 10, 5, 5)
    keys, amps = _state(10, 5, 5, 63504, 1e6, 3)
    ctx.set_state(keys, amps)
    g = ctx.pool_gradients()
    auto = ctx.pool_stats()
    ctx.set_pool_method("join")
    ref = ctx.pool_gradients()
    assert auto["keys"] == ctx.pool_stats()["keys"] == 63504
    assert np.abs(g - ref).max() < REL
    ctx.close()
