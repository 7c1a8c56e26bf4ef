"""N_CUT selection of states in HBM (more than 4,096 stored determinants)
against a sort on the host: distinct amplitudes, equal ones (the smaller keys
stay), exact zeros, amplitudes that agree in their leading bits, and cuts at
the ends of the range; then adjoint gradients whose replays select the same."""
import numpy as np
import pytest

import oracle
from paper_2411_07920_amd.inputs import draw_ansatz, draw_synthetic_state, enumerate_pool, make_integrals, reference_key

pytestmark = pytest.mark.gpu

N, NE = 16, 8


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import swcs
    h, eri = make_integrals(N, N, 71)
    c = swcs.make_context(N, NE // 2, NE // 2, h, eri, enumerate_pool(N), reference_key(NE))
    yield c
    c.close()


def _amps(kind, n, rng):
    a = rng.standard_normal(n) * 10.0 ** rng.uniform(-9, 0, n)
    if kind == "equal":
        a[:] = 0.25
        a[::3] = -0.25
    elif kind == "steps":  # a few thousand of each of some values
        a = rng.choice([1e-3, -1e-3, 2e-5, 0.5, -3e-8], n)
    elif kind == "zeros":
        a[rng.random(n) < 0.7] = 0.0
    elif kind == "close":  # equal in exponent and the first 24 bits
        a = 0.75 + rng.integers(0, 1 << 20, n) * 2.0 ** -50
        a[::2] *= -1.0
    return a


@pytest.mark.parametrize("kind", ["distinct", "equal", "steps", "zeros", "close"])
@pytest.mark.parametrize("n,cuts", [(4097, (1, 1024, 4096)), (60000, (1, 1025, 30000, 59999, 60000, 70000))])
def test_selection_against_sort(ctx, kind, n, cuts):
    rng = np.random.default_rng(n)
    keys, _ = draw_synthetic_state(N, NE // 2, NE // 2, n, 5)
    amps = _amps(kind, n, rng)
    pool = enumerate_pool(N)
    # an operator that acts on none of the determinants: the gate changes nothing
    lo, hi = 1 << 1, 1 << 31  # beta single from orbital 0 to orbital 15
    free = ((keys & np.uint64(lo)) != 0) == ((keys & np.uint64(hi)) != 0)
    keys, amps = keys[free], amps[free]
    extra, _ = draw_synthetic_state(N, NE // 2, NE // 2, 3 * n, 6)
    extra = extra[((extra & np.uint64(lo)) != 0) == ((extra & np.uint64(hi)) != 0)]
    extra = np.setdiff1d(extra, keys)[: n - len(keys)]
    keys = np.concatenate([keys, extra])
    amps = np.concatenate([amps, _amps(kind, len(extra), rng)])
    assert len(keys) == n
    op = int(np.flatnonzero((pool == np.array([31, 1, -1, -1])).all(1))[0])
    for cut in cuts:
        ctx.set_state(keys, amps)
        print(f"[ncut] {kind} {n} cut {cut}", flush=True)
        got_n = ctx.apply_gates([op], [0.3], 0.0, cut)
        k, a = ctx.get_state()
        order = np.lexsort((keys, -np.abs(amps)))[:cut]
        order = order[np.argsort(keys[order])]
        assert got_n == len(order) and np.array_equal(k, keys[order]) and np.array_equal(a, amps[order])


@pytest.mark.parametrize("kind", ["distinct", "equal", "steps", "zeros", "close"])
@pytest.mark.parametrize("n", [1, 2, 257, 1500, 4096])
def test_selection_in_lds(ctx, kind, n):
    """The same of states that stay in LDS (up to 4,096 determinants): bins of
    up to and more than 256 entries, cuts at both ends."""
    rng = np.random.default_rng(n + 1)
    # one spin-orbital left empty and one filled: the gate's operator acts on
    # none of these determinants
    keys, _ = draw_synthetic_state(N, NE // 2, NE // 2, 8 * n + 400, 7)
    lo, hi = 1 << 1, 1 << 31
    keys = keys[((keys & np.uint64(lo)) != 0) == ((keys & np.uint64(hi)) != 0)][:n]
    assert len(keys) == n
    amps = _amps(kind, n, rng)
    op = int(np.flatnonzero((enumerate_pool(N) == np.array([31, 1, -1, -1])).all(1))[0])
    for cut in sorted({1, max(1, n // 3), max(1, n - 1), n, n + 5}):
        ctx.set_state(keys, amps)
        print(f"[ncut] lds {kind} {n} cut {cut}", flush=True)
        got_n = ctx.apply_gates([op], [0.3], 0.0, cut)
        k, a = ctx.get_state()
        order = np.lexsort((keys, -np.abs(amps)))[:cut]
        order = order[np.argsort(keys[order])]
        assert got_n == len(order) and np.array_equal(k, keys[order]) and np.array_equal(a, amps[order])


def test_adjoint_replays_select_alike():
    """Gradients at N_CUT on a chain whose state leaves LDS: plain rows, and
    with angles of 0 so that exact zeros are at the cut."""
    from paper_2411_07920_amd import swcs
    n, na, nb = 9, 4, 3
    h, eri = make_integrals(n, n, 72)
    pool = enumerate_pool(n)
    ref = sum(1 << (2 * p) for p in range(na)) | sum(1 << (2 * p + 1) for p in range(nb))
    ops, theta = draw_ansatz(len(pool), 260, -0.6, 0.6, 73)
    c = swcs.make_context(n, na, nb, h, eri, pool, ref)
    orc = oracle.Oracle(n, na, nb, h, eri)
    for zero in (False, True):
        th = theta.copy()
        if zero:
            th[::2] = 0.0
        for cut in (700, 4500):
            print(f"[ncut] adjoint cut {cut} zeros {zero}", flush=True)
            st = oracle.Oracle.apply_ansatz(pool, ops, th, 0.0, ref, ncut=cut)
            c.apply_ansatz(ops, th, 0.0, ncut=cut)
            assert c.state_counts()[0] > 4096
            k, a = c.get_state()
            k_ref, a_ref = st.export()
            assert np.array_equal(k, k_ref) and np.array_equal(a, a_ref)
            dE, E = c.param_gradients(len(ops))
            dE_ref, _ = orc.param_gradients(pool, ops, th, 0.0, ref, ncut=cut)
            assert abs(E - orc.energy(st)[0]) < 1e-10 and np.abs(dE - dE_ref).max() < 1e-10
    c.close()
