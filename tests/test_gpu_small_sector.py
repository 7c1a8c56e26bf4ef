"""Chains of sectors smaller than the single-workgroup kernel's capacity (the
arrays then hold the sector, not the capacity) against the oracle: the
smallest sectors, threshold and N_CUT pruning, chains that fill the sector,
and arrays held below the sector, which stay with the multi-block gates."""
import math

import numpy as np
import pytest

import oracle
from paper_2411_07920_amd.inputs import draw_ansatz, enumerate_pool, make_integrals

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,na,nb,M", [(2, 1, 1, 3), (3, 2, 1, 9), (4, 4, 1, 7), (6, 3, 3, 120), (7, 3, 2, 90),
                                       (8, 4, 4, 200)])
def test_against_oracle(n, na, nb, M):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import swcs
    h, eri = make_integrals(n, n, 80 + n)
    pool = enumerate_pool(n)
    ref = sum(1 << (2 * p) for p in range(na)) | sum(1 << (2 * p + 1) for p in range(nb))
    ops, theta = draw_ansatz(len(pool), M, -0.7, 0.7, 81 + n)
    sector = math.comb(n, na) * math.comb(n, nb)
    c = swcs.make_context(n, na, nb, h, eri, pool, ref)
    orc = oracle.Oracle(n, na, nb, h, eri)
    for cap in (0, sector // 2):
        for eps, cut in ((0.0, 0), (1e-2, 0), (0.0, max(1, sector // 3))):
            print(f"[small] {n} {na}+{nb} cap {cap} eps {eps} cut {cut}", flush=True)
            c.set_capacity(cap)
            st = oracle.Oracle.apply_ansatz(pool, ops, theta, eps, ref, ncut=cut)
            try:
                c.apply_ansatz(ops, theta, eps, ncut=cut)
            except swcs.SwcsError as e:
                assert cap and e.code == swcs.SWCS_E_CAPACITY
                continue
            k, a = c.get_state()
            k_ref, a_ref = st.export()
            assert np.array_equal(k, k_ref) and np.array_equal(a, a_ref)
            dE, E = c.param_gradients(M)
            dE_ref, _ = orc.param_gradients(pool, ops, theta, eps, ref, ncut=cut)
            assert abs(E - orc.energy(st)[0]) < 1e-10 and np.abs(dE - dE_ref).max() < 1e-10
    c.close()


@pytest.mark.parametrize("n,ne,M", [(3, 2, 12), (4, 4, 40), (5, 6, 60), (7, 6, 90)])
def test_generators_against_oracle(n, ne, M):
    """Overlapping spin-complemented generators in the single-workgroup chain
    and its adjoint: every generator of the smallest pools, then sectors of up
    to 1,225 determinants filled through stars."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import spin, swcs
    h, eri = make_integrals(n, n, 90 + n)
    pool = enumerate_pool(n)
    gp = spin.spin_complemented(pool)
    ref = (1 << ne) - 1
    rng = np.random.default_rng(91 + n)
    over = np.flatnonzero(gp.overlap)
    gens = rng.integers(0, len(gp), M)
    gens[::2] = rng.choice(over, len(gens[::2]))
    theta = rng.uniform(-0.8, 0.8, M)
    rows = spin.gen_rows(gp, gens)
    orc = oracle.Oracle(n, ne // 2, ne // 2, h, eri)
    c = swcs.make_context(n, ne // 2, ne // 2, h, eri, pool, ref)
    for eps, cut in ((0.0, 0), (2e-2, 0), (0.0, 5)):
        print(f"[small] generators {n} {ne} eps {eps} cut {cut}", flush=True)
        st = oracle.Oracle.apply_gen_ansatz(pool, rows, theta, eps, ref, cut)
        assert c.apply_generators(rows, theta, eps, cut) == len(st)
        k, a = c.get_state()
        k_ref, a_ref = st.export()
        assert np.array_equal(k, k_ref) and np.array_equal(a, a_ref)
        dE, E = c.param_gradients(M)
        dE_ref, E_ref = orc.gen_param_gradients(pool, rows, theta, eps, ref, cut)
        assert abs(E - E_ref) < 1e-10 and np.abs(dE - dE_ref).max() < 1e-10
    c.close()
