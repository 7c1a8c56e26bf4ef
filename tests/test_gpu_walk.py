"""Adjoint gradients of chains that grow past what the walk over the logs keeps
in LDS (16,384 entries): the gates before that touch pairs with entries that a
later gate appends (pruned partners), plain and generator chains, against the
oracle."""
import numpy as np
import pytest

import oracle
from paper_2411_07920_amd import spin
from paper_2411_07920_amd.inputs import draw_ansatz, enumerate_pool, make_integrals

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gens,eps", [(False, 2e-4), (True, 2e-4)])
def test_walk_past_lds(gens, eps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import swcs
    n, na, nb, M = 10, 5, 5, 130
    h, eri = make_integrals(n, n, 95)
    pool = enumerate_pool(n)
    ref = (1 << (na + nb)) - 1
    c = swcs.make_context(n, na, nb, h, eri, pool, ref)
    orc = oracle.Oracle(n, na, nb, h, eri)
    ops, theta = draw_ansatz(len(pool), M, -0.8, 0.8, 96)
    if gens:
        gp = spin.spin_complemented(pool)
        rng = np.random.default_rng(97)
        g = rng.integers(0, len(gp), M)
        g[::3] = rng.choice(np.flatnonzero(gp.overlap), len(g[::3]))
        rows = spin.gen_rows(gp, g)
        c.apply_generators(rows, theta, eps)
        st = oracle.Oracle.apply_gen_ansatz(pool, rows, theta, eps, ref)
        dE_ref, E_ref = orc.gen_param_gradients(pool, rows, theta, eps, ref)
    else:
        c.apply_ansatz(ops, theta, eps)
        st = oracle.Oracle.apply_ansatz(pool, ops, theta, eps, ref)
        dE_ref, E_ref = orc.param_gradients(pool, ops, theta, eps, ref)
    stored, alive = c.state_counts()
    print(f"[walk] {stored} stored, {alive} alive", flush=True)
    assert alive == len(st)
    dE, E = c.param_gradients(M)
    assert abs(E - E_ref) < 1e-10 and np.abs(dE - dE_ref).max() < 1e-10
    assert stored > 16384
    c.close()
