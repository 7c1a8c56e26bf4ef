"""Per-gate active counts (swcs_gate_active) of chains that the single-workgroup kernel
took over from the multi-block one: sectors below its capacity and overlapping
generators, against a count over the stored keys before each gate."""
import numpy as np
import pytest

import oracle
from paper_2411_07920_amd import spin
from paper_2411_07920_amd.inputs import enumerate_pool, make_integrals

pytestmark = pytest.mark.gpu


def _acts(row, keys):
    P, Q, R, S = (int(x) for x in row)
    cre, ann = ((1 << P | 1 << Q), (1 << R | 1 << S)) if R >= 0 else (1 << P, 1 << Q)
    cre, ann = np.uint64(cre), np.uint64(ann)
    return (((keys & ann) == ann) & ((keys & cre) == 0)) | (((keys & cre) == cre) & ((keys & ann) == 0))


@pytest.mark.parametrize("n,ne,M,generators", [(3, 2, 10, False), (6, 4, 30, False), (7, 6, 40, False),
                                               (4, 4, 30, True), (7, 6, 40, True), (9, 6, 30, True)])
def test_counts(n, ne, M, generators):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import swcs
    h, eri = make_integrals(n, n, 90 + n)
    pool = enumerate_pool(n)
    ref = (1 << ne) - 1
    rng = np.random.default_rng(91 + n)
    theta = rng.uniform(-0.8, 0.8, M)
    c = swcs.make_context(n, ne // 2, ne // 2, h, eri, pool, ref)
    want = []
    if generators:  # overlapping ones: a unitary each
        gp = spin.spin_complemented(pool)
        rows = spin.gen_rows(gp, rng.choice(np.flatnonzero(gp.overlap), M))
        for g in range(M):
            keys = oracle.Oracle.apply_gen_ansatz(pool, rows[:g], theta[:g], 0.0, ref, 0).export()[0]
            want.append(int((_acts(pool[rows[g][0]], keys) | _acts(pool[rows[g][1]], keys)).sum()))
        c.apply_generators(rows, theta)
    else:
        ops = rng.choice(len(pool), M).astype(np.int32)
        for g in range(M):
            keys = oracle.Oracle.apply_ansatz(pool, ops[:g], theta[:g], 0.0, ref).export()[0]
            want.append(int(_acts(pool[ops[g]], keys).sum()))
        c.apply_ansatz(ops, theta)
    assert c.state_counts()[0] <= 4096 and sum(want) > 0
    assert c.gate_active(M).tolist() == want
    c.close()
