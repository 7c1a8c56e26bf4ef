"""Sorted export of states around the counts where the radix sort changes its
tiling (65,536 and 1,048,576 entries) and its scan goes from one block to many
(4,096 counts), against a sort on the host."""
import numpy as np
import pytest

from paper_2411_07920_amd.inputs import draw_synthetic_state, enumerate_pool, make_integrals, reference_key

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


@pytest.fixture(scope="module")
def drawn():
    return np.asarray(draw_synthetic_state(N, NE // 2, NE // 2, (1 << 20) + 4097, 5)[0])


@pytest.mark.parametrize("n", [1, 2, 4096, 4097, 65535, 65536, 65537, (1 << 20) - 1, 1 << 20, (1 << 20) + 4097])
def test_export_sorted(ctx, drawn, n):
    rng = np.random.default_rng(n)
    keys = rng.permutation(drawn)[:n]
    amps = rng.standard_normal(n)
    ctx.set_state(keys, amps)
    k, a = ctx.get_state()
    o = np.argsort(keys)
    assert np.array_equal(k, keys[o]) and np.array_equal(a, amps[o])


@pytest.mark.parametrize("n", [3, 1000, 4095, 4096, 4097])
def test_export_of_pruned_states(ctx, n):
    """Dead entries among the stored ones, on both sides of the export's switch
    from one workgroup to the radix sort."""
    keys = np.random.default_rng(n).permutation(np.asarray(draw_synthetic_state(N, NE // 2, NE // 2, 3 * n, 8)[0]))[:n]
    amps = np.random.default_rng(n + 1).standard_normal(n)
    amps[::3] *= 1e-6
    ctx.set_state(keys, amps)
    op = int(np.flatnonzero((enumerate_pool(N) == np.array([31, 1, -1, -1])).all(1))[0])
    ctx.apply_gates([op], [0.0], 1e-3)  # an angle of 0 moves nothing; the threshold prunes
    k, a = ctx.get_state()
    keep = np.abs(amps) >= 1e-3
    o = np.argsort(keys[keep])
    assert np.array_equal(k, keys[keep][o]) and np.array_equal(a, amps[keep][o])
