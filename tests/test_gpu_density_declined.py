"""States that are too crowded for the density matrix are found so once, by the sample
or by the pass itself, and joined; the finding does not outlive the state."""
import itertools
import math

import numpy as np
import pytest

from test_gpu_density import _context, _state

pytestmark = pytest.mark.gpu


def _active(n, core, active, occ, count, seed):
    """Determinants of `core` filled orbitals and occ + occ electrons in the next
    `active` ones."""
    strings = [sum(1 << (2 * p) for p in range(core)) | sum(1 << (2 * (core + p)) for p in c)
               for c in itertools.combinations(range(active), occ)]
    keys = np.array([a | b << 1 for a in strings for b in strings], dtype=np.uint64)
    rng = np.random.default_rng(seed)
    return rng.permutation(keys)[:count], rng.standard_normal(count) * 10.0 ** rng.uniform(-4, 0, count)


@pytest.mark.parametrize("by", ["sample", "bucket"])
def test_finding_belongs_to_the_state(by):
    """By the sample: 4,600 determinants of 9 active orbitals, 3,660 pairs each
    against 3,240 connections.  By the pass: a subset with more than 1,024."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import swcs
    if by == "sample":
        n, na, nb = 14, 8, 8
        states = {"crowded": _active(n, 2, 9, 6, 4600, 3), "sparse": _state(n, na, nb, 4600, 1e6, 4)}
    else:
        n, na, nb = 32, 2, 2
        states = {"crowded": _state(n, na, nb, 100000, 1e6, 3)}
    ctx, pool = _context(swcs, n, na, nb)
    want = {}
    ctx.set_pool_method("join")
    for name, s in states.items():
        ctx.set_state(*s)
        want[name] = ctx.pool_gradients()
    ctx.set_pool_method("auto")
    for name in ("crowded", "sparse", "crowded"):
        if name not in states:
            continue
        ctx.set_state(*states[name])
        for _ in range(3):
            g = ctx.pool_gradients()
            keys = ctx.pool_stats()["keys"]
            print(f"[declined] {name}: {keys} keys", flush=True)
            assert (keys == len(states[name][0]) * math.comb(na + nb, 3)) == (name == "sparse")
            assert np.abs(g - want[name]).max() < 1e-12 * np.abs(want[name]).max()
    # a gate changes the state: looked at again, with the same finding
    ctx.apply_gates(np.array([0]), np.array([0.1]))
    g = ctx.pool_gradients()
    ctx.set_pool_method("join")
    ref = ctx.pool_gradients()
    assert np.abs(g - ref).max() < 1e-12 * np.abs(ref).max()
    ctx.close()
