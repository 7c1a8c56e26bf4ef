"""Which pass forms sigma_P of a large state: AUTO takes the spin strings where the
tests against hole pairs mean to cover them, and leaves a crowded full sector to hole
pairs.  Each pass has a kernel timer of its own."""
import pytest

from test_gpu_strings import _state
from paper_2411_07920_amd.inputs import enumerate_pool, make_integrals

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,na,nb,count,strings", [
    (26, 8, 8, 40000, True), (16, 5, 1, 60000, True), (15, 6, 5, 40000, True), (13, 2, 7, 70000, True),
    (32, 3, 3, 20000, True), (32, 16, 16, 5000, True), (32, 5, 4, 20000, True), (11, 5, 4, 152460, True),
    (24, 0, 10, 20000, True), (12, 6, 6, 853776, False)])
def test_route(n, na, nb, count, strings):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_07920_amd import swcs
    h, eri = make_integrals(n, n, n)
    ref = sum(1 << (2 * p) for p in range(na)) | sum(1 << (2 * p + 1) for p in range(nb))
    c = swcs.make_context(n, na, nb, h, eri, enumerate_pool(n), ref)
    c.set_state(*_state(n, na, nb, count, 7 * n + na))
    runs = {}
    for method in ("auto", "hole_pairs"):
        c.set_sigma_method(method)
        for kernel in ("strings", "holepair"):
            c.timer_start(kernel)
            c.energy()
            runs[method, kernel] = c.timer_stop()[0]
    print(f"[route] {n} orbitals, {na}+{nb}: {runs}", flush=True)
    assert runs["hole_pairs", "strings"] == 0 and runs["hole_pairs", "holepair"] == 3
    assert runs["auto", "strings"] == (2 if strings else 0)
    assert runs["auto", "holepair"] == (0 if strings else 3)
    c.close()
