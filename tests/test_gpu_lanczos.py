"""A lone large solve (Gram-Schmidt passes joined in one reading of the Krylov
space) against the same solve in a mix (separate passes): the same bits."""
import pytest

from workloads import lattice, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402


@pytest.mark.parametrize("reorth", ["full", "selective"])
def test_joined_passes_give_the_separate_passes_bits(reorth):
    """24 sites without symmetry (2,704,156 states, above the bound of the
    batched kernels); 8, 9 and 49 vectors and more lie on both sides of the
    sizes of the joined kernel."""
    t = terms.heisenberg_terms(lattice.ring_bonds(24, 1.0, 0.2))
    b = ls.Basis(24, 12, [list(range(24))], [0], [[1.0, 0.0]])
    assert b.dim >= 1 << 21
    op = ls.ls_operator_create(b, t)
    for m in (8, 9, 52):
        print(f"[gpu] lanczos {reorth} {m}", flush=True)
        alone = op.lanczos(m, tol=0.0, seed=3, reorth=reorth)
        pair = [ls.Solver(op, m, tol=0.0, seed=3, reorth=reorth), ls.Solver(op, m, tol=0.0, seed=3, reorth=reorth)]
        ls.Solver.step_all(pair, steps=m)
        for s in pair:
            r = s.result()
            assert r["done"] and r["e0"] == alone["e0"] and r["resid"] == alone["resid"], (m, r, alone)
            s.close()
    op.close()
    b.close()
