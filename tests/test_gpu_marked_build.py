"""Builds that mark their members, at the sizes where the marks of a lane or
the walk degenerate, against the oracle: representatives and stabilizers."""
import numpy as np
import pytest

import oracle
from workloads import configs, lattice, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402


def _half_turn(n, inv=0):
    gens = [([(i + 2) % n for i in range(n)], 0, 1.0)]
    if inv:
        gens.append((list(range(n)), 1, complex(inv)))
    return lattice.close_group(n, gens)


def _pair_swap(n, chi):
    return lattice.close_group(n, [([1, 0] + list(range(2, n)), 0, complex(chi))])


@pytest.mark.parametrize("name,n,w,group", [
    ("swap", 2, 1, lambda: _pair_swap(2, 1)), ("swap", 3, -1, lambda: _pair_swap(3, -1)),
    ("swap0", 5, 0, lambda: _pair_swap(5, 1)), ("swapfull", 5, 5, lambda: _pair_swap(5, 1)),
    ("none", 6, 0, lambda: _pair_swap(6, -1)), ("swap64", 64, 2, lambda: _pair_swap(64, -1)),
    ("swap64all", 64, 64, lambda: _pair_swap(64, 1)), ("swap64less", 64, 63, lambda: _pair_swap(64, 1)),
    ("turn24", 24, 12, lambda: _half_turn(24)), ("turn24i", 24, 12, lambda: _half_turn(24, -1)),     # 3 candidates a lane at least
    ("turn20", 20, -1, lambda: _half_turn(20)), ("turn34", 34, 6, lambda: _half_turn(34)),
    ("plain18", 18, 9, lambda: lattice.trivial_group(18)), ("plain15", 15, -1, lambda: lattice.trivial_group(15)),
    ("relabel20", 20, 10, lambda: lattice.relabel_group(lattice.ring_group(20, 0, 1, 1), np.random.default_rng(3).permutation(20))),
    ("torus4x6", 24, 11, lambda: lattice.torus_group(4, 6, 0, 0, "c2v")), ("torus5x5", 25, 12, lambda: lattice.torus_group(5, 5, 1, 0, "none"))],
    ids=lambda v: str(v) if not callable(v) else "")
def test_members_and_stabilizers(name, n, w, group):
    g = group()
    sec = configs.sector_from_arrays(f"{name}_{n}_{w}", n, w, g.perm, g.flip, g.chi, terms.heisenberg_terms([(0, 1, 1.0)]))
    print(f"[gpu] {sec.name}", flush=True)
    reps, stab = oracle.enumerate_basis(oracle.Problem(sec))
    b = ls.ls_basis_build(sec)
    r, s = b.copy()
    assert np.array_equal(r.cpu().numpy().view(np.uint64), reps)
    assert np.array_equal(s.cpu().numpy().view(np.uint16), stab)
    assert ls.ls_sector_count(sec)[0] == len(reps)
