"""Row groups in steps (several lanes a row, elements exchanged through LDS
round by round) against the two-column product, whose rows one lane sums."""
import numpy as np
import pytest

import oracle
from workloads import configs, lattice, rng, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402


def _all_bonds(n):
    return [(i, j, 1.0) for i in range(n) for j in range(i)]


@pytest.mark.parametrize("name,n,w,group,bonds", [
    ("plain12", 12, 6, lambda: lattice.trivial_group(12), _all_bonds(12)),            # 66 steps: 3 rounds of 32
    ("plain17", 17, 8, lambda: lattice.trivial_group(17), _all_bonds(17)),            # 136 steps: 9 rounds of 16
    ("ring18", 18, 9, lambda: lattice.ring_group(18, 0, 1, 1), _all_bonds(18)),
    ("ring18k2", 18, 8, lambda: lattice.ring_group(18, 2, 0, 0), _all_bonds(18)),     # complex
    ("torus3x6", 18, 9, lambda: lattice.torus_group(3, 6, 0, 0, "full", None, 1), _all_bonds(18)),
    ("torus4x6", 24, 12, lambda: lattice.torus_group(4, 6, 0, 1, "none"), lattice.torus_bonds(4, 6, 1.0, 0.5))],
    ids=lambda v: v if isinstance(v, str) else "")
def test_many_rounds(name, n, w, group, bonds):
    """Every round overwrites the LDS words that the one before it read."""
    g = group()
    sec = configs.sector_from_arrays(name, n, w, g.perm, g.flip, g.chi, terms.heisenberg_terms(bonds))
    print(f"[gpu] {name}", flush=True)
    P = oracle.Problem(sec)
    reps, stab = oracle.enumerate_basis(P)
    b = ls.ls_basis_build(sec)
    op = ls.ls_operator_create(b, sec.terms)
    x = torch.from_numpy(rng.vector(8, len(reps), 2, complex_=op.is_complex)).cuda()
    want = op.matvec(x)[:, 0]
    x1 = x[:, 0].contiguous()
    for _ in range(20):
        assert torch.equal(op.matvec(x1), want)
    ref = oracle.matvec(P, reps, stab, np.ascontiguousarray(x1.cpu().numpy()))
    # a few roundings an element, under 200 elements a row
    assert np.abs(want.cpu().numpy() - ref).max() <= 1e-13 * max(1.0, np.abs(ref).max())
    op.check()


@pytest.mark.parametrize("name,group,w", [("plain", lambda: lattice.trivial_group(12), 6),
                                          ("real", lambda: lattice.ring_group(12, 0, 1, 1), 6),
                                          ("complex", lambda: lattice.ring_group(12, 1, 0, 0), 5),
                                          ("torus", lambda: lattice.torus_group(3, 4, 0, 0, "full", None, 1), 6)],
                         ids=lambda v: v if isinstance(v, str) else "")
def test_signs_of_zero(name, group, w):
    """A step that does not act on a row leaves its sum alone, also a sum of
    -0: vectors of zeros and of a few entries, bit for bit."""
    g = group()
    bonds = lattice.torus_bonds(3, 4, -1.0) if name == "torus" else lattice.ring_bonds(12, -1.0)
    sec = configs.sector_from_arrays(name, 12, w, g.perm, g.flip, g.chi, terms.heisenberg_terms(bonds))
    print(f"[gpu] {name}", flush=True)
    b = ls.ls_basis_build(sec)
    op = ls.ls_operator_create(b, sec.terms)
    dtype = torch.complex128 if op.is_complex else torch.float64
    negative = 0
    for few in (0, 3):
        for zero in (0.0, -0.0):
            x = torch.full((b.dim, 2), zero, dtype=dtype, device="cuda")
            x[:few] = 1.0
            want = op.matvec(x)[:, 0].contiguous().view(torch.int64)
            assert torch.equal(op.matvec(x[:, 0].contiguous()).view(torch.int64), want)
            negative += int((want == -2 ** 63).sum())
    assert negative > 0 or op.is_complex     # (complex sums with an element end at +0)
