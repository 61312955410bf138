"""Batches of one sector built with the hash index and with the bucket search
in one process: the cached choice of one basis is not the other's."""
import numpy as np
import pytest

from workloads import configs, lattice, rng, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402


@pytest.mark.parametrize("first", ["hash", "buckets"])
def test_choices_of_both_layouts(monkeypatch, first):
    n = 20 if first == "hash" else 19
    g = lattice.ring_group(n, 1, 0, 0)
    sec = configs.sector_from_arrays(f"ring{n}", n, n // 2, g.perm, g.flip, g.chi,
                                     terms.heisenberg_terms(lattice.ring_bonds(n, 1.0, 0.4)))
    order = ["hash", "buckets"] if first == "hash" else ["buckets", "hash"]
    ops = []
    for layout in order:
        print(f"[gpu] {sec.name} {layout}", flush=True)
        if layout == "buckets":
            monkeypatch.setenv("LS_ED_SEARCH", "buckets")
        else:
            monkeypatch.delenv("LS_ED_SEARCH", raising=False)
        b = ls.ls_basis_build(sec)
        assert b.dim >= 4096      # smaller sectors are not tuned
        op = ls.ls_operator_create(b, sec.terms)
        x = torch.from_numpy(rng.vector(3, b.dim, 2, complex_=op.is_complex)).cuda()
        y = torch.empty_like(x)
        B = ls.Batch([op], [2])
        B.matvec([x], [y])
        assert torch.equal(y, op.matvec(x))
        op.check()
        ops.append((op, B))
