"""The hash index over blocks of keys (stateToIndex) against the oracle's
lookup, bit for bit: every representative, and keys that share its block,
its group or neighbouring groups -- of the sector's weight and of others --
so that a wrong number inside a block or a group found in the wrong line
shows."""
import numpy as np
import pytest

import oracle
from workloads import configs, lattice, rng, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402


def _ring(n, w, k, refl, inv):
    g = lattice.ring_group(n, k, refl, inv)
    return configs.sector_from_arrays(f"ring{n}_w{w}", n, w, g.perm, g.flip, g.chi,
                                      terms.heisenberg_terms([(0, 1, 1.0)]))


def _torus(lx, ly, w, kx):
    g = lattice.torus_group(lx, ly, kx, 0, "none", None, 0)
    return configs.sector_from_arrays(f"torus{lx}x{ly}_w{w}", lx * ly, w, g.perm, g.flip, g.chi,
                                      terms.heisenberg_terms([(0, 1, 1.0)]))


@pytest.mark.parametrize("sec", [_ring(2, 1, 0, 0, 1), _ring(6, 3, 0, 0, 0), _ring(9, -1, 0, 1, 0),
                                 _ring(14, -1, 3, 0, 0), _ring(20, 10, 0, 1, 1), _ring(23, 11, 5, 0, 0),
                                 _ring(40, 4, 0, 1, 0), _ring(57, 3, 0, 1, 0), _ring(60, 4, 7, 0, 0),
                                 _ring(64, 3, 1, 0, 0), _torus(4, 5, 10, 2), _torus(6, 6, 5, 3)],
                         ids=lambda s: s.name)
def test_lookup_in_and_around_blocks(sec):
    print(f"[index] {sec.name}", flush=True)
    reps, stab = oracle.enumerate_basis(oracle.Problem(sec))
    b = ls.ls_basis_build(sec)
    n = sec.n_sites
    full = np.uint64((1 << n) - 1) if n < 64 else np.uint64(2 ** 64 - 1)
    some = reps[rng.counter_u64(3, np.arange(4000, dtype=np.uint64)) % np.uint64(max(1, len(reps)))]
    near = [reps, some ^ np.uint64(3), some ^ np.uint64(5), some ^ np.uint64(1), some ^ np.uint64(96),
            some ^ np.uint64(1 << 7), some ^ np.uint64(3 << 9), some + np.uint64(1), some - np.uint64(1),
            rng.counter_u64(9, np.arange(4000, dtype=np.uint64)), np.array([0, full], np.uint64)]
    keys = np.concatenate([k & full for k in near]).astype(np.uint64)
    got = b.index_lookup(torch.from_numpy(keys.view(np.int64)).cuda()).cpu().numpy()
    assert np.array_equal(got, oracle.index_lookup(reps, keys))
    b.close()
