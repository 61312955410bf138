"""state_info on both sides of the line between the torus search and the walk
of all images, with characters that are trivial, signs and phases, against
the oracle."""
import numpy as np
import pytest

import oracle
from workloads import configs, lattice, rng, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402


@pytest.mark.parametrize("lx,ly,w,kx,point,chars,inv", [
    (6, 5, 6, 0, "c2v", None, 0), (6, 5, 5, 0, "c2v", None, 0), (6, 5, 6, 0, "c2v", dict(mx=-1), 0),   # 6, 5 up: search, walk
    (5, 5, 19, 0, "full", None, 0), (5, 5, 20, 0, "full", dict(rot=-1), 0), (5, 5, 6, 0, "full", dict(mx=-1, my=-1), 0),
    (4, 4, 8, 0, "full", None, 1), (4, 4, 8, 0, "full", dict(rot=-1), -1), (4, 6, 12, 0, "c2v", None, 1),
    (6, 4, 12, 3, "none", None, -1), (4, 8, 4, 1, "none", None, 0), (2, 8, -1, 0, "c2v", dict(my=-1), 1),
    (5, 4, -1, 0, "c2v", None, 1), (6, 6, 5, 0, "full", dict(rot=-1), 0), (6, 6, 31, 0, "full", None, 0)])
def test_search_and_walk(lx, ly, w, kx, point, chars, inv):
    n = lx * ly
    g = lattice.torus_group(lx, ly, kx, 0, point, chars, inv)
    sec = configs.sector_from_arrays(f"states{lx}x{ly}_w{w}", n, w, g.perm, g.flip, g.chi,
                                     terms.heisenberg_terms(lattice.torus_bonds(lx, ly)))
    print(f"[gpu] {sec.name} {point} {chars} {inv}", flush=True)
    P = oracle.Problem(sec)
    b = ls.ls_basis_build(sec)
    reps = b.copy()[0].cpu().numpy().view(np.uint64)[:3000]
    full = np.uint64((1 << n) - 1)
    words = rng.counter_u64(4, np.arange(3000, dtype=np.uint64)) & full
    sparse = (words & rng.counter_u64(5, np.arange(3000, dtype=np.uint64)) & rng.counter_u64(6, np.arange(3000, dtype=np.uint64))) & full
    rows = np.array([sum(((1 << lx) - 1) << (lx * y) for y in range(ly) if (m >> y) & 1) for m in range(1 << ly)], np.uint64)
    turned = ((reps << np.uint64(3)) | (reps >> np.uint64(n - 3))) & full
    states = np.concatenate([reps, turned, words, sparse, rows, ~rows & full, np.array([0, full, full + np.uint64(1)], np.uint64)])
    got = [t.cpu().numpy() for t in b.state_info(torch.from_numpy(states.view(np.int64)).cuda())]
    want = oracle.state_info(P, states)
    assert np.array_equal(got[0].view(np.uint64), want[0])
    chi = np.asarray(want[1])
    chi = np.stack([chi.real, chi.imag], axis=1) if np.iscomplexobj(chi) else chi.reshape(len(states), 2)
    assert np.abs(got[1] - chi).max() <= 1e-9          # characters are given to 1e-9
    assert np.abs(got[2] - want[2]).max() <= 1e-15     # one division and one root
