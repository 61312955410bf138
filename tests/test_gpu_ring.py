"""The ring search (longest runs of a doubled word) against the oracle."""
import numpy as np
import pytest

import oracle
from workloads import configs, lattice, rng, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402


def _check_states(sec, b):
    """state_info of members, random words of the weight and of others, and
    words with bits past the sites, against the oracle."""
    P = oracle.Problem(sec)
    reps, _ = oracle.enumerate_basis(P)
    n = sec.n_sites
    words = rng.counter_u64(4, np.arange(3000, dtype=np.uint64)) & np.uint64((1 << n) - 1)
    pick = rng.counter_u64(5, np.arange(3000, dtype=np.uint64)) % np.uint64(len(reps))
    k = (rng.counter_u64(6, np.arange(3000, dtype=np.uint64)) % np.uint64(n)).astype(np.uint64)
    full = np.uint64((1 << n) - 1)
    turned = ((reps[pick] << k) | (reps[pick] >> (np.uint64(n) - k))) & full
    states = np.concatenate([reps[:2000], turned, words, np.array([0, full, 1], np.uint64)]).astype(np.uint64)
    got = [t.cpu().numpy() for t in b.state_info(torch.from_numpy(states.view(np.int64)).cuda())]
    want = oracle.state_info(P, states)
    assert np.array_equal(got[0].view(np.uint64), want[0])
    w = want[1]
    w = np.stack([w.real, w.imag], axis=1) if np.iscomplexobj(w) else w.reshape(len(states), 2)
    assert np.abs(got[1] - w).max() <= 1e-9          # characters are given to 1e-9
    assert np.abs(got[2] - want[2]).max() <= 1e-15   # one division and one root


@pytest.mark.parametrize("n,w,k,refl,inv", [
    (4, 2, 0, 1, 1), (5, 2, 0, 1, 0), (6, 3, 3, 0, -1), (10, -1, 0, 1, 1), (11, -1, 3, 0, 0), (16, 8, 8, 1, 1),
    (17, 2, 0, 1, 0), (18, 9, 0, 1, -1), (21, 10, 4, 0, 0), (31, 3, 0, 1, 0), (32, 3, 5, 0, 0), (32, 29, 0, 1, 0),
    (33, 3, 0, 1, 0), (36, 4, 9, 0, 0), (40, 3, 0, 1, 0), (48, 45, 0, 1, 0), (54, 3, 0, 1, 0), (55, 3, 2, 0, 0),
    (63, 3, 0, 1, 0), (63, 3, 1, 0, 0)])
def test_ring_search(n, w, k, refl, inv):
    """Words with runs up to and beyond what the doubled word shows, constant
    and alternating words, with and without spin inversion and mirror, both
    word sizes: basis, indices and products (bit-equal to the stored form)."""
    g = lattice.ring_group(n, k, refl, inv)
    sec = configs.sector_from_arrays(f"ring{n}_w{w}_k{k}_{refl}_{inv}", n, w, g.perm, g.flip, g.chi,
                                     terms.heisenberg_terms(lattice.ring_bonds(n, 1.0, 0.3)))
    print(f"[gpu] {sec.name}", flush=True)
    P = oracle.Problem(sec)
    reps, stab = oracle.enumerate_basis(P)
    b = ls.ls_basis_build(sec)
    assert np.array_equal(b.copy()[0].cpu().numpy().view(np.uint64), reps)
    op, st = ls.ls_operator_create(b, sec.terms), ls.ls_operator_create(b, sec.terms)
    ls.ls_operator_store(st)
    x = rng.vector(5, len(reps), 2, complex_=op.is_complex)
    y = op.matvec(torch.from_numpy(x).cuda())
    assert torch.equal(st.matvec(torch.from_numpy(x).cuda()), y)
    y1 = op.matvec(torch.from_numpy(np.ascontiguousarray(x[:, 0])).cuda())
    assert torch.equal(y[:, 0], y1)
    ref_y = oracle.matvec(P, reps, stab, np.ascontiguousarray(x[:, 0]))
    # a few roundings an element, under 130 elements a row
    assert np.abs(y1.cpu().numpy() - ref_y).max() <= 1e-13 * max(1.0, np.abs(ref_y).max())
    op.check()
    _check_states(sec, b)
