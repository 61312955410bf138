"""The torus search (merged pair table) against the oracle."""
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


@pytest.mark.parametrize("lx,ly,w,kx,point,inv", [
    (2, 3, 3, 0, "full", 1), (2, 16, 4, 1, "none", 0), (3, 2, 3, 0, "full", 1), (3, 6, 9, 0, "full", 1),
    (4, 4, 8, 0, "c2v", 1), (4, 4, 7, 2, "none", 0), (4, 5, 10, 0, "full", -1), (5, 5, 12, 0, "full", 0),
    (5, 5, 5, 2, "none", 0), (6, 4, 12, 0, "full", 1), (6, 6, 4, 0, "full", 0), (6, 6, 4, 0, "c2v", 0),
    (6, 10, 3, 0, "full", 0), (6, 10, 3, 1, "none", 0)])
def test_torus_search_shapes(lx, ly, w, kx, point, inv):
    """The torus search over shapes, point groups and momenta against the
    oracle: products of two columns and one, generated and stored, at the
    shapes where a table or a row operation degenerates (two rows, two
    columns, rows that do not fit 32 bits below the top two)."""
    g = lattice.torus_group(lx, ly, kx, 0, point, None, inv)
    sec = configs.sector_from_arrays(f"torus{lx}x{ly}_w{w}_{point}_k{kx}_{inv}", lx * ly, w, g.perm, g.flip, g.chi,
                                     terms.heisenberg_terms(lattice.torus_bonds(lx, ly, 1.0, 0.35)))
    print(f"[gpu] {sec.name}", flush=True)
    P = oracle.Problem(sec)
    reps, stab = oracle.enumerate_basis(P)
    b = ls.ls_basis_build(sec)
    assert np.array_equal(b.copy()[0].cpu().numpy().view(np.uint64), reps)
    op = ls.ls_operator_create(b, sec.terms)
    x = rng.vector(5, len(reps), 2, complex_=op.is_complex)
    y = op.matvec(torch.from_numpy(x).cuda())
    y1 = op.matvec(torch.from_numpy(np.ascontiguousarray(x[:, 0])).cuda())
    assert torch.equal(y[:, 0], y1)
    ref_y = oracle.matvec(P, reps, stab, np.ascontiguousarray(x[:, 0]))
    # every element is off by a few roundings of its value, a row sums under 200 of them
    assert np.abs(y1.cpu().numpy() - ref_y).max() <= 1e-13 * max(1.0, np.abs(ref_y).max())
    st = ls.ls_operator_create(b, sec.terms)
    ls.ls_operator_store(st)
    assert torch.equal(st.matvec(torch.from_numpy(x).cuda()), y)
    op.check()
    _check_states(sec, b)


@pytest.mark.parametrize("extra", ["pairs", "single", "ising", "split"])
@pytest.mark.parametrize("lx,ly,w,inv", [(4, 4, 8, 1), (5, 6, 4, 0), (6, 6, 5, 0)])
def test_steps_and_lists_agree(lx, ly, w, inv, extra):
    """Large enough or not, in steps or in lists: operators whose terms form
    steps (exchanges, both directions in a row), whose directions are apart
    (lists), with diagonal terms only, and with unequal coefficients in the
    two directions (no pair), against the oracle and the stored form."""
    g = lattice.torus_group(lx, ly, 0, 0, "full", None, inv)
    t = terms.heisenberg_terms(lattice.torus_bonds(lx, ly, 1.0, 0.35))
    diag, off = t[t["flip"] == 0], t[t["flip"] != 0]
    if extra == "single":     # one direction of all bonds, then the other
        t = np.concatenate([diag, off[0::2], off[1::2]])
    elif extra == "ising":
        t = diag
    elif extra == "split":    # every direction twice, as halves: equal coefficients on one state
        half = off.copy()
        half["re"] /= 2
        t = np.concatenate([diag, np.repeat(half, 2)])
    sec = configs.sector_from_arrays(f"steps{lx}x{ly}", lx * ly, w, g.perm, g.flip, g.chi, t)
    print(f"[gpu] {sec.name} {extra}", flush=True)
    P = oracle.Problem(sec)
    reps, stab = oracle.enumerate_basis(P)
    b = ls.ls_basis_build(sec)
    op, st = ls.ls_operator_create(b, t), ls.ls_operator_create(b, t)
    ls.ls_operator_store(st)
    for cols in (1, 2, 5):
        x = torch.from_numpy(np.ascontiguousarray(rng.vector(6, len(reps), cols).reshape(len(reps), cols))).cuda()
        y = op.matvec(x)
        assert torch.equal(y, st.matvec(x))
        B = ls.Batch([op], [cols])
        yb = torch.empty_like(x)
        B.matvec([x], [yb])
        assert torch.equal(yb, y)
        want = oracle.matvec(P, reps, stab, np.ascontiguousarray(x[:, 0].cpu().numpy()))
        # a few roundings an element, under 300 elements a row
        assert np.abs(y[:, 0].cpu().numpy() - want).max() <= 1e-13 * max(1.0, np.abs(want).max())
    op.check()
