"""Tori whose mirrors or quarter turns come with a spin inversion that is not
in the group by itself: row operations and base images with a flip of their
own, in the enumeration, state_info, generated and stored products and the
count, against the oracle."""
import numpy as np
import pytest

import oracle
from workloads import configs, lattice, rng, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402
from paper_2308_16712_amd._lib import sector_count  # noqa: E402


def _group(lx, ly, mx=None, my=None, rot=None, inv=None):
    """Translations, and mirrors / the quarter turn as (flip, character)."""
    def perm(f):
        p = [0] * (lx * ly)
        for y in range(ly):
            for x in range(lx):
                p[x + lx * y] = (f(x, y)[0] % lx) + lx * (f(x, y)[1] % ly)
        return p
    gens = [(perm(lambda x, y: (x + 1, y)), 0, 1.0), (perm(lambda x, y: (x, y + 1)), 0, 1.0)]
    for spec, f in ((mx, lambda x, y: (-x, y)), (my, lambda x, y: (x, -y)), (rot, lambda x, y: (-y, x)),
                    (inv, lambda x, y: (x, y))):
        if spec:
            gens.append((perm(f), spec[0], complex(spec[1])))
    return lattice.close_group(lx * ly, gens)


@pytest.mark.parametrize("lx,ly,w,spec", [
    (6, 3, 9, dict(mx=(1, 1))), (6, 3, 9, dict(mx=(1, -1))), (6, 4, -1, dict(my=(1, 1))), (6, 2, 6, dict(mx=(1, 1), my=(1, -1))),
    (4, 6, 12, dict(mx=(1, 1), my=(0, 1))), (4, 6, 12, dict(mx=(0, -1), my=(1, 1))), (5, 4, 10, dict(mx=(1, 1), my=(1, 1))),
    (3, 6, -1, dict(mx=(1, -1), my=(0, 1))), (4, 4, 8, dict(mx=(0, 1), my=(0, 1), rot=(1, 1))),
    (4, 4, 8, dict(mx=(1, 1), my=(1, 1), rot=(0, 1))), (4, 4, -1, dict(mx=(1, -1), my=(1, -1), rot=(1, 1)))], ids=lambda v: str(v) if not isinstance(v, dict) else
    "-".join(f"{k}{v[k][0]}{v[k][1]:+d}" for k in v))
def test_flipped_operations(lx, ly, w, spec):
    n = lx * ly
    g = _group(lx, ly, **spec)
    sec = configs.sector_from_arrays(f"flip{lx}x{ly}", n, w, g.perm, g.flip, g.chi,
                                     terms.heisenberg_terms(lattice.torus_bonds(lx, ly, 1.0, 0.35)))
    print(f"[gpu] {sec.name} {w} {spec}", flush=True)
    P = oracle.Problem(sec)
    reps, stab = oracle.enumerate_basis(P)
    b = ls.ls_basis_build(sec)
    r, s = b.copy()
    assert np.array_equal(r.cpu().numpy().view(np.uint64), reps)
    assert np.array_equal(s.cpu().numpy().view(np.uint16), stab)
    assert ls.ls_sector_count(sec)[0] == len(reps)
    assert sector_count(n, w, g.perm, g.flip, g.chi, noalloc=True)[0] == len(reps)
    words = rng.counter_u64(4, np.arange(3000, dtype=np.uint64)) & np.uint64((1 << n) - 1)
    states = np.concatenate([reps[:2000], words, np.array([0, (1 << n) - 1], np.uint64)])
    got = [t.cpu().numpy() for t in b.state_info(torch.from_numpy(states.view(np.int64)).cuda())]
    want = oracle.state_info(P, states)
    assert np.array_equal(got[0].view(np.uint64), want[0])
    assert np.abs(got[1][:, 0] - np.asarray(want[1]).reshape(len(states), -1)[:, 0].real).max() <= 1e-9
    assert np.abs(got[2] - want[2]).max() <= 1e-15   # one division and one root
    op, st = ls.ls_operator_create(b, sec.terms), ls.ls_operator_create(b, sec.terms)
    ls.ls_operator_store(st)
    assert op.search_kind()[0] == "torus"
    x = rng.vector(5, len(reps), 2)
    y = op.matvec(torch.from_numpy(x).cuda())
    assert torch.equal(st.matvec(torch.from_numpy(x).cuda()), y)
    assert torch.equal(op.matvec(torch.from_numpy(np.ascontiguousarray(x[:, 0])).cuda()), y[:, 0])
    ref = oracle.matvec(P, reps, stab, np.ascontiguousarray(x[:, 0]))
    # a few roundings an element, under 200 elements a row
    assert np.abs(y[:, 0].cpu().numpy() - ref).max() <= 1e-13 * max(1.0, np.abs(ref).max())
    op.check()
