"""Tori whose cosets are no row operations of each other: up to eight base
images, up to 128 base images and y-shifts, and term lists that fill the LDS
beside their flip images, against the oracle."""
import numpy as np
import pytest

import oracle
from workloads import configs, lattice, rng, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402

LX = 4


def _sector(ly, w, shears, steps, k=0):
    """Translations of a 4-wide torus (momentum k along x), (x, y) -> (x + y,
    y) and y -> m y for m in `shears`; bonds along `steps` (invariant)."""
    n = LX * ly

    def perm(f):
        p = [0] * n
        for y in range(ly):
            for x in range(LX):
                u, v = f(x, y)
                p[x + LX * y] = (u % LX) + LX * (v % ly)
        return p
    gens = [(perm(lambda x, y: (x + 1, y)), 0, np.exp(2j * np.pi * k / LX)), (perm(lambda x, y: (x, y + 1)), 0, 1.0)]
    if "turn" in shears:
        gens.append((perm(lambda x, y: (x + y, y)), 0, 1.0))
    gens += [(perm(lambda x, y, m=m: (x, m * y)), 0, 1.0) for m in shears if m != "turn"]
    g = lattice.close_group(n, gens)
    bonds = [((x + LX * y), ((x + a) % LX) + LX * ((y + b) % ly), 1.0 + 0.1 * a + 0.01 * b)
             for a, b in steps for y in range(ly) for x in range(LX)]
    return configs.sector_from_arrays(f"bases4x{ly}_w{w}", n, w, g.perm, g.flip, g.chi, terms.heisenberg_terms(bonds)), g


@pytest.mark.parametrize("ly,w,shears,steps,k,kind", [
    (16, 3, ("turn", 9), [(1, 0), (0, 8)], 0, "torus"),          # 8 base images, 128 base images and y-shifts
    (16, 4, ("turn", 9), [(1, 0), (0, 8)], 0, "torus"),
    (16, 3, (9,), [(1, 0), (0, 8)], 1, "torus"),                 # complex
    (16, 3, ("turn", 9), [(1, 0), (0, 4)], 0, "torus"),          # lists beside 8 flip images a term
    (12, 4, ("turn",), [(1, 0), (0, 4)], 0, "torus"),            # 4 base images, 48
    (8, 5, ("turn", 5), [(1, 0), (0, 4)], 0, "torus")],          # 8 base images, 64
    ids=lambda v: str(v).replace(" ", ""))
def test_many_base_images(ly, w, shears, steps, k, kind):
    sec, g = _sector(ly, w, shears, steps, k)
    print(f"[gpu] {sec.name} {g.size} elements {len(sec.terms)} terms", flush=True)
    P = oracle.Problem(sec)
    reps, stab = oracle.enumerate_basis(P)
    b = ls.ls_basis_build(sec)
    r, s = b.copy()
    assert np.array_equal(r.cpu().numpy().view(np.uint64), reps)
    assert np.array_equal(s.cpu().numpy().view(np.uint16), stab)
    op, st = ls.ls_operator_create(b, sec.terms), ls.ls_operator_create(b, sec.terms)
    assert op.search_kind()[0] == kind
    ls.ls_operator_store(st)
    x = rng.vector(5, len(reps), 2, complex_=op.is_complex).reshape(len(reps), 2)
    dev = torch.from_numpy(x).cuda()
    y = op.matvec(dev)
    assert torch.equal(st.matvec(dev), y)
    assert torch.equal(op.matvec(dev[:, 0].contiguous()), y[:, 0])
    B = ls.Batch([op], [2])
    yb = torch.empty_like(dev)
    B.matvec([dev], [yb])
    assert torch.equal(yb, y)
    ref = oracle.matvec(P, reps, stab, np.ascontiguousarray(x[:, 0]))
    # a few roundings an element, under 200 elements a row
    assert np.abs(y[:, 0].cpu().numpy() - ref).max() <= 1e-13 * max(1.0, np.abs(ref).max())
    push = op.matvec_push(dev[:, 0].contiguous())
    assert np.abs(push.cpu().numpy() - ref).max() <= 1e-13 * max(1.0, np.abs(ref).max())
    op.check()
    got = b.state_info(r)
    assert torch.equal(got[0], r)
