"""The hash index of sectors with few keys a group (one block a line) and of
keys whose group number needs more bits than an entry beside stabilizer
sizes has: lookups, products and dropped keys against the oracle.  The group
turns ten low sites, which leaves one representative or a few in a group."""
import numpy as np
import pytest

import oracle
from workloads import configs, lattice, rng, terms

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2308_16712_amd as ls  # noqa: E402


def _low_cycle(n, w, length=10, k=0):
    p = [(i + 1) % length if i < length else i for i in range(n)]
    g = lattice.close_group(n, [(p, 0, np.exp(2j * np.pi * k / length))])
    bonds = [(i, (i + 1) % length, 1.0) for i in range(length)] + [(i, i + 1, 0.5) for i in range(length, n - 1)] + \
        [(i, length, 0.25) for i in range(length)]
    return configs.sector_from_arrays(f"cycle{length}of{n}_w{w}_k{k}", n, w, g.perm, g.flip, g.chi,
                                      terms.heisenberg_terms(bonds))


@pytest.mark.parametrize("args", [(20, 10), (40, 4), (40, 4, 10, 3), (53, 3), (54, 3), (56, 3), (58, 3), (64, 3),
                                  (64, 3, 10, 1), (64, 61), (64, 64), (64, 63), (64, 2, 33), (64, 3, 7)],
                         ids=lambda a: "-".join(map(str, a)))
def test_sparse_and_wide(args):
    sec = _low_cycle(*args)
    print(f"[index] {sec.name}", flush=True)
    P = oracle.Problem(sec)
    reps, stab = oracle.enumerate_basis(P)
    b = ls.ls_basis_build(sec)
    r, s = b.copy()
    assert np.array_equal(r.cpu().numpy().view(np.uint64), reps)
    n = sec.n_sites
    full = np.uint64((1 << n) - 1) if n < 64 else np.uint64(2 ** 64 - 1)
    near = [reps] + [reps ^ np.uint64(m) for m in (1, 3, 5, 96, 128, 3 << 9, 1 << (n - 1), 3 << (n - 2))]
    near += [reps + np.uint64(1), reps - np.uint64(1), rng.counter_u64(9, np.arange(4000, dtype=np.uint64)),
             np.array([0, full], np.uint64)]
    keys = np.concatenate([k & full for k in near]).astype(np.uint64)
    dev = torch.from_numpy(keys.view(np.int64)).cuda()
    want = oracle.index_lookup(reps, keys)
    assert np.array_equal(b.index_lookup(dev).cpu().numpy(), want)
    op = ls.ls_operator_create(b, sec.terms)
    x = rng.vector(5, len(reps), 2, complex_=op.is_complex).reshape(len(reps), 2)
    y = op.matvec(torch.from_numpy(x).cuda())
    ref = oracle.matvec(P, reps, stab, np.ascontiguousarray(x[:, 0]))
    # a few roundings an element, under 100 elements a row
    assert np.abs(y[:, 0].cpu().numpy() - ref).max() <= 1e-13 * max(1.0, np.abs(ref).max())
    op.check()
    if len(reps) > 2:
        out = [len(reps) // 2, len(reps) // 2 + 1]
        for i in out:
            b.test_drop_key(i)
        got = b.index_lookup(dev).cpu().numpy()
        assert np.array_equal(got, np.where(np.isin(want, out), -1, want))
    b.close()
