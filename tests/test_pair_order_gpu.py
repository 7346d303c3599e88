"""The pair list's order on both sides of the rule between ordering a row's
pairs by a bitmap and sorting all of them (few and many pairs a row, up to and
past the samples that a bitmap holds)."""
import numpy as np
import pytest
import torch

from synth import jw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,masks", [(12, 4095, 3), (17, 32769, 1), (17, 60001, 8), (17, 60001, 120),
                                       (18, 131072, 2), (18, 131072, 400), (18, 131073, 6)])
def test_pairs_in_order(n, m, masks):
    import paper_2408_07625_amd as pe
    rng = np.random.default_rng(m + masks)
    flips = rng.choice(np.arange(1, 1 << n), size=masks, replace=False).astype(np.uint64)
    keys = rng.choice(1 << n, size=m, replace=False).astype(np.uint64)
    ham = jw.PauliHamiltonian(n, rng.normal(size=masks), flips[:, None], np.zeros((masks, 1), dtype=np.uint64))
    where = np.full(1 << n, -1, dtype=np.int64)
    where[keys.astype(np.int64)] = np.arange(m)
    i, j, g = [], [], []
    for k, f in enumerate(flips):
        to = where[(keys ^ f).astype(np.int64)]
        hit = np.flatnonzero(to >= 0)
        i.append(hit)
        j.append(to[hit])
        g.append(np.full(hit.size, k))
    i, j, g = (np.concatenate(v) for v in (i, j, g))
    order = np.lexsort((j, i))
    eng = pe.Engine(0)
    eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
    eng.set_samples(torch.from_numpy(keys.view(np.int64)[:, None].copy()).cuda())
    for variant in ("terms", "batch") if m < 50000 else ("terms",):
        for got, want in zip(eng.find_pairs(variant), (i, j, g)):
            np.testing.assert_array_equal(got.cpu().numpy(), want[order])
    eng.close()
