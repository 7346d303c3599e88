"""The list of coupled states outside U from the bitmap over the key space, at
the edges of the tiles it is counted by: fewer words than a thread takes, one
whole tile, one more."""
import numpy as np
import pytest
import torch

import oracle
from synth import jw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, m", [(3, 2), (5, 4), (6, 5), (7, 9), (8, 40), (15, 300), (16, 300), (18, 70)])
def test_misses_by_tiles(n, m):
    import paper_2408_07625_amd as pe
    rng = np.random.default_rng(100 + n)
    ham = jw.random_pauli(n, min(60, 2 ** n), rng, max_flip=min(n, 4))
    keys = rng.choice(2 ** n, m, replace=False).astype(np.uint64)[:, None]
    eng = pe.Engine(0)
    try:
        eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
        eng.set_samples(torch.from_numpy(keys.view(np.int64)).cuda())
        got = eng.find_misses().cpu().numpy().view(np.uint64)
    finally:
        eng.close()
    np.testing.assert_array_equal(got, oracle.find_misses(ham, keys))
