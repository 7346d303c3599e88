"""Matrix elements of pairs whose groups have many terms each, alone and beside
short ones: a lane sums its own run, or the wave one run after another."""
import numpy as np
import pytest
import torch

import oracle
from synth import jw

pytestmark = pytest.mark.gpu


def hamiltonian(n, lengths, rng):
    """One mask of two bits per length; real and imaginary strings."""
    c, xy, yz = [], [], []
    flips = [(p, q) for p in range(n) for q in range(p)]
    for k, length in enumerate(lengths):
        p, q = flips[k]
        z = rng.choice(1 << n, size=length, replace=False)
        xy += [(1 << p) | (1 << q)] * length
        yz += z.tolist()
    c = rng.normal(size=len(xy))
    col = lambda v: np.array(v, dtype=np.uint64)[:, None]  # noqa: E731
    return jw.PauliHamiltonian(n, c, col(xy), col(yz))


@pytest.mark.parametrize("lengths", [[16] * 12, [17] * 12, [63, 64, 65] * 4, [255, 256, 257] * 3, [300] * 9,
                                     [2] * 30 + [400], [1, 20, 300] * 4])
def test_runs(lengths):
    import paper_2408_07625_amd as pe
    n = 10
    rng = np.random.default_rng(len(lengths) + sum(lengths))
    ham = hamiltonian(n, lengths, rng)
    keys = rng.permutation(1 << n)[:700].astype(np.uint64)[:, None]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    eng = pe.Engine(0)
    eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
    eng.set_samples(dev(keys.view(np.int64)))
    i, j, _ = eng.find_pairs("terms")
    h = eng.pair_elements(i, j).cpu().numpy()
    x, y = (keys[t.cpu().numpy(), 0].astype(np.int64) for t in (i, j))
    parity = lambda v: np.bitwise_xor.reduce([(v >> b) & 1 for b in range(n)])  # noqa: E731
    ref = np.zeros(h.size, dtype=complex)
    for c, m, z in zip(ham.coeff, ham.xy[:, 0].astype(np.int64), ham.yz[:, 0].astype(np.int64)):
        hit = (x ^ y) == m
        ref[hit] += c * 1j ** bin(m & z).count("1") * (1 - 2 * parity(y[hit] & z))
    # sums of at most 400 terms in another order
    assert np.abs(h - ref).max() <= 400 * np.finfo(float).eps * np.abs(ham.coeff).sum()
    # the stored list holds the same elements
    L = rng.normal(size=keys.shape[0]) + 1j * rng.uniform(0, 6, size=keys.shape[0])
    eng.store_pairs("terms")
    e, _ = eng.local_energy(dev(L), None, "stored")
    want = oracle.local_energy(ham, keys, L)
    assert np.abs(e.cpu().numpy() - want).max() <= 1e-9 * max(1.0, np.abs(want).max())
    eng.close()
