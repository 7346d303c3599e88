"""The spin-string join at sizes around its row tiles (8 and 16 rows) and around
whole and partial words of the bitmap that orders a pair list, on problems
whose masks are many enough for the join to serve so few samples."""
import functools

import numpy as np
import pytest
import torch

import oracle
from synth import jw, samples

pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=1)
def hamiltonian(n):
    return jw.random_jw(n, jw.rng_for(85, n))[0]


@pytest.fixture(scope="module")
def engines():
    import paper_2408_07625_amd as pe
    made = {}

    def of(n):
        if n not in made:
            for e in made.values():
                e.close()
            made.clear()
            ham = hamiltonian(n)
            made[n] = pe.Engine(0)
            made[n].set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
        return made[n]
    yield of
    for e in made.values():
        e.close()


# 32 qubits: narrow keys, heavy and light strings; 64: no heavy strings; 66: two words
@pytest.mark.parametrize("n,m,variant", [(32, m, "trie") for m in (1087, 1088, 1089, 2047, 2048, 2049)] +
                         [(32, 16385, "terms"), (32, 131077, "terms")] +
                         [(64, m, "trie") for m in (63, 64, 65)] + [(64, m, "terms") for m in (511, 512, 513, 520)] +
                         [(66, m, "trie") for m in (57, 63, 65)] + [(66, 510, "terms")])
def test_edges(engines, n, m, variant):
    eng, ham = engines(n), hamiltonian(n)
    rng = jw.rng_for(86, n * 100000 + m)
    keys, rank = samples.excitation_batch(n, 12, m, rng)
    lp = samples.log_amplitudes(rank, rng)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    L = dev(lp)
    eng.set_tuning()
    eng.set_samples(dev(keys.view(np.int64)))
    joined = eng.local_energy(L, None, variant)[0].clone()
    pairs = [t.clone() for t in eng.find_pairs(variant)]
    eng.set_tuning(rows_per_wave=8)
    plain = eng.local_energy(L, None, "terms")[0].clone()
    eng.set_tuning()
    # the join adds in another order: the same bits throughout would be the loop's
    assert (joined != plain).any()
    rows = (0, min(m, 600))
    ref = oracle.local_energy(ham, keys, lp, rows=rows)
    assert np.abs(joined.cpu().numpy()[:ref.size] - ref).max() <= 1e-9 * max(1.0, np.abs(ref).max())
    assert (joined - plain).abs().max().item() <= 1e-9 * max(1.0, plain.abs().max().item())
    inside = pairs[0].cpu().numpy() < rows[1]
    for got, want in zip(pairs, oracle.find_pairs(ham, keys, rows=rows)):
        np.testing.assert_array_equal(got.cpu().numpy()[inside], want)
