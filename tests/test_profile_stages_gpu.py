"""Every launch of a step belongs to a profiled stage: what a call builds of the
samples on first use (U's orders for the join, its sorted copy for LoopOverTrie)
counts as their preparation, once."""
import numpy as np
import pytest
import torch

from synth import jw, samples

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant,rows,parts", [("terms", 0, 2), ("batch", 0, 2), ("terms", 8, 1), ("trie", 8, 2)])
def test_preparation_is_a_stage(variant, rows, parts):
    import paper_2408_07625_amd as pe
    n, m = 28, 30011
    ham, _, _ = jw.random_jw(n, jw.rng_for(72, 0))
    keys, rank = samples.excitation_batch(n, 14, m, jw.rng_for(72, 1))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    k, L = dev(keys.view(np.int64)), dev(samples.log_amplitudes(rank, jw.rng_for(72, 2)))
    eng = pe.Engine(0)
    eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
    eng.set_tuning(rows_per_wave=rows)
    eng.profile(True)
    for _ in range(2):
        eng.set_samples(k)
        for _ in range(2):
            eng.local_energy(L, None, variant)
    prof = eng.profile_read()
    assert prof["samples"][1] == 2 * parts and prof["samples"][0] > 0
    assert prof["pairs"][1] == 4
    eng.close()
