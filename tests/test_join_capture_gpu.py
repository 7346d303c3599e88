"""Samples set by a captured graph: each replay prepares what the key buffer
then holds, and calls after it see those samples, whatever earlier calls built
for the samples before."""
import numpy as np
import pytest
import torch

import oracle
from synth import jw, samples

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["terms", "batch"])
def test_samples_set_by_a_graph(variant):
    import paper_2408_07625_amd as pe
    n, m = 28, 30011
    ham, _, _ = jw.random_jw(n, jw.rng_for(71, 0))
    sets = [samples.excitation_batch(n, 14, m, jw.rng_for(71, 1 + s))[0] for s in range(3)]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rng = np.random.default_rng(3)
    lp = rng.normal(-1.0, 0.3, size=m) + 1j * rng.uniform(0, 6, size=m)
    L, keys = dev(lp), dev(sets[0].view(np.int64))
    eng = pe.Engine(0)
    eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
    eng.set_samples(keys)
    eng.local_energy(L, None, variant)   # every buffer is there
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        eng.set_samples(keys, check=False)
    for s in (0, 1, 2, 1):
        keys.copy_(dev(sets[s].view(np.int64)))
        graph.replay()
        for _ in range(2):
            e, _ = eng.local_energy(L, None, variant)
            ref = oracle.local_energy(ham, sets[s], lp, rows=(0, 100))
            assert np.abs(e.cpu().numpy()[:100] - ref).max() <= 1e-9 * max(1.0, np.abs(ref).max())
        n_pairs = eng.count_pairs(variant)
        eng.set_tuning(rows_per_wave=8)
        assert eng.count_pairs("terms") == n_pairs
        eng.set_tuning()
    eng.close()
