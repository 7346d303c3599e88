"""The pair counts of a batch are part of its run, also those of problems that
the spin-string join serves: reading them launches nothing."""
import numpy as np
import pytest
import torch

from launches import launched
from synth import jw, samples

pytestmark = pytest.mark.gpu


def test_counts_belong_to_the_run():
    import paper_2408_07625_amd as pe
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    probs, want = [], []
    for k, (n, ne, m) in enumerate([(28, 14, 33001), (12, 6, 150), (28, 14, 20011)]):
        rng = jw.rng_for(95 + k, 0)
        ham, _, _ = jw.random_jw(n, rng)
        keys, rank = samples.excitation_batch(n, ne, m, rng)
        probs.append({"n_qubits": n, "coeff": ham.coeff, "xy": ham.xy, "yz": ham.yz,
                      "keys": dev(keys.view(np.int64)), "logpsi": dev(samples.log_amplitudes(rank, rng))})
        eng = pe.Engine(0)
        eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
        eng.set_tuning(rows_per_wave=8)
        eng.set_samples(probs[-1]["keys"])
        want.append(eng.count_pairs("terms"))
        eng.close()
    b = pe.Batch(probs)
    b.set_graph(False)
    b.run("fp64")
    got = []
    assert launched(lambda: got.append(b.pair_counts())) == []
    np.testing.assert_array_equal(got[0], want)
    b.set_graph(True)
    for _ in range(3):
        for precision in ("fp32c", "fp64"):
            b.run(precision)
            np.testing.assert_array_equal(b.pair_counts(), want)
    b.close()
