"""Conventional local energy over sets of many popcount signatures (a spin-blocked
order of the qubits), where U's radius is what keeps candidates from being
looked up, and on both sides of the rule by candidates and coupled states."""
import numpy as np
import pytest
import torch

import oracle
from synth import jw, samples

pytestmark = pytest.mark.gpu


def blocked(n, a):
    """Qubit 2 k + s to k + s n / 2."""
    q = np.arange(n, dtype=np.uint64)
    to = q // np.uint64(2) + (q % np.uint64(2)) * np.uint64(n // 2)
    bits = (a[:, :1] >> q) & np.uint64(1)
    return (bits << to).sum(axis=1, dtype=np.uint64)[:, None]


@pytest.mark.parametrize("n,ne,m,part", [(20, 4, 200, 0), (30, 4, 500, 0), (36, 4, 130, 0), (30, 6, 6000, 1),
                                         (30, 6, 6000, 0)])
def test_radius(n, ne, m, part):
    import paper_2408_07625_amd as pe
    rng = np.random.default_rng(n + ne + m)
    ham, _, _ = jw.random_jw(n, rng)
    keys, _ = samples.excitation_batch(n, ne, m, rng)
    ham = jw.PauliHamiltonian(n, ham.coeff, blocked(n, ham.xy), blocked(n, ham.yz))
    keys = blocked(n, keys)
    eng = pe.Engine(0)
    eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
    eng.set_samples(torch.from_numpy(np.ascontiguousarray(keys).view(np.int64)).cuda())
    V = eng.find_misses()
    if part:   # as many states more as samples
        V = V[torch.randperm(V.shape[0], device="cuda")[:m + 1]].contiguous()
    lp = rng.normal(scale=0.3, size=m + V.shape[0]) + 1j * rng.uniform(0, 6, size=m + V.shape[0])
    L, Lv = (torch.from_numpy(v).cuda() for v in (lp[:m].copy(), lp[m:].copy()))
    X = np.concatenate([keys, V.cpu().numpy().view(np.uint64)])
    ref = oracle.local_energy(ham, X, lp, rows=(0, min(m, 200)))
    for precision, tol in (("fp64", 1e-9), ("fp32c", 1e-6)):
        e, _ = eng.local_energy_full(L, V, Lv, None, precision)
        got = e.cpu().numpy()[:ref.size]
        assert np.abs(got - ref).max() <= tol * max(1.0, np.abs(ref).max())
    eng.close()
