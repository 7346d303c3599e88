"""Matrix elements of samples whose keys have bits past the last qubit: the
call is asynchronous and eloc_check reports them afterwards, so the element
kernel meets them.  Such a bit in x ^ x' is in no XY mask: no pair."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from synth import jw, samples

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ne", [(12, 6), (13, 6), (66, 14)])
def test_elements_past_the_qubits(n, ne):
    import paper_2408_07625_amd as pe
    rng = jw.rng_for(70 + n, 0)
    ham, _, _ = jw.random_jw(n - n % 2, rng)
    keys, _ = samples.excitation_batch(n - n % 2, ne, 40, rng)
    good = keys.copy()
    top = keys.shape[1] - 1
    high = np.uint64(0xFFFFFFFFFFFFFFFF) << np.uint64(n % 64)
    picks = [high, np.uint64(1) << np.uint64(n % 64), np.uint64(3) << np.uint64(62), np.uint64(5) << np.uint64(61),
             np.uint64(0xF) << np.uint64(60)]
    for k, bits in enumerate(picks):
        keys[10 + k, top] |= bits
    i, j = (t.reshape(-1).astype(np.int32) for t in np.meshgrid(np.arange(40), np.arange(40), indexing="ij"))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    eng = pe.Engine(0)
    eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
    eng.set_samples(dev(keys.view(np.int64)), check=False)
    di, dj = dev(i), dev(j)
    h = torch.full((i.size,), 7.0, dtype=torch.complex128, device="cuda")
    off = torch.empty(i.size + 1, dtype=torch.int64, device="cuda")
    eng._sync_stream()
    assert eng.lib.eloc_pair_elements(eng.handle, i.size, p(di), p(dj), p(h), p(off), None, 0) == 0
    with pytest.raises(pe.ElocError) as ex:
        eng.check()
    assert ex.value.status == "EINVAL"
    # pairs of keys with the same bits past the qubits are as without them
    past = keys[:, top] & high
    same = past[i] == past[j]
    groups = {}
    for t, m in enumerate(map(tuple, ham.xy.tolist())):
        groups.setdefault(m, []).append(t)
    got, count = h.cpu().numpy(), np.diff(off.cpu().numpy())
    bits = lambda v: sum(bin(int(x)).count("1") for x in v)  # noqa: E731
    for t in range(i.size):
        terms = groups.get(tuple((good[i[t]] ^ good[j[t]]).tolist()), []) if same[t] else []
        ref = sum(ham.coeff[l] * 1j ** ((bits(ham.xy[l] & ham.yz[l]) + 2 * bits(good[j[t]] & ham.yz[l])) % 4)
                  for l in terms)
        assert count[t] == len(terms)
        assert abs(got[t] - ref) <= 1e-12 * max(1.0, sum(abs(ham.coeff[l]) for l in terms))
    # the context goes on with valid samples
    eng.set_samples(dev(good.view(np.int64)))
    L = rng.normal(size=40) + 1j * rng.uniform(0, 6, size=40)
    e, _ = eng.local_energy(dev(L))
    ref = oracle.local_energy(ham, good, L)
    assert np.abs(e.cpu().numpy() - ref).max() <= 1e-9 * max(1.0, np.abs(ref).max())
    eng.close()
