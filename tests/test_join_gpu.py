"""The spin-string join against the oracle and against the plain loops.

The join serves every variant where the Hamiltonian's masks factor by spin and
there are enough candidates; a context with a tuned launch shape
(rows_per_wave) keeps the loops, whose results it must give: pair lists
exactly, sums within the tolerances of the other parity tests."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from synth import configs, jw, samples

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-9, "fp32c": 1e-6}


@pytest.fixture(scope="module")
def pe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_07625_amd as pe
    return pe


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def molecule(n, ne, m, seed):
    rng = jw.rng_for(seed, 0)
    ham, _, _ = jw.random_jw(n, rng)
    keys, rank = samples.excitation_batch(n, ne, m, rng)
    return ham, keys, samples.log_amplitudes(rank, rng)


def mixed():
    """A 20-qubit molecule with further strings: masks of one to three bits
    (no ids by position), odd |Y|; samples of every sector."""
    rng = jw.rng_for(63, 0)
    ham, _, _ = jw.random_jw(20, rng)
    extra = jw.random_pauli(20, 60, rng, max_flip=3)
    ham = jw.PauliHamiltonian(20, np.concatenate([ham.coeff, extra.coeff]), np.concatenate([ham.xy, extra.xy]),
                              np.concatenate([ham.yz, extra.yz]))
    keys, _ = samples.excitation_batch(20, 10, 6001, rng)
    other = np.setdiff1d(rng.choice(1 << 20, size=4000, replace=False).astype(np.uint64), keys[:, 0])
    keys = np.concatenate([keys, other[:3000, None]])
    lp = rng.normal(-1.0, 0.5, size=keys.shape[0]) + 1j * rng.uniform(0, 2 * np.pi, size=keys.shape[0])
    return ham, np.ascontiguousarray(keys[rng.permutation(keys.shape[0])]), lp


def diagonal_free():
    """A 20-qubit molecule without its diagonal strings, few samples of a
    spin-up string (most buckets hold one)."""
    rng = jw.rng_for(64, 0)
    ham, _, _ = jw.random_jw(20, rng)
    keep = (ham.xy != 0).any(axis=1)
    ham = jw.PauliHamiltonian(20, ham.coeff[keep], ham.xy[keep], ham.yz[keep])
    keys = rng.choice(1 << 20, size=9001, replace=False).astype(np.uint64)[:, None]
    lp = rng.normal(size=9001) * 0.3 + 1j * rng.uniform(0, 6.28, size=9001)
    return ham, keys, lp


# name: problem, variant (LoopOverTrie's candidates count most, so that small
# problems take the join), rows for the oracle
CASES = {
    "28q": (lambda: molecule(28, 14, 30011, 60), "terms", 500),
    # strings of 32 bits: no spare bit, no heavy / light split
    "64q": (lambda: molecule(64, 12, 1501, 61), "batch", 60),
    "66q": (lambda: molecule(66, 14, 1301, 62), "trie", 60),
    "mixed20q": (mixed, "trie", 2000),
    "nodiag20q": (diagonal_free, "trie", 2000),
}


@pytest.fixture(scope="module", params=sorted(CASES))
def case(request, pe):
    make, variant, rows = CASES[request.param]
    ham, keys, lp = make()
    eng = pe.Engine(0)
    eng.set_hamiltonian(ham.n_qubits, ham.coeff, ham.xy, ham.yz)
    eng.set_samples(dev(keys.view(np.int64)))
    yield eng, ham, keys, lp, variant if request.param != "64q" else "terms", rows
    eng.close()


def loops(eng):
    """The plain loops on the same context."""
    eng.set_tuning(rows_per_wave=8)
    return "terms"


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
def test_energy_and_adjoint(case, precision):
    eng, ham, keys, lp, variant, rows = case
    rng = np.random.default_rng(5)
    L = dev(lp)
    W = dev(rng.integers(1, 9, size=keys.shape[0]).astype(np.float64))
    e, st = (t.clone() for t in eng.local_energy(L, W, variant, precision))
    g = eng.adjoint(L, e, st, 0.3 - 0.7j, W, variant, precision).clone()
    again, _ = eng.local_energy(L, W, variant, precision)
    assert torch.equal(e, again)   # bitwise reproducible
    plain = loops(eng)
    e2, st2 = (t.clone() for t in eng.local_energy(L, W, plain, precision))
    g2 = eng.adjoint(L, e, st, 0.3 - 0.7j, W, plain, precision).clone()
    eng.set_tuning()
    ref = oracle.local_energy(ham, keys, lp, rows=(0, rows))
    scale = max(1.0, np.abs(ref).max())
    assert np.abs(e.cpu().numpy()[:rows] - ref).max() <= TOL[precision] * scale
    scale = max(1.0, e2.abs().max().item())
    assert (e - e2).abs().max().item() <= TOL[precision] * scale
    assert (st - st2).abs().max().item() <= TOL[precision] * max(1.0, st2.abs().max().item())
    assert (g - g2).abs().max().item() <= TOL[precision] * max(1.0, g2.abs().max().item())


def test_join_is_taken(case):
    """The two routes add a row's pairs in different orders: the same bits in
    every row of thousands would mean that the loops served both."""
    eng, ham, keys, lp, variant, rows = case
    L = dev(lp)
    joined = eng.local_energy(L, None, variant)[0].clone()
    plain = eng.local_energy(L, None, loops(eng))[0].clone()
    eng.set_tuning()
    assert (joined != plain).any()


def test_pair_list(case):
    eng, ham, keys, lp, variant, rows = case
    got = [t.clone() for t in eng.find_pairs(variant)]
    n = eng.store_pairs(variant)
    e, _ = (t.clone() for t in eng.local_energy(dev(lp), None, "stored", "fp64"))
    plain = loops(eng)
    want = eng.find_pairs(plain)
    e2, _ = eng.local_energy(dev(lp), None, plain, "fp64")
    eng.set_tuning()
    assert n == got[0].numel() == want[0].numel()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    assert (e - e2).abs().max().item() <= TOL["fp64"] * max(1.0, e2.abs().max().item())


def test_invalid_samples(pe):
    """A repeated key and a key past the last qubit are reported, and the
    context goes on with valid samples."""
    ham, keys, lp = molecule(28, 14, 30011, 60)
    eng = pe.Engine(0)
    eng.set_hamiltonian(28, ham.coeff, ham.xy, ham.yz)
    for at, value, status in ((7, keys[3, 0], "EDUP"), (9, np.uint64(0xFFFFFFFFFFFFFFFF), "EINVAL")):
        bad = keys.copy()
        bad[at, 0] = value
        eng.set_samples(dev(bad.view(np.int64)), check=False)
        eng.local_energy(dev(lp), check=False)
        with pytest.raises(pe.ElocError) as ex:
            eng.check()
        assert ex.value.status == status
    eng.set_samples(dev(keys.view(np.int64)))
    e, _ = eng.local_energy(dev(lp))
    ref = oracle.local_energy(ham, keys, lp, rows=(0, 200))
    assert np.abs(e.cpu().numpy()[:200] - ref).max() <= TOL["fp64"]
    eng.close()


@pytest.mark.parametrize("built", [False, True])
def test_noalloc_under_capture(pe, built):
    """The allocation-free pass captured in a graph, before and after the
    samples' index was built: every replay gives the eager result, and so do
    eager calls between the replays."""
    ham, keys, lp = molecule(28, 14, 30011, 60)
    eng = pe.Engine(0)
    eng.set_hamiltonian(28, ham.coeff, ham.xy, ham.yz)
    k, L = dev(keys.view(np.int64)), dev(lp)
    eng.set_samples(k)
    if built:
        eng.local_energy(L)
    out = torch.zeros(keys.shape[0], dtype=torch.complex128, device="cuda")
    stats = torch.zeros(4, dtype=torch.float64, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        eng._sync_stream()
        rc = eng.lib.eloc_local_energy_noalloc(eng.handle, pe.VARIANTS["terms"], pe.PRECISIONS["fp64"], p(L), None,
                                               p(out), p(stats))
    assert rc == 0
    e, st = (t.clone() for t in eng.local_energy(L))
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, e) and torch.equal(stats, st)
        e2, _ = eng.local_energy(L)
        assert torch.equal(e2, e)
    eng.close()


def test_pair_elements(case):
    """H and the per-term phases of coupled and uncoupled pairs, against the
    oracle (long and short runs, places of every kind)."""
    eng, ham, keys, lp, variant, rows = case
    i, j, _ = eng.find_pairs(variant)
    rng = np.random.default_rng(9)
    pick = dev(rng.choice(i.numel(), size=min(i.numel(), 3000), replace=False))
    i, j = i[pick], j[pick]
    far = dev(rng.integers(0, keys.shape[0], size=(2, 200)).astype(np.int32))
    i, j = torch.cat([i, far[0]]), torch.cat([j, far[1]])
    h, off, k = eng.pair_elements(i, j, phases=True)
    ni, nj = i.cpu().numpy(), j.cpu().numpy()
    groups = {}
    for t, m in enumerate(map(tuple, ham.xy.tolist())):
        groups.setdefault(m, []).append(t)
    off, k, h = off.cpu().numpy(), k.cpu().numpy(), h.cpu().numpy()
    bits = lambda v: sum(int(x).bit_count() if hasattr(int, "bit_count") else bin(int(x)).count("1") for x in v)  # noqa: E731
    for t in range(0, ni.size, 7):
        terms = groups.get(tuple((keys[ni[t]] ^ keys[nj[t]]).tolist()), [])
        ph = [(bits(ham.xy[l] & ham.yz[l]) + 2 * bits(keys[nj[t]] & ham.yz[l])) % 4 for l in terms]
        assert off[t + 1] - off[t] == len(terms)
        assert k[off[t]:off[t + 1]].tolist() == ph
        ref = sum(ham.coeff[l] * 1j ** p for l, p in zip(terms, ph))
        scale = max(1.0, sum(abs(ham.coeff[l]) for l in terms))
        assert abs(h[t] - ref) <= 1e-12 * scale


@pytest.mark.parametrize("m", [1, 63, 2047, 2049, 4097])
def test_pair_order(pe, m):
    """The pair list is ordered by (row, column) at bitmap sizes around whole
    and partial words, with and without the join."""
    ham, keys, lp = molecule(20, 10, 4097, 65)
    keys = keys[:m]
    eng = pe.Engine(0)
    eng.set_hamiltonian(20, ham.coeff, ham.xy, ham.yz)
    eng.set_samples(dev(keys.view(np.int64)))
    want = oracle.find_pairs(ham, keys)
    for variant in ("terms", "batch", "trie"):
        for a, b in zip(eng.find_pairs(variant), want):
            np.testing.assert_array_equal(a.cpu().numpy(), b)
    eng.close()
