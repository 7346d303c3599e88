"""Preparing the samples over more keys than one round of workgroups, and the
rules that tell which coupled states have a non-zero element."""
import numpy as np
import pytest
import torch

import oracle
from synth import jw

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_07625_amd as pe
    return pe


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n", [24, 70])
@pytest.mark.parametrize("m", [1, 256, 257, 262145, 300001])
def test_many_keys(pe, n, m):
    """Z strings and X flips, whose local energies numpy gives by a sorted
    search; a duplicate and a bit past n_qubits at the last key are found."""
    rng = np.random.default_rng(n + m)
    W = (n + 63) // 64
    low = rng.choice(1 << 24, size=m, replace=False).astype(np.uint64)
    keys = np.zeros((m, W), dtype=np.uint64)
    keys[:, 0] = low
    if W == 2:
        keys[:, 1] = low & np.uint64(63)
    xy = np.zeros((4, W), dtype=np.uint64)
    yz = np.zeros((4, W), dtype=np.uint64)
    yz[0, 0], yz[1, 0], xy[2, 0], xy[3, 0] = 0b1011, 1 << 20, 0b11, 1 << 22
    c = np.array([0.7, -0.3, 0.45, 0.2])
    lp = rng.normal(scale=0.5, size=m) + 1j * rng.uniform(0, 6, m)
    parity = lambda v: np.array([bin(int(t)).count("1") & 1 for t in v])
    ref = sum(c[t] * (1 - 2 * parity(low & yz[t, 0])) for t in (0, 1)).astype(complex)
    order = np.argsort(low)
    for t in (2, 3):
        other = low ^ xy[t, 0]
        if W == 2:   # the second word repeats the low six bits, which the flip of bits 0 and 1 does not change there
            hit = ((other ^ low) & np.uint64(63)) == 0
        else:
            hit = np.ones(m, dtype=bool)
        at = np.minimum(np.searchsorted(low[order], other), m - 1)
        j = order[at]
        hit &= low[j] == other
        ref = ref + np.where(hit, c[t] * np.exp(lp[j] - lp), 0.0)
    eng = pe.Engine(0)
    eng.set_hamiltonian(n, c, xy, yz)
    eng.set_samples(_dev(keys.view(np.int64)))
    e, _ = eng.local_energy(_dev(lp))
    # four terms of magnitude up to exp of the spread: rounding only
    np.testing.assert_allclose(e.cpu().numpy(), ref, rtol=1e-12, atol=1e-12 * np.abs(ref).max())
    if m > 1:
        bad = keys.copy()
        bad[m - 1] = bad[0]
        with pytest.raises(pe.ElocError, match="EDUP"):
            eng.set_samples(_dev(bad.view(np.int64)))
    bad = keys.copy()
    bad[m - 1, W - 1] |= np.uint64(1 << (n % 64))
    with pytest.raises(pe.ElocError, match="EINVAL"):
        eng.set_samples(_dev(bad.view(np.int64)))
    eng.close()


@pytest.mark.parametrize("n", [9, 30, 31, 66])
@pytest.mark.parametrize("tol", [0.0, 1e-10, 0.3])
def test_miss_rules(pe, n, tol):
    """Groups whose Z masks differ by sums of none to five masks, real and
    imaginary strings, equal and opposite coefficients (elements that cancel)."""
    rng = np.random.default_rng(n)
    W = (n + 63) // 64
    rows = []
    used = set()
    for masks in range(6):
        for _ in range(6):
            flip = tuple(sorted(rng.choice(n, size=3, replace=False)))
            if flip in used:
                continue
            used.add(flip)
            base = rng.choice(n, size=2, replace=False)
            span = [rng.choice(n, size=2, replace=False) for _ in range(masks)]
            for pick in range(min(1 << masks, 12)):
                z = np.zeros(n, dtype=np.uint8)
                z[base] ^= 1
                for k in range(masks):
                    if (pick >> k) & 1:
                        z[span[k]] ^= 1
                rows.append((rng.choice([-0.25, 0.25, 0.25, 0.5]), flip, tuple(np.nonzero(z)[0])))
    seen, c, xy, yz = set(), [], [], []
    for h, flip, z in rows:
        if (flip, z) in seen:
            continue
        seen.add((flip, z))
        x, y = [0] * W, [0] * W
        for q in flip:
            x[q // 64] |= 1 << (int(q) % 64)
        for q in z:
            y[q // 64] |= 1 << (int(q) % 64)
        c.append(h), xy.append(x), yz.append(y)
    ham = jw.PauliHamiltonian(n, np.array(c), np.array(xy, dtype=np.uint64), np.array(yz, dtype=np.uint64))
    m = 37
    bits = rng.integers(0, 2, size=(m, n))
    keys = np.zeros((m, W), dtype=np.uint64)
    for q in range(n):
        keys[:, q // 64] |= bits[:, q].astype(np.uint64) << np.uint64(q % 64)
    keys = np.unique(keys, axis=0)
    eng = pe.Engine(0)
    eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
    eng.set_samples(_dev(keys.view(np.int64)))
    got = eng.find_misses(tol).cpu().numpy().view(np.uint64)
    np.testing.assert_array_equal(got, oracle.find_misses(ham, keys, tol))
    eng.close()
