"""The loops of the variants at full size.  The spin-string join serves these
problems in place of every variant; a set launch shape keeps the loops, which
serve Hamiltonians whose masks do not factor by spin, tuned contexts and the
case without memory for the join."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu as G
from synth import jw
from test_gpu import eng, large_golden  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.fixture
def loops(eng):  # noqa: F811
    eng.set_tuning(rows_per_wave=8)
    try:
        yield eng
    finally:
        eng.set_tuning()


@pytest.mark.parametrize("variant", ["terms", "batch", "trie"])
def test_medium(loops, medium_workload, variant):
    G.check_workload(loops, medium_workload, variants=(variant,),
                     rows=[(0, 300), (31000, 31133), (65536 - 217, 65536)])


@pytest.mark.parametrize("variant", ["terms", "batch", "trie"])
def test_large_golden(loops, large_workload, large_golden, variant):  # noqa: F811
    """52 qubits, 2^20 samples (LoopOverTerms by its table's partitions): the
    oracle's energies, total pair count and row digests."""
    G.test_large_workload_golden(loops, large_workload, large_golden, variant)


@pytest.mark.parametrize("variant", ["terms", "batch"])
def test_wide(loops, wide_workload, variant):
    G.test_wide_workload_sampled(loops, wide_workload, variant)


def test_wide_pairs(loops, wide_workload):
    G.test_wide_workload_pairs_sampled(loops, wide_workload)


def test_unfactored_masks(eng):  # noqa: F811
    """Masks that are no products of spin parts, 2^20 samples, nothing tuned: the
    loop by partitions of a table past 8 MB, forward and adjoint."""
    rng = np.random.default_rng(61)
    n, m = 40, 1 << 20
    ham = jw.random_pauli(n, 500, rng, max_flip=3)
    base = rng.integers(0, 1 << n, size=m // 8, dtype=np.uint64)
    flips = ham.xy[rng.integers(0, 500, size=m + m // 4), 0]
    keys = np.unique(np.concatenate([base, base[rng.integers(0, base.size, size=flips.size)] ^ flips]))
    keys = rng.permutation(keys)[:m][:, None]
    lp = rng.normal(scale=0.3, size=keys.shape[0]) + 1j * rng.uniform(0, 6, size=keys.shape[0])
    G.load(eng, ham, keys)
    L = G.dev(lp)
    rows = (keys.shape[0] - 150, keys.shape[0])
    ref = oracle.local_energy(ham, keys, lp, rows=rows)
    e, st = (t.clone() for t in eng.local_energy(L))
    assert np.abs(e.cpu().numpy()[rows[0]:] - ref).max() <= G.TOL64 * max(1.0, np.abs(ref).max())
    e32, _ = eng.local_energy(L, precision="fp32c")
    assert np.abs(e32.cpu().numpy()[rows[0]:] - ref).max() <= G.TOL32 * max(1.0, np.abs(ref).max())
    g = eng.adjoint(L, e, st, 0.4 + 1.0j).cpu().numpy()
    want = oracle.adjoint(ham, keys, lp, ref, 0.4 + 1.0j, energy_value=complex(st[0].item(), st[1].item()), rows=rows)
    assert np.abs(g[rows[0]:] - want).max() <= G.TOL64 * max(1.0, np.abs(want).max())
    i, j, _ = eng.find_pairs("terms")
    lo = int(torch.searchsorted(i, torch.tensor([rows[0]], dtype=torch.int32, device="cuda")))
    pi, pj, _ = oracle.find_pairs(ham, keys, rows=rows)
    np.testing.assert_array_equal(i[lo:].cpu().numpy(), pi)
    np.testing.assert_array_equal(j[lo:].cpu().numpy(), pj)
