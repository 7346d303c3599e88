"""Conventional local energy with lanes over rows, against the loop over
groups on the same states: ragged row tiles, both exact table formats, tables
with and without partitions, odd-Y terms."""
import numpy as np
import pytest
import torch

from synth import jw, samples

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, ne, m, odd", [
    (12, 6, 1, False),       # one row
    (14, 6, 65, False),      # a tile and one row; few groups
    (13, 0, 63, True),       # odd-Y terms, no single signature
    (24, 12, 2500, False),   # partitioned table, whole tiles in every class
    (24, 12, 1200, False),   # partitioned table, too few rows for its classes
    (36, 4, 130, False),     # 64-bit slots
])
def test_rows_against_loop(n, ne, m, odd):
    import paper_2408_07625_amd as pe
    rng = np.random.default_rng(n * 1000 + m)
    if odd:
        ham = jw.random_pauli(n, 400, rng, max_flip=3)
        keys = rng.choice(2 ** n, m, replace=False).astype(np.uint64)[:, None]
    else:
        ham, _, _ = jw.random_jw(n, rng)
        keys, _ = samples.excitation_batch(n, ne, m, rng)
    eng = pe.Engine(0)
    try:
        eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
        eng.set_samples(torch.from_numpy(np.ascontiguousarray(keys).view(np.int64)).cuda())
        V = eng.find_misses()
        assert V.shape[0] >= 4 * m
        spread = 1.0
        gen = torch.Generator(device="cuda").manual_seed(n)

        def log_psi(k):
            return torch.complex(spread * torch.rand(k, device="cuda", dtype=torch.float64, generator=gen),
                                 6.3 * torch.rand(k, device="cuda", dtype=torch.float64, generator=gen))
        L, Lv = log_psi(m), log_psi(V.shape[0])
        # two orders of the same sum of at most as many terms as H has
        bound = 2 * len(ham.coeff) * 2.0 ** -53 * np.abs(ham.coeff).sum() * np.exp(spread)
        for prec, tol in (("fp64", bound), ("fp32c", 1e-6 * np.abs(ham.coeff).sum())):
            print(f"n={n} m={m} V={V.shape[0]} {prec}", flush=True)
            eng.set_tuning(rows_per_wave=8)
            ref, ref_st = eng.local_energy_full(L, V, Lv, None, prec)
            ref, ref_st = ref.clone(), ref_st.clone()
            eng.set_tuning()
            for _ in range(2):
                e, st = eng.local_energy_full(L, V, Lv, None, prec)
                assert (e - ref).abs().max().item() <= tol
                assert (st[:2] - ref_st[:2]).abs().max().item() <= tol
    finally:
        eng.close()
