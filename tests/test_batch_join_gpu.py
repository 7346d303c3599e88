"""Batches with problems large enough for the spin-string join beside ones
that are not: against the single launches with their loops, through replayed
graphs with eager work between, eagerly, under other schedules, and with
invalid samples in a joined problem."""
import numpy as np
import pytest
import torch

from synth import jw, samples

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-9, "fp32c": 1e-6}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(scope="module")
def made():
    """(n_qubits, electrons, samples): joined at 26 and 28 qubits."""
    import paper_2408_07625_amd as pe
    out = []
    for k, (n, ne, m) in enumerate([(12, 6, 150), (28, 14, 33001), (16, 8, 900), (26, 12, 30000), (36, 18, 800)]):
        rng = jw.rng_for(90 + k, 0)
        ham, _, _ = jw.random_jw(n, rng)
        keys, rank = samples.excitation_batch(n, ne, m, rng)
        out.append((n, ham, keys, samples.log_amplitudes(rank, rng)))
    probs = [{"n_qubits": n, "coeff": ham.coeff, "xy": ham.xy, "yz": ham.yz, "keys": dev(keys.view(np.int64)),
              "logpsi": dev(lp)} for n, ham, keys, lp in out]
    return pe, out, probs


def single(pe, n, ham, keys, lp, precision):
    """The loops of a single launch (rows_per_wave set: no join)."""
    eng = pe.Engine(0)
    eng.set_hamiltonian(n, ham.coeff, ham.xy, ham.yz)
    eng.set_tuning(rows_per_wave=8)
    eng.set_samples(dev(keys.view(np.int64)))
    e, s = eng.local_energy(dev(lp), precision=precision)
    pairs = eng.count_pairs("terms")
    eng.close()
    return e.cpu().numpy(), s.cpu().numpy(), pairs


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
def test_batch_with_joins(made, precision):
    pe, problems, probs = made
    ref = [single(pe, *p, precision) for p in problems]
    b = pe.Batch(probs)
    other = torch.zeros(1 << 20, device="cuda")

    def check(what):
        counts = b.pair_counts()
        for k, (e, s, pairs) in enumerate(ref):
            tol = TOL[precision] * max(1.0, np.abs(e).max())
            assert np.abs(b.eloc[k].cpu().numpy() - e).max() <= tol, (what, k)
            assert np.abs(b.stats[k].cpu().numpy()[:3] - s[:3]).max() <= tol * max(1.0, abs(s[2])), (what, k)
            assert counts[k] == pairs, (what, k)

    for replay in range(3):
        b.run(precision)
        check(("graph", replay))
        other.mul_(2).add_(1)   # eager work between the replays
        for t in b.eloc:
            t.zero_()
        torch.cuda.synchronize()
    b.set_graph(False)
    b.run(precision)
    check("eager")
    b.set_schedule(rows_per_wave=4, item_candidates=1 << 16, batch_ratio=1.0)
    b.run(precision)
    check("rows 4")
    b.set_schedule(rows_per_wave=8, item_candidates=1 << 16, batch_ratio=1.0, blocks_per_cu=4)
    b.run(precision)
    check("joined again")
    b.close()


def test_invalid_samples_in_a_joined_problem(made):
    pe, problems, probs = made
    keys = problems[1][2].copy()
    keys[31000] = keys[5]
    bad = dict(probs[1], keys=dev(keys.view(np.int64)))
    b = pe.Batch([probs[0], bad, probs[2]])
    with pytest.raises(pe.ElocError, match="EDUP"):
        b.run("fp64")
    b.close()
