"""The sampler where the 24-bit prefix at a level's cut holds more candidates
than the selection ranks in LDS: the levels run once, and give the oracle's
samples."""
import numpy as np
import pytest
import torch

from launches import count, launched
from oracle import sampler as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eng():
    import paper_2408_07625_amd as pe
    e = pe.Engine(0)
    yield e
    e.close()


def _weights(m):
    return {n: torch.from_numpy(np.ascontiguousarray(getattr(m, n))).cuda()
            for n in ("W1", "b1", "W2", "b2", "W3", "b3")}


def test_many_candidates_of_one_prefix(eng):
    """One outcome of every qudit has nearly all of the probability, so the
    states with two others (23 814 of them) lie near -80 000, where a 24-bit
    prefix spans 16."""
    N, D, K = 24, 6, 5000
    m = S.random_model(N, D, 64, np.random.default_rng(7), -1, -1, scale=0.3)
    m.b3[...] = 0.0
    m.b3[:, 0] = 20000.0
    ref_keys, ref_l, ref_T = S.ar_gumbel_top_k(m, K, seed=5)
    prefix = ref_T.view(np.uint64) >> np.uint64(40)
    assert (prefix == prefix[-1]).sum() > 4096 and np.unique(ref_T).size == K
    w, got = _weights(m), []
    names = launched(lambda: got.append(eng.sample(N, D, w, K, seed=5)))
    keys, logp, pert = got[0]
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64), S.keys_to_words(ref_keys, N))
    np.testing.assert_allclose(logp.cpu().numpy(), ref_l, rtol=1e-10, atol=1e-10)
    np.testing.assert_allclose(pert.cpu().numpy(), ref_T, rtol=1e-10, atol=1e-10)
    assert count(names, "k_ar_net") <= N // D


@pytest.mark.parametrize("K", [1 << 14, 1 << 21])
def test_large_sets_take_the_levels_once(eng, K):
    """A flat tail: the prefix at the cut holds about K / 512 candidates."""
    N, D = 36, 6
    m = S.random_model(N, D, 64, np.random.default_rng(8), -1, -1, scale=1.0)
    w, got = _weights(m), []
    names = launched(lambda: got.append(eng.sample(N, D, w, K, seed=9)))
    keys, logp, pert = (t.cpu().numpy() for t in got[0])
    assert count(names, "k_ar_net") <= N // D
    assert keys.shape[0] == K and np.unique(keys[:, 0]).size == K
    assert (np.diff(pert) < 0).all()   # in order, no two the same
    # the first of a larger set are those of a smaller one
    few = eng.sample(N, D, w, 1 << 13, seed=9)
    np.testing.assert_array_equal(few[0].cpu().numpy(), keys[:1 << 13])
