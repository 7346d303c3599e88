"""The sampler's selection at the edges of its forms against the sampling
oracle: levels that keep everything, tiles of candidates with remainders, equal
values (at the cut, among the kept ones, more of them than the selection
ranks), no allowed state."""
import numpy as np
import pytest
import torch

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


def _check(eng, m, N, D, K, seed, n_up=-1, n_down=-1):
    keys, logp, pert = eng.sample(N, D, _weights(m), K, seed=seed, n_up=n_up, n_down=n_down)
    ref_keys, ref_l, ref_T = S.ar_gumbel_top_k(m, K, seed=seed)
    ref = S.keys_to_words(ref_keys, N)
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64), ref)
    np.testing.assert_allclose(logp.cpu().numpy(), ref_l, rtol=1e-10, atol=1e-10)
    np.testing.assert_allclose(pert.cpu().numpy(), ref_T, rtol=1e-10, atol=1e-10)


@pytest.mark.parametrize("N,D,K,n_up,n_down", [
    (1, 1, 1, -1, -1), (6, 6, 1, -1, -1), (12, 6, 64, -1, -1), (12, 6, 65, -1, -1), (13, 1, 100, -1, -1),
    (18, 6, 4095, -1, -1), (18, 6, 4097, 3, 4), (16, 2, 3000, 4, 4), (66, 3, 500, 20, 20)])
def test_select_edges(eng, N, D, K, n_up, n_down):
    m = S.random_model(N, D, 64, np.random.default_rng(N * K), n_up, n_down, scale=1.2)
    _check(eng, m, N, D, K, 77 + K, n_up, n_down)


@pytest.mark.parametrize("K", [3, 40, 256, 4096, 20000])
def test_equal_values(eng, K):
    """Outcomes 2 and 3 of each qudit at 1e18 below the others: their Gumbel
    variables are lost in rounding, so their values tie, within a level and at
    its cut."""
    N, D = 16, 2
    m = S.random_model(N, D, 64, np.random.default_rng(5), -1, -1, scale=0.5)
    b3 = np.zeros_like(m.b3)
    b3[:, :2] = 1e18
    m.b3[...] = b3
    _check(eng, m, N, D, K, 11)


def test_no_allowed_state(eng):
    m = S.random_model(12, 6, 64, np.random.default_rng(1), 3, 3, scale=1.0)
    keys, _, _ = eng.sample(12, 6, _weights(m), 100, seed=1, n_up=7, n_down=3)
    assert keys.shape[0] == 0
