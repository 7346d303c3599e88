"""The SR selection by tournament and the blocked solve at the edges of their
forms: chunk counts, a kept list past the LDS sort, ties over chunks; row
tiles of the Gram and of the Cholesky, columns ragged against a slab."""
import numpy as np
import pytest
import torch

from oracle import sr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eng():
    import paper_2408_07625_amd as pe
    e = pe.Engine(0)
    yield e
    e.close()


def _values(rng, n, form):
    if form == "random":
        return rng.normal(size=n)
    if form == "descending":
        return -np.arange(n, dtype=float)
    if form == "ascending":
        return np.arange(n, dtype=float)
    if form == "equal":
        return np.full(n, -3.25)
    # the large values in an eighth of the chunks (of 32 neighbours, 2048 in
    # turn), with many ties: the kept list is n / 8 long
    v = rng.normal(size=n) - 100.0
    top = (np.arange(n) // 32) % 2048 < 256
    v[top] = rng.integers(0, 3, size=int(top.sum()))
    return v


@pytest.mark.parametrize("n,n_sr,form", [
    (2, 2, "equal"), (31, 7, "random"), (33, 33, "ascending"), (4096, 256, "descending"), (65536, 256, "equal"),
    (65537, 100, "ascending"), (300001, 256, "descending"), (300001, 256, "few"), (300001, 1, "few"),
    ((1 << 22), 100, "equal"), ((1 << 22) + 1, 100, "few"), (70000, 257, "random")])
def test_select_forms(eng, n, n_sr, form):
    rng = np.random.default_rng(n + n_sr)
    L = _values(rng, n, form) + 1j * rng.uniform(0, 6, n)
    got = eng.sr_select(torch.from_numpy(L).cuda(), n_sr).cpu().numpy()
    np.testing.assert_array_equal(got, sr.select(L, n_sr))


def test_select_infinities(eng):
    """-inf (a vanishing amplitude) sorts last, in index order."""
    L = np.full(5000, -np.inf) + 0j
    L[[4999, 17, 2048]] = [-1.0, -2.0, 3.0]
    got = eng.sr_select(torch.from_numpy(L).cuda(), 6).cpu().numpy()
    np.testing.assert_array_equal(got, [2048, 4999, 17, 0, 1, 2])


@pytest.mark.parametrize("n_sr,n_p", [(7, 63), (8, 64), (39, 65), (40, 130), (63, 129), (64, 700), (71, 300), (72, 301),
                                      (103, 640), (104, 333), (111, 450), (112, 451), (135, 500), (136, 501),
                                      (255, 900), (256, 20011)])
def test_solve_forms(eng, n_sr, n_p):
    """Sets on both sides of each number of row tiles at which the Gram or the
    Cholesky changes form.  The two solves differ by rounding only, bounded by
    the condition number of Re S + lambda times a few FP64 epsilons."""
    rng = np.random.default_rng(n_sr)
    lam = 1e-2
    O = rng.normal(size=(n_sr, n_p)) + 1j * rng.normal(size=(n_sr, n_p))
    L = rng.normal(size=n_sr) + 1j * rng.uniform(0, 6, n_sr)
    F = rng.normal(size=n_p)
    w = sr.weights(L)
    D = (O - (w @ O)[None, :]) * np.sqrt(w)[:, None]
    X = np.concatenate([D.real, D.imag])
    G = X @ X.T
    A = G + lam * np.eye(len(X))
    ref = (F - X.T @ np.linalg.solve(A, X @ F)) / lam
    ev = np.linalg.eigvalsh(G)
    cond = (ev.max() + lam) / lam
    tol = 64 * np.finfo(float).eps * cond
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (O.real, O.imag, L, F)]
    d = eng.sr_solve(*dev, lam).cpu().numpy()
    err = np.abs(d - ref).max() / np.abs(ref).max()
    print(f"sr n_sr={n_sr} n_p={n_p}: rel err {err:.2e} (tol {tol:.1e})")
    assert err <= tol
    again = eng.sr_solve(*dev, lam).cpu().numpy()
    np.testing.assert_array_equal(d, again)
