"""Short interleaved systems that Gaussian elimination without pivoting solves and that are
far from diagonal dominance: a unit first diagonal value, zeros below it, and off-diagonals
whose products are -1, so that every pivot of the elimination from the top is 1.  (A method
that starts eliminations inside the system divides by zero.)  Against a dense solve in FP64; the
condition number is 42 at 32 rows and the elimination does not grow: 42 eps is 2.5e-6 in
FP32 and 5e-15 in FP64, the bars are twice that."""
import numpy as np
import pytest

from tests.conftest import rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def adw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2006_10142_amd as m
    m._lib.load()
    return m


@pytest.mark.parametrize("n,dtype", [(n, "f32") for n in (2, 4, 5, 8, 9, 16, 17, 31, 32)] + [(n, "f64") for n in (2, 5, 8, 9, 15, 16)])
@pytest.mark.parametrize("batch,pad,noalloc", [(2, 0, False), (70, 3, True), (1025, 0, False)])
def test_elimination_from_the_top(adw, n, dtype, batch, pad, noalloc):
    print(f"short lines n={n} {dtype} batch={batch}", flush=True)
    nt, tol = (np.float32, 5e-6) if dtype == "f32" else (np.float64, 1e-14)
    rng = np.random.default_rng(n)
    es = batch + pad
    sign = np.where(rng.random((n, es)) < 0.5, -1.0, 1.0)
    a, c = sign.copy(), np.zeros((n, es))
    c[:-1] = -1.0 / a[1:]
    b = np.zeros((n, es))
    b[0] = 1.0
    d = rng.standard_normal((n, es)).astype(nt)
    mat = np.zeros((batch, n, n))
    k = np.arange(n)
    mat[:, 0, 0] = 1.0
    mat[:, k[1:], k[:-1]] = a[1:, :batch].T
    mat[:, k[:-1], k[1:]] = c[:-1, :batch].T
    ref = np.linalg.solve(mat, d[:, :batch].T.astype(np.float64)[:, :, None])[:, :, 0].T
    A, B, C, D = (torch.from_numpy(np.ascontiguousarray(v.astype(nt))).cuda() for v in (a, b, c, d))
    adw.tridiag_solve_batched(A, B, C, D, n, batch, 1, es, noalloc=noalloc)
    got = D.cpu().numpy()
    assert rel_l2(got[:, :batch], ref) <= tol and np.array_equal(got[:, batch:], d[:, batch:])


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", [1, 3, 8, 9, 16, 17, 24, 25, 31, 32, 33])
@pytest.mark.parametrize("batch,pad", [(31, 0), (33, 1), (129, 2), (100001, 0)])
def test_dominant_systems(adw, oracle_lib, n, dtype, batch, pad):
    """Around the lengths and the count where the kernel changes; the bars of the longer
    interleaved systems (1e-5, 1e-13).  The last count in one system of 50."""
    print(f"short dominant lines n={n} {dtype} batch={batch}", flush=True)
    nt = np.float32 if dtype == "f32" else np.float64
    rng = np.random.default_rng(n + batch)
    es = batch + pad
    a, c, d = (rng.uniform(-1, 1, (n, es)).astype(nt) for _ in range(3))
    b = (np.abs(a) + np.abs(c) + 0.5).astype(nt)
    pick = np.arange(0, batch, 50) if batch > 1000 else np.arange(batch)
    ref = np.asarray(oracle_lib.tridiag_batched(*(np.ascontiguousarray(v[:, pick]) for v in (a, b, c, d)), n, pick.size, 1,
                                                pick.size)).reshape(n, pick.size)
    a[0] = c[-1] = np.nan
    for v in (a, b, c):
        v[:, batch:] = np.nan
    A, B, C, D = (torch.from_numpy(v).cuda() for v in (a, b, c, d))
    adw.tridiag_solve_batched(A, B, C, D, n, batch, 1, es)
    got = D.cpu().numpy()
    assert np.isfinite(got[:, :batch]).all() and np.array_equal(got[:, batch:], d[:, batch:])
    assert rel_l2(got[:, pick], ref) <= (1e-13 if dtype == "f64" else 1e-5)


@pytest.mark.parametrize("n,pad,shift", [(8192, 0, 0), (6148, 0, 0), (7001, 3, 0), (7260, 0, 1)])
def test_large_contiguous_calls(adw, n, pad, shift):
    """Calls past 550 MB with rows on 16-byte boundaries (whole and partial vectors at their
    end) and off them: the residual of every system, 1e-6 as for the other large calls."""
    print(f"large contiguous lines n={n} pad={pad} shift={shift}", flush=True)
    batch, pitch = int(5.6e8 / 16 / n) + 1, n + pad
    g = torch.Generator(device="cuda").manual_seed(n)
    size = batch * pitch + 4
    a, c, d = (torch.rand(size, device="cuda", generator=g)[shift:] - 0.5 for _ in range(3))
    b = a.abs() + c.abs() + 0.5
    x = d.clone()
    if shift:                                          # (an expression's result starts its own storage)
        a, b, c, x = (torch.cat([t.new_zeros(shift), t])[shift:] for t in (a, b, c, x))
    adw.tridiag_solve_batched(a, b, c, x, n, batch, pitch, 1)
    v = lambda t: t[:batch * pitch].view(batch, pitch)[:, :n]
    res = v(b) * v(x) - v(d)
    res[:, 1:] += v(a)[:, 1:] * v(x)[:, :-1]
    res[:, :-1] += v(c)[:, :-1] * v(x)[:, 1:]
    assert (res.norm() / v(d).norm()).item() <= 1e-6
    if pad:
        assert torch.equal(x[:batch * pitch].view(batch, pitch)[:, n:], d[:batch * pitch].view(batch, pitch)[:, n:])
