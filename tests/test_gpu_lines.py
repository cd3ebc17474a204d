"""GPU line kernels at the sizes where their splits change, against the FP64 oracle.

One step from u_prev = 2 u_curr, whose result is the ADI increment itself, on random
coefficients.  Tolerances: the factors I - beta K L of a line are diagonally dominant
with condition number at most 1 + 4 r, so a backward-stable solve of both factors is
off by a few eps (1 + 4 r_max) relative; with r_max = 4.5, 1e-13 in FP64 and 2e-5 in
FP32 leave a factor of ten over 2 * 19 eps.
"""
import numpy as np
import pytest

from tests.conftest import rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-5}


@pytest.fixture(scope="module")
def adw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2006_10142_amd as m
    m._lib.load()
    return m


def increment(adw, oracle_lib, dtype, nx, ny, rmax, smin=1.0, one_pass=None):
    """(relative error of one step's increment, the handle's info)."""
    nt, tt = (np.float32, torch.float32) if dtype == "f32" else (np.float64, torch.float64)
    rng = np.random.default_rng(nx * 31 + ny)
    h = 1.0 / (max(nx, ny) + 1)
    dt = np.sqrt(2 * rmax) * h / 3.0
    c = rng.uniform(smin, 3.0, (ny, nx)).astype(nt)
    uc = rng.standard_normal((ny, nx)).astype(nt)
    up = (2 * uc.astype(np.float64)).astype(nt)
    src = np.array([(ny - 1) * nx + nx - 1, 0, (ny // 2) * nx + nx // 3], np.int32)
    amp = (np.array([[1.0, -0.5, 2.0]]) / (h * h)).astype(nt)
    f = np.bincount(src, weights=amp[0].astype(np.float64), minlength=nx * ny).reshape(ny, nx)
    ref = oracle_lib.step_parts(c.astype(np.float64) ** 2, up, uc, h, dt, f=f)["d"]
    wave = adw.Wave(nx, ny, h, dt, c=torch.from_numpy(c).cuda(), dtype=tt)
    if one_pass is not None:
        wave.set_tuning(fused_step=one_pass)
    a, b = wave.step(torch.from_numpy(up).cuda(), torch.from_numpy(uc).cuda(), 1,
                     src_idx=torch.from_numpy(src).cuda(), src_amp=torch.from_numpy(amp).cuda())
    torch.cuda.synchronize()
    info = wave.info()
    wave.close()
    return rel_l2(b.cpu().numpy(), ref), info


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx", [1, 7, 9, 511, 513, 1025, 2049, 4095, 4097, 8192])
def test_entry_pivots_of_long_rows(adw, oracle_lib, dtype, nx):
    """Rows around the widths where the pivot kernel's thread group changes (512 x 2^k)
    and its last segment is partial; r up to 4.5, where the pivots are remembered over
    many segments."""
    print(f"entry pivots {dtype} nx={nx}", flush=True)
    err, _ = increment(adw, oracle_lib, dtype, nx, 5, 4.5)
    assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 3), (5, 40), (66, 31), (515, 33), (1501, 97), (2051, 20), (8190, 6), (8191, 5), (100, 2000)])
def test_rows_of_any_length(adw, oracle_lib, dtype, nx, ny):
    """Rows that end inside a 16-byte vector and start off 16-byte boundaries, on the
    exact two-pass step of every line-group width."""
    print(f"rows of any length {dtype} {nx}x{ny}", flush=True)
    err, info = increment(adw, oracle_lib, dtype, nx, ny, 4.5)
    assert info["fused_step"] == 0 and err <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(3, 128), (17, 129), (9, 255), (5, 257), (1017, 30), (1016, 513), (2041, 66),
                                   (4081, 40), (4080, 9), (4, 1023), (33, 1025), (7, 2048), (6, 2049), (4200, 1030)])
def test_whole_columns(adw, oracle_lib, dtype, nx, ny):
    """Columns around the lengths where the rows a thread holds double (64 x 2^k), and
    widths around those where the columns of a workgroup change, ragged last blocks
    included; 2049 rows take the chunked solve."""
    print(f"whole columns {dtype} {nx}x{ny}", flush=True)
    err, info = increment(adw, oracle_lib, dtype, nx, ny, 4.5, one_pass=False)
    assert info["kernels_per_step"] == (2 if ny <= 2048 else 4) and err <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(1, 1), (9, 5), (64, 130), (511, 20), (513, 66), (1031, 17), (2048, 9), (2049, 9),
                                   (12, 1030), (5, 2049)])
def test_time_dependent_step(adw, oracle_lib, dtype, nx, ny):
    """One step with a changing coefficient at r up to 4.5 (more sources than a strip
    stages, receivers on the first and last nodes and outside the grid), then one plain
    step on the coefficient it left; rows of more than 2048 nodes and columns of more
    than 2048 rows take the separate launches."""
    print(f"time-dependent step {dtype} {nx}x{ny}", flush=True)
    nt = np.float32 if dtype == "f32" else np.float64
    rng = np.random.default_rng(nx + 7 * ny)
    n, h = nx * ny, 1.0 / (max(nx, ny) + 1)
    dt = 3.0 * h                                        # r = dt^2 kappa / (2 h^2), kappa in [0.1, 1]
    ka, kb = (rng.uniform(0.1, 1.0, (ny, nx)).astype(nt) for _ in range(2))
    up, uc = (rng.standard_normal((ny, nx)).astype(nt) for _ in range(2))
    src = rng.integers(0, n, 40).astype(np.int32)
    amp = (rng.standard_normal(40) / (h * h)).astype(nt)
    f = np.bincount(src, weights=amp.astype(np.float64), minlength=n).reshape(ny, nx)
    rec = np.array([0, n - 1, n // 2, -1, n, n - 1], np.int32)
    u1 = oracle_lib.step_tdc(ka, kb, up, uc, h, dt, f=f)
    u2 = oracle_lib.run(kb.astype(np.float64), uc, u1, h, dt, 1)[1]

    def cu(a):
        return torch.from_numpy(a).cuda()
    wave = adw.Wave(nx, ny, h, dt, kappa=1.0, dtype=torch.float32 if dtype == "f32" else torch.float64)
    tr = cu(np.zeros(rec.size, nt))
    a, b = wave.step_tdc(cu(up), cu(uc), cu(ka), cu(kb), src_idx=cu(src), src_amp=cu(amp), rec_idx=cu(rec), traces=tr)
    got1 = b.cpu().numpy()
    a, b = wave.step(a, b, 1)
    got2, tr = b.cpu().numpy(), tr.cpu().numpy()
    wave.close()
    assert rel_l2(got1, u1) <= TOL[dtype] and rel_l2(got2, u2) <= TOL[dtype]
    inside = [0, 1, 2, 5]
    assert np.array_equal(tr[inside], got1.ravel()[rec[inside]]) and np.isnan(tr[[3, 4]]).all()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,batch,pad,shift", [(127, 70, 0, 1), (129, 9, 3, 1), (1023, 5, 1, 3), (2050, 3, 1, 2),
                                               (4095, 3, 0, 1), (4097, 2, 2, 1), (8191, 2, 0, 3)])
def test_contiguous_lines_of_any_alignment(adw, oracle_lib, dtype, n, batch, pad, shift):
    """Contiguous systems that start off 16-byte boundaries and end inside a vector, with
    gaps between them, around the lengths where the thread group changes."""
    print(f"contiguous lines {dtype} n={n} batch={batch} pad={pad} shift={shift}", flush=True)
    nt = np.float32 if dtype == "f32" else np.float64
    rng = np.random.default_rng(n)
    size = (batch - 1) * (n + pad) + n
    a, c, d = (rng.uniform(-1, 1, size).astype(nt) for _ in range(3))
    b = (np.abs(a) + np.abs(c) + 0.5).astype(nt)
    ref = oracle_lib.tridiag_batched(a, b, c, d, n, batch, n + pad, 1)
    A, B, C, D = (torch.from_numpy(np.concatenate([np.zeros(shift, nt), v])).cuda()[shift:] for v in (a, b, c, d))
    adw.tridiag_solve_batched(A, B, C, D, n, batch, n + pad, 1)
    got = D.cpu().numpy()
    assert rel_l2(got, ref) <= (1e-13 if dtype == "f64" else 1e-5)
    gap = np.ones(size, bool)
    for s in range(batch):
        gap[s * (n + pad):s * (n + pad) + n] = False
    assert np.array_equal(got[gap], d[gap])


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,batch,pad", [(1, 70, 0), (2, 17, 3), (5, 33, 1), (15, 32769, 0), (128, 47, 0), (129, 16, 5),
                                         (257, 9, 0), (513, 15, 1), (1024, 2041, 0), (1000, 4097, 0), (1025, 1021, 3),
                                         (2048, 5, 0), (1030, 5001, 0), (2049, 3, 1), (4096, 6, 0), (2100, 513, 0),
                                         (2100, 1025, 0), (4097, 5, 2)])
def test_interleaved_lines(adw, oracle_lib, dtype, n, batch, pad):
    """Interleaved systems around the lengths and counts where the kernel and its split
    change, with gaps between the rows; what lies outside a system is not read (NaN)."""
    print(f"interleaved lines {dtype} n={n} batch={batch} pad={pad}", flush=True)
    nt = np.float32 if dtype == "f32" else np.float64
    rng = np.random.default_rng(n)
    es = batch + pad
    a, c, d = (rng.uniform(-1, 1, (n, es)).astype(nt) for _ in range(3))
    b = (np.abs(a) + np.abs(c) + 0.5).astype(nt)
    ref = oracle_lib.tridiag_batched(a, b, c, d, n, batch, 1, es)
    a[0] = c[-1] = np.nan
    for v in (a, b, c):
        v[:, batch:] = np.nan
    A, B, C, D = (torch.from_numpy(v).cuda() for v in (a, b, c, d))
    adw.tridiag_solve_batched(A, B, C, D, n, batch, 1, es)
    got, ref = D.cpu().numpy(), np.asarray(ref).reshape(n, es)
    assert rel_l2(got[:, :batch], ref[:, :batch]) <= (1e-13 if dtype == "f64" else 1e-5)
    assert np.array_equal(got[:, batch:], d[:, batch:])


def test_lines_past_the_caches(adw):
    """Line solves whose arrays exceed the last-level cache (their kernels read past it):
    the residual of 3500 systems of 8192 unknowns, contiguous and interleaved."""
    n, batch = 8192, 3500
    for sys_stride, elem_stride in ((n, 1), (1, batch)):
        print(f"lines past the caches {sys_stride} {elem_stride}", flush=True)
        g = torch.Generator(device="cuda").manual_seed(3)
        a, c, d0 = (torch.rand(n * batch, device="cuda", generator=g) - 0.5 for _ in range(3))
        b = a.abs() + c.abs() + 0.5
        d = d0.clone()
        adw.tridiag_solve_batched(a, b, c, d, n, batch, sys_stride, elem_stride)
        shape = (batch, n) if elem_stride == 1 else (n, batch)
        a, b, c, d0, x = (t.view(shape) if elem_stride == 1 else t.view(shape).t() for t in (a, b, c, d0, d))
        res = b * x - d0
        res[:, 1:] += a[:, 1:] * x[:, :-1]
        res[:, :-1] += c[:, :-1] * x[:, 1:]
        assert (res.norm() / d0.norm()).item() <= 1e-6
