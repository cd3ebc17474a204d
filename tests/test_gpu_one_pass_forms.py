"""One-pass steps beside the tuned one: FP32 column strips with 16 halo rows and columns for
r in (0.18, 0.81], FP32 tiles and FP32 and FP64 strips on rows that are no multiple of 16
bytes, against the FP64 oracle.

Tolerances: an FP32 step is a few eps (1 + 4 r_max), eps = 6e-8, of the increment (8 of
them at r_max = 0.81: 2e-6), and the truncation is at most half an ulp of max|w|, some
ten times the increment's rms (6e-7); 5e-6 covers both.  Three steps add up: 1.5e-5.
FP64 (eps = 1.1e-16, the same two terms): 1e-14 and 3e-14.
"""
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


def cu(a, shift=0):
    t = torch.empty(a.size + shift, dtype=torch.from_numpy(a).dtype, device="cuda")[shift:].view(a.shape)
    return t.copy_(torch.from_numpy(a))


def problem(nx, ny, rmax, nt):
    rng = np.random.default_rng(nx * 31 + ny)
    n, h = nx * ny, 1.0 / (max(nx, ny) + 1)
    dt = np.sqrt(2 * rmax) * h / 3.0
    c = rng.uniform(1.0, 3.0, (ny, nx)).astype(nt)
    c[ny // 2, :] = c[:, nx // 2] = 3.0                       # r = rmax along a whole row and column
    uc = rng.standard_normal((ny, nx)).astype(nt)
    up = (2 * uc.astype(np.float64)).astype(nt)
    src = np.concatenate([[0, n - 1, nx - 1, n - nx], n // 2 + np.arange(40) % 7]).astype(np.int32)   # 40 in one tile
    amp = (rng.standard_normal((3, src.size)) / (h * h)).astype(nt)
    rec = np.array([0, nx - 1, n - nx, n - 1, n // 2, n // 2 + 1], np.int32)
    return h, dt, c, up, uc, src, amp, rec


@pytest.mark.parametrize("nx,ny,rmax", [
    (48, 1540, 0.2), (64, 1536, 0.809), (216, 1537, 0.5), (424, 1600, 0.809), (12, 8190, 0.809), (1004, 1251, 0.809),
    (3256, 770, 0.5), (1001, 1251, 0.809), (65, 1537, 0.5), (2503, 1007, 0.809),   # strips with the wide halo
    (33, 2049, 0.179), (65, 1100, 0.179), (241, 1250, 0.17), (2047, 147, 0.179), (3001, 101, 0.179), (723, 417, 0.179),
    (1502, 200, 0.179),                                       # tiles on rows of any length
    (2051, 1953, 0.179), (4001, 1001, 0.17),                  # strips on rows of any length
    (33, 2001, -0.1328), (65, 1100, -0.1328),                 # FP64 (r < 0)
    (1001, 801, -0.12), (9, 8191, -0.1328), (8191, 99, -0.1328)])
@pytest.mark.parametrize("shift", [0, 1])
def test_step_and_traces(adw, oracle_lib, nx, ny, rmax, shift):
    """One step's increment, then the field and traces of three; levels off 16-byte
    boundaries (shift 1) keep the exact step."""
    print(f"one-pass forms {nx}x{ny} r={rmax} shift={shift}", flush=True)
    nt, tt, tol = (np.float32, torch.float32, 5e-6) if rmax > 0 else (np.float64, torch.float64, 1e-14)
    h, dt, c, up, uc, src, amp, rec = problem(nx, ny, abs(rmax), nt)
    kap = c.astype(np.float64) ** 2
    f = np.bincount(src, weights=amp[0].astype(np.float64), minlength=nx * ny).reshape(ny, nx)
    d = oracle_lib.step_parts(kap, up, uc, h, dt, f=f)["d"]
    _, u3, tr3 = oracle_lib.run(kap, up, uc, h, dt, 3, src_idx=src, src_amp=amp, rec_idx=rec)
    wave = adw.Wave(nx, ny, h, dt, c=cu(c), dtype=tt)
    i = wave.info()
    assert (i["kernels_per_step"], i["fused_step"], i["fused_allowed"]) == (1, 0, 0)
    _, b = wave.step(cu(up, shift), cu(uc, shift), 1, src_idx=cu(src), src_amp=cu(amp[:1]))
    assert rel_l2(b.cpu().numpy(), d) <= tol
    tr = cu(np.zeros((3, rec.size), nt))
    _, b = wave.step(cu(up, shift), cu(uc, shift), 3, src_idx=cu(src), src_amp=cu(amp), rec_idx=cu(rec), traces=tr)
    assert rel_l2(b.cpu().numpy(), u3) <= 3 * tol and rel_l2(tr.cpu().numpy(), tr3) <= 3 * tol
    wave.close()


def test_when_the_exact_step_runs(adw):
    """Outside the bounds, on small grids, with the exact step or a plan of it asked for,
    and after a step that changes the coefficient."""
    def launches(nx, ny, rmax, dtype=torch.float32, **tuning):
        h = 1.0 / (max(nx, ny) + 1)
        w = adw.Wave(nx, ny, h, np.sqrt(2 * rmax) * h, c=1.0, dtype=dtype)
        if tuning:
            w.set_tuning(**tuning)
        k = w.info()["kernels_per_step"]
        w.close()
        return k
    assert launches(64, 1600, 0.5) == 1 and launches(65, 1600, 0.17) == 1
    assert launches(64, 1600, 0.82) > 1 and launches(65, 1600, 0.82) > 1
    assert launches(64, 1600, 0.5, torch.float64) > 1 and launches(65, 1600, 0.135, torch.float64) > 1
    assert launches(1024, 1024, 0.5) > 1 and launches(449, 449, 0.17) > 1 and launches(40, 1600, 0.5) > 1
    assert launches(513, 513, 0.13, torch.float64) > 1 and launches(65, 1600, 0.13, torch.float64) == 1
    for plan in (dict(fused_step=False), dict(y_chunk_rows=16), dict(x_threads_per_line=64)):
        assert launches(64, 1600, 0.5, **plan) > 1 and launches(65, 1600, 0.17, **plan) > 1
    h = 1.0 / 1601
    w = adw.Wave(64, 1600, h, h, c=1.0, dtype=torch.float32)
    k = torch.ones(1600, 64, device="cuda")
    u = torch.zeros(1600, 64, device="cuda")
    w.step_tdc(u, u.clone(), k, k)
    assert w.info()["kernels_per_step"] > 1
    w.set_kappa(k)
    assert w.info()["kernels_per_step"] == 1
    w.close()


@pytest.mark.parametrize("sizes", [[(1, 9), (33, 70), (257, 64), (5, 300), (243, 65), (8, 8)],
                                   [(3203, 3201), (3201, 3203), (3999, 2501), (6667, 1601)]])
def test_batched_rows_of_any_length(adw, sizes):
    """The batched forms on rows of any length (tiles; column strips from 40 M nodes) against
    the batch's exact step, eager and replayed: five FP32 steps apart by rounding and half
    an ulp of truncation each, 3e-6."""
    print(f"batched rows of any length {sizes}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    h = [1.0 / (max(s) + 1) for s in sizes]
    c = [1.0 + 2.0 * torch.rand(ny, nx, device="cuda", generator=g) for nx, ny in sizes]
    u0 = [torch.randn(ny, nx, device="cuda", generator=g) for nx, ny in sizes]
    out = []
    for exact, graph in ((False, False), (False, True), (True, False)):
        b = adw.Batch(sizes, h, [0.19 * x for x in h], c)      # r <= 0.163
        assert b.plan()["fused_allowed"] == 0 and b.plan()["fused_step"] == 0
        if exact:
            b.set_plan(fused_step=False)
        b.bind([u.clone() for u in u0], [u.clone() for u in u0])
        if graph:
            b.graph(True)
        b.step(5)
        out.append([x.clone() for x in b.levels()[1]])
        b.close()
    for a, r, e in zip(*out):
        assert torch.equal(a, r) and ((a - e).norm() / e.norm()).item() <= 3e-6
