"""Launch plans of the exact step with line groups of 512 threads, alone and with the
y-chunk elimination fused in, against the oracle, to the bars of test_gpu_parity.py (FP64
1e-12, FP32 1e-5 after a run; ten steps here)."""
import numpy as np
import pytest

from tests.conftest import rel_l2
from paper_2006_10142_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def adw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2006_10142_amd as m
    m._lib.load()
    return m


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(300, 211), (2049, 75), (3001, 33), (4096, 64)])
@pytest.mark.parametrize("fused,m", [(False, 16), (True, 16), (True, 32)])
def test_line_groups_of_512_threads(adw, oracle_lib, dtype, nx, ny, fused, m):
    print(f"512 threads {nx}x{ny} {dtype} fused={fused} m={m}", flush=True)
    nt, tt, tol = (np.float32, torch.float32, 1e-5) if dtype == "f32" else (np.float64, torch.float64, 1e-12)
    h = 1.0 / (max(nx, ny) + 1)
    dt = 0.5 * h
    c = wl.smooth_field(nx, ny, 1.0, 3.0, seed=21).astype(nt)
    u0 = wl.gaussian_pulse(nx, ny, sigma=0.1).astype(nt)
    wave = adw.Wave(nx, ny, h, dt, c=torch.from_numpy(c).cuda(), dtype=tt)
    wave.set_tuning(512, 3, fused, m, fused_step=False)
    i = wave.info()
    assert (i["x_threads_per_line"], i["y_fused"], i["kernels_per_step"]) == (512, int(fused), 3 if fused else 4)
    a = torch.from_numpy(u0).cuda()
    b = wave.start(a)
    a, b = wave.step(a, b, 10)
    kap = c.astype(np.float64) ** 2
    u1 = oracle_lib.start(kap, u0, h, dt)
    _, ref, _ = oracle_lib.run(kap, u0, u1, h, dt, 10)
    assert rel_l2(b.cpu().numpy(), ref) <= tol
    wave.close()


@pytest.mark.parametrize("nx,ny,rmax,dtype", [(64, 1600, 0.5, "f32"), (300, 211, 2.0, "f32"), (300, 211, 2.0, "f64"),
                                              (65, 1600, 0.13, "f64")])
def test_undone_plans_step_as_a_new_handle(adw, nx, ny, rmax, dtype):
    """A chunked y plan, a new coefficient while it holds, then fused_step "auto": steps of
    both kinds (the automatic one and the exact one) have the bits of a new handle's."""
    print(f"undone plans {nx}x{ny} {dtype}", flush=True)
    tt = torch.float32 if dtype == "f32" else torch.float64
    g = torch.Generator(device="cuda").manual_seed(3)
    h = 1.0 / (max(nx, ny) + 1)
    k = (0.5 + 0.5 * torch.rand(ny, nx, device="cuda", generator=g)).to(tt)
    u = torch.randn(ny, nx, device="cuda", generator=g).to(tt)
    v = torch.randn(ny, nx, device="cuda", generator=g).to(tt)
    got = []
    for undo in (True, False):
        w = adw.Wave(nx, ny, h, np.sqrt(2 * rmax) * h, c=1.0, dtype=tt)
        if undo:
            w.set_tuning(x_rows_per_strip=5, y_chunk_rows=32)
        w.set_kappa(k)
        if undo:
            w.set_tuning(fused_step="auto")
        _, a = w.step(u.clone(), v.clone(), 1)
        b = w.start(u)                                        # the exact line solves
        got.append((w.info(), a.clone(), b.clone()))
        w.close()
    assert got[0][0] == got[1][0] and torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][2], got[1][2])
