"""Steps captured in a graph by the caller, with the coefficient replaced between replays:
every replay against the oracle.  Tolerances: r is 2 at most, a step is a few eps (1 + 4 r)
of its increment and two steps add up: 1e-5 in FP32, 1e-13 in FP64 (a one-pass step of 16
halo nodes would be off by 4e-5 at r = 2, of 8 by 1e-2)."""
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


@pytest.mark.parametrize("nx,ny,r0,dtype", [(64, 1600, 0.5, "f32"), (65, 1600, 0.17, "f32"), (65, 1600, 0.13, "f64")])
def test_replays_on_new_coefficients(adw, oracle_lib, nx, ny, r0, dtype):
    print(f"captured steps {nx}x{ny} {dtype}", flush=True)
    nt, tt, tol = (np.float32, torch.float32, 1e-5) if dtype == "f32" else (np.float64, torch.float64, 1e-13)
    h = 1.0 / (max(nx, ny) + 1)
    dt = np.sqrt(2 * r0) * h                                  # r = r0 kappa
    rng = np.random.default_rng(11)
    k0 = np.ones((ny, nx), nt)
    k1 = ((2.0 / r0) * rng.uniform(0.5, 1.0, (ny, nx))).astype(nt)
    u0 = wl.gaussian_pulse(nx, ny, sigma=0.1).astype(nt)
    wave = adw.Wave(nx, ny, h, dt, kappa=torch.from_numpy(k0).cuda(), dtype=tt)
    assert wave.info()["kernels_per_step"] == 1
    a, b = torch.from_numpy(u0).cuda(), torch.from_numpy(0.99 * u0).to(tt).cuda()
    first = a.clone(), b.clone()
    wave.step(a, b, 2)                                        # the kernels are loaded
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        wave.step(a, b, 2)
    for kap in (k0, k1, k0, k1):
        wave.set_kappa(torch.from_numpy(kap).cuda())
        a.copy_(first[0])
        b.copy_(first[1])
        for _ in range(2):                                    # two replays of two steps
            up, uc = a.cpu().numpy(), b.cpu().numpy()
            g.replay()
            _, ref, _ = oracle_lib.run(kap.astype(np.float64), up.astype(np.float64), uc.astype(np.float64), h, dt, 2)
            assert rel_l2(b.cpu().numpy(), ref) <= tol
    wave.close()
