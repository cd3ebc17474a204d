"""Plain steps on the coefficient a time-dependent step left, with plans set in between,
against the oracle: the coefficient's largest r (2) is far outside every truncation bound
(a one-pass step of 8 halo nodes would be off by 1e-2, of 16 by 4e-5).  Tolerances: a step
is a few eps (1 + 4 r_max) = 9 eps of its increment, 1e-5 in FP32 and 1e-13 in FP64 hold
it with an order to spare."""
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


@pytest.mark.parametrize("nx,ny,r0,dtype", [(256, 256, 0.1, "f32"), (64, 1600, 0.5, "f32"), (256, 256, 0.1, "f64")])
@pytest.mark.parametrize("plan", [dict(x_rows_per_strip=4), dict(fused_lane_nodes=-1), dict(fused_tile_cols=-1),
                                  dict(fused_segment_rows=-1)])
def test_step_on_an_unmeasured_coefficient(adw, oracle_lib, nx, ny, r0, dtype, plan):
    print(f"after tdc {nx}x{ny} {dtype} {plan}", flush=True)
    nt, tt, tol = (np.float32, torch.float32, 1e-5) if dtype == "f32" else (np.float64, torch.float64, 1e-13)
    h = 1.0 / (max(nx, ny) + 1)
    dt = np.sqrt(2 * r0) * h                                  # r = r0 kappa
    rng = np.random.default_rng(7)
    k0 = np.ones((ny, nx), nt)
    k1 = ((2.0 / r0) * rng.uniform(0.5, 1.0, (ny, nx))).astype(nt)
    u0 = wl.gaussian_pulse(nx, ny, sigma=0.1).astype(nt)
    wave = adw.Wave(nx, ny, h, dt, kappa=torch.from_numpy(k0).cuda(), dtype=tt)
    assert wave.info()["kernels_per_step"] == 1
    a, b = torch.from_numpy(u0).cuda(), torch.from_numpy(u0).cuda()
    a, b = wave.step_tdc(a, b, kappa_prev=torch.from_numpy(k0).cuda(), kappa_next=torch.from_numpy(k1).cuda())
    up, uc = a.cpu().numpy(), b.cpu().numpy()
    wave.set_tuning(**plan)
    a, b = wave.step(a, b, 1)
    _, ref, _ = oracle_lib.run(k1.astype(np.float64), up.astype(np.float64), uc.astype(np.float64), h, dt, 1)
    assert rel_l2(b.cpu().numpy(), ref) <= tol
    wave.close()


@pytest.mark.parametrize("nx,ny", [(60, 200), (301, 211), (1000, 1000), (1999, 2040), (2048, 130)])
def test_pivots_are_those_of_set_kappa(adw, nx, ny):
    """The FP32 pivots a time-dependent step leaves are those set_kappa builds (composed in
    FP64, rounded once): the plain exact step after either has the same bits.  r up to 2,
    where maps composed in FP32 are further off than a sequential sweep."""
    print(f"pivots after tdc {nx}x{ny}", flush=True)
    tt = torch.float32
    g = torch.Generator(device="cuda").manual_seed(nx + ny)
    h = 1.0 / (max(nx, ny) + 1)
    k = (1.0 / 9.0 + 8.0 / 9.0 * torch.rand(ny, nx, device="cuda", generator=g)).to(tt)
    u = torch.randn(ny, nx, device="cuda", generator=g).to(tt)
    v = torch.randn(ny, nx, device="cuda", generator=g).to(tt)
    out = []
    for by_step in (True, False):
        w = adw.Wave(nx, ny, h, 2.0 * h, c=1.0, dtype=tt)      # r = 2 kappa
        w.set_tuning(fused_step=False)
        if by_step:
            w.step_tdc(u.clone(), v.clone(), kappa_prev=k, kappa_next=k)
        else:
            w.set_kappa(k)
        _, b = w.step(u.clone(), v.clone(), 1)
        out.append(b.clone())
        w.close()
    assert torch.equal(*out)


@pytest.mark.parametrize("nx,ny", [(100, 1700), (100, 2000), (33, 1999), (33, 2000), (480, 1652), (128, 2000), (40, 2048)])
def test_narrow_columns(adw, oracle_lib, nx, ny):
    """Exact FP32 steps on both sides of the rule between whole columns and the chunked
    y-solve, before and after a time-dependent step (which takes whole columns), r up to 2;
    the step's own tolerance (see above)."""
    print(f"narrow columns {nx}x{ny}", flush=True)
    rng = np.random.default_rng(nx + ny)
    h = 1.0 / (max(nx, ny) + 1)
    dt = 2.0 * h                                              # r = 2 kappa
    ka, kb = (rng.uniform(1 / 9, 1.0, (ny, nx)).astype(np.float32) for _ in range(2))
    up, uc = (rng.standard_normal((ny, nx)).astype(np.float32) for _ in range(2))

    def cu(a):
        return torch.from_numpy(a).cuda()
    wave = adw.Wave(nx, ny, h, dt, kappa=cu(ka), dtype=torch.float32)
    _, b = wave.step(cu(up), cu(uc), 1)
    _, ref, _ = oracle_lib.run(ka.astype(np.float64), up.astype(np.float64), uc.astype(np.float64), h, dt, 1)
    assert rel_l2(b.cpu().numpy(), ref) <= 1e-5
    a, b = wave.step_tdc(cu(up), cu(uc), kappa_prev=cu(ka), kappa_next=cu(kb))
    u1 = oracle_lib.step_tdc(ka.astype(np.float64), kb.astype(np.float64), up.astype(np.float64), uc.astype(np.float64), h, dt)
    assert rel_l2(b.cpu().numpy(), u1) <= 1e-5
    got = b.cpu().numpy()
    _, b = wave.step(a, b, 1)
    _, ref, _ = oracle_lib.run(kb.astype(np.float64), uc.astype(np.float64), got.astype(np.float64), h, dt, 1)
    assert rel_l2(b.cpu().numpy(), ref) <= 1e-5
    wave.close()
