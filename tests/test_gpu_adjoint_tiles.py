"""The one-launch reverse step on tiles (224 columns by 22 rows at most) at the edges of
its tiles, against the oracle's adjoint, to the bars of test_gpu_adjoint.py (relative L2
1e-5 for FP32: the windows differ from the full lines by at most half an ulp a step)."""
import numpy as np
import pytest

from tests.conftest import rel_l2
from tests.test_gpu_adjoint import case, gpu_grad, oracle_grad

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def adw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2006_10142_amd as m
    m._lib.load()
    return m


@pytest.mark.parametrize("nx,ny", [(4, 21), (8, 23), (20, 1), (224, 22), (228, 44), (236, 45), (452, 30), (64, 67)])
@pytest.mark.parametrize("nsrc", [2, 90])
def test_reverse_step_tiles(adw, oracle_lib, nx, ny, nsrc):
    """One tile, one column or row more than whole tiles, grids smaller than a window;
    sources at tile corners (one node shared), more of them than a tile stages, and
    receivers sharing nodes on the first and last rows and columns."""
    print(f"reverse step tiles {nx}x{ny} nsrc={nsrc}", flush=True)
    c = case("f32", nx=nx, ny=ny, nsteps=12, seed=nx + ny, nonzero=True)
    n = nx * ny
    rng = np.random.default_rng(n)
    corner = [min(22, ny) * nx - 1, 0, n - 1, min(n - 1, 223), 0]
    c["src_idx"] = np.array((corner + list(rng.integers(0, min(n, 3 * nx), nsrc)))[:nsrc], np.int32)
    c["amp"] = (rng.standard_normal((12, nsrc)) * 30.0).astype(np.float32)
    rec = [0, n - 1, nx - 1, n - nx, n // 2, n // 2, min(n - 1, 22 * nx), min(n - 1, 21 * nx)]
    c["rec_idx"] = np.array(rec, np.int32)
    gk, ga, tr = gpu_grad(adw, c, 5, one_pass=True)
    rk, ra, rtr = oracle_grad(oracle_lib, c)
    assert rel_l2(tr, rtr) <= 1e-5 and rel_l2(gk, rk) <= 1e-5 and rel_l2(ga, ra) <= 1e-5


@pytest.mark.parametrize("dtype,one_pass", [("f32", True), ("f32", False), ("f64", True), ("f64", False)])
@pytest.mark.parametrize("nsteps", [4, 5, 9, 17])
def test_reverse_pass_repeats(adw, dtype, one_pass, nsteps):
    """1, 1, 2 and 4 segments of 5 steps: the first run of a handle (no segment storage
    yet), a second reverse pass of its record, and a later run that leaves its last
    levels in the storage, all with the same gradient bit for bit."""
    print(f"reverse pass repeats {dtype} one_pass={one_pass} nsteps={nsteps}", flush=True)
    c = case(dtype, nx=96, ny=40, nsteps=nsteps, nonzero=True)
    tt = torch.float32 if dtype == "f32" else torch.float64

    def cu(a):
        return torch.from_numpy(np.ascontiguousarray(a)).cuda()
    wave = adw.Wave(c["nx"], c["ny"], c["h"], c["dt"], kappa=cu(c["kappa"]), dtype=tt)
    wave.set_tuning(fused_step=one_pass)
    kw = dict(src_idx=cu(c["src_idx"]), src_amp=cu(c["amp"]), rec_idx=cu(c["rec_idx"]))
    got = []
    for _ in range(2):
        tr = wave.adjoint_forward(cu(c["up"]), cu(c["uc"]), nsteps, checkpoint_every=5, **kw)
        for _ in range(2):
            gk, ga = wave.adjoint_backward(tr, want_amp=True, **kw)
            got.append((tr.clone(), gk, ga))
    torch.cuda.synchronize()
    wave.close()
    for g in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], g))
