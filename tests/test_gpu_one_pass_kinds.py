"""Every kind of one-pass launch where it is reached by name on small grids: the kinds that
leave u^{n+1} in a buffer of their own (the adjoint's kept levels), and the batched forms
on rows of any length, against the oracle.  Bars of test_gpu_adjoint.py and
test_gpu_batch.py (relative L2 1e-5 for FP32, 1e-12 for FP64 after a run)."""
import numpy as np
import pytest

from tests.conftest import rel_l2
from tests.test_gpu_adjoint import case, oracle_grad
from tests.test_gpu_batch import make_batch, oracle_run, run_batch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def adw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2006_10142_amd as m
    m._lib.load()
    return m


@pytest.mark.parametrize("dtype,kind", [("f32", dict(fused_lane_nodes=8)), ("f32", dict(fused_lane_nodes=4)),
                                        ("f32", dict(fused_tile_cols=496, fused_lane_nodes=8)),
                                        ("f32", dict(fused_segment_rows=32)),
                                        ("f32", dict(fused_segment_rows=100, fused_tile_cols=64)), ("f64", {}),
                                        ("f64", dict(fused_segment_rows=100, fused_tile_cols=32))])
@pytest.mark.parametrize("nx,ny", [(508, 130), (72, 201)])
def test_kept_levels_of_every_kind(adw, oracle_lib, dtype, kind, nx, ny):
    """Four segments of three steps: the first reverse pass recomputes the last two with the
    forward run's step, the second run leaves them in the storage itself; one gradient,
    that of the oracle."""
    print(f"kept levels {dtype} {kind} {nx}x{ny}", flush=True)
    c = case(dtype, nx=nx, ny=ny, nsteps=11, seed=nx, nonzero=True)
    tol = 1e-5 if dtype == "f32" else 1e-12
    # (sources beside receivers: eleven steps carry 1e-35 from the case's own to its receivers)
    c["src_idx"] = (c["rec_idx"][:2] + np.array([1, nx])).astype(np.int32)

    def cu(a):
        return torch.from_numpy(np.ascontiguousarray(a)).cuda()
    wave = adw.Wave(nx, ny, c["h"], c["dt"], kappa=cu(c["kappa"]), dtype=torch.float32 if dtype == "f32" else torch.float64)
    wave.set_tuning(fused_step=True, **kind)
    i = wave.info()
    assert i["fused_step"] == 1 and all(i[k] == v for k, v in kind.items())
    kw = dict(src_idx=cu(c["src_idx"]), src_amp=cu(c["amp"]), rec_idx=cu(c["rec_idx"]))
    got = []
    for _ in range(2):
        tr = wave.adjoint_forward(cu(c["up"]), cu(c["uc"]), 11, checkpoint_every=3, **kw)
        gk, ga = wave.adjoint_backward(2.0 * (tr - cu(c["target"])), want_amp=True, **kw)
        got.append((gk.clone(), ga.clone(), tr.clone()))
    torch.cuda.synchronize()
    wave.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))
    for g, r in zip(got[0], oracle_grad(oracle_lib, c)):
        assert rel_l2(g.cpu().numpy(), r) <= tol


@pytest.mark.parametrize("form", ["tiles", "strips", "exact"])
def test_batched_forms_match_oracle(adw, oracle_lib, form):
    sizes = [(1, 9), (9, 1), (33, 517), (101, 37), (241, 64), (243, 1030), (257, 211), (483, 65), (999, 50)]
    print(f"batched {form}", flush=True)
    sims = make_batch("f32", sizes=sizes, seed=3)
    got, info = run_batch(adw, sims, "f32", 25, plan=dict(fused_form=form))
    assert info["fused_form"] == adw.Batch.FORMS[form]
    for s, g in zip(sims, got):
        assert rel_l2(g, oracle_run(oracle_lib, s, 25)) <= 1e-5, (s["nx"], s["ny"])
