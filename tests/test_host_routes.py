"""Which kernels the host code queues, on the recording HIP runtime (no GPU): the forms a
handle takes after calls that change its state."""
import pytest

from tests import recorder

ONE_PASS = ("k_fused", "k_fused4", "k_fusedr")


@pytest.mark.parametrize("nx,ny,rmax,f64", [(256, 256, 0.1, 0), (256, 256, 0.1, 1), (64, 1600, 0.5, 0),
                                            (65, 1600, 0.17, 0), (65, 1600, 0.13, 1),
                                            (2056, 2100, 0.1, 0), (2056, 2100, 0.1, 1)])
def test_no_one_pass_step_on_an_unmeasured_coefficient(nx, ny, rmax, f64):
    """A time-dependent step leaves a coefficient whose largest r is unknown: no call but
    set_kappa brings a one-pass form back.  (2056 columns: the time-dependent step of
    separate launches.)"""
    got = recorder.run(f'''
out = []
for kw in (dict(x_rows_per_strip=4), dict(y_chunk_rows=16), dict(fused_lane_nodes=-1), dict(fused_tile_cols=-1),
           dict(fused_segment_rows=-1), dict(fused_tile_cols=64), dict(fused_step=1), dict()):
    w = wave({nx}, {ny}, {rmax}, {f64})
    before = short(step(w))
    a, b = ct.c_void_p(A), ct.c_void_p(B)
    _lib.check(lib.adi_wave_step_tdc(w, ct.byref(a), ct.byref(b), C, D, None, None))
    st = tune(w, **kw)
    i = info(w)
    after = short(step(w))
    rid = ct.c_ulonglong()
    _lib.check(lib.adi_adjoint_forward(w, A, B, None, None, 2, 1, ct.byref(rid)))
    forward = short(names())
    _lib.check(lib.adi_wave_set_kappa(w, C, 1.0))
    out.append([kw, before, st, i["fused_step"] + i["fused_allowed"], i["r_max"], after, forward, short(step(w))])
''')
    for kw, before, st, flags, rmax_got, after, forward, restored in got:
        assert before[0] in ONE_PASS and flags == 0 and rmax_got < 0
        assert (st == -4) == ("fused_step" in kw)                  # asked for by name: refused
        assert not set(after + forward) & set(ONE_PASS), (kw, after, forward)
        plan = {"x_rows_per_strip", "y_chunk_rows"} & set(kw)
        assert restored[0] in ONE_PASS or (plan and before[0] != restored[0])


ADJOINT = '''
def forward(w, nsteps, every, s=0):
    rid = ct.c_ulonglong()
    names()
    _lib.check(lib.adi_adjoint_forward(w, A, B, None, None, nsteps, every, ct.byref(rid)))
    return short(names())

def backward(w):
    """status, steps of the forward run's kind queued again, exact steps queued"""
    names()
    st = lib.adi_adjoint_backward(w, 0, None, None, None, D, None)
    k = short(names())
    return st, k.count("k_fused4") + k.count("k_fusedr"), k.count("k_xsweep")
'''


@pytest.mark.parametrize("rmax,f64", [(0.1, 0), (0.1, 1)])
def test_reverse_pass_after_one_that_failed(rmax, f64):
    """Four segments of two steps whose last two are in the segment storage; a reverse pass
    that fails at each of its event records in turn.  The next one may take the kept levels
    only if no earlier segment was recomputed over them."""
    got = recorder.run(ADJOINT + f'''
out = []
for n in range(9):
    w = wave(256, 256, {rmax}, {f64})
    forward(w, 8, 2)
    first = backward(w)
    forward(w, 8, 2)
    rec.rec_fail_event(n)
    failed = backward(w)
    rec.rec_fail_event(-1)
    out.append([first, failed, backward(w)])
    _lib.check(lib.adi_wave_destroy(w))
''')
    for first, failed, again in got:
        assert first == [0, 4, 4] and failed[0] == -3 and again[0] == 0
        assert again[1:] == ([4, 4] if failed[2] else [0, 4])
    assert {f[2] for _, f, _ in got} >= {0, 2, 4}


@pytest.mark.parametrize("nx,ny,rmax,f64", [(64, 1600, 0.5, 0), (65, 1600, 0.17, 0), (2051, 1953, 0.17, 0),
                                            (65, 1600, 0.13, 1)])
def test_captured_steps_take_any_coefficient(nx, ny, rmax, f64):
    """A graph of steps replays the kernels it was captured with after set_kappa has given
    the handle another coefficient: where the exact step was captured before these forms
    were there, it still is.  The forms come back outside the capture."""
    got = recorder.run(f'''
w = wave({nx}, {ny}, {rmax}, {f64})
eager = short(step(w, 2))
_lib.check(lib.adi_wave_set_stream(w, 5))
rec.rec_capturing(1)
captured = short(step(w, 2))
rec.rec_capturing(0)
out = [eager, captured, short(step(w, 2))]
''')
    eager, captured, after = got
    assert len(eager) == 2 and set(eager) <= set(ONE_PASS) and after == eager
    assert captured.count("k_xsweep") == 2 and not set(captured) & set(ONE_PASS)


def test_captured_forward_run_keeps_no_levels():
    """A captured forward run may be replayed between an eager one and its reverse pass, and
    after the segment storage has been replaced: it writes checkpoints only, and from then
    on every reverse pass recomputes.  A captured reverse pass may be replayed twice."""
    got = recorder.run(ADJOINT + '''
w = wave(256, 256, 0.1)
_lib.check(lib.adi_wave_set_stream(w, 5))
forward(w, 8, 2)
out = [backward(w)]
forward(w, 8, 2)
out.append(backward(w))                 # levels kept by the eager run
forward(w, 8, 2)
rec.rec_capturing(1)
out.append(backward(w))
forward(w, 8, 2)
rec.rec_capturing(0)
out.append(backward(w))
forward(w, 8, 2)                        # the graph of the run above may be replayed after this one
out.append(backward(w))
''')
    assert got == [[0, 4, 4], [0, 0, 4], [0, 4, 4], [0, 4, 4], [0, 4, 4]]


@pytest.mark.parametrize("f64", [0, 1])
def test_reported_line_groups_are_accepted(f64):
    """x_threads_per_line as adi_wave_get_info reports it can be set again, also after other
    widths, on rows of every width."""
    got = recorder.run(f'''
out = []
for nx in (8, 512, 513, 1025, 2048, 2049, 3000, 4096, 4097, 8192):
    w = wave(nx, 64, 2.0, {f64})
    tr = info(w)["x_threads_per_line"]
    sts = [tune(w, x_threads_per_line=tr), tune(w, x_threads_per_line=1024), tune(w, x_threads_per_line=tr)]
    out.append([nx, tr, sts, info(w)["x_threads_per_line"], step(w)[0]])
    _lib.check(lib.adi_wave_destroy(w))
''')
    for nx, tr, sts, again, kernel in got:
        assert sts == [0, 0, 0] and again == tr and f"Li{tr}E" in kernel, (nx, tr, sts)
    assert {tr for _, tr, *_ in got} == {64, 128, 256, 512, 1024}


def test_a_refused_tuning_changes_nothing():
    """Every refused call of adi_wave_set_tuning, with valid settings beside the bad one,
    leaves the plan and the step as they were."""
    got = recorder.run('''
out = []
good = dict(x_rows_per_strip=4, y_chunk_rows=32, fused_step=2, fused_tile_cols=64, fused_segment_rows=64)
for nx, ny, r in ((64, 1600, 0.5), (256, 256, 0.1), (65, 1600, 0.17), (128, 128, 2.0)):
    w = wave(nx, ny, r)
    before = [info(w), step(w)]
    for bad in (dict(line_solver=3), dict(line_solver=-1), dict(x_threads_per_line=96), dict(y_chunk_rows=8),
                dict(fused_step=3), dict(fused_lane_nodes=5), dict(fused_tile_cols=12), dict(fused_segment_rows=4)):
        st = tune(w, **{**good, **bad})
        out.append([nx, ny, bad, st, [info(w), step(w)] == before])
''')
    for nx, ny, bad, st, same in got:
        assert st == -1 and same, (nx, ny, bad)


@pytest.mark.parametrize("nx,ny,rmax,f64", [(64, 1600, 0.5, 0), (65, 1600, 0.17, 0), (65, 1600, 0.13, 1),
                                            (256, 256, 0.1, 0), (128, 128, 2.0, 0), (128, 128, 2.0, 1),
                                            (3000, 300, 2.0, 0), (3000, 4100, 2.0, 0), (300, 5000, 2.0, 1)])
def test_plans_can_be_undone(nx, ny, rmax, f64):
    """fused_step -1 brings the automatic choice back after any plan: the kernels of a new
    handle, with the pivots or planes they read built again."""
    got = recorder.run(f'''
out = []
for kw in (dict(x_rows_per_strip=5), dict(x_threads_per_line=1024), dict(y_fused=2), dict(y_chunk_rows=16),
           dict(y_chunk_rows=32), dict(fused_step=2), dict(x_rows_per_strip=5, y_chunk_rows=32, fused_step=2)):
    w = wave({nx}, {ny}, {rmax}, {f64})
    first = [info(w), step(w)]
    st = [tune(w, **kw)]
    names()
    st.append(tune(w, fused_step=-1))
    built = short(names())
    again = [info(w), step(w)]
    _lib.check(lib.adi_wave_set_kappa(w, C, 1.0))
    whole = first[0]["kernels_per_step"] == 2
    out.append([kw, st, again == first, [info(w), step(w)] == first, whole, built])
''')
    for kw, st, same, after_kappa, whole, built in got:
        assert st == [0, 0] and same and after_kappa, kw
        if whole and ("y_fused" in kw or "y_chunk_rows" in kw):
            assert "k_ycol_pivots" in built, (kw, built)


BATCH = '''
import paper_2006_10142_amd as adw

def batch(sizes, rmax=0.1):
    rec.rec_set_rmax(rmax)
    n = len(sizes)
    h = ct.c_void_p()
    _lib.check(lib.adi_batch_create(ct.byref(h), n, (ct.c_int * n)(*[s[0] for s in sizes]),
                                    (ct.c_int * n)(*[s[1] for s in sizes]), (ct.c_double * n)(*[0.1] * n),
                                    (ct.c_double * n)(*[0.1] * n), None, (ct.c_double * n)(*[1.0] * n), 0, None))
    b = adw.Batch.__new__(adw.Batch)
    b._h, b.count, b.sizes, b._code = h, n, sizes, 0
    lev = [(ct.c_void_p * n)(*[base + (k << 32) for k in range(n)]) for base in (A, B)]
    _lib.check(lib.adi_batch_bind(h, *lev))
    return b

def runs(b):
    names()
    b.step(1)
    got = names()
    return "exact" if len(got) == 3 else "strips" if "k_fusedr" in got[0] else "tiles"

def times(*ms):
    rec.rec_times((ct.c_float * len(ms))(*ms), len(ms))

RAGGED = [(33, 70), (257, 64), (243, 65)]
'''


@pytest.mark.parametrize("ms,form", [((1, 5, 9), "tiles"), ((5, 1, 9), "strips"), ((5, 5, 1), "exact")])
def test_batch_autotune_cache_keeps_the_form(ms, form, tmp_path):
    """The form the autotuner chose is in the plan and in the cache file, a second tuning
    times all of them again, and a file made for another coefficient is no error."""
    cache = str(tmp_path / "plans.json")
    got = recorder.run(BATCH + f'''
a = batch(RAGGED)
times(*{ms})
a.autotune(2, cache={cache!r})
b = batch(RAGGED)
b.autotune(2, cache={cache!r})
names()
times(5, 1, 9)                             # strips are the fastest now
a.autotune(2)
again = runs(a)
c = batch(RAGGED, 0.5)                     # no form applies
c.autotune(2, cache={cache!r})
out = [runs(b), b.plan()["fused_items"], again, runs(c), c.plan()["fused_form"]]
''')
    assert got[0] == form and got[2:] == ["strips", "exact", 0]
    # tiles of at most 240 columns by 64 rows: 1 x 2 + 2 x 1 + 2 x 2; strips: 1 + 2 + 2
    assert form == "exact" or got[1] == (8 if form == "tiles" else 5)


def test_batch_form_plans():
    """Forms set by name, the exact step asked for and given up again, plans read and set
    again, and what is refused."""
    got = recorder.run(BATCH + '''
out = []
b = batch(RAGGED)
out.append([runs(b), b.plan()["fused_form"]])
for kw in (dict(fused_form="strips"), dict(fused_form="tiles"), dict(fused_form="exact"), dict(fused_form="auto"),
           dict(fused_step=False), dict(x_threads_per_line=128), dict(fused_form="auto")):
    b.set_plan(**kw)
    p = _lib.AdiBatchPlan()
    _lib.check(lib.adi_batch_get_plan(b._h, ct.byref(p)))
    _lib.check(lib.adi_batch_set_plan(b._h, ct.byref(p)))
    out.append([runs(b), b.plan()["fused_form"]])
c = batch([(64, 64), (128, 64)])           # the tuned one-pass step
out.append([runs(c) != "exact", c.plan()["fused_form"]])
for d in (c, batch(RAGGED, 0.5)):
    for form in (1, 2, 3, -1, 4, -2):
        p = _lib.AdiBatchPlan()
        _lib.check(lib.adi_batch_get_plan(d._h, ct.byref(p)))
        p.fused_form = form
        out.append(lib.adi_batch_set_plan(d._h, ct.byref(p)))
b.set_plan(fused_step=False)
times(1, 1, 9)
b.autotune(2)
out.append(runs(b))                        # the exact step as asked for: only its plans are timed
''')
    assert got[:8] == [["tiles", 1], ["strips", 2], ["tiles", 1], ["exact", 3], ["tiles", 1], ["exact", 3],
                       ["exact", 3], ["tiles", 1]]
    assert got[8] == [True, 0] and got[9:21] == 2 * [-4, -4, -4, -4, -1, -1] and got[21] == "exact"


def test_batch_autotune_tunes_the_exact_step_too():
    """Where a form is the fastest, the exact step that fused_step 2 takes has the fastest of
    its own plans, as it had before there were forms."""
    got = recorder.run(BATCH + '''
b = batch(RAGGED)
times(1, 1, 9, 4, 9, 9, 9, 3, 9)          # tiles, strips, 128, 256, 1024 threads, then x grids 0, 256, 512 ...
b.autotune(2)
p = b.plan()
out = [runs(b), p["x_threads_per_line"], p["x_grid"]]
''')
    assert got == ["tiles", 256, 512]


@pytest.mark.parametrize("nx,ny,rmax,f64", [(64, 1600, 0.5, 0), (3000, 2999, 0.8, 0), (65, 1600, 0.17, 0),
                                            (723, 417, 0.17, 0), (2051, 1953, 0.17, 0), (65, 1600, 0.13, 1),
                                            (1001, 801, 0.13, 1), (256, 256, 0.1, 0), (2048, 2048, 0.1, 0),
                                            (4096, 4096, 0.1, 0), (2048, 2048, 0.1, 1)])
def test_reported_tiles_are_those_launched(nx, ny, rmax, f64):
    """The tile plan in adi_wave_get_info is the one of the step that runs: its tiles cover
    the grid, its count is the launch's (rounded up to whole XCD bands)."""
    got = recorder.run(f'''
w = wave({nx}, {ny}, {rmax}, {f64})
i = info(w)
rec.rec_clear()
a, b = ct.c_void_p(A), ct.c_void_p(B)
_lib.check(lib.adi_wave_step(w, ct.byref(a), ct.byref(b), None, None, 1))
k = rec.rec_log().decode().splitlines()[0].split()
out = [i, short(k[:1])[0], int(k[1])]
''')
    i, kernel, grid = got
    assert i["kernels_per_step"] == 1 and kernel in ONE_PASS
    assert grid == (i["fused_tiles"] + 7) // 8 * 8
    assert (i["fused_segment_rows"] > 0) == (kernel == "k_fusedr")
    assert i["fused_lane_nodes"] == (2 if f64 else 8 if kernel == "k_fused" else 4)
    rows = i["fused_segment_rows"] or 64
    across = i["fused_tiles"] // -(-ny // rows)
    assert across * -(-ny // rows) == i["fused_tiles"]
    wide = min(i["fused_strips_wide"], across)
    cols = wide * i["fused_tile_cols"] + (across - wide) * (i["fused_tile_cols"] - 8)
    assert nx <= cols < nx + 8 * across + i["fused_tile_cols"]


def test_narrow_fp32_columns():
    """Exact FP32 steps of narrow grids, both sides of each line of the rule: the chunked
    y-solve (4 launches) from about 1650 rows on, whole columns (2) below, on up to 24 and
    more than 480 columns, on rows of whole 512 bytes, with more rows in the last chunk, and
    in FP64.  The time-dependent step takes whole columns on all of them, and leaves the
    chunked y-solve the planes of the new coefficient."""
    got = recorder.run('''
out = []
for nx, ny, f64, want in ((100, 1650, 0, 2), (100, 1651, 0, 4), (100, 1700, 0, 4), (100, 1704, 0, 2), (100, 1708, 0, 2),
                          (100, 1999, 0, 2), (100, 2000, 0, 4), (100, 2048, 0, 4), (100, 2049, 0, 4), (24, 2000, 0, 2),
                          (25, 2000, 0, 4), (480, 2000, 0, 4), (481, 2000, 0, 2), (128, 2000, 0, 2), (256, 2048, 0, 2),
                          (160, 1696, 0, 4), (100, 2000, 1, 2), (100, 1700, 1, 2)):
    w = wave(nx, ny, 2.0, f64)
    k = len(step(w))
    a, b = ct.c_void_p(A), ct.c_void_p(B)
    names()
    _lib.check(lib.adi_wave_step_tdc(w, ct.byref(a), ct.byref(b), C, D, None, None))
    out.append([nx, ny, want, k, info(w)["kernels_per_step"], short(names()), short(step(w))])
''')
    for nx, ny, want, k, reported, tdc, after in got:
        assert k == reported == want == len(after), (nx, ny, k)
        if ny > 2048:
            continue
        assert tdc == ["k_tdc_x", "k_ycol"] + (["k_ystatic1", "k_ystatic2"] if want == 4 else []), (nx, ny, tdc)


def test_interleaved_systems_in_very_great_number():
    """Up to 2^31 - 1 interleaved systems: one launch as far as a launch's threads and the
    kernel's 32-bit system numbers reach, the three of the partition solve beyond."""
    got = recorder.run('''
out = []
for n, batch in ((1, (1 << 24) - 3), (1, (1 << 24) + 1), (1, (1 << 31) - 1), (16, 1 << 30), (33, 140000000), (200, 1 << 24),
                 (1000, (1 << 24) + 1)):
    for f64 in (0, 1):
        rec.rec_clear()
        st = lib.tridiag_solve_batched(f64, n, batch, A, B, C, D, 1, batch, None)
        log = [l.split() for l in rec.rec_log().decode().splitlines()]
        out.append([n, batch, f64, st, short([l[0] for l in log]), [int(l[1]) * int(l[2]) for l in log]])
''')
    for n, batch, f64, st, kernels, threads in got:
        assert st == 0 and all(0 < t < 1 << 32 for t in threads), (n, batch, threads)
        assert (kernels == ["k_tri_cols"]) == (batch <= 1 << 24), (n, batch, kernels)
        assert threads[0] >= batch
