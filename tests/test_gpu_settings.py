"""Settings of a plan's forms on the GPU: whatever was set, the results are the
oracle's, |x - x_oracle| <= 1e-12 A (A: the oracle's abs-sum of the entry)."""
import numpy as np
import pytest

import oracle
from paper_1905_00480_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

RTOL = 1e-12


def _bd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_00480_amd import binding
    binding.load_library()
    return binding


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _check(t, ref, ab, what):
    torch.cuda.synchronize()
    err = np.abs(t.cpu().numpy().ravel() - ref.ravel())
    bound = RTOL * ab.ravel() + 1e-300
    assert np.all(err <= bound), "%s: %d entries off, max |d| %.3e" % (
        what, int((err > bound).sum()), float(err.max()))


@pytest.mark.parametrize("tile", [0, 8, 32])
def test_deterministic_expansion_after_the_band_tile_is_set(tile):
    bd = _bd()
    s = wl.small_mixed()
    psi, w = wl.psi_for(s), wl.coeffs_for(s)
    d_psi, d_w = _dev(psi), _dev(w)
    ref, ab = oracle.expand(*s.geometry(), w, psi, with_abs=True)
    plan = bd.Plan.from_system(s, flags=bd.FLAG_DETERMINISTIC)
    first = plan.expand(d_w, d_psi.clone())
    plan.set_expand_tile(tile)
    again = plan.expand(d_w, d_psi.clone())
    _check(again, ref, ab, "band tile %d" % tile)
    assert torch.equal(first, again)
    plan.set_expand(bd.EXPAND_OWNER, 0, 16)  # a form of its own, then the tile
    plan.set_expand_tile(tile)
    _check(plan.expand(d_w, d_psi.clone()), ref, ab, "owner form, band tile %d" % tile)
    plan.set_expand(bd.EXPAND_OWNER)
    assert torch.equal(first, plan.expand(d_w, d_psi.clone()))
    plan.close()


@pytest.mark.parametrize("flags", ["f64", "det"])
def test_results_through_a_round_trip_of_settings(flags):
    """Each form that the settings name gives the oracle's results, and the
    settings of a new plan, given back, its bits."""
    bd = _bd()
    fl = bd.FLAG_DETERMINISTIC if flags == "det" else 0
    s = wl.small_mixed()
    psi, w = wl.psi_for(s), wl.coeffs_for(s)
    d_psi, d_w = _dev(psi), _dev(w)
    refs = oracle.project(*s.geometry(), psi, with_abs=True)
    exp = oracle.expand(*s.geometry(), w, psi, with_abs=True)
    plan = bd.Plan.from_system(s, flags=fl)
    forms, sc, tile, ex = plan.forms(), plan.schedule(), plan.expand_tile(), plan.expand_form()
    c0, e0 = plan.project(d_psi).clone(), plan.expand(d_w, d_psi.clone())

    def check(what):
        _check(plan.project(d_psi), *refs, what)
        _check(plan.expand(d_w, d_psi.clone()), *exp, what)

    plan.set_schedule(bd.SCHED_SINGLE_LPT, 0, 4096)
    plan.set_expand_tile(8)
    plan.set_expand(*((ex[0], 0, 16) if fl else (ex[0], 4, 8)))
    check("named forms")
    plan.set_schedule(*sc)
    plan.set_expand_tile(tile)
    check("band tile back")
    plan.set_expand(*ex)
    assert plan.forms() == forms and plan.expand_form() == ex
    assert torch.equal(plan.project(d_psi), c0)
    e1 = plan.expand(d_w, d_psi.clone())
    _check(e1, *exp, "all back")
    if plan.forms()[2] == bd.FORM_TILES:  # (blocks add with atomics)
        assert torch.equal(e0, e1)
    plan.close()


@pytest.mark.parametrize("flags", ["f32", "det"])
def test_projection_and_tuner_without_room_for_the_scratch(flags):
    """A plan whose plane sums do not fit what is left of the card (80 atoms of
    cut-off 10 and 200 planes, 640 values per point: 5.4 GB of about 3.2) projects
    without them, and the tuner does not refuse it.  The bands repeat 32 of a
    small plan.  Both sum at most 3200 terms, so they agree within 2 * 3300
    roundings of h^3 sum |psi P|, which is at most the norm of psi (P has norm 1)."""
    bd = _bd()
    f32 = flags == "f32"
    fl = bd.FLAG_FP32 if f32 else bd.FLAG_DETERMINISTIC
    nbands = 1280 if f32 else 640
    rng = np.random.default_rng(5)
    pos = rng.uniform(0.2, 0.6, size=(80, 3))
    pos[:, 2] = rng.uniform(18.0, 22.0, size=80)
    geo = dict(n=(4, 4, 200), h=0.2, periodic=(False,) * 3, pos=pos, sigma=np.full(80, 6.0),
               numax=np.full(80, 10, dtype=np.int32), rbox=np.full(80, 30.0), flags=fl)
    dt = torch.float32 if f32 else torch.float64
    small = torch.from_numpy(rng.standard_normal((3200, 32))).to("cuda", dt)
    plan = bd.Plan(nbands=32, **geo)
    ref = plan.project(small.reshape(-1)).reshape(-1, 1, 32).clone()
    plan.close()
    torch.cuda.empty_cache()
    left = 3 << 30
    taken = torch.empty(torch.cuda.mem_get_info()[0] - left, dtype=torch.uint8, device="cuda")
    free = torch.cuda.mem_get_info()[0]
    plan = bd.Plan(nbands=nbands, **geo)
    assert plan.forms()[0] == bd.FORM_PLANES
    assert plan.info["expand_scratch_doubles"] * 8 > free
    psi = small.repeat(1, nbands // 32).reshape(-1)
    c = torch.full((plan.coeff_doubles,), float("nan"), dtype=dt, device="cuda")
    norm = float((0.2 ** 3 * (small.double() ** 2).sum(dim=0)).max()) ** 0.5
    tol = 2 * 3300 * (2.0 ** -24 if f32 else 2.0 ** -53) * norm
    for step in range(2):
        plan.project(psi, c)
        torch.cuda.synchronize()
        for rows in c.reshape(-1, nbands // 32, 32).split(1024):
            at = rows.data_ptr() - c.data_ptr()
            r0 = at // (c.element_size() * nbands)
            assert float((rows - ref[r0:r0 + rows.shape[0]]).abs().max()) <= tol
        if step == 0:
            if f32:  # (slow on the work items of deterministic plans)
                r = plan.tune(psi, c, reps=1)
                assert r["candidates"] >= 2 and r["project_form"] == bd.PROJECT_ITEMS
            c.fill_(float("nan"))
    plan.close()
    del taken
    torch.cuda.empty_cache()


def test_tuners_come_back_to_the_default_forms():
    """Where planes and tiles are several times faster than the other forms (six
    atoms of cut-off 5, 32 bands, 32^3: 20 us against 60 and more) the tuners
    find them, whatever was set before, with settings that name them."""
    bd = _bd()
    s = wl.small_periodic(natoms=6, nbands=32)
    psi, w = wl.psi_for(s), wl.coeffs_for(s)
    d_psi, d_w = _dev(psi), _dev(w)
    plan = bd.Plan.from_system(s)
    c = torch.empty(plan.coeff_doubles, dtype=torch.float64, device="cuda")
    forms, sc, ex = plan.forms(), plan.schedule(), plan.expand_form()
    assert forms[0] == bd.FORM_PLANES and forms[2] == bd.FORM_TILES
    for setting in (lambda: plan.set_schedule(bd.SCHED_SINGLE_LPT, 0, 4096),
                    lambda: plan.set_project(bd.PROJECT_BLOCKS), lambda: None):
        setting()
        r = plan.tune(d_psi, c, reps=10)
        assert plan.forms() == forms and plan.schedule() == sc
        assert r["project_form"] == plan.project_form()[0] == bd.PROJECT_ITEMS
        _check(plan.project(d_psi), *oracle.project(*s.geometry(), psi, with_abs=True), "tuned")
    for setting in (lambda: plan.set_expand(bd.EXPAND_BLOCKS, 2, 8),
                    lambda: plan.set_expand(bd.EXPAND_ROWS), lambda: plan.set_expand_tile(8),
                    lambda: None):
        setting()
        plan.tune_expand(d_w, d_psi.clone(), reps=10)
        assert plan.forms() == forms and plan.expand_form() == ex
        _check(plan.expand(d_w, d_psi.clone()),
               *oracle.expand(*s.geometry(), w, psi, with_abs=True), "tuned")
    plan.close()


@pytest.mark.parametrize("nbands", [1, 3, 7, 20])
def test_expansion_tuner_from_the_owner_form(nbands):
    """Where the owner form is the fastest, it is left with its own strips (and
    not the last block shape that was timed)."""
    bd = _bd()
    s = wl.make_system("own", (40, 36, 33), 0.2, (True, False, True), 9, 0.6, 4, nbands, 77)
    psi, w = wl.psi_for(s), wl.coeffs_for(s)
    ref = oracle.expand(*s.geometry(), w, psi, with_abs=True)
    for width in (16, 32):
        plan = bd.Plan.from_system(s)
        plan.set_expand(bd.EXPAND_OWNER, 0, width)
        own = plan.expand_form()
        plan.tune_expand(_dev(w), _dev(psi), reps=3)
        if plan.forms()[2] == bd.EXPAND_OWNER:
            assert plan.expand_form() == own
        _check(plan.expand(_dev(w), _dev(psi)), *ref, "after tuning from %s" % (own,))
        plan.close()


@pytest.mark.parametrize("nu,nbands", [(nu, b) for nu in range(11) for b in (20, 33)])
def test_named_forms_at_every_cutoff(nu, nbands):
    """The forms that the defaults leave to explicit settings: work items in one
    launch and one per cut-off, blocks, rows and strips."""
    bd = _bd()
    s = wl.make_system("named", (26, 23, 21), 0.2, (True, True, False), 4, 0.6, nu, nbands,
                       800 + nu + nbands)
    psi, w = wl.psi_for(s), wl.coeffs_for(s)
    d_psi, d_w = _dev(psi), _dev(w)
    prj = oracle.project(*s.geometry(), psi, with_abs=True)
    exp = oracle.expand(*s.geometry(), w, psi, with_abs=True)
    for flags in (0, bd.FLAG_DETERMINISTIC):
        plan = bd.Plan.from_system(s, flags=flags)
        for sched in (bd.SCHED_BY_NU, bd.SCHED_SINGLE_LPT):
            plan.set_schedule(sched, 0, 8192)
            assert plan.forms()[:2] == (bd.PROJECT_ITEMS, 0)
            _check(plan.project(d_psi), *prj, "schedule %d" % sched)
        _, rows, x = plan.expand_form()
        named = [(bd.EXPAND_OWNER, 0, 16)]
        if not flags:
            named += [(bd.EXPAND_BLOCKS, max(1, rows // 2), x), (bd.EXPAND_BLOCKS, rows, x // 2),
                      (bd.EXPAND_ROWS, 0, 0)]
        for form in named:
            plan.set_expand(*form)
            assert plan.forms()[2] == form[0]
            _check(plan.expand(d_w, d_psi.clone()), *exp, "expansion %s" % (form,))
        plan.close()


def test_projection_tuner_on_deterministic_and_bloch_plans():
    """As above; a deterministic plan is back at its bits."""
    bd = _bd()
    s = wl.small_periodic(natoms=6, nbands=32)
    psi = wl.psi_for(s)
    for flags, d_psi in ((bd.FLAG_DETERMINISTIC, _dev(psi)), (bd.FLAG_BLOCH, _dev(psi + 1j * psi))):
        plan = bd.Plan.from_system(s, flags=flags)
        forms, sc = plan.forms(), plan.schedule()
        c0 = plan.project(d_psi).clone()
        plan.set_schedule(bd.SCHED_SINGLE_LPT, 0, 4096)
        assert plan.forms()[0] == bd.PROJECT_ITEMS
        plan.tune(d_psi, torch.empty_like(c0), reps=10)
        assert plan.forms() == forms and plan.schedule() == sc
        assert torch.equal(plan.project(d_psi), c0)
        plan.close()
