"""Resident 2D time stepping (many steps per launch, fields in registers)
against the streaming kernels: both do the same operations per node, so data,
images and CGNR iterates agree bit for bit.  Sizes sit at the edges of the
rows per lane (64 lanes of 2 .. 6 rows), of the slabs (8 waves of 1 .. 3
columns) and of the exchanged columns; shot counts make the plan pick narrow,
wide and mixed launches."""
import numpy as np
import pytest

from gpu_common import require_gpu, to_dev
from paper_2508_10405_amd import lsrtm, synth

pytestmark = pytest.mark.gpu


def _run(torch, w, resident, **opts):
    ctx = lsrtm.context_for(w, tile=1, **opts)
    ctx.set_option(lsrtm.OPT_RESIDENT, resident)
    dm = to_dev(torch, w.dm)
    out = []
    for _ in range(2):           # the second round reads checkpoints, graphs and cached replays
        out.append(ctx.forward())
        out.append(ctx.born(dm))
        out.append(ctx.adjoint(out[-1]))
    x, mis = ctx.cgnr(out[1], 2)
    out += [x, torch.tensor(mis)]
    ctx.close()
    return out


# (padded nz, padded nx, npml, shots, steps, interval, options)
CASES = [
    (28, 7, 3, 2, 20, 7, {}),                    # slabs narrower than a wave's halo
    (65, 40, 8, 3, 31, 0, {}),                   # two rows per lane, one past 64
    (128, 64, 6, 40, 24, 10, {}),                # exactly 64 lanes of two rows
    (129, 130, 13, 3, 40, 16, {"graph": False}),
    (192, 97, 20, 50, 24, 9, {"ckpt_dtype": "bf16"}),
    (193, 89, 20, 2, 33, 11, {"ckpt_dtype": "f16"}),
    (256, 203, 20, 24, 24, 8, {"replay_cache_mb": 600}),
    (257, 120, 20, 3, 24, 8, {"replay_cache_mb": 4000}),
    (320, 161, 13, 24, 20, 7, {"ckpt_per_group": True, "shots_per_launch": 5}),
    (321, 100, 0, 2, 16, 5, {}),                 # no absorbing strips
    (384, 75, 20, 30, 16, 6, {"shots_per_launch": 7, "replay_cache_mb": 4000}),
]


@pytest.mark.parametrize("nz,nx,npml,nshot,nt,k,opts", CASES)
def test_bitwise_equal_to_streaming(nz, nx, npml, nshot, nt, k, opts):
    torch = require_gpu()
    w = synth.small((nz - 2 * npml, nx - 2 * npml), nt=nt, npml=npml, seed=nz + nx, nshot=nshot, uneven=nshot > 2)
    a = _run(torch, w, 0, ckpt_every=k, **opts)
    b = _run(torch, w, 1, ckpt_every=k, **opts)
    for i, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), (i, float((x - y).abs().max()))


def test_switching_schedules_on_one_context():
    """The replay cache is kept in a layout per schedule: switching between
    them on one context refills it."""
    torch = require_gpu()
    w = synth.small((100, 120), nt=40, npml=10, seed=5, nshot=4)
    ctx = lsrtm.context_for(w, tile=1, ckpt_every=9, replay_cache_mb=2000)
    dm = to_dev(torch, w.dm)
    ref = None
    for resident in (1, 0, 0, 1, 1, 0):
        ctx.set_option(lsrtm.OPT_RESIDENT, resident)
        d = ctx.born(dm)
        got = (d, ctx.adjoint(d), ctx.born(dm))
        if ref is None:
            ref = got
        assert all(torch.equal(x, y) for x, y in zip(got, ref)), resident
    ctx.close()


def test_many_receivers_on_one_slab():
    """More receivers than threads on a slab, several on one node, and
    receivers on the first and last node of each axis."""
    torch = require_gpu()
    w = synth.small((60, 60), nt=30, npml=6, seed=9, nshot=2)
    rng = np.random.default_rng(3)
    full = np.stack(np.meshgrid(np.arange(60), np.arange(20, 36), indexing="ij"), -1).reshape(-1, 2)
    dup = full[rng.integers(0, len(full), 200)]
    edge = np.array([[0, 0], [59, 0], [0, 59], [59, 59]])
    w.rec = [np.concatenate([full, dup, edge]), full[::7]]
    a, b = _run(torch, w, 0, ckpt_every=8), _run(torch, w, 1, ckpt_every=8)
    for i, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), i


def test_more_launches_than_ids():
    """Segments of one step: the launches of one migration (two a segment)
    outnumber the ids that tell their exchanged words apart."""
    torch = require_gpu()
    w = synth.small((90, 60), nt=270, npml=6, seed=13, nshot=2)
    a = _run(torch, w, 0, ckpt_every=1)
    b = _run(torch, w, 1, ckpt_every=1)
    assert all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_interval_of_rounded_checkpoints(dtype):
    """16-bit checkpoints round the state at every interval, so the interval
    that the planner picks is that of a plan without the resident layout's
    larger replay buffer (the fused schedule's, which has no resident form)."""
    torch = require_gpu()
    w = synth.small((117, 60), nt=300, npml=6, seed=21, nshot=3)
    picked = []
    for fused in (False, True):
        ctx = lsrtm.context_for(w, tile=1, ckpt_dtype=dtype, fused=fused)
        picked.append(ctx.sizes()["ckpt_every"])
        ctx.close()
    assert picked[0] == picked[1]


def test_groups_of_whole_rounds():
    """Groups of unequal size (9 and 7 of 16 shots, 7 of them to a round):
    data and image are those of one shot per launch."""
    torch = require_gpu()
    w = synth.small((48, 765), nt=12, npml=6, seed=17, nshot=16)
    got = []
    for spl in (9, 1):
        ctx = lsrtm.context_for(w, tile=1, shots_per_launch=spl, ckpt_every=5)
        if spl > 1:
            assert ctx.sizes()["shots_per_launch"] == 9 and ctx.sizes()["groups"] == 2
        d = ctx.born(to_dev(torch, w.dm))
        got.append((d, ctx.adjoint(d)))
        ctx.close()
    assert all(torch.equal(x, y) for x, y in zip(*got))


@pytest.mark.parametrize("nz,nx,npml,nshot", [(320, 203, 20, 24), (300, 203, 20, 24), (240, 100, 0, 30), (128, 60, 9, 2)])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_not_finite_values_stay_in_their_cone(nz, nx, npml, nshot, bad):
    """One Inf or NaN among the data, in the perturbation and in a wavelet, and
    a march too short for it to reach the whole grid: the same values are
    finite, and equal, on either schedule (wide launches keep the z strips'
    memories in LDS slots that many lanes share, narrow ones in registers)."""
    torch = require_gpu()
    nt = 5
    w = synth.small((nz - 2 * npml, nx - 2 * npml), nt=nt, npml=npml, seed=nz, nshot=nshot)
    at = (nz - 2 * npml - 8, nx // 2 - npml)             # in the last lane with rows outside the z strips
    w.rec[0][0] = at
    w.src[0] = at
    got = []
    for resident in (0, 3):
        ctx = lsrtm.context_for(w, tile=1, ckpt_every=nt)
        ctx.set_option(lsrtm.OPT_RESIDENT, resident)
        dm = to_dev(torch, w.dm)
        d = ctx.born(dm)
        y = d.clone()
        y[(nt - 1) * len(w.rec[0])] = bad                # last step, first receiver of shot 0
        dm[0, at[1], at[0]] = bad
        out = [ctx.adjoint(y), ctx.born(dm)]
        wav = to_dev(torch, w.wavelet)
        wav[0, 3] = bad
        ctx.set_acquisition(w.win, w.src, w.rec, wav)
        out.append(ctx.forward())
        assert ctx.resident()["last"] == (resident > 0)
        got.append(out)
        ctx.close()
    for i, (a, b) in enumerate(zip(*got)):
        fin = torch.isfinite(a)
        assert 0 < int(fin.sum()) < fin.numel(), i
        assert torch.equal(fin, torch.isfinite(b)), (i, int(fin.sum()), int(torch.isfinite(b).sum()))
        assert torch.equal(a[fin], b[fin]), i


def test_small_contexts_side_by_side():
    """Contexts on streams and threads of their own whose launches fit the GPU
    together (one shot each, 30 workgroups) do not take turns; their results
    are those of one alone."""
    import threading
    import time
    torch = require_gpu()
    n, calls = 4, 25
    w = synth.small((100, 200), nt=1000, npml=20, seed=3, nshot=1)
    jobs = []
    for _ in range(n):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            ctx = lsrtm.context_for(w, tile=1)
            dm = to_dev(torch, w.dm)
            d = ctx.born(dm)
            ref = ctx.born(dm).clone()
        torch.cuda.synchronize()
        jobs.append((st, ctx, dm, d, ref))

    def run(job):
        st, ctx, dm, d, _ = job
        with torch.cuda.stream(st):
            for _ in range(calls):
                ctx.born(dm, d)
            st.synchronize()

    def timed(which):
        ts = [threading.Thread(target=run, args=(j,)) for j in which]
        t = time.perf_counter()
        for th in ts:
            th.start()
        for th in ts:
            th.join()
        return time.perf_counter() - t
    timed(jobs)
    one, all_ = min(timed(jobs[:1]) for _ in range(3)), min(timed(jobs) for _ in range(3))
    print(f"one context {one * 1e3 / calls:.2f} ms a call, {n} side by side {all_ * 1e3 / calls:.2f}", flush=True)
    for _, ctx, _, d, ref in jobs:
        assert torch.equal(d, ref)
        ctx.close()
    assert all_ < 0.7 * n * one


@pytest.mark.parametrize("nz,nx,npml,nshot,nt,k,opts", CASES)
def test_calls_run_resident(nz, nx, npml, nshot, nt, k, opts):
    """Wherever the windows fit (3), first and later calls do run on the
    resident kernels, without one that gives up, and give the streaming ones'
    bits."""
    torch = require_gpu()
    w = synth.small((nz - 2 * npml, nx - 2 * npml), nt=nt, npml=npml, seed=nz + nx, nshot=nshot, uneven=nshot > 2)
    a = _run(torch, w, 0, ckpt_every=k, **opts)
    b = _run(torch, w, 3, ckpt_every=k, **opts)
    for i, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), (i, float((x - y).abs().max()))
    ctx = lsrtm.context_for(w, tile=1, ckpt_every=k, **opts)
    ctx.set_option(lsrtm.OPT_RESIDENT, 3)
    dm = to_dev(torch, w.dm)
    on = {"planned": True, "last": True, "gave_up": 0}
    for _ in range(2):
        d = ctx.forward()
        assert ctx.resident() == on
        d = ctx.born(dm, d)
        assert ctx.resident() == on
        ctx.adjoint(d)
        assert ctx.resident() == on
    ctx.cgnr(d, 1)
    assert ctx.resident() == on
    ctx.close()


@pytest.mark.parametrize("opts", [{}, {"graph": False}, {"replay_cache_mb": 2000}, {"ckpt_dtype": "bf16"},
                                  {"ckpt_per_group": True, "shots_per_launch": 2}, {"timing": True}])
def test_launches_that_find_no_room(opts):
    """A call whose launches give up runs again on the streaming kernels, in
    the middle of a CGNR run too: the results are theirs bit for bit, also
    those of the calls after it.  It is counted, and the next calls do not try
    again until the pause is over."""
    torch = require_gpu()
    w = synth.small((100, 120), nt=40, npml=10, seed=6, nshot=4)
    got = []
    for resident in (0, 2, 1):
        ctx = lsrtm.context_for(w, tile=1, ckpt_every=9, **opts)
        dm = to_dev(torch, w.dm)
        out = []
        gave_up = 0
        for call in (ctx.forward, lambda: ctx.born(dm), lambda: ctx.adjoint(out[1]), lambda: ctx.born(dm),
                     lambda: ctx.adjoint(out[0])):
            ctx.set_option(lsrtm.OPT_RESIDENT, resident)      # ends the pause
            out.append(call())
            gave_up += resident == 2
            assert ctx.resident() == {"planned": resident > 0, "last": resident == 1, "gave_up": gave_up}
        out.append(ctx.adjoint(out[0]))
        assert ctx.resident()["gave_up"] == gave_up
        x = ctx.cgnr_begin(out[1])
        for it in range(3):
            if resident == 2:
                ctx.set_option(lsrtm.OPT_RESIDENT, 2 if it == 1 else 1)
            out.append(torch.tensor(ctx.cgnr_iterate(x)))
            gave_up += resident == 2 and it == 1
            assert ctx.resident()["gave_up"] == gave_up
        out.append(x)
        got.append(out)
        if "timing" in opts:
            # the samples of the launches that gave up are not counted
            d = ctx.adjoint(out[0])
            ctx.set_option(lsrtm.OPT_RESIDENT, resident)
            ctx.adjoint(out[0])
            assert ctx.stats()["adj_a"][1] == w.nt or resident != 1
            assert (ctx.stats()["adj_b"][1] > 0) == (resident != 1)
        ctx.close()
    for other in got[1:]:
        for i, (a, b) in enumerate(zip(got[0], other)):
            assert torch.equal(a, b), i


def test_streaming_passes_of_resident_plans_are_tuned(tmp_path, monkeypatch):
    """Passes of a resident plan need no tile, so none is tuned for them; the
    pseudo-Hessian pass and a call that found no room take the streaming
    kernels, whose tile is tuned before the first of these (the tuner adds a
    line to its file)."""
    torch = require_gpu()
    w = synth.small((60, 80), nt=20, npml=8, seed=4, nshot=2)
    dm = to_dev(torch, w.dm)
    for i, streaming in enumerate((lambda c: c.pseudo_hessian(), lambda c: c.born(dm))):
        file = tmp_path / f"tune{i}.txt"
        monkeypatch.setenv("LSRTM_TUNE_CACHE", str(file))
        ctx = lsrtm.context_for(w)
        ctx.born(dm)
        ctx.adjoint(ctx.forward())
        assert ctx.resident()["last"] and not file.exists()
        ctx.set_option(lsrtm.OPT_RESIDENT, 2)
        for _ in range(2):
            streaming(ctx)
            assert len(file.read_text().splitlines()) == 1
        ctx.close()


def _context(torch, w, resident, **opts):
    """Planned with the option set (or None for the default)."""
    ctx = lsrtm.Context(tuple(reversed(w.lnvp.shape)), w.h, w.nt, w.dt, npml=w.npml, pml_R=w.pml_R, pml_f0=w.pml_freq,
                        **opts)
    if resident is not None:
        ctx.set_option(lsrtm.OPT_RESIDENT, resident)
    ctx.set_model(to_dev(torch, w.lnvp), to_dev(torch, w.lnip))
    ctx.set_acquisition(w.win, w.src, w.rec, to_dev(torch, w.wavelet))
    return ctx


@pytest.mark.parametrize("opts", [{"ckpt_every": 60}, {}, {"ckpt_dtype": "bf16"}, {"ckpt_dtype": "bf16", "ckpt_every": 60}])
def test_budgets_that_held_the_plan_still_do(opts):
    """The resident kernels' replay buffer takes four times the memory at 32
    padded rows.  A budget that holds a plan without it holds one with the
    option on, with the same checkpoint layout; the results are the same."""
    torch = require_gpu()
    w = synth.small((20, 400), nt=60, npml=6, seed=31, nshot=8, nrec=40)
    dm = to_dev(torch, w.dm)
    seen = set()
    ref = None
    for budget in list(range(66, 100, 2)) + list(range(100, 460, 20)):
        plans = []
        for resident in (0, 3):
            try:
                ctx = _context(torch, w, resident, mem_budget_mb=budget, **opts)
            except lsrtm.LsrtmError as e:
                assert e.status == lsrtm.ENOMEM
                plans.append(None)
                continue
            sz = ctx.sizes()
            assert sz["plan_bytes"] <= budget << 20
            plans.append(sz["ckpt_per_group"])
            if resident:
                on = ctx.resident()["planned"]
                if (on, sz["ckpt_per_group"], sz["groups"]) not in seen:
                    d = ctx.born(dm)
                    got = (d, ctx.adjoint(d)) if "ckpt_dtype" not in opts else (d,)
                    ref = ref or got
                    assert ctx.resident()["last"] == on
                    assert all(torch.equal(a, b) for a, b in zip(ref, got))
                seen.add((on, sz["ckpt_per_group"], sz["groups"]))
            ctx.close()
        assert plans[0] == plans[1], (budget, plans)
    assert {on for on, _, _ in seen} == {True, False}


def test_plans_without_the_resident_layout():
    """With the option off, and where a slab has more receivers than its LDS
    holds, the replay buffer has the size that the streaming kernels need, the
    groups are balanced, and turning the option off and on re-plans."""
    torch = require_gpu()
    k = 10
    w = synth.small((20, 765), nt=40, npml=6, seed=32, nshot=16, nrec=40)
    off, on = (_context(torch, w, r, ckpt_every=k, shots_per_launch=9) for r in (0, 3))
    assert off.sizes()["shots_per_launch"] == 8 and on.sizes()["shots_per_launch"] == 9
    padded, plain = 777 * 2 * 64, 777 * 32
    grp = lambda n: n * (plain * (7 + 7 + 2) * 4)
    assert on.sizes()["plan_bytes"] - off.sizes()["plan_bytes"] == grp(9) - grp(8) + k * 3 * 4 * (9 * padded - 8 * plain)
    sizes = on.sizes()
    on.set_option(lsrtm.OPT_RESIDENT, 0)
    assert on.sizes() == off.sizes() and not on.resident()["planned"]
    on.set_option(lsrtm.OPT_RESIDENT, 3)
    assert on.sizes() == sizes and on.resident()["planned"]
    for ctx in (off, on):
        ctx.close()
    many = synth.small((20, 60), nt=20, npml=6, seed=33, nshot=2)
    many.rec[0] = np.stack([np.random.default_rng(1).integers(0, 20, 12000), np.full(12000, 30)], axis=1)
    for dup, fits in ((many.rec[0], False), (many.rec[0][:4000], True)):
        many.rec[0] = dup
        ctx, ref = (_context(torch, many, r, ckpt_every=7) for r in (3, 0))
        assert ctx.resident()["planned"] == fits
        if not fits:
            assert ctx.sizes()["plan_bytes"] == ref.sizes()["plan_bytes"]
        d = ctx.born(to_dev(torch, many.dm))
        assert torch.equal(d, ref.born(to_dev(torch, many.dm)))
        assert torch.equal(ctx.adjoint(d), ref.adjoint(d))
        assert ctx.resident()["last"] == fits
        ctx.close()
        ref.close()


# (padded nz, padded nx, npml, shots, steps), whether forward, Born, migration take the resident kernels; with a replay
# cache Born passes and migrations, which share it, go together
ROUTES = [
    ((8, 240, 0, 256, 100), (False, False, False)),      # 4 of 64 lanes, 256 shots
    ((28, 757, 10, 64, 100), (False, False, False)),
    ((40, 260, 10, 256, 100), (False, True, False)),     # together 0.98 of the streaming estimate
    ((28, 80, 6, 32, 12), (True, False, True)),          # together 0.83
    ((64, 280, 20, 64, 12), (False, False, False)),      # a short march
    ((28, 260, 10, 4, 100), (True, True, True)),         # few shots
    ((140, 240, 20, 1, 1000), (True, True, True)),
    ((280, 777, 20, 14, 100), (True, True, True)),
]


@pytest.mark.parametrize("shape,expect", ROUTES)
@pytest.mark.parametrize("opts", [{}, {"replay_cache_mb": 4000}])
def test_route_by_estimate(shape, expect, opts):
    """Which kernels a kind of call takes by itself, and that calls of a plan
    on mixed routes share checkpoints and cached replays rightly."""
    torch = require_gpu()
    nz, nx, npml, nshot, nt = shape
    if shape[0] == 28 and nshot == 32:
        opts = dict(opts, ckpt_every=20)                 # one segment
    if "replay_cache_mb" in opts and expect[1] != expect[2]:
        expect = (expect[0],) + (shape[0] == 28,) * 2
    w = synth.small((nz - 2 * npml, nx - 2 * npml), nt=nt, npml=npml, seed=nz, nshot=nshot, nrec=30)
    dm = to_dev(torch, w.dm)
    got, every = [], []
    for resident in (1, 0):
        ctx = _context(torch, w, None if resident else 0, mem_budget_mb=30000, **opts)
        out, route = [], []
        for call in (ctx.forward, lambda: ctx.born(dm), lambda: ctx.adjoint(out[1]), lambda: ctx.born(dm),
                     lambda: ctx.adjoint(out[1]), ctx.forward):
            out.append(call())
            route.append(ctx.resident()["last"])
        assert tuple(route) == ((*expect, *expect[1:], expect[0]) if resident else (False,) * 6)
        assert ctx.resident()["planned"] == (bool(resident) and any(expect))
        every.append(ctx.sizes()["ckpt_every"])
        x, mis = ctx.cgnr(out[1], 1)
        got.append(out + [x, torch.tensor(mis)])
        ctx.close()
    for i, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), i
    # calls that stay streaming write no more checkpoints for the others' sake
    assert "replay_cache_mb" in opts or all(expect) or every[0] >= every[1]


def test_autotune_times_the_kernels_of_the_passes(tmp_path, monkeypatch):
    """One small shot, whose fused steps are one launch and two-phase streaming
    steps two: the tuner compares the fused steps with the resident ones that
    its passes take, and a tuning file of the streaming kernels is not theirs."""
    torch = require_gpu()
    w = synth.small((100, 200), nt=200, npml=20, seed=8, nshot=1)
    dm = to_dev(torch, w.dm)
    ms = []
    for resident in (0, 1):
        file = tmp_path / f"tune{resident}.txt"
        monkeypatch.setenv("LSRTM_TUNE_CACHE", str(file))
        ctx = _context(torch, w, resident)
        pts = ctx.sizes()["padded_points"]
        if resident:
            file.write_text(f"nd=2 nshot=1 pts={pts} nt=200 n=100x200x1 npml=20|1 0 1 -1 -1\n")
        res = ctx.autotune(nsteps=8, groups=True)
        ms.append(res["ms_per_step"])
        if resident:
            assert ctx.sizes()["fused"] == 0
            assert ctx.resident()["planned"]
            d = ctx.born(dm)
            assert ctx.resident()["last"]
        else:
            d_ref = ctx.born(dm)
        print("autotune", resident, res, ctx.sizes()["fused"], flush=True)
        ctx.close()
    assert 0.0 < ms[1] < ms[0]
    assert torch.equal(d, d_ref)


def test_born_passes_keep_off_the_other_layout():
    """A Born pass on the streaming kernels while the replay cache holds the
    resident kernels' layout (its launch found no room) does not read it."""
    torch = require_gpu()
    w = synth.small((100, 120), nt=40, npml=10, seed=12, nshot=4)
    dm = to_dev(torch, w.dm)
    ctx = _context(torch, w, 1, ckpt_every=9, replay_cache_mb=2000)
    d = ctx.born(dm)
    img = ctx.adjoint(d)
    assert ctx.resident()["last"] and ctx.sizes()["replay_cache_segments"] > 0
    assert torch.equal(ctx.born(dm), d)
    ctx.set_option(lsrtm.OPT_RESIDENT, 2)
    for _ in range(2):                    # gives up, then the pause
        assert torch.equal(ctx.born(dm), d)
        assert not ctx.resident()["last"]
    ctx.set_option(lsrtm.OPT_RESIDENT, 1)
    assert torch.equal(ctx.born(dm), d) and torch.equal(ctx.adjoint(d), img)
    ctx.close()


def test_calls_that_share_a_cache_go_together():
    """Born passes and migrations of a plan with a replay cache take the same
    kernels, also where the estimate has one of them faster on the others (32
    small shots, 12 steps in one segment): every Born pass after a migration
    reads the cached replays."""
    torch = require_gpu()
    w = synth.small((16, 68), nt=12, npml=6, seed=14, nshot=32, nrec=20)
    dm = to_dev(torch, w.dm)
    got = []
    for resident in (None, 0):
        ctx = _context(torch, w, resident, ckpt_every=20, replay_cache_mb=2000)
        assert ctx.sizes()["replay_cache_segments"] == 1
        out, route = [], []
        for call in (lambda: ctx.born(dm), lambda: ctx.adjoint(out[0]), lambda: ctx.born(dm), lambda: ctx.adjoint(out[0]),
                     lambda: ctx.born(dm)):
            out.append(call())
            route.append(ctx.resident()["last"])
        assert route == [resident is None] * 5
        got.append(out)
        ctx.close()
    for i, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), i


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_cached_replays_of_rounded_checkpoints(dtype):
    """Born passes take the segments that the replay cache holds from there,
    with the rounding of 16-bit checkpoints: as many segments as without the
    resident layout, after launches that found no room and during the pause too."""
    torch = require_gpu()
    w = synth.small((100, 120), nt=60, npml=10, seed=15, nshot=6)
    dm = to_dev(torch, w.dm)
    planned = set()
    for mb in (4, 30, 60, 90, 130, 2000):
        got = []
        for resident in (0, 1):
            ctx = _context(torch, w, resident, ckpt_dtype=dtype, ckpt_every=9, replay_cache_mb=mb, shots_per_launch=4)
            held = ctx.sizes()["replay_cache_segments"]
            out = []
            # the option before each call: 2 gives up, 1 after it ends the pause, None leaves it
            for kind, option in (("f", 1), ("b", 1), ("a", 1), ("b", 1), ("b", 2), ("b", None), ("a", None), ("b", None),
                                 ("b", 1), ("a", 1), ("b", 1), ("f", 2), ("b", None), ("b", 1), ("a", 2), ("b", None), ("b", 1),
                                 ("a", 1), ("b", 1)):
                if resident and option is not None:
                    ctx.set_option(lsrtm.OPT_RESIDENT, option)
                out.append(ctx.forward() if kind == "f" else ctx.born(dm) if kind == "b" else ctx.adjoint(out[0]))
            got.append(out)
            if resident:
                planned.add(ctx.resident()["planned"])
                segments.append(held)
            else:
                segments = [held]
            ctx.close()
        assert dtype == "f32" or segments[0] == segments[1]
        for i, (a, b) in enumerate(zip(*got)):
            assert torch.equal(a, b), (mb, i, segments)
    assert True in planned


@pytest.mark.parametrize("nz,nx,npml,nshot", [(12, 42, 0, 3), (65, 60, 0, 2), (257, 60, 4, 3), (320, 203, 20, 24)])
def test_subnormal_images(nz, nx, npml, nshot):
    """Data so small that the images are subnormal: the same bits."""
    torch = require_gpu()
    w = synth.small((nz - 2 * npml, nx - 2 * npml), nt=14, npml=npml, seed=nz, nshot=nshot)
    for s in range(nshot):               # about the last rows, whose half nodes are their own
        w.rec[s][:, 0] = nz - 2 * npml - 1 - np.arange(len(w.rec[s])) % 3
        w.src[s] = (nz - 2 * npml - 2, w.src[s][1])
    got = []
    for resident in (0, 3):
        ctx = _context(torch, w, resident, ckpt_every=5)
        d = ctx.born(to_dev(torch, w.dm))
        top = float(ctx.adjoint(d).abs().max())
        got.append([ctx.adjoint(d * (s / top)) for s in (1e-36, 1e-38, 1e-40, 1e-42)])
        assert 0.0 < float(got[-1][-2].abs().max()) < 1.2e-38
        assert ctx.resident()["last"] == (resident > 0)
        ctx.close()
    for i, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32)), (i, int((a != b).sum()))
