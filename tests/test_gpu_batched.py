"""Batched form: many independent solves in one context, graph replay of
chunks of sweeps, persistent launch shapes and the autotuner.

Launch shapes and graph replay only change how the same kernels are issued:
every variant must give bit-identical amplitudes and energies.  The 40-solve
batch (N in {14, 38, 54, 66} x 10 densities, cutoffs drawn from a seeded
generator) must reproduce each solve run alone in its own context, and its
smallest members the oracle.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ccd = pytest.importorskip("paper_1611_06765_amd.ccd")

DENS = [round(0.02 * (k + 1), 2) for k in range(10)]
C4_SEED = 20161121


def c4_cutoffs(seed=C4_SEED):
    """Cutoff n^2 <= nmax2 of each of the 40 solves, in the order
    (N, density) = (14, 0.02), (14, 0.04), ..., (66, 0.20)."""
    return np.random.default_rng(seed).integers(12, 37, size=40)


def c4_problems(seed=C4_SEED):
    cut = c4_cutoffs(seed)
    out = []
    for a, n in enumerate([14, 38, 54, 66]):
        for b, r in enumerate(DENS):
            out.append(ccd.problem(n, int(cut[10 * a + b]), r))
    return out


def _ctx(probs):
    import torch
    assert torch.cuda.is_available()
    return ccd.Context(probs, stream=torch.cuda.current_stream().cuda_stream).bind()


def _all_t(ctx):
    return [ctx.get_amplitudes(p) for p in range(ctx.n)]


MIXED_SET = [(38, 12, 0.06), (66, 20, 0.16), (14, 20, 0.10), (66, 36, 0.16)]


def test_graph_replay_bit_identical_to_eager():
    probs = [ccd.problem(*x) for x in MIXED_SET[:3]]
    a = _ctx(probs)
    ra = a.iterate(mixing=0.6, tol=0.0, max_iter=7, history=True)
    b = _ctx(probs)
    rb = b.iterate(mixing=0.6, tol=0.0, max_iter=7, history=True, check_every=3, graph=True)
    assert np.array_equal(ra["history"], rb["history"])
    for x, y in zip(_all_t(a), _all_t(b)):
        assert np.array_equal(x, y)
    # replaying the cached graphs again continues the same iteration
    ra = a.iterate(mixing=0.6, tol=0.0, max_iter=7, history=True)
    rb = b.iterate(mixing=0.6, tol=0.0, max_iter=7, history=True, check_every=3, graph=True)
    assert np.array_equal(ra["history"], rb["history"])


def test_check_every_does_not_change_convergence():
    probs = [ccd.problem(*x) for x in MIXED_SET[:3]]
    a = _ctx(probs)
    ra = a.iterate(mixing=0.5, tol=1e-8, max_iter=300, history=True)
    b = _ctx(probs)
    rb = b.iterate(mixing=0.5, tol=1e-8, max_iter=300, history=True, check_every=16, graph=True)
    assert ra["status"] == rb["status"] == ccd.CCD_OK
    assert np.array_equal(ra["sweeps"], rb["sweeps"])
    assert np.array_equal(ra["history"], rb["history"], equal_nan=True)
    for p in range(len(probs)):
        assert a.energy(p) == b.energy(p)


@pytest.mark.parametrize("precision,mixed_tol,rule", [(0, 0.0, 0), (0, 0.0, 1), (2, 1e-2, 1)])
def test_chunk_lengths_do_not_change_the_solve(precision, mixed_tol, rule):
    """The host shortens a chunk of sweeps to the sweeps it predicts the
    slowest live problem still needs (no graph replay); the device alone
    decides when each problem stops, so reading its flags after every sweep,
    every 8 sweeps with that prediction, or once per 64 gives the same sweep
    counts, energy histories and energies, in FP64 and in a BF16 phase with
    FP64 refinement (two phases, each with its own prediction)."""
    probs = [ccd.problem(*x) for x in MIXED_SET[:3]]
    out = []
    for every in (1, 8, 64):
        c = _ctx(probs)
        r = c.iterate(mixing=0.5, tol=0.0, tol_rel=1e-9, stop_rule=rule, max_iter=300, history=True,
                      check_every=every, precision=precision, mixed_tol=mixed_tol, refine_sweeps=2)
        assert r["status"] == ccd.CCD_OK
        out.append((r, [c.energy(p) for p in range(len(probs))]))
    for r, e in out[1:]:
        assert np.array_equal(out[0][0]["sweeps"], r["sweeps"])
        assert np.array_equal(out[0][0]["history"], r["history"], equal_nan=True)
        assert out[0][1] == e


TABLES = [
    [1, 1, 1, 1, 1, 1, 0, 0, 0, 0],
    [2, 2, 2, 2, 2, 2, 1, 1, 1, 1],
    [4, 4, 4, 4, 4, 4, 1, 0, 1, 0],
    [0, 0, 0, 0, 0, 0, 1, 1, 1, 1],
]


@pytest.mark.parametrize("prec", [ccd.CCD_PREC_FP64, ccd.CCD_PREC_BF16])
def test_launch_shapes_bit_identical(prec):
    """Persistent grids and the alternative ring tile shapes, all four ring
    size buckets populated (the n^2 <= 36 member has pair blocks of order > 64)."""
    probs = [ccd.problem(*x) for x in MIXED_SET]
    ref = _ctx(probs)
    info = ref.info(3)
    assert info["max_ph"] > 64
    ref.iterate(mixing=0.7, tol=0.0, max_iter=3, precision=prec)
    want = _all_t(ref)
    for tab in TABLES:
        c = _ctx(probs)
        c.set_tuning(tab)
        assert np.array_equal(c.get_tuning(), tab)
        c.iterate(mixing=0.7, tol=0.0, max_iter=3, precision=prec)
        for x, y in zip(want, _all_t(c)):
            assert np.array_equal(x, y), tab


def test_problems_stopping_at_different_sweeps_under_every_launch_shape():
    """Inside a run the energy step of a sweep (which clears the flag of a
    problem that has converged) runs as extra blocks of the next sweep's
    chi_klij launch, beside that launch's own items and the rings.  With
    problems stopping at different sweeps, persistent grids (workgroups that
    take several items) and flags read every sweep or every 8 sweeps, every
    sweep count, energy history and energy equals that of the default shapes
    with the flags read after every sweep."""
    probs = [ccd.problem(n, n2, rho) for n, n2 in ((14, 8), (38, 12), (54, 16), (66, 20))
             for rho in (0.05, 0.1, 0.2)]

    def solve(tab, every, graph=False):
        c = _ctx(probs)
        c.set_tuning(tab)
        r = c.iterate(mixing=0.5, tol=0.0, tol_rel=1e-9, stop_rule=1, max_iter=300, history=True,
                      check_every=every, graph=graph)
        assert r["status"] == ccd.CCD_OK
        return r, [c.energy(p) for p in range(len(probs))]

    ref, e_ref = solve([0] * ccd.CCD_TUNE_LEN, 1)
    assert len(set(ref["sweeps"].tolist())) > 3  # the problems stop at different sweeps
    for tab in [[0] * ccd.CCD_TUNE_LEN] + TABLES:
        for every, graph in ((1, False), (8, False), (8, True)):
            r, e = solve(tab, every, graph)
            assert np.array_equal(ref["sweeps"], r["sweeps"]), (tab, every, graph)
            assert np.array_equal(ref["history"], r["history"], equal_nan=True), (tab, every, graph)
            assert e_ref == e, (tab, every, graph)


def test_autotune_keeps_the_iteration():
    probs = [ccd.problem(*x) for x in MIXED_SET]
    ref = _ctx(probs)
    ref.iterate(mixing=0.5, tol=0.0, max_iter=4)
    c = _ctx(probs)
    c.iterate(mixing=0.5, tol=0.0, max_iter=2)
    tab, best = c.autotune(ccd.CCD_PREC_FP64, reps=3)
    assert np.all(best >= 0.0) and best[ccd.CCD_TUNE_LADDER] > 0.0
    for k, v in enumerate(tab):
        assert v in ((0, 1, 2, 4) if k < ccd.CCD_TUNE_RING_NW32 else (0, 1))
    c.iterate(mixing=0.5, tol=0.0, max_iter=2, graph=True, check_every=2)
    for x, y in zip(_all_t(ref), _all_t(c)):
        assert np.array_equal(x, y)
    with pytest.raises(ccd.CCDError):
        c.set_tuning([3] + [0] * 9)


def test_c4_batch_matches_separate_solves_and_oracle():
    """The 40-solve batch, FP64, two sweeps: each member equals the same solve
    in its own context bit for bit; the N = 14 members match the oracle."""
    from oracle import oracle
    probs = c4_problems()
    big = _ctx(probs)
    h = big.iterate(mixing=0.5, tol=0.0, max_iter=2, history=True, check_every=2, graph=True)["history"]
    for p, pr in enumerate(probs):
        one = _ctx([pr])
        h1 = one.iterate(mixing=0.5, tol=0.0, max_iter=2, history=True)["history"]
        assert np.array_equal(h[p], h1[0]), p
    cut = c4_cutoffs()
    for b in (0, 4, 9):
        o3 = oracle.O3(oracle.PNM(14, int(cut[b]), DENS[b]))
        for s in range(2):
            e = o3.sweep(0.5)
            assert abs(h[b, s] - e) <= 1e-10 * abs(e), (b, s, h[b, s], e)


def test_c4_mixed_batched_converges_to_fp64():
    """The 40 solves batched, BF16 contractions then FP64 refinement, graph
    replay and tuned shapes: every energy within 1e-6 of the FP64 solve."""
    probs = c4_problems()
    ref = _ctx(probs)
    r = ref.iterate(mixing=0.5, tol=1e-9, max_iter=600, check_every=8, graph=True)
    assert r["status"] == ccd.CCD_OK
    mix = _ctx(probs)
    mix.autotune(ccd.CCD_PREC_BF16, reps=2)
    m = mix.iterate(mixing=0.5, tol=1e-9, max_iter=600, precision=ccd.CCD_PREC_BF16, mixed_tol=1e-3,
                    refine_sweeps=3, check_every=8, graph=True)
    assert m["status"] == ccd.CCD_OK
    for p in range(len(probs)):
        e64, em = ref.energy(p)[2], mix.energy(p)[2]
        assert abs(em - e64) <= 1e-6 * abs(e64), (p, em, e64)


def test_extrapolated_stop_rule_bounds_the_error():
    """stop_rule 1: from the MBPT2 start and from a perturbed start (which
    excites every mode), stopping at tol_rel = 1e-7 leaves each energy within
    1e-6 of the converged one; the plain |dE| test is never stricter."""
    probs = [ccd.problem(66, 20, 0.16), ccd.problem(38, 12, 0.06)]
    ref = _ctx(probs)
    ref.iterate(mixing=0.5, tol=1e-11, max_iter=2000, check_every=16)
    e_ref = [ref.energy(p)[2] for p in range(2)]
    for scale in (1.0, 1.6):
        a = _ctx(probs)
        b = _ctx(probs)
        for c in (a, b):
            if scale != 1.0:
                for p in range(2):
                    c.set_amplitudes(c.get_amplitudes(p) * scale, p)
        ra = a.iterate(mixing=0.5, tol=0.0, tol_rel=1e-7, stop_rule=1, max_iter=2000)
        rb = b.iterate(mixing=0.5, tol=0.0, tol_rel=1e-7, stop_rule=0, max_iter=2000)
        assert ra["status"] == rb["status"] == ccd.CCD_OK
        assert np.all(ra["sweeps"] >= rb["sweeps"])
        for p in range(2):
            assert abs(a.energy(p)[2] - e_ref[p]) <= 1e-6 * abs(e_ref[p]), (scale, p)


# sizes at the edges of the merged launches: one hole pair; small pairs only; pairs of
# order 32, 48, 64; of order 66 (kept in 68 rows); of order above 68 (a twist)
_EDGE = [[(2, 1, 0.1)], [(14, 4, 0.1), (14, 11, 0.07)], [(38, 12, 0.1)], [(54, 12, 0.12), (2, 9, 0.1)],
         [(66, 20, 0.16), (66, 20, 0.08), (66, 20, 0.12)], [(66, 36, 0.16)],
         [(66, 36, 0.16, 41.47, (0.725, 0.725, 0.725))]]


@pytest.mark.parametrize("specs", _EDGE, ids=lambda s: "-".join(f"{x[0]}_{x[1]}" for x in s))
@pytest.mark.parametrize("prec", [ccd.CCD_PREC_FP64, ccd.CCD_PREC_FP32, ccd.CCD_PREC_BF16])
def test_three_launch_sweep_equals_the_separate_launches(specs, prec):
    """The default sweep (three launches on one stream) against the families
    as launches of their own, bit for bit, for each term alone and all
    together: energies of every sweep and all amplitudes."""
    probs = [ccd.problem(*x) for x in specs]
    a, b = _ctx(probs), _ctx(probs)
    b.set_tuning([0, 0, 0, 0, 0, 4, 0, 0, 0, 0])
    for mask in (1, 2, 4, 8, 16, 32, 64, 127):
        out = []
        for c in (a, b):
            c.reset_amplitudes()
            out.append(c.iterate(mixing=0.5, max_iter=3, precision=prec, terms=mask, history=True, check_every=2))
        assert np.array_equal(out[0]["history"], out[1]["history"]), mask
        for p in range(len(probs)):
            assert np.array_equal(a.get_amplitudes(p), b.get_amplitudes(p)), (mask, p)


# problems that stop at different sweeps: several of one group, several groups, one with
# small pairs only beside large ones
_STOPS = [[(14, 4, r) for r in (0.02, 0.2, 0.1)], [(66, 20, 0.16), (66, 20, 0.02), (14, 4, 0.05), (38, 12, 0.1)],
          [(2, 1, 0.1), (66, 36, 0.06), (54, 12, 0.2)]]


@pytest.mark.parametrize("specs", _STOPS, ids=lambda s: "-".join(f"{x[0]}_{x[1]}" for x in s))
@pytest.mark.parametrize("prec", [ccd.CCD_PREC_FP64, ccd.CCD_PREC_BF16])
@pytest.mark.parametrize("every", [1, 2, 8])
def test_problems_that_stop_early_equal_their_own_contexts(specs, prec, every):
    """Problems leave the sweep's lists as they stop.  Sweeps, energies and
    amplitudes equal those of a context of the problem's own bit for bit, also
    after more sweeps of all problems, whose first one reads whichever of the two
    amplitude buffers a problem ended in."""
    probs = [ccd.problem(*x) for x in specs]
    opt = dict(mixing=0.5, tol_rel=2e-8, max_iter=120, stop_rule=1, precision=prec, history=True, refine_sweeps=1,
               mixed_tol=1e-2 if prec else 0.0, check_every=every)
    def solve(c, more):
        r = c.iterate(**opt)
        t = [c.get_amplitudes(p) for p in range(c.n)]
        m = c.iterate(mixing=0.5, max_iter=more, history=True)
        return r["sweeps"], r["history"], t, m["history"], [c.get_amplitudes(p) for p in range(c.n)]
    batch = _ctx(probs)
    runs = [solve(batch, 3)]
    batch.reset_amplitudes()
    runs.append(solve(batch, 2))
    assert len(set(runs[0][0])) > 1
    for p, prob in enumerate(probs):
        alone = _ctx([prob])
        for more, run in zip((3, 2), runs):
            alone.reset_amplitudes()
            ref = solve(alone, more)
            assert run[0][p] == ref[0][0]
            assert np.array_equal(run[1][p], ref[1][0], equal_nan=True)
            assert np.array_equal(run[2][p], ref[2][0])
            assert np.array_equal(run[3][p], ref[3][0])
            assert np.array_equal(run[4][p], ref[4][0])


@pytest.mark.parametrize("specs", [[(14, 64, r) for r in np.linspace(0.05, 0.2, 14)],
                                   [(38, 12, r) for r in np.linspace(0.05, 0.2, 12)] + [(2, 64, 0.1)]],
                         ids=["14_64", "38_12"])
def test_ladder_on_four_waves_equals_eight(specs):
    """Batches with more than 1024 ladder items (four waves an item) against each
    problem alone (eight), bit for bit, also at the largest cutoff's table of 257
    entries: the pp ladder, the hh ladder and all terms."""
    probs = [ccd.problem(*x) for x in specs]
    batch = _ctx(probs)
    for mask in (1, 18, 127):
        batch.reset_amplitudes()
        e = batch.iterate(mixing=0.5, max_iter=3, terms=mask, history=True)["history"]
        for p in (0, len(probs) // 2, len(probs) - 1):
            alone = _ctx([probs[p]])
            r = alone.iterate(mixing=0.5, max_iter=3, terms=mask, history=True)
            assert np.array_equal(e[p], r["history"][0]), (mask, p)
            assert np.array_equal(batch.get_amplitudes(p), alone.get_amplitudes(0)), (mask, p)


@pytest.mark.parametrize("specs", [[(14, 4, 0.1)], [(14, 12, 0.1)], [(54, 16, 0.1)], [(66, 36, 0.1)],
                                   [(54, 16, 0.1), (14, 4, 0.1), (14, 12, 0.1), (2, 1, 0.1)],
                                   [(14, 12, 0.1), (14, 4, 0.1)]],
                         ids=lambda s: "-".join(f"{x[0]}_{x[1]}" for x in s))
def test_amplitudes_come_back_as_they_were_set(specs):
    """Downloads of 6 and 68 KB (one kernel into pinned memory of that size), 1.0 and
    7.9 MB (through two and four slots, the last one partly filled), alone and in
    contexts whose other problems need another area: the same bits."""
    c = _ctx([ccd.problem(*x) for x in specs])
    rng = np.random.default_rng(5)
    t = [rng.normal(0.0, 1e-2, c.info(p)["n_amplitudes"]) for p in range(c.n)]
    for _ in range(2):
        for p in range(c.n):
            c.set_amplitudes(t[p], p)
        for p in range(c.n):
            assert np.array_equal(c.get_amplitudes(p), t[p]), p
        t = [x[::-1].copy() for x in t]


def test_a_problem_without_amplitudes():
    """Eight neutrons in the 14 states of n^2 <= 1 under a general twist have no pair
    excitation that keeps the momentum: nothing to copy, no correlation, and no
    difference to the problem beside it."""
    c = _ctx([ccd.problem(14, 4, 0.16), ccd.problem(8, 1, 0.1, twist=(0.1, 0.2, 0.3))])
    one = _ctx([ccd.problem(14, 4, 0.16)])
    assert c.info(1)["n_amplitudes"] == 0
    for ctx in (c, one):
        ctx.iterate(mixing=0.5, tol=1e-8, max_iter=60, check_every=4)
    assert c.get_amplitudes(1).size == 0
    c.set_amplitudes(np.empty(0), 1)
    assert c.energy(1)[1:] == (0.0, 0.0)
    assert np.array_equal(c.get_amplitudes(0), one.get_amplitudes(0))
    assert c.energy(0) == one.energy(0)


def _kernels(run, always="k_update"):
    """names of the kernels that a call launches (always: one that it launches in any case)"""
    from torch.profiler import ProfilerActivity, profile
    import torch
    run()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        run()
        torch.cuda.synchronize()
    names = " ".join(e.key for e in p.key_averages())
    if always not in names:
        pytest.skip("the profiler sees no kernels here")
    return names


def _twists(n, nmax2, mesh):
    return [ccd.problem(n, nmax2, 0.12, twist=t) for t in ccd.twist_mesh(mesh)[0]]


@pytest.mark.parametrize("probs,separate", [(lambda: [ccd.problem(66, 36, 0.16)], False),
                                            (lambda: [ccd.problem(14, 4, 0.1)] * 100, False),
                                            (lambda: [ccd.problem(14, 4, 0.1)] * 500, True),
                                            (lambda: _twists(14, 10, 4), False), (lambda: _twists(14, 10, 5), True)],
                         ids=["one", "100 boxes", "500 boxes", "64 twists", "125 twists"])
def test_large_batches_run_as_separate_launches(probs, separate):
    """The three launches of k_front hold fewer waves of small pairs at a time
    than the pairs' own launches, and lose to them where there are many."""
    c = _ctx(probs())
    names = _kernels(lambda: c.iterate(mixing=0.5, max_iter=2))
    assert ("k_front" in names, "k_ringp_small" in names) == (not separate, separate), names


@pytest.mark.parametrize("probs", [lambda: [ccd.problem(14, 4, r) for r in np.linspace(0.03, 0.2, 500)],
                                   lambda: _twists(14, 10, 5),
                                   lambda: _twists(38, 12, 4) + [ccd.problem(66, 12, 0.03)]],
                         ids=["500 boxes", "125 twists", "64 twists and a box"])
def test_large_batches_equal_their_own_contexts(probs):
    """Batches that start as separate launches and, as their problems stop, go on
    with shorter lists and then as three launches: sweeps, energies and
    amplitudes of problems alone in their contexts, bit for bit."""
    probs = probs()
    batch = _ctx(probs)
    opt = dict(mixing=0.5, tol_rel=2e-8, max_iter=150, stop_rule=1, history=True, check_every=4)
    r = batch.iterate(**opt)
    more = batch.iterate(mixing=0.5, max_iter=3, history=True)["history"]
    assert len(set(r["sweeps"].tolist())) > 1
    for p in sorted({0, 1, len(probs) // 2, len(probs) - 2, len(probs) - 1, int(np.argmax(r["sweeps"])),
                     int(np.argmin(r["sweeps"]))}):
        alone = _ctx([probs[p]])
        a = alone.iterate(**opt)
        assert a["sweeps"][0] == r["sweeps"][p]
        assert np.array_equal(a["history"][0], r["history"][p], equal_nan=True)
        assert np.array_equal(alone.iterate(mixing=0.5, max_iter=3, history=True)["history"][0], more[p])
        assert np.array_equal(alone.get_amplitudes(), batch.get_amplitudes(p))


def test_autotuner_finds_the_default_shapes_from_any_table():
    """A small box's default sweep takes a quarter of the time of separate
    launches, whatever their shapes; a search from a table that is not 0 in
    several slots, each of them changed by itself, ends with it all the same."""
    c = _ctx([ccd.problem(14, 4, 0.1)])
    for table in ([0, 0, 0, 0, 1, 1, 0, 0, 0, 0], [1, 1, 0, 0, 0, 0, 1, 0, 0, 0], [2] * 6 + [1] * 4) * 2:
        c.set_tuning(table)
        found, _ = c.autotune(ccd.CCD_PREC_FP64, reps=1)
        assert not found.any(), (table, found)


@pytest.mark.parametrize("probs", [[(66, 36, 0.16)], [(66, 20, 0.05), (66, 20, 0.16)]], ids=["one", "two"])
def test_timing_of_the_launches_that_a_solve_makes(probs):
    """CCD_TIME_LAUNCHES leaves the three-launch sweep as it is (the energy of a run's
    last sweep is one launch more); True makes every family a launch of its own.
    Both change no bits."""
    probs = [ccd.problem(*x) for x in probs]
    want = _ctx(probs).iterate(mixing=0.5, max_iter=6, history=True, check_every=6)["history"]
    for mode, names in ((ccd.CCD_TIME_LAUNCHES, {"direct": 6, "ladder": 6, "update": 6, "energy": 1}),
                        (True, {"direct": 6, "dsum": 6, "ring_small": 6, "ring32": 6, "ring48": 6, "ring64": 6,
                                "ladder": 6, "update": 6, "energy": 6})):
        c = _ctx(probs)
        c.set_timing(mode)
        got = c.iterate(mixing=0.5, max_iter=6, history=True, check_every=6)["history"]
        kt = {k: v[1] for k, v in c.kernel_times().items() if v[1]}
        assert np.array_equal(got, want)
        assert {k: kt.get(k, 0) for k in names} == names, kt
        assert ("ring64" in kt) == (mode is True)
        assert all(ms > 0 for ms, n in c.kernel_times().values() if n)
