"""Solves that cross the limits of the solvers' plans while they run or lie beyond them: a
mixed solve whose live systems fall below the size from which the runs of iterations end with
a queued true-residual update; multi-shift solves with one shift, whose deferred steps lie
over another vector, with several launches per iteration; batches that start above the size
of one merged launch and shrink below it, and with more classes than one takes.

Parity bar as in test_gpu_solvers.py: the FP64 true relative residual recomputed by the
oracle is <= tol, and the library's own agrees with it to the rounding of two evaluations."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_00426_amd as stg  # noqa: E402
import seeded_inputs as si  # noqa: E402
from oracle import oracle_np as on  # noqa: E402

from gpu_common import say, to_dev  # noqa: E402

TOL = 1e-10
STG_TUNE_FIELDS_PER_LAUNCH, STG_TUNE_CG_FORM = 6, 10


@pytest.fixture(params=[0, 2])
def cg_form(request):
    stg.stg_set_tuning(STG_TUNE_CG_FORM, request.param)
    yield request.param
    stg.stg_set_tuning(STG_TUNE_CG_FORM, 0)


def _check(dims, links, mass, b, x, s, sigma=0.0):
    assert s["status"] == 0
    if not b.any():
        assert not x.any()
        return
    res = on.true_relative_residual(dims, links, on.standard_phases(dims), mass, b, x,
                                    sigma=sigma)
    slack = 64 * 2.0 ** -53 * (1 + (mass ** 2 + sigma + 16)
                               * np.linalg.norm(x) / np.linalg.norm(b))
    assert res <= TOL + slack, (sigma, res)
    assert abs(s["true_rel_resid"] - res) <= slack


@pytest.mark.parametrize("poll", [0, 1, 8])
@pytest.mark.parametrize("lofmt", ["c64_12", "bf16_12"])
def test_mixed_solve_falls_below_the_queued_size(lofmt, poll, cg_form):
    # 72 x 2048 half sites at first; 62 of the systems start from a solution to 1e-4 and
    # leave the other ten, far below 2^17 site-fields, to run on
    dims, mass, nrhs = (8, 8, 8, 8), 0.1, 72
    links = si.su3_links(dims, 1701, 71)
    b = si.gaussian_field(dims, nrhs, 426, 71)
    hi = stg.pack_gauge(dims, to_dev(links), "c128_12")
    lo = stg.pack_gauge(dims, to_dev(links), lofmt)
    x0, _, _ = stg.cg_solve(hi, mass, to_dev(b), tol=1e-4)
    late = np.arange(3, nrhs, 7)
    x0[torch.from_numpy(late).to(x0.device)] = 0
    x, st, stats = stg.cg_solve(hi, mass, to_dev(b), x=x0, lo=lo, tol=TOL, poll_every=poll)
    x = x.cpu().numpy()
    early = [s["iters"] for j, s in enumerate(stats) if j not in late]
    say(f"{lofmt} poll {poll} form {cg_form}: {max(early)} iterations at most, then "
        f"{stats[3]['iters']}")
    assert st == 0 and max(early) < min(stats[j]["iters"] for j in late)
    for j in range(nrhs):
        _check(dims, links, mass, b[j], x[j], stats[j])


@pytest.mark.parametrize("cap", [0, 1, 2])
@pytest.mark.parametrize("nrhs", [9, 13])
@pytest.mark.parametrize("lofmt", [None, "c64_12"])
def test_one_shift_in_several_launches(lofmt, nrhs, cap):
    dims, mass, shifts = (4, 2, 6, 4), 0.1, [0.02]
    links = si.su3_links(dims, 1701, 72, nrhs)
    b = si.gaussian_field(dims, nrhs, 426, 72, nrhs)
    # systems that end at different times, one from the start, in the second launch
    b[1:4] += 40 * np.roll(b[0], 1, axis=-1)
    b[8] = 0.0
    hi = stg.pack_gauge(dims, to_dev(links), "c128_12")
    lo = stg.pack_gauge(dims, to_dev(links), lofmt) if lofmt else None
    stg.stg_set_tuning(STG_TUNE_FIELDS_PER_LAUNCH, cap)
    try:
        x, st, stats = stg.multishift_cg_solve(hi, mass, shifts, to_dev(b), lo=lo, tol=TOL)
    finally:
        stg.stg_set_tuning(STG_TUNE_FIELDS_PER_LAUNCH, 0)
    x = x.cpu().numpy()
    assert st == 0
    for j in range(nrhs):
        _check(dims, links, mass, b[j], x[0, j], stats[0][j], sigma=shifts[0])
        if lofmt is None:  # the stage meets the tolerance by itself: no wrong step
            s = stats[0][j]
            assert s["iters"] - s["ms_iters"] <= max(4, 0.1 * s["ms_iters"])


@pytest.mark.parametrize("lofmt", [None, "c64_12"])
def test_four_shifts_with_a_zero_system_in_the_second_launch(lofmt):
    dims, mass, nrhs = (4, 2, 6, 4), 0.1, 11
    shifts = [1.0, 1e-3, 0.1, 5.0]
    links = si.su3_links(dims, 1701, 73)
    b = si.gaussian_field(dims, nrhs, 426, 73)
    b[9] = 0.0
    hi = stg.pack_gauge(dims, to_dev(links), "c128_12")
    lo = stg.pack_gauge(dims, to_dev(links), lofmt) if lofmt else None
    x, st, stats = stg.multishift_cg_solve(hi, mass, shifts, to_dev(b), lo=lo, tol=TOL)
    x = x.cpu().numpy()
    assert st == 0
    for k, sigma in enumerate(shifts):
        for j in range(nrhs):
            _check(dims, links, mass, b[j], x[k, j], stats[k][j], sigma=sigma)


def _solve(dims, nrhs, mass, lofmt, seed, hi_phases=None):
    links = si.su3_links(dims, 1701, 74, seed)
    b = si.gaussian_field(dims, nrhs, 426, 74, seed)
    sv = {"hi": stg.pack_gauge(dims, to_dev(links), "c128_12", hi_phases), "mass": mass,
          "b": to_dev(b)}
    if lofmt:
        sv["lo"] = stg.pack_gauge(dims, to_dev(links), lofmt)
    return sv, (dims, links, mass, b)


@pytest.mark.parametrize("poll", [0, 1, 8])
@pytest.mark.parametrize("lofmt", [None, "c64_12"])
def test_batch_shrinks_below_the_merged_size(lofmt, poll, cg_form):
    # 9 chunks x 128 tiles of the large solve, whose heavy mass ends it first, and 17 others
    plan = [((16, 16, 16, 16), 34, 2.0), ((8, 6, 4, 6), 3, 0.1), ((4, 4, 4, 4), 5, 0.05),
            ((4, 8, 8, 6), 2, 0.1)]
    made = [_solve(*p, lofmt, i) for i, p in enumerate(plan)]
    xs, st, stats = stg.cg_solve_batch([sv for sv, _ in made], tol=TOL, poll_every=poll)
    heavy = max(s["iters"] for s in stats[0])
    light = min(s["iters"] for row in stats[1:] for s in row)
    say(f"batch {lofmt} poll {poll} form {cg_form}: {heavy} iterations, then {light}")
    assert st == 0 and heavy < light
    for i, (_, (dims, links, mass, b)) in enumerate(made):
        x = xs[i].cpu().numpy()
        for j in range(b.shape[0]):
            if i == 0 and j not in (0, 3, 17, 32, 33):
                assert stats[i][j]["status"] == 0 and stats[i][j]["true_rel_resid"] <= TOL
                continue
            _check(dims, links, mass, b[j], x[j], stats[i][j])


@pytest.mark.parametrize("poll", [0, 1])
def test_batch_with_more_classes_than_one_launch_takes(poll, cg_form):
    # 1 to 4 fields with standard phases, and 1 and 2 fields whose FP64 gauge field stores
    # them: six classes that the inner hop could merge, four that the FP64 one could
    plan = [((4, 4, 4, 4), 1, 0.1, False), ((4, 2, 6, 4), 2, 0.1, False),
            ((6, 4, 4, 2), 3, 0.2, False), ((4, 4, 2, 8), 4, 0.05, False),
            ((4, 6, 4, 4), 1, 0.1, True), ((2, 4, 4, 6), 2, 0.3, True)]
    made = []
    for i, (dims, nrhs, mass, stored) in enumerate(plan):
        ph = to_dev(np.ascontiguousarray(on.standard_phases(dims))) if stored else None
        made.append(_solve(dims, nrhs, mass, "c64_12", 10 + i, ph))
    xs, st, stats = stg.cg_solve_batch([sv for sv, _ in made], tol=TOL, poll_every=poll)
    assert st == 0
    for i, (_, (dims, links, mass, b)) in enumerate(made):
        x = xs[i].cpu().numpy()
        for j in range(b.shape[0]):
            _check(dims, links, mass, b[j], x[j], stats[i][j])
