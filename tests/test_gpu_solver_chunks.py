"""Solves of several systems whose fields share launches across shifts: the refinement of
the multi-shift solve takes its live systems in chunks of up to 8, whatever shift they
belong to, while their right-hand side is the one of their group; and the shifted vectors
of its first stage, which are updated once for 1, 2, 4 or 8 iterations.

Parity bar as in test_gpu_solvers.py: the FP64 true relative residual recomputed by the
oracle is <= tol for every system, also when the shifts are not in order (finished and
live systems then alternate) and when a zero right-hand side is finished from the start."""
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


@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("poll", [0, 1, 3])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 5])
@pytest.mark.parametrize("lofmt", [None, "c64_12", "bf16_12"])
def test_refinement_across_shifts(lofmt, nrhs, poll, zero):
    dims, mass = (4, 6, 2, 8), 0.1
    shifts = [3.0, 1e-3, 0.5, 2e-2, 10.0, 1e-4, 0.1]
    links = si.su3_links(dims, 1701, 31, nrhs)
    phases = on.standard_phases(dims)
    b = si.gaussian_field(dims, nrhs, 426, 31, nrhs)
    if zero:
        b[nrhs - 1] = 0.0
    hi = stg.pack_gauge(dims, to_dev(links), "c128_12")
    lo = stg.pack_gauge(dims, to_dev(links), lofmt) if lofmt else None
    say(f"refinement {lofmt} nrhs {nrhs} poll {poll} zero {zero}")
    x, st, stats = stg.multishift_cg_solve(hi, mass, shifts, to_dev(b), lo=lo, tol=TOL,
                                           poll_every=poll)
    x = x.cpu().numpy()
    assert st == 0
    for k, sigma in enumerate(shifts):
        for j in range(nrhs):
            assert stats[k][j]["status"] == 0
            if not b[j].any():
                assert not x[k, j].any()
                continue
            res = on.true_relative_residual(dims, links, phases, mass, b[j], x[k, j], sigma=sigma)
            # the library's own residual, to the rounding of two FP64 evaluations
            slack = 64 * 2.0 ** -53 * (1 + (mass ** 2 + sigma + 16)
                                       * np.linalg.norm(x[k, j]) / np.linalg.norm(b[j]))
            assert res <= TOL + slack, (sigma, j, res)
            assert abs(stats[k][j]["true_rel_resid"] - res) <= slack


@pytest.mark.parametrize("poll", [1, 5])
@pytest.mark.parametrize("nshift", [1, 2, 3, 4, 9])
@pytest.mark.parametrize("lofmt", [None, "c64_12"])
def test_deferred_shift_updates(lofmt, nshift, poll):
    # 1 to 9 shifts: every length of the ring of residuals (1, 2, 4 and 8 in FP64); the
    # first stage ends anywhere in the ring.  The multi-shift stage in FP64 meets the
    # tolerance by itself: a refinement that had to iterate would show a wrong update.
    dims, mass, nrhs = (6, 4, 2, 8), 0.1, 2
    shifts = list(si.log_shifts(nshift, 1e-3, 5.0))
    links = si.su3_links(dims, 1701, 33)
    phases = on.standard_phases(dims)
    b = si.gaussian_field(dims, nrhs, 426, 33)
    hi = stg.pack_gauge(dims, to_dev(links), "c128_12")
    lo = stg.pack_gauge(dims, to_dev(links), lofmt) if lofmt else None
    x, st, stats = stg.multishift_cg_solve(hi, mass, shifts, to_dev(b), lo=lo, tol=TOL,
                                           poll_every=poll)
    x = x.cpu().numpy()
    assert st == 0
    for k, sigma in enumerate(shifts):
        for j in range(nrhs):
            s = stats[k][j]
            res = on.true_relative_residual(dims, links, phases, mass, b[j], x[k, j], sigma=sigma)
            assert res <= 1.01 * TOL, (sigma, j, res)
            say(f"  {lofmt} nshift {nshift} sigma {sigma:.2e}: stage {s['ms_iters']} "
                f"iters {s['iters']} resid {res:.2e}")
            if lofmt is None:
                # the recurrence's residual may leave a few steps to the refinement
                assert s["iters"] - s["ms_iters"] <= max(4, 0.1 * s["ms_iters"])
