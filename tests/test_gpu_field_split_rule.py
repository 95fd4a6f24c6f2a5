"""The automatic launch shape of hops with 4 and 8 fields on either side of the sizes where
it changes (Vh = 8192 and 65536: field split or direction split, fields per wave, layer
order, here with 34 x3 planes), against the one-thread-per-site launch.

Tolerance: the two differ in the order of additions only.  An output entry is a sum of 48
real products of entries of unitary links and O(1) fields and 24 more rounded operations per
third-row entry, so |difference| <= 128 u times the largest entry, u the unit roundoff."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_00426_amd as stg  # noqa: E402
import seeded_inputs as si  # noqa: E402

from gpu_common import say, to_dev  # noqa: E402

STG_TUNE_THREADS_PER_SITE = 3


@pytest.mark.parametrize("dims", [(8, 8, 16, 14), (8, 8, 16, 16), (16, 16, 16, 32),
                                  (16, 16, 16, 34)])
@pytest.mark.parametrize("fmt", ["c128_12", "c64_12", "bf16_12"])
def test_automatic_shape(dims, fmt):
    vh = si.half_volume(dims)
    links = to_dev(si.su3_links(dims, 1701, 61, vh))
    g = stg.pack_gauge(dims, links, fmt)
    dt = torch.complex128 if fmt == "c128_12" else torch.complex64
    u = 2.0 ** -53 if fmt == "c128_12" else 2.0 ** -24
    for nr in (4, 8, 12):
        v = to_dev(si.gaussian_field(dims, nr, 426, 61, vh)).to(dt)
        for name in ("oe", "normal"):
            def run():
                if name == "oe":
                    return stg.dirac_apply_oe(g, v)
                return stg.stg_apply_normal(g, 0.1, v)
            got = run()
            stg.stg_set_tuning(STG_TUNE_THREADS_PER_SITE, 1)
            try:
                want = run()
            finally:
                stg.stg_set_tuning(STG_TUNE_THREADS_PER_SITE, 0)
            hops = 2 if name == "normal" else 1
            err = float((got - want).abs().max() / want.abs().max())
            say(f"{fmt} {dims} {nr} fields {name}: {err:.2e}")
            assert err <= 128 * hops * u
