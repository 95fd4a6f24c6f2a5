"""Launches of 4 fields keep the direction split where it is the faster one (FP64-12 links up
to Vh = 16384, FP32-12 and BF16-12 ones below 8192), and take the field split just above.

The two add a site's eight products in different orders, so on random fields their results
differ in the last bits somewhere, and the automatic launch has to be bitwise the one that is
asked for.  8 fields take the field split everywhere: there the fields per wave and the site
order leave every bit as it is, which holds between all of them."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_00426_amd as stg  # noqa: E402
import seeded_inputs as si  # noqa: E402

from gpu_common import to_dev  # noqa: E402

STG_TUNE_LAYER_GROUP, STG_TUNE_FIELD_SPLIT = 7, 9


def _gauge_and_field(dims, fmt, nr):
    vh = si.half_volume(dims)
    g = stg.pack_gauge(dims, to_dev(si.su3_links(dims, 1701, 63, vh)), fmt)
    dt = torch.complex128 if fmt == "c128_12" else torch.complex64
    return g, to_dev(si.gaussian_field(dims, nr, 426, 63, vh)).to(dt)


def _with(g, v, split, group=0):
    stg.stg_set_tuning(STG_TUNE_FIELD_SPLIT, split)
    stg.stg_set_tuning(STG_TUNE_LAYER_GROUP, group)
    try:
        return stg.stg_apply_normal(g, 0.1, v)
    finally:
        stg.stg_set_tuning(STG_TUNE_FIELD_SPLIT, 0)
        stg.stg_set_tuning(STG_TUNE_LAYER_GROUP, 0)


@pytest.mark.parametrize("fmt,dims,split", [
    ("c128_12", (8, 8, 8, 8), -1), ("c128_12", (12, 12, 12, 12), -1),
    ("c128_12", (16, 16, 16, 8), -1), ("c128_12", (14, 12, 14, 14), 1),
    ("c64_12", (8, 8, 16, 14), -1), ("c64_12", (8, 8, 16, 16), 1),
    ("bf16_12", (8, 8, 16, 14), -1), ("bf16_12", (8, 8, 16, 16), 1)])
def test_four_fields(fmt, dims, split):
    g, v = _gauge_and_field(dims, fmt, 4)
    auto = _with(g, v, 0)
    assert torch.equal(auto, _with(g, v, split))
    assert not torch.equal(auto, _with(g, v, -split))


@pytest.mark.parametrize("dims", [(12, 12, 14, 14), (14, 16, 16, 8), (16, 16, 8, 14),
                                  (16, 16, 8, 16), (14, 12, 14, 14)])
def test_eight_fields(dims):
    g, v = _gauge_and_field(dims, "c128_12", 8)
    auto = _with(g, v, 0)
    for split, group in ((1, 0), (1, 4), (2, 0)):
        assert torch.equal(auto, _with(g, v, split, group)), (split, group)
