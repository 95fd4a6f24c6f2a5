"""The automatic launch of several fields is as accurate as the direction split of 4 fields
and, with 8, as one field per wave.

4 fields: the direction split sums a site's directions by themselves and adds the four sums.
The field split of FP64-12 links, which larger lattices take, does the same in the same
order, so with standard phases (factors of 1 and -1) the results are bitwise equal on either
side of its line; FP32-12 and BF16-12 links keep the direction split.  One chain over all
eight products, as the field split runs for 8 fields, would be off from 64 bits by up to
1.8 times as much, and differs in some bits on any random field.  8 fields: the fields per
wave and the order of sites leave every bit as it is."""
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


@pytest.mark.parametrize("fmt", ["c128_12", "c64_12", "bf16_12"])
@pytest.mark.parametrize("dims", [(4, 2, 6, 4), (8, 8, 8, 8), (12, 12, 12, 12), (16, 16, 16, 8),
                                  (14, 12, 14, 14), (16, 16, 16, 32)])
@pytest.mark.parametrize("nr", [4, 6])
def test_four_fields(nr, dims, fmt):
    g, v = _gauge_and_field(dims, fmt, nr)
    auto = _with(g, v, 0)
    assert torch.equal(auto, _with(g, v, -1))
    if fmt == "c128_12":
        assert torch.equal(auto[:4], _with(g, v[:4].contiguous(), 1))
        assert torch.equal(auto[:4], _with(g, v[:4].contiguous(), 2))


@pytest.mark.parametrize("dims", [(12, 12, 14, 14), (14, 16, 16, 8), (16, 16, 8, 14),
                                  (16, 16, 8, 16), (14, 12, 14, 14)])
def test_eight_fields(dims):
    g, v = _gauge_and_field(dims, "c128_12", 8)
    auto = _with(g, v, 0)
    for split, group in ((1, 0), (1, 4), (2, 0)):
        assert torch.equal(auto, _with(g, v, split, group)), (split, group)
