"""The binding reads a lattice's extents at every call, in whatever form they come (anything
that int() takes), although it keeps the structure that it passes to the library.  No GPU is
used: stg_links_bytes is host arithmetic."""
import numpy as np
import pytest
import torch

import paper_1701_00426_amd as stg


def _bytes(dims):
    return stg.stg_links_bytes(dims, stg._lib.STG_LINK_C128_12)


@pytest.mark.parametrize("form", [list, tuple, np.array, torch.tensor,
                                  lambda d: [np.array(n) for n in d],
                                  lambda d: tuple(torch.tensor(n) for n in d),
                                  lambda d: [float(n) for n in d],
                                  lambda d: [str(n) for n in d]],
                         ids=["list", "tuple", "array", "tensor", "0-d arrays", "0-d tensors",
                              "floats", "texts"])
def test_forms_of_extents(form):
    for dims in ([4, 6, 2, 8], [8, 8, 8, 8]):
        assert _bytes(form(dims)) == 8 * 6 * 16 * np.prod(dims) // 2
        assert stg.half_volume(form(dims)) == np.prod(dims) // 2


def test_changed_extents_are_read_again():
    dims = tuple(torch.tensor(4) for _ in range(4))
    small = _bytes(dims)
    dims[3].fill_(8)
    assert _bytes(dims) == 2 * small


def test_many_lattices():
    for n in range(2, 802, 2):  # more than are kept
        assert _bytes((2, 2, 4, n)) == 8 * 6 * 16 * 8 * n
    assert _bytes((2, 2, 4, 2)) == 8 * 6 * 16 * 16
