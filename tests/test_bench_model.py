"""The byte model of the multi-shift stage that bench.py reports, on cases counted by hand."""
import bench


def _stats(iters):
    return [[{"ms_iters": n} for n in row] for row in iters]


def test_shifted_vectors_move_once_per_ring():
    dims, vec = (2, 2, 2, 4), 3 * 8          # Vh = 16, 24 B per vector and site
    m = bench.multishift_stage_bytes(dims, _stats([[17], [8], [1]]), 8)
    assert m["shift_iters_total"] == 26 and m["base_iters"] == [17]
    # rings of 8 that the systems touch: 3 + 1 + 1; the residuals of 17 iterations
    assert m["ms_shift_update"] == 16 * vec * (17 + 4 * 5)
    assert m["p_update"] == m["ms_r_update"] == 16 * vec * 3 * 17
    assert m["hops"] == 16 * (2 * 17 * 8 * 48 + 17 * 5 * vec)


def test_shorter_ring_and_several_fields():
    dims, vec = (2, 2, 2, 4), 3 * 16
    m = bench.multishift_stage_bytes(dims, _stats([[4, 3], [2, 0]]), 16, slots=2)
    assert m["ms_shift_update"] == 16 * vec * ((4 + 3) + 4 * (2 + 2 + 1 + 0))
    assert m["hop_launch_pairs"] == 4
