"""Host check of the byte model of cycles whose small 3D levels run in bricks."""
import bench


def test_vcycle_bytes_of_levels_in_bricks():
    """128^3: the finest level per color, 64^3 in bricks of one step a launch, 32^3
    and 16^3 of two, the tail from 8^3 down."""
    lk = [("per-cell", 256, 4096), ("per-cell", 1, 2048), ("per-cell", 2, 256), ("per-cell", 2, 32)] + \
        [("tail", 0, 0)] * 3
    m = [128 ** 3 // 8 ** l for l in range(7)]
    # no launch forms the right-hand side of level 1: its first brick launch does
    want = (44 * 8 + 8 * (6 + 9 / 8) + 8 * (6 + 6 / 8)) * m[0]
    for l, launches in ((1, 2), (2, 1), (3, 1)):
        # each launch reads 8 values and writes 3; the first pre launch writes f,
        # the last the restricted u, ub and fr, the first post launch prolongs
        want += 8 * (2 * launches * 11 + 3 + 9 / 8 + 6 / 8) * m[l]
    want += 8 * (9 * m[4] + 2 * sum(m[4:]))
    assert abs(bench.vcycle_bytes(3, (128,) * 3, lk) - want) < 1e-6 * want
