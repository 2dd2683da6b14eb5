"""Launches of whole calls at the ends of the documented ranges, without a GPU.

A dispatch takes fewer than 2^32 threads along x, so a launch that would have more
is cut into several.
"""

import pytest

from tests import launches

LIMIT = 1 << 32


@pytest.fixture(scope="module")
def tmp(tmp_path_factory):
    return tmp_path_factory.mktemp("stub")


# (dtype, n, k, items): images whose band transform has more items of 1024
# threads than one dispatch takes: 240 (228) columns of a band of 32 (64) rows an
# item, of the 128-row bands a group of 64 shifts.
@pytest.mark.parametrize("dtype,n,k,items", [(0, 32, 1024, 4370 * 1024),
                                             (0, 64, 1000, 4600 * 1000),
                                             (0, 128, 500, 4600 * 500 * 2),
                                             (1, 64, 511, 4600 * 511 * 2),
                                             (1, 128, 255, 4600 * 255 * 4)])
def test_transform_of_the_widest_images_fits_its_dispatches(tmp, dtype, n, k, items):
    got = launches.record(f"""
fhtp._check(fhtp.lib().fhtp_fht_bands(PTR, {dtype}, {n * k}, {1 << 20}, {k}, PTR, PTR, 1 << 60, None),
            "fht_bands")
results = take()
""", tmp)
    assert {launches.name(m) for m, _, _ in got} == {"fht_split_kernel"}
    assert sum(grid for _, grid, _ in got) == items
    assert items * 1024 >= LIMIT
    for _, grid, block in got:
        assert block == 1024 and grid * block < LIMIT
    # a dispatch that is not the last ends where the workgroups' order repeats
    assert all(grid % 1024 == 0 for _, grid, _ in got[:-1])


# The 128-row blocks of 512- and 1024-row bands: the split transform has no grid to
# choose, so rules that differ in fht_grid leave them in one launch.
@pytest.mark.parametrize("dtype", [0, 1])
def test_grid_rules_do_not_part_launches_without_a_grid_choice(tmp, dtype):
    got = launches.record(f"""
from paper_1912_01884_amd import autotune
shapes = [(1024, 300, 2, {dtype}), (2048, 300, 2, {dtype})]
bends = [fhtp.make_bend(3)] * 2
for grid in (0, 1):
    fhtp.tune_set([autotune.rule(log2n=9, fht_grid=grid)])
    results.append(batch(shapes, bends))
""", tmp)
    for run in got:
        assert [launches.name(m) for m, _, _ in run].count("fht_split_kernel") == 1


# Packs of the widest images, of few rows: 64 workgroups of 1024 threads for each 1024
# columns of a pack's scanned windows, 32 of its column recurrence.
@pytest.mark.parametrize("count,h,bend", [(64, 2, "fhtp.make_bend(1 << 20)"),
                                          (65, 4, "fhtp.make_bend(None, 0.3)"),
                                          (256, 4, "fhtp.make_bend(None, 0.3)"),
                                          (130, 4, "fhtp.make_bend(1 << 20)"),
                                          (256, 4, "fhtp.make_bend(1 << 20)")])
def test_steps_of_packs_of_the_widest_images_fit_their_dispatches(tmp, count, h, bend):
    got = launches.record(f"""
results = batch([({h}, {1 << 20}, 2, 0)] * {count}, [{bend}] * {count})
""", tmp)
    for m, grid, block in got:
        assert 0 < grid * block < LIMIT, launches.name(m)
    steps = [(grid, block) for m, grid, block in got
             if launches.name(m) not in ("fht_reg_kernel", "walk", "walk_colmax", "angle_windows")]
    assert sum(grid * block for grid, block in steps) >= count * (1 << 20) * 4


# Scanned windows of every band height: a batch's images of one width of back-pointers
# and of tables share the launches of their steps.
@pytest.mark.parametrize("bend", ["fhtp.make_bend(None, 0.3)", "fhtp.make_bend(25)"])
def test_heights_of_a_batch_share_their_step_launches(tmp, bend):
    low = [(16 * 5, 200), (32 * 9, 500), (64 * 4, 333), (128 * 3, 90)]
    tall = [(256 * 4, 70), (512 * 2, 140), (1024 * 6, 33)]
    shapes = [(h, w, k, 1) for (h, w), k in zip(low + tall, (5, 9, 4, 3, 4, 2, 6))]
    got = launches.record(f"results = batch({shapes}, [{bend}] * {len(shapes)})", tmp)
    steps = [launches.name(m) for m, _, _ in got if launches.name(m).startswith("dp_step")]
    # the longest chain of each width of back-pointers
    assert len(steps) == (9 - 1) + (6 - 1)


# Which kernel takes an image's scanned windows, on both sides of each line.
@pytest.mark.parametrize("n,w,bend,pin,scan", [
    (1, 3000, "fhtp.make_bend(5)", True, True),
    (2, 12287, "fhtp.make_bend(None, 0.3)", True, False),
    (2, 12288, "fhtp.make_bend(None, 0.3)", True, True),
    (16, 16383, "fhtp.make_bend(None, 0.3)", False, False),
    (16, 16384, "fhtp.make_bend(None, 0.3)", False, True),
    (16, 16384, "fhtp.make_bend(17)", False, False),
    (8, 16384, "fhtp.make_bend(None, 0.3)", True, False),
    (8, 16385, "fhtp.make_bend(None, 0.3)", True, True),
    (16, 24575, "fhtp.make_bend(None, 0.02)", False, False),
    (16, 24576, "fhtp.make_bend(None, 0.02)", True, True),
    (32, 40959, "fhtp.make_bend(None, 0.02)", False, False),
    (32, 40960, "fhtp.make_bend(None, 0.02)", False, True),
    (32, 16385, "fhtp.make_bend(None, 0.1)", False, True),
    (32, 24575, "fhtp.make_bend(None, 0.3)", False, False),
    (32, 24576, "fhtp.make_bend(None, 0.3)", False, True),
    (32, 49151, "fhtp.make_bend(17)", False, False),
    (32, 49152, "fhtp.make_bend(17)", False, True),
    (8, 8191, "fhtp.make_bend(1 << 20)", True, False),
    (8, 8192, "fhtp.make_bend(1 << 20)", True, True),
    (32, 8192, "fhtp.make_bend(1 << 20)", True, False),
    (32, 8193, "fhtp.make_bend(1 << 20)", True, True),
    (64, 60000, "fhtp.make_bend(None, 0.02)", False, False),
    (64, 60000, "fhtp.make_bend(1 << 20)", True, False),
    (256, 4095, "fhtp.make_bend(None, 0.005)", False, False),
    (256, 4096, "fhtp.make_bend(None, 0.005)", False, True),
    (256, 16384, "fhtp.make_bend(17)", False, False),
    (512, 8192, "fhtp.make_bend(17)", True, True),
    (512, 8192, "fhtp.make_bend(40)", False, False),
    (1024, 300, "fhtp.make_bend(17)", False, True),
    (1024, 300, "fhtp.make_bend(18)", False, False),
    (1024, 16384, "fhtp.make_bend(40)", False, True),
    (1024, 16384, "fhtp.make_bend(60)", False, False),
    (1024, 16384, "fhtp.make_bend(1 << 20)", True, False),
])
def test_kernel_of_scanned_windows(tmp, n, w, bend, pin, scan):
    opt = "fhtp.make_options(pin=(1, 5))" if pin else "None"
    got = launches.record(f"results = detect({3 * n}, {w}, 3, 1, {bend}, {opt})", tmp)
    names = [launches.name(m) for m, _, _ in got]
    steps = [m for m in names if m.startswith("dp_step")]
    assert steps == ["dp_step_generic" if scan else "dp_step_blocks"] * 2
    # the block kernel's first step makes the windows of up to 511 displacements
    angle = "None, " in bend
    assert names.count("angle_windows") == (1 if angle and (scan or n > 256) else 0)


# The column recurrence: the fewest columns a workgroup that fill the chip at most once,
# 64 where even they do more, by the columns of the whole launch in a batch.
@pytest.mark.parametrize("w,count,cols", [(2048, 1, 8), (2049, 1, 16), (4097, 1, 32), (8192, 1, 32),
                                          (8193, 1, 64), (100000, 1, 64), (1000, 8, 32),
                                          (1000, 9, 64)])
def test_columns_of_the_recurrence(tmp, w, count, cols):
    call = (f"detect(256, {w}, 2, 1, fhtp.make_bend(1 << 20))" if count == 1 else
            f"batch([(256, {w}, 2, 1)] * {count}, [fhtp.make_bend(1 << 20)] * {count})")
    got = launches.record(f"results = {call}", tmp)
    grids = [grid for m, grid, _ in got if launches.name(m) == "dp_colmax"]
    assert grids == [count * -(-w // cols)] * 2


# Images of different widths, whose stripes of the pair kernel's order differ: the
# stripe is each image's own, and they share their launches.
@pytest.mark.parametrize("steps,kernel,count", [(2, "dp_pair_fixed", 3), (3, "dp_triple_fixed", 2)])
def test_widths_of_a_batch_share_their_launches(tmp, steps, kernel, count):
    shapes = [(512, w, 8, 1) for w in (700, 8200, 9500, 11000, 12500, 16000)]
    got = launches.record(f"""
from paper_1912_01884_amd import autotune
fhtp.tune_set([autotune.rule(window=0, steps={steps}, stripe=4, w_max=1000),
               autotune.rule(window=0, steps={steps})])
results = batch({shapes}, [fhtp.make_bend(4)] * {len(shapes)})
""", tmp)
    assert [launches.name(m) for m, _, _ in got].count(kernel) == count


# 8-bit bands: both directions in a workgroup above 384 workgroups of them.
@pytest.mark.parametrize("n,groups", [(32, 1), (64, 1), (128, 2)])
def test_directions_of_the_transform(tmp, n, groups):
    got = launches.record(f"""
for k in (384 // {groups}, 384 // {groups} + 1):
    fhtp._check(fhtp.lib().fhtp_fht_bands(PTR, 0, {n} * k, 60, k, PTR, PTR, 0, None), "fht_bands")
    results += take()
""", tmp)
    assert [m.split("fht_split_kernelI")[1].split("E")[1] for m, _, _ in got] == ["Lb0", "Lb1"]
    assert [grid for _, grid, _ in got] == [384 * 2, 384 + groups]
