"""GPU parity of the index stage on class matrices given directly (a mask of every such size would not fit), bit-exact
against the oracle: run index, lists and schedules, by rows and by columns, around the sizes at which the path changes."""
import numpy as np
import pytest
import torch

from gpu_util import assert_class_index_equal, device_us, index_of_classes, index_to_numpy

pytestmark = pytest.mark.gpu


def _bbm():
    import paper_2409_15097_amd as bbm
    return bbm


def _classes(Mb, nbr, nbc, density=0.3, seed=0):
    rng = np.random.default_rng(1000 * nbr + nbc + seed)
    return (rng.integers(1, 3, (Mb, nbr, nbc)) * (rng.random((Mb, nbr, nbc)) < density)).astype(np.uint8)


def _check(cls, fused):
    bbm = _bbm()
    idx = index_of_classes(cls)
    if fused:
        bbm.bbm_build_index(idx)
    else:
        bbm.bbm_build_runs(idx)
        bbm.bbm_build_sparse_index(idx)
    bbm.bbm_build_col_index(idx)
    torch.cuda.synchronize()
    got = index_to_numpy(idx)
    assert_class_index_equal(got, cls)
    return got


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("Mb,nbr,nbc", [
    (1, 1, 1), (1, 3, 5), (3, 1, 5), (1, 4, 4), (1, 5, 4),                      # below, at and above 16 class bytes
    (1, 512, 4), (1, 513, 4), (600, 1, 1), (300, 2, 2), (1, 700, 3),            # rows of 1 to 4 blocks, one load for several rows
    (90, 7, 5), (70, 8, 7), (65, 8, 8), (57, 9, 9), (256, 15, 15), (2, 2000, 15), (40, 13, 16)])
def test_rows_of_few_blocks(Mb, nbr, nbc, fused):
    """Fewer than 16 blocks a row: several rows in one 16-byte load, the last loads moved back to end with the matrix."""
    cls = _classes(Mb, nbr, nbc)
    cls[-1, -1, -1] = 2
    cls[0, :, 0] = 1                                                            # a column that the schedule may cut
    _check(cls, fused)


def test_rows_of_15_blocks_cost_what_rows_of_16_do():
    """Counted with a load per byte, 256 planes of 15 x 15 blocks took 1.8 (rows) and 2.7 times (columns) as long as
    16 x 16; with 16-byte loads 1.05."""
    bbm = _bbm()
    t = {}
    for n in (15, 16):
        idx = index_of_classes(_classes(256, n, n))
        t[n] = [device_us(lambda: build(idx)) for build in (bbm.bbm_build_index, bbm.bbm_build_col_index)]
    assert t[15][0] < 1.4 * t[16][0] and t[15][1] < 1.6 * t[16][1], t


def _with_long_lines(Mb, nbr, nbc, density, seed=0):
    """Short lists but for a few full rows and columns in different planes (lines that the schedules cut), an empty column and
    an empty row."""
    rng = np.random.default_rng(nbr + nbc + seed)
    cls = _classes(Mb, nbr, nbc, density, seed)
    cls[:, nbr // 3] = 0
    cls[:, :, nbc // 5] = 0
    for m in range(Mb):
        cls[m, rng.integers(0, nbr, 2)] = 1 + m % 2
        cls[m, :, rng.integers(0, nbc, 2)] = 2 - m % 2
    return cls


@pytest.mark.parametrize("Mb,nbr,nbc,density", [
    (1, 1, 1023, 0.3), (1, 1, 1024, 0.3), (1, 1, 1025, 0.9), (3, 2, 1535, 0.3), (1, 3, 1536, 0.02), (5, 3, 1551, 0.001), (1, 128, 1024, 0.05),
    (2, 16, 4095, 0.1), (1, 1, 131072, 0.01)])
def test_long_rows_listed_in_strips(Mb, nbr, nbc, density):
    """The list without the run index, rows of 1024 blocks and more: strips that are full, partial, empty, and empty up to
    the last one; parts that begin in any strip; the largest class matrix of the one launch."""
    cls = _classes(Mb, nbr, nbc, density)
    cls[0, 0, :nbc - 1] = 0
    cls[0, 0, -1] = 2
    cls[-1, -1, nbc // 3: nbc // 2] = 1
    if nbr > 2:
        cls[-1, 1] = 0                                                          # an empty row
        cls[0, 2] = 2                                                           # a full one, cut into parts
    _check(cls, fused=False)


def test_long_rows_are_not_walked_by_one_wave():
    """A row of 16384 blocks, walked by one wave, took 8.4 times as long as one of 1024; in strips 1.2 times."""
    bbm = _bbm()
    t = []
    for nbc in (1024, 16384):
        idx = index_of_classes(_classes(1, 1, nbc))
        t.append(device_us(lambda: bbm.bbm_build_sparse_index(idx)))
    assert t[1] < 3 * t[0], t


# by rows: list and schedule in the second of two launches, from 128 KiB of classes up to 1024 rows a plane and 4096 in all
@pytest.mark.parametrize("Mb,nbr,nbc,density", [
    (3, 199, 256, 0.02),           # lists of about 8: threshold at its floor, rows in launch-order groups of 4, the last one short
    (3, 199, 256, 0.6),            # long lists: rows ranked singly
    (4, 1024, 40, 0.05),           # the most rows
    (2, 130, 1100, 0.01)])         # lists over many ballot steps
def test_list_and_schedule_in_the_second_launch(Mb, nbr, nbc, density):
    assert Mb * nbr * nbc > 128 << 10 and nbr <= 1024 and Mb * nbr <= 4096      # past the one launch, within the two
    cls = _with_long_lines(Mb, nbr, nbc, density)
    got = _check(cls, fused=True)
    assert (got["sched"][1] == 32) == (density < 0.1 and nbc < 1000)            # the split threshold: at its floor, or above
    assert got["sched"][0] > 0 or density > 0.1                                 # rows were cut into parts
    _check(cls, fused=False)                                                    # the same in the separate kernels


# by columns: count, scan, fill and schedule in launches of their own, from 256 KiB of classes or 4096 columns on
@pytest.mark.parametrize("Mb,nbr,nbc,density", [
    (3, 330, 300, 0.02), (3, 330, 300, 0.5), (2, 70, 2100, 0.05), (3, 200, 1500, 0.03), (2, 2, 4097, 0.3), (1, 40, 8200, 0.02),
    (70, 2, 65, 0.5)])
def test_columns_in_several_launches(Mb, nbr, nbc, density):
    assert Mb * nbc > 4096 or Mb * nbr * nbc > 256 << 10
    cls = _with_long_lines(Mb, nbr, nbc, density)
    got = _check(cls, fused=True)
    if nbr >= 40 and density < 0.1:
        assert got["col_sched"][0] > 0                                          # columns were cut into parts


def test_column_index_past_4096_columns_costs_little_more():
    """With one wave scanning a plane's counts, 8192 columns took 4.2 times as long as the one launch of 4096; now 1.4 times."""
    bbm = _bbm()
    t = []
    for nbc in (4096, 8192):
        idx = index_of_classes(_classes(1, 16, nbc))
        t.append(device_us(lambda: bbm.bbm_build_col_index(idx)))
    assert t[1] < 2.5 * t[0], t
