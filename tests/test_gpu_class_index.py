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
