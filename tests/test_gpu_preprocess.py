"""GPU parity: block classes, BinBlkMat, packed bits, run index and sparse list, bit-exact against the oracle."""
import numpy as np
import pytest
import torch

from workloads import masks, small_variant, make_config
from gpu_util import index_to_numpy, assert_index_equal, device_us

pytestmark = pytest.mark.gpu


def _bbm():
    import paper_2409_15097_amd as bbm
    return bbm


def _run(mask_np, Br, Bc, row_stride=None, fused=True):
    bbm = _bbm()
    Mb, N, _ = mask_np.shape
    if row_stride is None:
        mask = torch.from_numpy(mask_np).cuda()
    else:
        buf = torch.zeros((Mb, N, row_stride), dtype=torch.uint8, device="cuda")
        buf[:, :, :N] = torch.from_numpy(mask_np).cuda()
        mask = buf[:, :, :N]
    idx = bbm.build_index(mask, Br, Bc, fused=fused)      # one-call entry point, or runs and list separately
    torch.cuda.synchronize()
    return idx


CASES = [
    ("C1", 256, 64, 64), ("C1", 256, 128, 64), ("C1", 256, 128, 32), ("C1", 256, 32, 128), ("C1", 256, 256, 256),
    ("C2", 1024, 128, 64), ("C2", 1024, 64, 64), ("C3", 640, 128, 64), ("C3", 640, 64, 16),
    ("C4", 2048, 128, 64), ("C4", 2048, 64, 64), ("C5", 2048, 128, 64), ("C5", 2048, 64, 64),
    ("C0d", 512, 128, 64), ("C0c", 512, 128, 64), ("C0c", 1024, 128, 32),
]


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("name,N,Br,Bc", CASES)
def test_index_bit_exact_small_variants(name, N, Br, Bc, fused):
    cfg = small_variant(name, N=N, B=2, H=1, with_qkv=False)
    idx = _run(cfg["mask"], Br, Bc, fused=fused)
    assert_index_equal(index_to_numpy(idx), cfg["mask"], Br, Bc)


@pytest.mark.parametrize("N,Br,Bc", [(200, 64, 64), (333, 128, 64), (1000, 128, 64), (77, 64, 64), (1, 64, 64),
                                     (1025, 100, 32), (2100, 7, 16), (64, 1, 64)])
def test_index_bit_exact_ragged_sizes(N, Br, Bc):
    rng = np.random.default_rng(N)
    blk = masks.random_blocks(64 * (-(-N // 64)), N, blk=32, p_empty=0.35, p_full=0.4)[0][:N, :N]
    mask = (blk * rng.integers(1, 255, blk.shape, dtype=np.uint8)).astype(np.uint8)[None]
    idx = _run(mask, Br, Bc)                       # rows that start at any byte unless N % 16 == 0
    assert_index_equal(index_to_numpy(idx), mask, Br, Bc)
    stride = 16 * (-(-N // 16)) + 16
    idx = _run(mask, Br, Bc, row_stride=stride, fused=False)    # padded, aligned rows with a ragged tail
    assert_index_equal(index_to_numpy(idx), mask, Br, Bc)


def test_all_zero_and_all_ones_masks():
    for fill in (0, 1):
        mask = np.full((2, 320, 320), fill, dtype=np.uint8)
        idx = _run(mask, 64, 64)
        assert_index_equal(index_to_numpy(idx), mask, 64, 64)


def test_long_rows_of_blocks_cross_ballot_chunks():
    """nbc > 64 so that runs and lists span several 64-block ballot chunks."""
    N, Bc = 2304, 16                                # nbc = 144
    mask = np.zeros((1, N, N), dtype=np.uint8)
    mask[0, :64, 16 * 10:16 * 140] = 1              # one run crossing two chunk boundaries
    mask[0, 64:128, :16 * 64] = 1                   # run ending exactly at a chunk boundary
    mask[0, 64:128, 16 * 64 + 5] = 1                # followed by a partial block
    mask[0, 128:192, 16 * 63:16 * 65] = 1           # two-block run straddling the boundary
    mask[0, 128:192, 16 * 100:16 * 102] = 1         # equal-length run later: leftmost must win
    mask[0, 192:256, 16 * 128:] = 1                 # run reaching the row end
    for fused in (True, False):
        idx = _run(mask, 64, Bc, fused=fused)      # 36 rows x 3 chunks: still one launch when fused
        assert_index_equal(index_to_numpy(idx), mask, 64, Bc)


def test_more_block_rows_than_the_schedule_sorts():
    """Br = 1 gives 4200 block rows (> 4096): the schedule lists them from the last row to the first, unsorted."""
    N = 4200
    rng = np.random.default_rng(5)
    mask = (rng.random((1, N, N)) < 0.002).astype(np.uint8)
    mask[0, 100:110] = 1                            # a few full-width rows: long lists that the schedule cuts
    mask[0, 3000:3003, ::2] = 1
    for fused in (True, False):
        idx = _run(mask, 1, 64, fused=fused)
        got = index_to_numpy(idx)
        assert_index_equal(got, mask, 1, 64)
        assert got["sched"][0] > 0                  # parts exist
        assert np.array_equal(got["sched"][-4 * N:].reshape(N, 4)[:, 0], np.arange(N - 1, -1, -1))


@pytest.mark.parametrize("name", ["C2", "C3", "C4", "C5"])
def test_index_bit_exact_full_size(name):
    cfg = make_config(name, with_qkv=False)
    for Br in (128, 64):
        idx = _run(cfg["mask"], Br, 64, fused=(Br == 128))
        assert_index_equal(index_to_numpy(idx), cfg["mask"], Br, 64)
        del idx


@pytest.mark.parametrize("Mb,N,Br,kind", [(3, 6000, 64, "window"), (2, 9000, 128, "packed"), (1, 14000, 128, "graph"), (5, 3333, 32, "window"),
                                          (2, 8192, 64, "blocks"), (1, 12000, 128, "window")])
def test_mid_size_class_matrices_list_and_schedule_in_one_launch(Mb, N, Br, kind):
    """Class matrices of 17 to 33 KB, built in one launch by either entry point.  Short rows (ranked in groups of four), long rows
    (ranked singly), rows the schedule cuts, several planes.  (Larger ones, whose second launch fills the lists and writes the
    schedule, are in test_gpu_class_index.py.)"""
    rng = np.random.default_rng(N + Br)
    i, j = np.arange(N)[:, None], np.arange(N)[None, :]
    mask = np.zeros((Mb, N, N), dtype=np.uint8)
    for m in range(Mb):
        if kind == "window":
            mask[m] = np.abs(i - j) <= 100 + 150 * m
            mask[m, rng.integers(0, N, 5)] = 1                      # global queries: rows the schedule cuts
            mask[m][:, rng.integers(0, N, 5)] = 1                   # global keys
        elif kind == "packed":
            edges = np.sort(rng.integers(0, N, 40))
            seg = np.searchsorted(edges, np.arange(N))
            mask[m] = (seg[:, None] == seg[None, :]) & (j <= i)
        elif kind == "graph":
            mask[m] = (rng.random((N, N)) < 0.0005) | (np.abs(i - j) < 3)
            mask[m, 4000:4040] = 1
        else:
            cls = rng.choice(3, size=(-(-N // 64), -(-N // 64)), p=[0.7, 0.2, 0.1])
            blk = np.kron(cls, np.ones((64, 64), dtype=np.int64))[:N, :N]
            mask[m] = (blk == 1) | ((blk == 2) & (rng.random((N, N)) < 0.3))
    for fused in (True, False):
        idx = _run(mask, Br, 64, fused=fused)
        got = index_to_numpy(idx)
        assert_index_equal(got, mask, Br, 64)
    assert got["sched"][1] >= 32 and (kind != "window" or got["sched"][0] > 0)       # the window masks have cut rows


@pytest.mark.parametrize("Nq,Nk,offset", [(64, 15, 0), (70, 16, 3), (129, 17, 0), (130, 255, 1), (130, 257, 0), (5, 511, 7), (300, 513, 0),
                                          (128, 272, 16), (2900, 2993, 5)])
def test_block_mask_at_any_address(Nq, Nk, offset):
    """Rows that start at any byte: row lengths around the 16-byte chunk and the two segment lengths, and a mask above the
    size from which such rows are read in the longer segments."""
    rng = np.random.default_rng(Nq + Nk)
    mask = ((rng.random((1, Nq, Nk)) < 0.2) * rng.integers(1, 256, (1, Nq, Nk))).astype(np.uint8)
    mask[:, :, :64] = np.minimum(mask[:, :, :64], 0 if Nk > 64 else 255)     # an all-zero block column
    mask[:, :min(Nq, 128), 64:128] = 255                                     # a full block (where the mask reaches it)
    buf = torch.zeros(Nq * (Nk + offset) + offset, dtype=torch.uint8, device="cuda")
    view = buf[offset:].view(1, Nq, Nk + offset)[:, :, :Nk]
    view.copy_(torch.from_numpy(mask))
    idx = _bbm().bbm_build_block_mask_rect(view, 128, 64)
    torch.cuda.synchronize()
    assert_index_equal(index_to_numpy(idx), mask, 128, 64)


@pytest.mark.parametrize("Br", [1, 7, 8, 9, 16, 17, 32, 33, 64, 65])
@pytest.mark.parametrize("Nq,Nk,Bc", [(67, 1023, 16), (130, 1100, 256), (257, 2049, 64), (2950, 2993, 32)])
def test_block_mask_at_the_edges_of_its_heights(Nq, Nk, Bc, Br):
    """Block heights around those at which segment length and batch change (8, 16, 32, 64), a last block row of few rows,
    the last mask above the size from which 64-row blocks take the longer segments."""
    rng = np.random.default_rng(Nq + Br)
    kind = rng.random((-(-Nq // Br), -(-Nk // Bc)))
    block = np.repeat(np.repeat(kind, Br, axis=0), Bc, axis=1)[:Nq, :Nk]
    mask = ((block < 0.2) | ((block < 0.5) & (rng.random((Nq, Nk)) < 0.02))).astype(np.uint8)[None]
    idx = _bbm().bbm_build_block_mask_rect(torch.from_numpy(mask).cuda(), Br, Bc)
    torch.cuda.synchronize()
    assert_index_equal(index_to_numpy(idx), mask, Br, Bc)


def test_low_blocks_cost_little_more_than_tall_ones():
    """The same 256 MiB are read at every block height.  Batches of 128 rows for all of them made 8-row blocks 6 times and
    32-row blocks 2.1 times as slow as 128-row ones; with batches no longer than the block 1.4 and 0.9 were measured."""
    bbm = _bbm()
    mask = torch.zeros((1, 16384, 16384), dtype=torch.uint8, device="cuda")
    mask[0, :, 5000:6000] = 1
    t = {}
    for Br in (8, 32, 128):
        idx = bbm.bbm_build_block_mask(mask, Br, 64)
        t[Br] = device_us(lambda: bbm.bbm_build_block_mask(mask, Br, 64, idx=idx))
    assert t[8] < 3 * t[128] and t[32] < 1.5 * t[128], t


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("Mb,Nq,Nk,Br,Bc", [
    (1, 10, 10, 64, 64), (2, 40, 239, 8, 16), (3, 520, 250, 64, 16), (1, 200, 8300, 64, 16),     # < 16, 15, 16, 519 block columns
    (2, 4600, 130, 1, 64), (1, 4099, 300, 1, 256), (17, 260, 64, 64, 64),                        # many lines, more planes than waves
    (1, 8300, 8210, 16, 16)])                                                                    # past the one-launch size
def test_index_and_columns_at_their_limits(Mb, Nq, Nk, Br, Bc, fused):
    """Row and column index around the one-launch kernel's limits: few and many blocks per line, line counts around a
    work-group's eight waves and its 4096 lines, class matrices past its size."""
    rng = np.random.default_rng(Nq * 7 + Nk)
    nbr, nbc = -(-Nq // Br), -(-Nk // Bc)
    kind = rng.random((Mb, nbr, nbc))
    kind[:, : max(1, nbr // 40)] *= 0.3                       # a few long lines (cut into parts)
    block = np.repeat(np.repeat(kind, Br, axis=1), Bc, axis=2)[:, :Nq, :Nk]
    mask = (block < 0.2).astype(np.uint8)
    mask[:, ::3, ::5] &= (block[:, ::3, ::5] < 0.1)
    bbm = _bbm()
    idx = bbm.build_index(torch.from_numpy(mask).cuda(), Br, Bc, fused=fused, columns=True)
    torch.cuda.synchronize()
    assert_index_equal(index_to_numpy(idx), mask, Br, Bc)
