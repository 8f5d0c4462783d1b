"""The one-call preprocessing (include/bbm_mask_index.h): argument checks on the CPU; on the GPU the same bits as its parts."""
import ctypes as C

import pytest
import torch

FAKE = C.c_void_p(0x1000)      # never dereferenced: validation fails first


def _call(bbm, mask=FAKE, Mb=1, Nq=64, Nk=64, stride=64, Br=64, Bc=64, cls=FAKE, runs=(FAKE,) * 5, lst=(FAKE, FAKE, None),
          cols=(None, None, None), arrivals=None):
    return bbm.lib.bbm_build_mask_index(mask, Mb, Nq, Nk, stride, Br, Bc, cls, None, None, *runs, *lst, *cols, arrivals, None)


def test_rejects_what_its_parts_reject():
    import paper_2409_15097_amd as bbm
    E, U = bbm.BBM_EINVAL, bbm.BBM_EUNSUPPORTED
    assert _call(bbm, mask=None) == E and _call(bbm, cls=None) == E
    assert _call(bbm, Mb=0) == E and _call(bbm, Nq=0) == E and _call(bbm, Nk=0) == E and _call(bbm, stride=63) == E
    assert _call(bbm, Br=0) == U and _call(bbm, Br=257) == U and _call(bbm, Bc=48) == U and _call(bbm, Bc=0) == U
    for t in range(5):
        assert _call(bbm, runs=tuple(None if i == t else FAKE for i in range(5))) == E
    assert _call(bbm, lst=(None, FAKE, None)) == E and _call(bbm, lst=(FAKE, None, None)) == E
    assert _call(bbm, lst=(FAKE, FAKE, C.c_void_p(0x1004))) == E
    assert _call(bbm, cols=(FAKE, None, None)) == E and _call(bbm, cols=(None, FAKE, None)) == E
    assert _call(bbm, cols=(FAKE, FAKE, C.c_void_p(0x1004))) == E and _call(bbm, cols=(C.c_void_p(0x1001), FAKE, None)) == E
    assert _call(bbm, arrivals=C.c_void_p(0x1002)) == E
    assert "arrivals" in bbm.bbm_last_error()


def _outputs(idx, columns):
    names = ["blk_class", "bin_blk_mat", "offset", "total_ones", "nz_lo", "nz_hi", "nz_cnt", "row_ptr"] + (["col_ptr"] if columns else [])
    out = {n: getattr(idx, n) for n in names}
    for n, ptr, nb in [("sched", idx.row_ptr, idx.nbr)] + ([("col_sched", idx.col_ptr, idx.nbc)] if columns else []):
        t = getattr(idx, n).view(-1)
        out[n + " header"], out[n + " order"] = t[:8], t[-4 * idx.Mb * nb:]
        out[n + " parts"] = t[8:8 + 8 * int(t[0])]
    for n, ptr in [("col_idx", idx.row_ptr)] + ([("row_idx", idx.col_ptr)] if columns else []):
        t = getattr(idx, n).view(idx.Mb, -1)
        for m in range(idx.Mb):
            out[f"{n} {m}"] = t[m, :int(ptr[m, -1])]
    return out


def _assert_same(got, want, columns):
    a, b = _outputs(got, columns), _outputs(want, columns)
    assert a.keys() == b.keys()
    for n in a:
        assert torch.equal(a[n], b[n]), n
    words = lambda i: i.packed_mask.view(i.Mb, -1, i.N)  # noqa: E731
    cls = want.blk_class.repeat_interleave(want.Br, 1)[:, :want.N]  # words of empty blocks are not written
    if want.Bc == 64:
        seen = (cls != 0).permute(0, 2, 1)
        assert torch.equal(words(got)[seen], words(want)[seen])


# rows of blocks x columns of blocks: the last sizes that one launch takes and the first that several do; planes; short and unaligned rows
SIZES = [(1, 5, 9, 128), (1, 64, 16, 64), (1, 129, 15, 128), (1, 1024, 1025, 128), (1, 1025, 1024, 128), (8, 100, 300, 128), (9, 100, 300, 128),
         (2, 1000, 4097, 256), (1, 512, 64 * 512, 64), (1, 512, 64 * 513, 64), (1, 40, 64 * 4096, 64), (1, 40, 64 * 4097, 64), (3, 130, 64, 64),
         (1, 300, 777, 96), (1, 4096, 4096, 128), (4, 700, 700, 64)]


@pytest.mark.gpu
@pytest.mark.parametrize("columns", [False, True])
@pytest.mark.parametrize("Mb,Nq,Nk,Br", SIZES)
def test_same_bits_as_the_parts_call_after_call(Mb, Nq, Nk, Br, columns):
    import paper_2409_15097_amd as bbm
    gen = torch.Generator(device="cuda").manual_seed(Nq + Nk)
    got = None
    for density in (0.002, 0.9999, 0.05, 0.0):   # one index, masks of other structure: nothing is left over from a call
        kind = torch.rand((Mb, -(-Nq // 64), -(-Nk // 64)), generator=gen, device="cuda").repeat_interleave(64, 1).repeat_interleave(64, 2)[:, :Nq, :Nk]
        mask = ((torch.rand((Mb, Nq, Nk), generator=gen, device="cuda") < density) | (kind < 0.2)).to(torch.uint8) if density else torch.zeros((Mb, Nq, Nk), dtype=torch.uint8, device="cuda")
        del kind
        print(f"mask index {Mb}x{Nq}x{Nk} Br={Br} columns={columns} density={density}", flush=True)
        got = bbm.build_index(mask, Br, 64, idx=got, columns=columns)
        want = bbm.build_index(mask, Br, 64, columns=columns, fused=False)
        _assert_same(got, want, columns)
        assert int(got.arrivals) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("first_in_the_graph", [False, True])
def test_recorded_calls_replay_with_eager_ones_in_between(first_in_the_graph):
    import dataclasses
    import paper_2409_15097_amd as bbm
    N = 1000
    i = torch.arange(N, device="cuda")
    masks = [((i[:, None] - i[None, :]).abs() <= w).to(torch.uint8)[None].contiguous() for w in (3, 200, 1000)]
    mask = masks[0].clone()
    idx = bbm.build_index(mask, 128, 64)
    if first_in_the_graph:                       # an index whose counter is not there yet when the call is recorded
        idx = dataclasses.replace(idx)
        assert idx.arrivals is None
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bbm.build_index(mask, 128, 64, idx=idx)
    for m in masks + masks:
        mask.copy_(m)
        graph.replay()
        _assert_same(idx, bbm.build_index(m, 128, 64, fused=False), False)
        mask.copy_(masks[1])
        bbm.build_index(mask, 128, 64, idx=idx)  # an eager call into the same index
        _assert_same(idx, bbm.build_index(masks[1], 128, 64, fused=False), False)


MARK = 1 << 20                                   # no call has that many work-groups: one that counts moves it, one that does not leaves it


def _band(N, w):
    i = torch.arange(N, device="cuda")
    return ((i[:, None] - i[None, :]).abs() <= w).to(torch.uint8)[None].contiguous()


@pytest.mark.gpu
@pytest.mark.parametrize("columns", [False, True])
@pytest.mark.parametrize("Mb,Nq,Nk,Br", SIZES)
def test_which_sizes_one_launch_takes(Mb, Nq, Nk, Br, columns):
    import paper_2409_15097_amd as bbm
    mask = (torch.rand((Mb, Nq, Nk), device="cuda") < 0.01).to(torch.uint8)
    idx = bbm.build_index(mask, Br, 64, columns=columns)
    idx.arrivals.fill_(MARK)
    bbm.build_index(mask, Br, 64, idx=idx, columns=columns)
    rows = Mb * -(-Nq // Br)
    one = not columns and rows <= 8 and rows * -(-Nk // 64) <= 4096 and not (Br == 64 and Mb * Nq * Nk > 8 << 20)
    work_groups = rows * -(-Nk // 256)
    assert int(idx.arrivals) == (work_groups - 1 if one else MARK)   # (an increment past its limit gives zero)


@pytest.mark.gpu
def test_calls_on_another_stream_do_not_share_the_counter():
    import paper_2409_15097_amd as bbm
    first, second = _band(1000, 3), _band(1000, 300)
    idx = bbm.build_index(first, 128, 64)
    idx.arrivals.fill_(MARK)                     # what a call under way on this stream might have left there
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    bbm.build_index(second, 128, 64, idx=idx, stream=other)
    other.synchronize()
    assert int(idx.arrivals) == MARK
    _assert_same(idx, bbm.build_index(second, 128, 64, fused=False), False)
    idx.arrivals.zero_()                         # and the stream that it belongs to goes on with it
    bbm.build_index(first, 128, 64, idx=idx)
    _assert_same(idx, bbm.build_index(first, 128, 64, fused=False), False)
    assert int(idx.arrivals) == 0


@pytest.mark.gpu
def test_recorded_calls_leave_the_counter_alone():
    import paper_2409_15097_amd as bbm
    mask = _band(1000, 3)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    idx = bbm.build_index(mask, 128, 64, stream=side)   # the counter belongs to the stream that is recorded below
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        bbm.build_index(mask, 128, 64, idx=idx)
    idx.arrivals.fill_(MARK)                     # an eager call whose work-groups have not all been counted
    for w in (200, 3, 1000):
        mask.copy_(_band(1000, w))
        graph.replay()
        _assert_same(idx, bbm.build_index(mask, 128, 64, fused=False), False)
    assert int(idx.arrivals) == MARK


@pytest.mark.gpu
def test_a_counter_is_not_made_while_the_stream_of_the_call_is_recorded():
    """The stream of the call is recorded, the current one is not."""
    import dataclasses
    import paper_2409_15097_amd as bbm
    mask = _band(1000, 3)
    idx = dataclasses.replace(bbm.build_index(mask, 128, 64))
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        with torch.cuda.stream(other):
            assert not torch.cuda.is_current_stream_capturing()
            bbm.build_index(mask, 128, 64, idx=idx, stream=side)
    assert idx.arrivals is None
    for w in (200, 3):
        mask.copy_(_band(1000, w))
        graph.replay()
        _assert_same(idx, bbm.build_index(mask, 128, 64, fused=False), False)
