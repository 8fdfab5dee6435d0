"""The C-ABI library loads, exports every symbol include/ilre.h declares, and its host-side argument
checks answer without a GPU.  No compute calls here."""
import ctypes
import os
import re

import pytest

import paper_2508_17892_amd as il
from paper_2508_17892_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    with open(os.path.join(ROOT, "include", "ilre.h")) as f:
        text = f.read()
    return sorted(set(re.findall(r"\b(ilre_[a-z_]+)\s*\(", text)))


def test_header_symbols_are_exported():
    lib = il.load()
    declared = _declared_functions()
    assert set(declared) == set(il.EXPORTS)
    for name in declared:
        assert getattr(lib, name) is not None


def test_opts_struct_matches_header_layout():
    # int32 x4, float, int32, int64 x4, pointer, size_t, pointer, int32 x2 on LP64
    assert ctypes.sizeof(binding.IlreOpts) == 4 * 4 + 4 + 4 + 8 * 4 + 8 + 8 + 8 + 4 + 4
    assert binding.IlreOpts.sink.offset == 80
    assert binding.IlreOpts.k_stride_head.offset == 24
    assert binding.IlreOpts.workspace.offset == 56


def test_workspace_bytes_grows_with_shape():
    a = il.ilre_workspace_bytes(4096, 32, 32, 8, 128, 3, il.ILRE_F32)
    b = il.ilre_workspace_bytes(1 << 20, 256, 32, 8, 128, 5, il.ILRE_BF16)
    assert 0 < a < b < (1 << 30)


@pytest.mark.parametrize("args,status", [
    ((0, 32, 32, 8, 128, 3, 0), il.ILRE_EINVAL),
    ((4096, 0, 32, 8, 128, 3, 0), il.ILRE_EINVAL),
    ((4096, 32, 30, 8, 128, 3, 0), il.ILRE_EINVAL),
    ((4096, 32, 32, 8, 64, 3, 0), il.ILRE_EUNSUPPORTED),
    ((4096, 32, 32, 8, 128, 3, 7), il.ILRE_EUNSUPPORTED),
    ((4096, 32, 32, 8, 128, 65, 0), il.ILRE_EINVAL),
])
def test_workspace_bytes_rejects_bad_shapes(args, status):
    with pytest.raises(il.IlreError) as e:
        il.ilre_workspace_bytes(*args)
    assert e.value.status == status
    assert il.ilre_last_error()


def _opts(**kw):
    o = binding.IlreOpts()
    o.struct_size = ctypes.sizeof(binding.IlreOpts)
    o.dtype = il.ILRE_BF16
    o.n_pool_kernels = 2
    for k, v in kw.items():
        setattr(o, k, v)
    return o


def test_argument_errors_need_no_device():
    lib = il.load()
    kern = (ctypes.c_int32 * 2)(3, 7)
    fake = ctypes.c_void_p(4096)          # never dereferenced: every call below fails validation first
    o = _opts()
    # null pointers
    assert lib.ilre_recall(None, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, ctypes.byref(o)) in (il.ILRE_EINVAL, il.ILRE_ENOMEM)
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, None, fake, ctypes.byref(o)) == il.ILRE_EINVAL
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, None) == il.ILRE_EINVAL
    # missing workspace
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, ctypes.byref(o)) == il.ILRE_ENOMEM
    assert "workspace" in il.ilre_last_error()
    # even kernel size, zero budget, budget over the limit, wrong struct size, bad score mode
    even = (ctypes.c_int32 * 2)(3, 4)
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, even, fake, fake, ctypes.byref(o)) == il.ILRE_EINVAL
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 0, kern, fake, fake, ctypes.byref(o)) == il.ILRE_EINVAL
    assert lib.ilre_recall(fake, fake, 100000, 8, 8, 2, 128, 9000, kern, fake, fake, ctypes.byref(o)) == il.ILRE_EUNSUPPORTED
    big = (ctypes.c_int32 * 2)(3, 4095)
    assert lib.ilre_recall(fake, fake, 100000, 8, 8, 2, 128, 64, big, fake, fake, ctypes.byref(o)) == il.ILRE_EUNSUPPORTED
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, ctypes.byref(_opts(struct_size=8))) == il.ILRE_EINVAL
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, ctypes.byref(_opts(score_mode=5))) == il.ILRE_EUNSUPPORTED
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, ctypes.byref(_opts(flags=64))) == il.ILRE_EUNSUPPORTED
    # undersized and misaligned workspace
    small = _opts(workspace=1 << 20, workspace_bytes=1024)
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, ctypes.byref(small)) == il.ILRE_ENOMEM
    odd = _opts(workspace=(1 << 20) + 8, workspace_bytes=1 << 30)
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, ctypes.byref(odd)) == il.ILRE_EINVAL
    # bad strides
    ok_ws = dict(workspace=1 << 20, workspace_bytes=1 << 30)
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, ctypes.byref(_opts(k_stride_token=100, **ok_ws))) == il.ILRE_EINVAL
    assert lib.ilre_recall(fake, fake, 1000, 8, 8, 2, 128, 64, kern, fake, fake, ctypes.byref(_opts(q_stride_token=132, **ok_ws))) == il.ILRE_EINVAL
    # staged entry points validate too
    assert lib.ilre_row_stats(fake, fake, 1000, 8, 8, 2, 128, None, fake, ctypes.byref(o)) == il.ILRE_EINVAL
    assert lib.ilre_col_scores(fake, fake, 1000, 8, 8, 2, 128, fake, fake, None, ctypes.byref(o)) == il.ILRE_EINVAL
    assert lib.ilre_select(None, 1000, 64, kern, fake, ctypes.byref(o)) == il.ILRE_EINVAL
    assert lib.ilre_select(fake, 1000, 64, kern, fake, ctypes.byref(o)) == il.ILRE_ENOMEM


def test_argument_errors_of_the_printed_form_rerope_and_gather():
    lib = il.load()
    fake = ctypes.c_void_p(4096)          # never dereferenced: every call below fails validation first
    o = _opts()
    mk, ak = (ctypes.c_int32 * 3)(2, 4, 8), (ctypes.c_int32 * 2)(1, 5)

    def sel(L=1000, sink=4, budget=64, mk_=mk, n_max=3, ak_=ak, n_avg=2, scores=fake, out=fake, opts=o):
        return lib.ilre_select_max_avg(scores, L, sink, budget, mk_, n_max, ak_, n_avg, out, None, ctypes.byref(opts))

    assert sel() == il.ILRE_ENOMEM                                   # everything valid except the missing workspace
    assert sel(scores=None) == il.ILRE_EINVAL
    assert sel(sink=-1) == il.ILRE_EINVAL and sel(sink=1001) == il.ILRE_EINVAL
    assert sel(budget=0) == il.ILRE_EINVAL
    assert sel(n_max=0) == il.ILRE_EINVAL and sel(ak_=None) == il.ILRE_EINVAL
    assert sel(mk_=(ctypes.c_int32 * 3)(2, 0, 8)) == il.ILRE_EINVAL
    assert sel(mk_=(ctypes.c_int32 * 3)(2, 4, 2048)) == il.ILRE_EUNSUPPORTED
    assert sel(ak_=(ctypes.c_int32 * 2)(1, 4096)) == il.ILRE_EUNSUPPORTED
    assert sel(n_max=3, n_avg=2, mk_=mk, ak_=ak, L=100000, budget=9000) == il.ILRE_EUNSUPPORTED
    wide = (ctypes.c_int32 * 9)(*range(1, 10))
    assert sel(mk_=wide, n_max=9, ak_=wide, n_avg=9) == il.ILRE_EUNSUPPORTED     # 81 combinations
    # sizing: grows with the number of average kernels, rejects what the entry points reject
    a = il.ilre_workspace_bytes_max_avg(1 << 20, 256, 32, 8, 128, 4, (2, 4, 8), 16, il.ILRE_BF16)
    b = il.ilre_workspace_bytes_max_avg(1 << 20, 256, 32, 8, 128, 4, (2, 4, 8), 4, il.ILRE_BF16)
    assert b < a < (1 << 30)
    with pytest.raises(il.IlreError):
        il.ilre_workspace_bytes_max_avg(1000, 8, 8, 2, 128, 4, (0,), 1, il.ILRE_BF16)

    def rope(L=1000, chunk=128, extra=4, base=10000.0, pairing=0, k_in=fake, k_out=fake, opts=o):
        return lib.ilre_rerope_keys(k_in, k_out, L, 2, 128, chunk, extra, base, None, pairing, ctypes.byref(opts))

    assert rope(k_in=None) == il.ILRE_EINVAL and rope(k_out=None) == il.ILRE_EINVAL
    assert rope(chunk=0) == il.ILRE_EINVAL and rope(extra=-1) == il.ILRE_EINVAL
    assert rope(base=0.0) == il.ILRE_EINVAL and rope(pairing=2) == il.ILRE_EUNSUPPORTED
    assert rope(k_in=ctypes.c_void_p(4100)) == il.ILRE_EINVAL                     # misaligned
    assert rope(opts=_opts(k_stride_token=100)) == il.ILRE_EINVAL
    assert lib.ilre_rerope_keys(fake, fake, 1000, 2, 64, 128, 4, 10000.0, None, 0, ctypes.byref(o)) == il.ILRE_EUNSUPPORTED

    assert lib.ilre_gather_ids(None, 1000, fake, 10, fake, ctypes.byref(o)) == il.ILRE_EINVAL
    assert lib.ilre_gather_ids(fake, 1000, fake, -1, fake, ctypes.byref(o)) == il.ILRE_EINVAL
    assert lib.ilre_gather_ids(fake, 1000, fake, 0, fake, ctypes.byref(o)) == il.ILRE_OK   # nothing to do, nothing launched
    assert il.ilre_last_error()


def test_row_stats_static_rejects_shapes_beyond_its_buffer():
    """The entry point that allocates nothing holds 4 MiB of scratch; a shape that needs more is refused on
    the host, before any device call."""
    lib = il.load()
    fake = ctypes.c_void_p(4096)          # never dereferenced
    o = _opts()
    # 64 kv heads x 16384 query tokens = 1M rows, one token split: 8 MiB of partial statistics
    rc = lib.ilre_row_stats_static(fake, fake, 1 << 20, 16384, 64, 64, 128, fake, fake, ctypes.byref(o))
    assert rc == il.ILRE_EUNSUPPORTED and "static buffer" in il.ilre_last_error()
    assert lib.ilre_row_stats_static(fake, fake, 1000, 8, 8, 2, 128, None, fake, ctypes.byref(o)) == il.ILRE_EINVAL
    assert lib.ilre_row_stats_static(fake, fake, 1000, 8, 8, 2, 64, fake, fake, ctypes.byref(o)) == il.ILRE_EUNSUPPORTED


def _splits(L, Lq, Hq, Hkv, block, dtype):
    """Token splits of a scoring pass, read off the size of the workspace."""
    nqb = -(-(Hq // Hkv) * Lq // block)

    def beside_the_selection(n, rows, heads, blocks):  # row statistics, a word a workgroup, edges of the splits, score vectors
        return 8 * rows * (n + 1) + 4 * (8 * -(-heads * n // 8) * blocks + n) + 4 * L * heads * blocks

    one = il.ilre_workspace_bytes(L, 1, 8, 8, 128, 3, il.ILRE_BF16)  # a split a tile of 64 tokens, up to 64
    selection = one - beside_the_selection(min(64, -(-L // 64)), 8, 8, 1)
    rest = il.ilre_workspace_bytes(L, Lq, Hq, Hkv, 128, 3, dtype) - selection
    n = min(range(1, 600), key=lambda n: abs(beside_the_selection(n, Hq * Lq, Hkv, nqb) - rest))
    assert abs(beside_the_selection(n, Hq * Lq, Hkv, nqb) - rest) < 3 * Hq * Lq  # (a split is 8 bytes a row, each region ends on 256)
    return n


@pytest.mark.parametrize("dtype,Lq,Hq,Hkv,block,room,least,most", [
    # query blocks that outnumber an XCD's places, or half of them: several rounds of workgroups
    (il.ILRE_BF16, 2080, 16, 2, 256, 64, 512, 2048), (il.ILRE_BF16, 1360, 64, 4, 256, 64, 512, 2048), (il.ILRE_BF16, 540, 32, 1, 512, 32, 256, 1024),
    (il.ILRE_BF16, 245, 71, 1, 512, 32, 256, 1024), (il.ILRE_F32, 260, 32, 1, 128, 64, 512, 2048), (il.ILRE_BF16, 1280, 40, 5, 512, 32, 256, 1024),
    # one round, as many as an XCD holds
    (il.ILRE_BF16, 90, 28, 4, 256, 64, 504, 504), (il.ILRE_BF16, 150, 28, 4, 256, 64, 480, 480), (il.ILRE_BF16, 170, 64, 8, 512, 32, 240, 240),
    (il.ILRE_BF16, 256, 32, 8, 512, 32, 256, 256), (il.ILRE_F32, 176, 64, 8, 128, 64, 440, 440),
])
def test_scoring_fills_the_chip_whatever_the_query_blocks(dtype, Lq, Hq, Hkv, block, room, least, most):
    """Workgroups of a scoring pass: no fewer than the chip has places where query blocks are many, and no more than a round of them where one fills it."""
    nqb = -(-(Hq // Hkv) * Lq // block)
    assert least <= _splits(131072, Lq, Hq, Hkv, block, dtype) * nqb * Hkv <= most
    assert 8 * room == (256 if block == 512 else 512)


@pytest.mark.parametrize("L,Lq,Hq,Hkv,splits", [
    # as few as the second pass merges itself (32) where no compute unit has more tiles of 32 tokens to do for it ...
    (4096, 32, 32, 8, 32), (2100, 32, 32, 8, 17), (4128, 32, 32, 8, 22), (6144, 128, 8, 2, 32), (3000, 32, 24, 6, 24),
    # ... and all there are where one would, or with many tiles
    (4096, 32, 16, 4, 64), (2100, 32, 24, 6, 33), (5000, 64, 20, 5, 40), (8192, 32, 32, 8, 64),
])
def test_fp32_splits_of_short_contexts(L, Lq, Hq, Hkv, splits):
    assert _splits(L, Lq, Hq, Hkv, 128, il.ILRE_F32) == splits


def test_walk_cases_sit_at_the_edge_of_the_bitmap():
    """The GPU cases of the walk name the number of tokens up to which its set is a bitmap; it is the library's."""
    import test_gpu_parity as parity_tests

    with open(os.path.join(ROOT, "paper_2508_17892_amd", "csrc", "select.hip")) as f:
        text = f.read()
    chunk, chunks = (int(re.search(rf"constexpr int {name} = (\d+);", text).group(1)) for name in ("kBitmapChunk", "kBitmapChunks"))
    assert parity_tests.BITMAP_TOKENS == chunks * chunk * 32
    bodies = {c[0] - c[1] - parity_tests.BITMAP_TOKENS for c in parity_tests.WALK_CASES}
    assert {-1, 0, 1} <= bodies
