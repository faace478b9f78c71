"""CPU-only checks of the C-ABI library: it loads, exports every symbol the
header declares, validates descriptions and shapes, and its host-side plan
(token order, cumulative lengths, index maps) agrees with the CPU reference."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import workloads
from oracle import encoder as oe
from oracle import preprocess as op
from paper_2603_26498_amd import binding as B
from paper_2603_26498_amd.runtime import VisionEncoder

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "tcmv.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(tcmv_[a-z0-9_]+)\s*\(", hdr))
    assert declared, "no declarations found"
    assert declared == set(B.SIGNATURES), declared ^ set(B.SIGNATURES)
    lib = C.CDLL(B.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name
    assert B.tcmv_version() >= 100
    assert B.error_name(-2) == "TCMV_E_BAD_SHAPE"


def test_library_exports_every_scheduler_symbol():
    from paper_2603_26498_amd import sched_binding as SB
    hdr = open(os.path.join(ROOT, "include", "tcms.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(tcms_[a-z0-9_]+)\s*\(", hdr))
    assert declared == set(SB.SIGNATURES), declared ^ set(SB.SIGNATURES)
    lib = C.CDLL(B.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name
    assert C.sizeof(SB.tcms_cluster_model) == 10 * 8 and C.sizeof(SB.tcms_regulator) == 9 * 8


def test_struct_sizes_match_header_layout():
    assert C.sizeof(B.tcmv_model_desc) == 13 * 4 + 4 + 24 + 4 * 4 + 4 + 4 + 4
    assert C.sizeof(B.tcmv_item) == 6 * 4 + 8
    assert C.sizeof(B.tcmv_weights) == 14 * 8


def test_description_validation():
    with pytest.raises(B.TcmvError) as e:
        B.tcmv_create(B.make_desc(dtype="bf16", layers=1, d=100, heads=3, mlp=64))
    assert e.value.code == B.TCMV_E_INVALID_ARG
    with pytest.raises(B.TcmvError) as e:
        B.tcmv_create(B.make_desc(dtype="bf16", layers=1, d=192, heads=4, mlp=256))      # head size 48
    assert e.value.code == B.TCMV_E_UNSUPPORTED and "head size" in str(e.value)
    with pytest.raises(B.TcmvError):
        B.tcmv_create(B.make_desc(dtype="f32", layers=1, d=64, heads=1, mlp=64, merge=3))
    ctx = B.tcmv_create(B.make_desc(dtype="f32", layers=1, d=64, heads=1, mlp=64, patch=7))
    assert B.tcmv_k_pad(B.make_desc(dtype="f32", layers=1, d=64, heads=1, mlp=64, patch=7)) == 148
    B.tcmv_destroy(ctx)
    assert B.tcmv_k_pad(B.make_desc(dtype="bf16", layers=1, d=64, heads=1, mlp=64, patch=14)) == 640
    assert B.tcmv_k_pad(B.make_desc(dtype="bf16", layers=1, d=64, heads=1, mlp=64, patch=14, tpatch=2)) == 1216


def _plan(desc, items):
    enc = VisionEncoder(desc)
    return enc, enc.plan(items, upload=False)


@pytest.mark.parametrize("idx", [1, 2, 3, 4, 5, 6, 7])
def test_plan_matches_reference_token_order(idx):
    wl = workloads.small_config(idx)
    enc, pl = _plan(wl.desc, wl.items)
    grids = oe.grids_of(wl.items, wl.desc)
    cu = oe.cu_seqlens_of(grids, wl.desc.use_cls)
    assert pl.cu_seqlens == cu.tolist()
    assert pl.info.n_tokens == cu[-1]
    assert pl.info.n_patch_rows == sum(g[0] * g[1] * g[2] for g in grids)
    assert pl.info.k == wl.desc.k and pl.info.k_pad % 2 == 0 and pl.info.k_pad >= wl.desc.k
    thw = pl.row_map(0)
    dst = pl.row_map(1)
    ref = np.concatenate([op.token_coords(*g, wl.desc.merge, wl.desc.window) for g in grids if g[0]] or [np.zeros((0, 3), int)])
    assert np.array_equal(thw >> 16, ref[:, 0]) and np.array_equal((thw >> 8) & 255, ref[:, 1])
    assert np.array_equal(thw & 255, ref[:, 2])
    # destination rows: patch rows in order, skipping one CLS row at the start of each segment
    exp, r = [], 0
    for g in grids:
        n = g[0] * g[1] * g[2]
        if n:
            r += 1 if wl.desc.use_cls else 0
            exp += list(range(r, r + n))
            r += n
    assert dst.tolist() == exp
    pos = pl.row_map(2)
    if wl.desc.pos == "sep2d":
        assert np.array_equal(pos & 0xFFFF, ref[:, 1]) and np.array_equal(pos >> 16, ref[:, 2])
    elif wl.desc.pos == "learned1d":
        seg0 = np.searchsorted(cu, dst, side="right") - 1
        assert np.array_equal(pos, dst - cu[seg0])
    m2 = wl.desc.merge ** 2
    assert pl.info.n_out_tokens == (cu[-1] // m2 if wl.desc.out_dim else 0)
    assert pl.info.hidden_bytes == cu[-1] * wl.desc.d * 4


def test_full_size_token_counts():
    """Plan sizes of the full workloads (no frames needed on the host)."""
    expect = {1: 197, 2: 18432, 4: 32768, 6: 65536, 7: 32768}
    for idx in (1, 2, 3, 4, 5, 6, 7):
        wl = workloads.full_config(idx, with_frames=False, with_weights=False)
        enc, pl = _plan(wl.desc, wl.items)
        cu = oe.cu_seqlens_of(oe.grids_of(wl.items, wl.desc), wl.desc.use_cls)
        assert pl.cu_seqlens == cu.tolist()
        if idx in expect:
            assert pl.info.n_tokens == expect[idx]
        if idx == 5:
            assert pl.info.n_segments == 26 and pl.info.n_items == 226
            assert all(a == b for a, b in zip(pl.cu_seqlens[26:], pl.cu_seqlens[27:]))   # text: no tokens


def test_bad_shapes_are_rejected():
    desc = workloads.qwen_like_desc(layers=1, d=320, heads=4, mlp=640, out_dim=192, max_grid=16)
    enc = VisionEncoder(desc)
    I = workloads.Item
    for bad in ([I(1, 1, 30, 28, 30, 28)],            # not a multiple of patch*merge
                [I(1, 1, 28, 28, 0, 28)],             # empty target
                [I(2, 3, 28, 28, 28, 28)],            # odd video length with temporal patch 2
                [I(1, 1, 28, 28, 28 * 17, 28)],       # grid side above the position table
                [I(1, 1, 0, 28, 28, 28)]):            # empty source
        with pytest.raises(B.TcmvError) as e:
            enc.plan(bad, upload=False)
        assert e.value.code == B.TCMV_E_BAD_SHAPE, bad
    with pytest.raises(B.TcmvError) as e:
        enc.plan([I(7, 1, 28, 28, 28, 28)], upload=False)
    assert e.value.code == B.TCMV_E_INVALID_ARG
    # empty and text-only plans are valid and empty
    for items in ([], [I(0, 0, 0, 0, 0, 0)] * 3):
        pl = enc.plan(items, upload=False)
        assert pl.info.n_tokens == 0 and pl.info.n_patch_rows == 0 and pl.cu_seqlens == [0] * (len(items) + 1)
    # more tokens than the kernels' 32-bit element offsets allow (tokens x widest row below 2^32): 14 images of
    # 254 x 254 patches with rows up to 5120 wide; one fewer image fits
    big = workloads.qwen_like_desc(layers=1, max_grid=254)
    side = 254 * 14
    with pytest.raises(B.TcmvError) as e:
        VisionEncoder(big).plan([I(1, 1, side, side, side, side)] * 14, upload=False)
    assert e.value.code == B.TCMV_E_BAD_SHAPE and "2^32" in str(e.value)
    assert VisionEncoder(big).plan([I(1, 1, side, side, side, side)] * 12, upload=False).info.n_tokens == 12 * 254 * 254
    # learned 1-D table too short
    d2 = workloads.ModelDesc(dtype="bf16", layers=1, d=128, heads=2, mlp=128, patch=14, pos="learned1d", max_pos=3)
    with pytest.raises(B.TcmvError) as e:
        VisionEncoder(d2).plan([I(1, 1, 28, 28, 28, 28)], upload=False)
    assert e.value.code == B.TCMV_E_BAD_SHAPE


def test_device_calls_fail_cleanly_without_weights_or_gpu():
    desc = workloads.qwen_like_desc(layers=1, d=320, heads=4, mlp=640, out_dim=192, max_grid=16)
    enc = VisionEncoder(desc)
    pl = enc.plan([workloads.Item(1, 1, 28, 28, 28, 28)], upload=False)
    rc = B.lib().tcmv_encode(enc.ctx, pl.handle, 256, 256, 256, 256, 1 << 30, None)
    assert rc == B.TCMV_E_NO_WEIGHTS
    rc = B.lib().tcmv_preprocess(enc.ctx, pl.handle, 256, 256, None)     # item has a null frame pointer
    assert rc == B.TCMV_E_INVALID_ARG
    assert "frame pointer" in B.tcmv_last_error(enc.ctx)
    assert B.tcmv_op_attention_workspace(B.TCMV_BF16, [0, 100, 100, 164], 128, 2) > 0


def test_plan_metadata_belongs_to_the_caller():
    """The library hands out the plan's index metadata as host bytes and never allocates device memory itself: the
    stage calls take the caller's device copy, and refuse a missing, misaligned or short one."""
    desc = workloads.qwen_like_desc(layers=1, d=320, heads=4, mlp=640, out_dim=192, max_grid=16)
    enc = VisionEncoder(desc)
    item = workloads.Item(1, 1, 28, 28, 28, 28)
    pl = enc.plan([item], upload=False)
    assert pl.meta is None and pl.info.meta_bytes > 0 and pl.info.meta_bytes % 256 == 0
    blob = B.tcmv_plan_meta(pl.handle)
    assert len(blob) == pl.info.meta_bytes
    # the normalisation table (3 x 256 values, bf16-representable for a bf16 model) is part of it
    tab = np.array([((v / 255.0) - 0.5) / 0.5 for v in range(256)], np.float32)
    tab = (tab.view(np.uint32) + 0x7FFF + ((tab.view(np.uint32) >> 16) & 1) & 0xFFFF0000).astype(np.uint32).view(np.float32)
    assert blob.find(tab.tobytes()) >= 0
    # an empty plan needs no metadata
    empty = enc.plan([workloads.Item(0, 0, 0, 0, 0, 0)], upload=False)
    assert empty.info.meta_bytes == 0 and B.tcmv_plan_meta(empty.handle) == b""
    assert B.lib().tcmv_plan_upload(empty.handle, None, 0, None) == B.TCMV_OK
    # argument checks come before any device work
    assert B.lib().tcmv_plan_upload(pl.handle, None, pl.info.meta_bytes, None) == B.TCMV_E_INVALID_ARG
    assert B.lib().tcmv_plan_upload(pl.handle, 256 + 16, pl.info.meta_bytes, None) == B.TCMV_E_INVALID_ARG
    assert B.lib().tcmv_plan_upload(pl.handle, 256, pl.info.meta_bytes - 1, None) == B.TCMV_E_WORKSPACE_TOO_SMALL
    assert B.lib().tcmv_plan_upload(None, 256, 0, None) == B.TCMV_E_INVALID_ARG
    rc = B.lib().tcmv_preprocess(enc.ctx, pl.handle, None, 256, None)
    assert rc == B.TCMV_E_INVALID_ARG


def test_attention_index_is_host_data():
    cu = [0, 100, 100, 164]
    n = B.lib().tcmv_op_attention_index_bytes(B.TCMV_BF16, (C.c_int64 * 4)(*cu), 3, 128, 2)
    assert n > 0 and n % 256 == 0
    idx = B.tcmv_op_attention_index(B.TCMV_BF16, cu, 128, 2)
    assert len(idx) == n
    vcol = np.frombuffer(idx[:164 * 4], np.int32)
    # every row has its own column in the transposed-V buffer; the second non-empty segment starts at a multiple of 64
    assert len(set(vcol.tolist())) == 164 and vcol[:100].max() < 128 and vcol[100:].min() == 128
    buf = C.create_string_buffer(16)
    assert B.lib().tcmv_op_attention_index(B.TCMV_BF16, (C.c_int64 * 4)(*cu), 3, 128, 2, buf, 16) == B.TCMV_E_WORKSPACE_TOO_SMALL
    assert B.lib().tcmv_op_attention_index_bytes(B.TCMV_BF16, (C.c_int64 * 4)(0, 5, 3, 9), 3, 128, 2) == 0


def test_windowed_plan_whose_transposed_values_do_not_fit_32_bit_offsets_is_refused():
    """Every window is padded to 64 columns of the transposed values, so a plan with small windows needs far more
    columns than it has tokens; the offset guard must count them."""
    desc = workloads.ModelDesc(dtype="bf16", layers=1, d=2048, heads=32, mlp=2048, patch=14, tpatch=1, merge=1,
                               pos="none", window=2, full_every=0)
    enc = VisionEncoder(desc)
    # 8 x 8 grids: 16 windows of 4 tokens -> 1024 columns for 64 tokens
    items = [workloads.Item(1, 1, 112, 112, 112, 112)] * 3000
    with pytest.raises(B.TcmvError) as e:
        enc.plan(items, upload=False)
    assert e.value.code == B.TCMV_E_BAD_SHAPE and "transposed" in str(e.value)
    assert enc.plan(items[:1000], upload=False).info.n_tokens == 1000 * 64


# rows per work item that were measured to be the fastest of 256 and 512 (the choice between them), and the limits of the rule
@pytest.mark.parametrize("heads,dh,lens,rows", [
    (16, 80, [4096], 256), (16, 80, [1024] * 4, 256), (8, 80, [8192], 256),               # one 256-row item per CU
    (16, 80, [4608], 512), (16, 80, [5120], 512), (16, 80, [6144], 512), (16, 80, [7680], 512), (16, 80, [8192], 512),
    (16, 80, [1024] * 6, 512), (16, 80, [1024, 1024, 5120], 512), (8, 80, [9728], 512),
    (16, 64, [5120], 256), (16, 64, [6144], 256), (16, 64, [8192], 512), (16, 32, [6144], 256),
    (16, 80, [3840], 128), (16, 80, [4352], 256), (16, 96, [8192], 128)])
def test_rows_of_an_attention_work_item(heads, dh, lens, rows):
    cu = [0] + [int(c) for c in np.cumsum(lens)]
    assert B.tcmv_op_attention_rows(B.TCMV_BF16, cu, heads * dh, heads) == rows


# tiny requests: 64-row items over four groups of waves only with a tile of keys for each group and CUs to spare; elsewhere
# they lost time (8 x 64 tokens 3 %, 4 x 256 tokens of 16 heads 1 % and 8 % of what touching weights gains)
@pytest.mark.parametrize("heads,dh,lens,rows", [
    (16, 80, [256], 64), (16, 80, [193], 64), (16, 80, [192], 128), (16, 80, [64], 128), (16, 80, [1], 128), (16, 80, [64] * 4, 128),
    (16, 80, [256] * 2, 64), (16, 80, [256] * 3, 128), (16, 64, [256] * 4, 128), (16, 80, [257], 128), (6, 64, [256] * 6, 64)])
def test_rows_of_tiny_requests(heads, dh, lens, rows):
    cu = [0] + [int(c) for c in np.cumsum(lens)]
    assert B.tcmv_op_attention_rows(B.TCMV_BF16, cu, heads * dh, heads) == rows


def _host_plan(desc, sizes):
    """Plan of still images given in patches (no weights, nothing uploaded) and the encoder that owns it."""
    p = desc.patch
    return _plan(desc, [workloads.Item(workloads.IMAGE, 1, h * p, w * p, h * p, w * p, None) for h, w in sizes])


def test_route_queries_answer_on_the_host():
    enc, pl = _host_plan(workloads.qwen_like_desc(), [(16, 16)])
    names = {c: B.tcmv_plan_gemm_kernel(pl.handle, c, 0) for c in ("qkv_gemm", "out_gemm", "fc1_gemm", "fc2_gemm")}
    assert names["qkv_gemm"] == names["fc1_gemm"] == "64x64" and names["out_gemm"] == names["fc2_gemm"] == "64x64 slices"
    assert B.tcmv_plan_gemm_kernel(pl.handle, "layernorm", 0) is None and B.tcmv_plan_gemm_kernel(pl.handle, "qkv_gemm", 32) is None
    assert B.tcmv_plan_key_norms(pl.handle, 0) == 0 and B.tcmv_plan_key_norms(pl.handle, -1) < 0
    assert B.tcmv_op_gemm_kernel(B.EPI_STORE, 32768, 3840, 1280) == "256x320 persistent"
    assert B.tcmv_op_gemm_kernel(B.EPI_STORE, 100, 100, 100) is None       # k must be a multiple of 64
    enc, pl = _host_plan(workloads.small_config(1).desc, [(14, 14)])       # fp32: no bf16 kernel
    assert B.tcmv_plan_gemm_kernel(pl.handle, "qkv_gemm", 0) is None and B.tcmv_plan_key_norms(pl.handle, 0) == 0


# products on which an earlier estimate took a kernel 8 - 40 % slower than the one named (weights read from memory)
@pytest.mark.parametrize("epi,m,n,k,kernel", [
    (B.EPI_STORE, 8192, 3072, 128, "128x128"), (B.EPI_STORE, 4096, 3072, 128, "128x128"), (B.EPI_STORE, 12288, 1024, 128, "128x128"),
    (B.EPI_STORE, 1024, 3072, 512, "128x128 k/2"), (B.EPI_STORE, 8192, 1024, 256, "256x128"), (B.EPI_STORE, 2048, 3072, 512, "256x128"),
    (B.EPI_GATED, 576, 8192, 1024, "256x128"), (B.EPI_GATED, 640, 8192, 1024, "256x128"), (B.EPI_GELU, 1280, 4096, 1024, "256x128"),
    (B.EPI_RESID, 8192, 1024, 128, "128x128"), (B.EPI_RESID, 10240, 1024, 1024, "128x128"), (B.EPI_RESID, 11520, 1024, 1024, "128x128"),
    (B.EPI_RESID, 8464, 1280, 1280, "128x128"), (B.EPI_RESID, 9216, 1152, 1280, "128x128"), (B.EPI_RESID, 2304, 1280, 1280, "64x64"),
    (B.EPI_RESID, 2688, 1024, 1024, "64x64"), (B.EPI_RESID, 10240, 1152, 4352, "128x128")])
def test_kernels_of_products_that_an_estimate_got_wrong(epi, m, n, k, kernel):
    assert B.tcmv_op_gemm_kernel(epi, m, n, k) == kernel


# products that lose time when they are cut behind their whole rounds, although an earlier estimate cut them (whole and cut,
# microseconds: 23766 x 1152 x 1280 95.5 / 101.5, 32529 x 1024 x 1024 92 / 100, 13186 x 3584 x 5120 376 / 423, 8807 rows 255 / 280,
# 12877 x 5120 x 5120 525 / 544, 70138 x 2048 x 2048 641 / 713, 14374 rows 136 / 153; 21910 x 1280 x 1280 loses behind
# 256x256 tiles, 93.9 / 101.3, and gains behind 256x320 ones)
@pytest.mark.parametrize("epi,m,n,k,kernel", [
    (B.EPI_RESID, 23766, 1152, 1280, "256x256 persistent"), (B.EPI_RESID, 26938, 1152, 1280, "256x320 persistent"),
    (B.EPI_RESID, 32529, 1024, 1024, "256x256 persistent"), (B.EPI_STORE, 13186, 3584, 5120, "256x256 persistent"),
    (B.EPI_STORE, 8807, 3584, 5120, "256x256 persistent"), (B.EPI_GELU, 12877, 5120, 5120, "256x256 persistent"),
    (B.EPI_RESID, 70138, 2048, 2048, "256x256 persistent"), (B.EPI_RESID, 14374, 2048, 2048, "256x256 persistent"),
    (B.EPI_RESID, 21910, 1280, 1280, "256x320 persistent + 128x128")])
def test_products_that_lose_when_cut_stay_whole(epi, m, n, k, kernel):
    assert B.tcmv_op_gemm_kernel(epi, m, n, k) == kernel


# side of one still image in patches -> kernels of the two products that accumulate (1280 wide, mlp 5120): slices of k where
# they pay together with the norm that adds them, in the tiles that are faster (896 rows: 31 us a layer with 128x128 tiles, 37
# with 64x64; 1760 rows: 51 unsplit, 51 in slices)
@pytest.mark.parametrize("side,out,fc2", [
    ((16, 16), "64x64 slices", "64x64 slices"), ((20, 24), "64x64 slices", "64x64 slices"), ((24, 32), "64x64", "128x128 slices"),
    ((28, 32), "64x64", "128x128 slices"), ((32, 32), "64x64", "128x128 slices"), ((36, 40), "64x64", "128x128 slices"),
    ((44, 48), "64x64", "128x128 k/2")])
def test_where_products_are_cut_along_k(side, out, fc2):
    enc, pl = _host_plan(workloads.qwen_like_desc(), [side])
    assert B.tcmv_plan_gemm_kernel(pl.handle, "out_gemm", 0) == out
    assert B.tcmv_plan_gemm_kernel(pl.handle, "fc2_gemm", 0) == fc2


# whether the reference-free attention pass and the key norms it needs pay for one image (sides in patches): with few heads
# or long segments they do although the work items are few, where they were measured to (and short ones do without)
@pytest.mark.parametrize("heads,dh,side,n,pays", [
    (4, 32, (120, 120), 1, True), (4, 64, (120, 120), 1, True), (4, 96, (120, 120), 1, True), (4, 80, (120, 120), 1, True),
    (8, 64, (84, 92), 1, True), (8, 96, (84, 92), 1, True), (8, 80, (84, 92), 1, True), (2, 64, (84, 92), 1, True),
    (16, 64, (44, 48), 1, True), (16, 64, (56, 56), 1, True), (12, 64, (64, 64), 1, True), (8, 64, (40, 64), 2, True),
    (16, 80, (32, 36), 1, False), (16, 80, (40, 44), 1, False), (16, 64, (32, 40), 1, False), (4, 96, (64, 64), 1, False),
    (8, 96, (32, 40), 4, False), (2, 32, (48, 48), 1, False), (16, 80, (64, 68), 1, True), (16, 96, (64, 72), 1, True)])
def test_where_key_norms_pay(heads, dh, side, n, pays):
    desc = workloads.ModelDesc(layers=1, d=heads * dh, heads=heads, mlp=256, patch=14, tpatch=1, merge=1)
    enc, pl = _host_plan(desc, [side] * n)
    norms = B.tcmv_plan_key_norms(pl.handle, 0)
    assert (norms > 0) == pays
    assert norms < 2 or dh in (64, 80)          # only whole heads of these sizes fit the write-out of the QKV product


# whether attention reads the weights behind it into the caches (one image, sides in patches): where model and request
# exceed the last-level cache or a layer fits the L2 caches; the others lost up to 12 % (2 layers of 2048, 64 tokens: 113 us
# without, 126 with)
@pytest.mark.parametrize("layers,d,heads,mlp,side,touches", [
    (12, 768, 12, 3072, (24, 24), 1), (8, 1024, 16, 4096, (16, 16), 1), (4, 1280, 16, 4352, (24, 24), 0), (4, 1280, 16, 5120, (48, 48), 0),
    (2, 2048, 32, 8192, (8, 8), 0), (5, 1280, 16, 5120, (16, 16), 0), (5, 1280, 16, 5120, (32, 32), 1), (6, 1280, 16, 5120, (8, 8), 1),
    (32, 1280, 16, 5120, (16, 16), 1), (32, 1280, 16, 5120, (63, 65), 0), (32, 1280, 16, 5120, (64, 64), 0)])
def test_where_attention_reads_the_weights_behind_it(layers, d, heads, mlp, side, touches):
    enc, pl = _host_plan(workloads.ModelDesc(layers=layers, d=d, heads=heads, mlp=mlp, patch=14, tpatch=1, merge=1), [side])
    norms = B.tcmv_plan_key_norms(pl.handle, 0) > 0                    # with key norms a second launch would have to do it
    assert B.tcmv_plan_touches_weights(pl.handle, 0) == (0 if norms else touches)
    assert B.tcmv_plan_touches_weights(pl.handle, layers) < 0


@pytest.mark.parametrize("heads,dh,side,norms", [(60, 64, 39, 0), (64, 64, 36, 0), (84, 64, 33, 0), (56, 64, 39, None), (60, 96, 66, 0), (28, 80, 99, None)])
def test_attention_too_wide_for_the_pass_over_the_keys_goes_without_norms(heads, dh, side, norms):
    """The separate pass holds at most 512 chunk sums and norms of a row: wider models keep running, without the norms
    (or with those of the QKV product)."""
    ctx = B.tcmv_create(B.make_desc(dtype="bf16", layers=1, d=1024, heads=heads, mlp=256, patch=14, tpatch=1, merge=1, head_dim=dh, attn_scale=0.1))
    plan = B.tcmv_plan_create(ctx, [(workloads.IMAGE, 1, side * 14, side * 14, side * 14, side * 14, None)])
    got = B.tcmv_plan_key_norms(plan, 0)
    B.tcmv_plan_destroy(plan)
    B.tcmv_destroy(ctx)
    assert got == norms if norms is not None else got > 0
    assert got != 1 or heads * (dh // 8 + 1) <= 512
