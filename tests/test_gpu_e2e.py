"""GPU parity of the three stages (through the C ABI) against the CPU
reference on reduced versions of the five workloads, plus the adversarial
end-to-end variants (non-zero biases, random gamma/beta) they are built with.

Tolerances.  Preprocessing and patch indexing: bit-exact.  fp32 model: 1e-4 of
the row maximum.  bf16 model: per token max|err|/max|ref| <= 2e-2 and cosine
>= 0.999 (the bar of the target), checked on every output row."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from oracle import encoder as oe
from paper_2603_26498_amd import binding as B
from paper_2603_26498_amd.runtime import VisionEncoder
from util import assert_tokens_close

pytestmark = pytest.mark.gpu


def run_gpu(wl):
    enc = VisionEncoder(wl.desc, wl.weights)
    pl = enc.plan(wl.items)
    patches = enc.preprocess(pl)
    hidden = enc.encode(pl, patches)
    out = enc.merge_project(pl, hidden) if wl.desc.out_dim else None
    torch.cuda.synchronize()
    return enc, pl, patches, hidden, out


def check_patches(wl, ref, patches):
    k = wl.desc.k
    got = patches.float().cpu().numpy()
    exp = np.concatenate([p for p in ref["patches"]], 0) if got.shape[0] else np.zeros((0, k), np.float32)
    assert got.shape[0] == exp.shape[0]
    assert np.array_equal(got[:, :k].view(np.uint32), exp.view(np.uint32)), "patches differ (must be bit-exact)"
    assert not got[:, k:].any(), "padding columns must be zero"


@pytest.mark.parametrize("idx", [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("affine", [False, True])
def test_small_workloads(idx, affine):
    wl = workloads.small_config(idx, random_affine=affine)
    ref = oracle.run(wl)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert pl.cu_seqlens == ref["cu_seqlens"].tolist()
    check_patches(wl, ref, patches)
    rel, cos = (1e-4, 0.999999) if wl.desc.dtype == "f32" else (2e-2, 0.999)
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], rel, cos, f"small{idx} hidden")
    if out is not None:
        assert_tokens_close(out.float().cpu().numpy(), ref["out"], rel, cos, f"small{idx} out")


def test_resize_paths_bit_exact_many_sizes():
    """Up- and down-scaling, odd source sizes, several items per launch."""
    desc = workloads.ModelDesc(dtype="bf16", layers=0, d=128, heads=2, mlp=128, patch=14, tpatch=2, merge=2)
    rng = np.random.default_rng(77)
    items = []
    for (n, sh, sw, dh, dw) in [(1, 37, 53, 28, 56), (2, 240, 426, 56, 84), (1, 31, 17, 84, 140), (4, 5, 1, 28, 28),
                                (1, 1080, 1920, 224, 448), (1, 56, 56, 56, 56), (2, 100, 100, 112, 28)]:
        items.append(workloads.Item(2 if n > 1 else 1, n, sh, sw, dh, dw, workloads.random_frames(rng, n, sh, sw)))
    wl = workloads.Workload("resize", desc, items, workloads.make_weights(desc, 1))
    enc = VisionEncoder(desc, wl.weights)
    pl = enc.plan(items)
    patches = enc.preprocess(pl)
    torch.cuda.synchronize()
    ref = oracle.run(wl, stages=("preprocess",))
    check_patches(wl, ref, patches)


@pytest.mark.parametrize("dtype,patch,tpatch,merge", [("f32", 16, 1, 1), ("f32", 7, 3, 1), ("bf16", 14, 1, 1),
                                                      ("bf16", 8, 2, 2), ("f32", 14, 2, 2)])
def test_preprocess_layouts_and_general_normalisation(dtype, patch, tpatch, merge):
    mean = tuple(float(np.float32(m)) for m in (0.485, 0.456, 0.406))
    std = tuple(float(np.float32(s)) for s in (0.229, 0.224, 0.225))
    desc = workloads.ModelDesc(dtype=dtype, layers=0, d=128, heads=2, mlp=128, patch=patch, tpatch=tpatch, merge=merge,
                               mean=mean, std=std)
    rng = np.random.default_rng(5)
    pm = patch * merge
    items = [workloads.Item(1, 1, 3 * pm, 2 * pm, 3 * pm, 2 * pm, workloads.random_frames(rng, 1, 3 * pm, 2 * pm)),
             workloads.Item(0, 0, 0, 0, 0, 0, None),
             workloads.Item(2, 2 * tpatch, pm, 4 * pm, pm, 4 * pm, workloads.random_frames(rng, 2 * tpatch, pm, 4 * pm))]
    wl = workloads.Workload("layout", desc, items, workloads.make_weights(desc, 1))
    enc = VisionEncoder(desc, wl.weights)
    pl = enc.plan(items)
    patches = enc.preprocess(pl)
    torch.cuda.synchronize()
    check_patches(wl, oracle.run(wl, stages=("preprocess",)), patches)


def _fma_form_reproduces_table(mean, std):
    """Whether bf16(fma(v, 1/(255 std), -mean/std)) in fp32 equals the contract's bf16(fp32((v/255 - mean)/std)) for
    every pixel value (the product v * scale fits a double exactly, so rounding the double sum once to fp32 is the
    fused multiply-add)."""
    v = np.arange(256, dtype=np.float64)
    table = workloads.snap_to_bf16_grid(((v / 255.0 - mean) / std).astype(np.float32))
    sc, of = np.float32(1.0 / (255.0 * std)), np.float32(-mean / std)
    return np.array_equal(table, workloads.snap_to_bf16_grid((v * np.float64(sc) + np.float64(of)).astype(np.float32)))


@pytest.mark.parametrize("first_channel,computed", [((0.5, 0.5), True), ((0.3121532201766968, 0.4928024709224701), False)])
def test_bf16_normalisation_computed_or_looked_up_is_the_table(first_channel, computed):
    """The bf16 strip kernel computes the normalised value with one fused multiply-add where that gives the table's
    768 values, and looks it up where it does not (here: one entry of the first channel differs).  Either way the
    patches are the reference's, bit for bit; copied and resampled strips, a video and still images."""
    mean = (first_channel[0], float(np.float32(0.456)), float(np.float32(0.406)))
    std = (first_channel[1], float(np.float32(0.224)), float(np.float32(0.225)))
    assert all(_fma_form_reproduces_table(m, s) for m, s in zip(mean, std)) == computed
    desc = workloads.ModelDesc(dtype="bf16", layers=0, d=128, heads=2, mlp=128, patch=14, tpatch=2, merge=2,
                               mean=mean, std=std)
    rng = np.random.default_rng(6)
    items = [workloads.Item(1, 1, 84, 532, 84, 532, workloads.random_frames(rng, 1, 84, 532)),       # 38 tokens wide: strips of 16, 16, 6
             workloads.Item(2, 4, 56, 476, 56, 476, workloads.random_frames(rng, 4, 56, 476)),       # 34 wide: 16, 16, 2
             workloads.Item(1, 1, 61, 333, 56, 308, workloads.random_frames(rng, 1, 61, 333)),       # resampled
             workloads.Item(2, 2, 100, 90, 84, 112, workloads.random_frames(rng, 2, 100, 90))]
    # every pixel value occurs in every channel of the first image
    items[0].frames.reshape(-1, 3)[:256] = np.arange(256, dtype=np.uint8)[:, None]
    wl = workloads.Workload("normalisation", desc, items, workloads.make_weights(desc, 1))
    enc = VisionEncoder(desc, wl.weights)
    pl = enc.plan(items)
    patches = enc.preprocess(pl)
    torch.cuda.synchronize()
    check_patches(wl, oracle.run(wl, stages=("preprocess",)), patches)


def test_text_only_and_empty_batches_launch_nothing():
    wl = workloads.small_config(5)
    enc = VisionEncoder(wl.desc, wl.weights)
    for items in ([], [workloads.Item(0, 0, 0, 0, 0, 0, None)] * 4):
        pl = enc.plan(items)
        p = enc.preprocess(pl)
        h = enc.encode(pl, p)
        o = enc.merge_project(pl, h)
        torch.cuda.synchronize()
        assert p.shape[0] == 0 and h.shape[0] == 0 and o.shape[0] == 0


def test_text_requests_do_not_disturb_other_requests():
    wl = workloads.small_config(5)
    only_visual = [it for it in wl.items if it.n_frames > 0]
    enc = VisionEncoder(wl.desc, wl.weights)
    res = []
    for items in (wl.items, only_visual):
        pl = enc.plan(items)
        h = enc.encode(pl, enc.preprocess(pl))
        res.append(enc.merge_project(pl, h).float().cpu().numpy())
    assert np.array_equal(res[0], res[1])


def test_permutation_equivariance_without_positions():
    """Permuting the patch rows of a segment permutes the encoder output rows."""
    desc = workloads.ModelDesc(dtype="bf16", layers=2, d=128, heads=2, mlp=256, patch=14, tpatch=1, merge=1)
    w = workloads.make_weights(desc, 3, random_affine=True)
    rng = np.random.default_rng(3)
    it = workloads.Item(1, 1, 70, 84, 70, 84, workloads.random_frames(rng, 1, 70, 84))
    enc = VisionEncoder(desc, w)
    pl = enc.plan([it])
    patches = enc.preprocess(pl)
    perm = torch.from_numpy(rng.permutation(patches.shape[0])).to(patches.device)
    a = enc.encode(pl, patches).clone()
    b = enc.encode(pl, patches[perm].contiguous())
    torch.cuda.synchronize()
    assert_tokens_close(b.cpu().numpy(), a[perm].cpu().numpy(), 2e-2, 0.999, "permutation")


def test_workspace_too_small_and_missing_projector_are_reported():
    wl = workloads.small_config(2)
    enc = VisionEncoder(wl.desc, wl.weights)
    pl = enc.plan(wl.items)
    patches = enc.preprocess(pl)
    small = enc.workspace(256)
    hidden = torch.empty((pl.info.n_tokens, wl.desc.d), device="cuda:0")
    with pytest.raises(B.TcmvError) as e:
        B.tcmv_encode(enc.ctx, pl.handle, pl.meta, patches, hidden, small, small.numel())
    assert e.value.code == B.TCMV_E_WORKSPACE_TOO_SMALL
    with pytest.raises(B.TcmvError) as e:
        B.tcmv_merge_project(enc.ctx, pl.handle, hidden, hidden, small, small.numel())
    assert e.value.code == B.TCMV_E_UNSUPPORTED


def test_results_are_deterministic_run_to_run():
    wl = workloads.small_config(3)
    a = run_gpu(wl)[4].float().cpu().numpy()
    b = run_gpu(wl)[4].float().cpu().numpy()
    assert np.array_equal(a, b)


def test_per_request_pipeline_matches_plan_by_plan_runs():
    """One plan per request, preprocessing of the next request overlapped with the
    encoding of the current one on a second stream: outputs must be the ones of
    running the requests one after the other, and each request's output must be
    its rows of the batched run (requests do not interact)."""
    for idx in (5, 6):
        wl = workloads.small_config(idx)
        enc = VisionEncoder(wl.desc, wl.weights)
        plans = [enc.plan([it]) for it in wl.items]
        seq = [enc.run(p).float().cpu().numpy() for p in plans]
        for _ in range(2):
            pip = enc.run_pipelined(plans)
            torch.cuda.synchronize()
            for a, b in zip(seq, pip):
                assert np.array_equal(a, b.float().cpu().numpy())
        whole = enc.plan(wl.items)
        out = enc.run(whole).float().cpu().numpy()
        m2 = wl.desc.merge ** 2
        r0 = 0
        for a, plan in zip(seq, plans):
            assert plan.info.n_out_tokens == a.shape[0] == plan.info.n_tokens // m2
            assert_tokens_close(out[r0:r0 + a.shape[0]], a, 2e-2, 0.999, f"{wl.name} request rows")
            r0 += a.shape[0]
        assert r0 == out.shape[0]


@pytest.mark.parametrize("std", [0.02, 0.08])
def test_long_segments_take_the_norm_bounded_attention_path(std):
    """Segments of 8192 and 2304 tokens make the library compute key norms and run attention without a softmax
    reference where the bound allows it; the result must not depend on which copy of the kernel ran."""
    desc = workloads.qwen_like_desc(layers=2, d=320, heads=4, mlp=640, out_dim=192, max_grid=48)
    rng = np.random.default_rng(9)
    items = [workloads.Item(2, 16, 448, 448, 448, 448, workloads.random_frames(rng, 16, 448, 448)),
             workloads.Item(1, 1, 672, 672, 672, 672, workloads.random_frames(rng, 1, 672, 672))]
    wl = workloads.Workload("long", desc, items, workloads.make_weights(desc, 31, std=std, random_affine=True))
    ref = oracle.run(wl, workers=4)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert pl.cu_seqlens == [0, 8192, 8192 + 2304]
    assert B.tcmv_plan_key_norms(pl.handle, 0) > 0
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, "long segments hidden")
    assert_tokens_close(out.float().cpu().numpy(), ref["out"], 2e-2, 0.999, "long segments out")


@pytest.mark.parametrize("heads,dh,side,n,kernel", [
    (2, 64, (57, 57), 1, "128x128"), (6, 64, (37, 87), 1, "128x128 k/2"), (18, 64, (36, 33), 2, "192x256"), (4, 64, (35, 38), 6, "256x128"),
    (8, 64, (39, 36), 4, "256x256 persistent"), (4, 80, (96, 43), 2, "256x160"), (8, 80, (40, 33), 6, "256x320 persistent")])
@pytest.mark.parametrize("spread", [0.36, 1.43])
@pytest.mark.parametrize("pos", ["rope2d", "none"])
def test_key_norms_from_the_write_out_of_every_kernel_that_computes_them(heads, dh, side, n, kernel, spread, pos):
    """Two layers with rotary positions or without (kernels of their own), RMSNorm and gated MLP, ragged rows: the QKV product squares and sums the keys on
    their way out, into alternating tables that the attention of the layer before clears.  Weights of standard deviation
    spread / sqrt(d) give queries and keys of standard deviation `spread` at every width, scores of spread^2 (bounded by
    the norms, or not).  Queries and keys are rounded to bf16 (2^-9 of each), which moves a score by about 2^-8 of itself and
    its probability by as much: 1 % for scores near 2, inside the bar; scores of 7 (spread 2.7) would miss it."""
    desc = workloads.ModelDesc(layers=2, d=heads * dh, heads=heads, mlp=128, patch=14, tpatch=1, merge=1, pos=pos, norm="rms", gated=1)
    rng = np.random.default_rng(heads + dh)
    items = [workloads.Item(workloads.IMAGE, 1, 14 * side[0], 14 * side[1], 14 * side[0], 14 * side[1],
                            workloads.random_frames(rng, 1, 14 * side[0], 14 * side[1])) for _ in range(n)]
    wl = workloads.Workload("key_norms", desc, items, workloads.make_weights(desc, 32, std=spread / desc.d ** 0.5, random_affine=True))
    ref = oracle.run(wl, workers=4)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert B.tcmv_plan_key_norms(pl.handle, 0) == 2 and B.tcmv_plan_gemm_kernel(pl.handle, "qkv_gemm", 0) == kernel
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, kernel)


@pytest.mark.parametrize("dh", [32, 64, 72, 80, 96])
@pytest.mark.parametrize("spread", [0.36, 1.43])
@pytest.mark.parametrize("rows,grids", [
    (64, [(1, 1), (3, 21), (8, 8), (5, 13), (8, 16), (12, 16), (10, 25), (16, 16)]),        # at most one tile of keys for a group
    (128, [(1, 1), (5, 8), (8, 8), (5, 13), (8, 16), (3, 43), (1, 193), (20, 35)])])        # groups of 0 to 6 tiles, the last one ragged
def test_attention_of_small_requests_with_the_keys_split_over_groups_of_waves(rows, grids, spread, dh):
    """One to 700 keys shared by four or two groups of waves, some of them without keys; scores up to about spread^2 (see above)."""
    heads = 8 if dh == 72 else 4 if dh == 80 else 2          # the width of the model is a multiple of 64
    desc = workloads.ModelDesc(layers=1, d=heads * dh, heads=heads, mlp=128, patch=14, tpatch=1, merge=1)
    rng = np.random.default_rng(rows + dh)
    items = [workloads.Item(workloads.IMAGE, 1, 14 * h, 14 * w, 14 * h, 14 * w, workloads.random_frames(rng, 1, 14 * h, 14 * w)) for h, w in grids]
    wl = workloads.Workload("key_groups", desc, items, workloads.make_weights(desc, 34, std=spread / desc.d ** 0.5, random_affine=True))
    ref = oracle.run(wl, workers=4)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert B.tcmv_op_attention_rows(B.TCMV_BF16, pl.cu_seqlens, heads * (enc.dh_lib or dh), heads) == rows and B.tcmv_plan_key_norms(pl.handle, 0) == 0
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, "key groups")


@pytest.mark.parametrize("dh", [32, 64, 80, 96])
@pytest.mark.parametrize("rows,grids", [
    (64, [(1, 1), (1, 5), (5, 8), (8, 8), (16, 16)]), (128, [(1, 1), (1, 5), (8, 16), (20, 35)]), (128, [(24, 24)] * 28 + [(1, 1)])])
def test_attention_over_equal_keys_gives_their_value(rows, grids, dh):
    """Pictures of one colour: all keys of a segment score alike, so every probability is 1 against the largest score (to
    1e-6, which bf16 rounds away) and the output is the value, whatever the queries and keys are: bit for bit what the
    model with zero queries and keys computes.  One key alone is the smallest case."""
    heads = 4 if dh == 80 else 8 if len(grids) > 8 else 2
    desc = workloads.ModelDesc(layers=1, d=heads * dh, heads=heads, mlp=128, patch=14, tpatch=1, merge=1)
    items = [workloads.Item(workloads.IMAGE, 1, 14 * h, 14 * w, 14 * h, 14 * w, np.full((1, 14 * h, 14 * w, 3), 37 + 29 * i % 200, np.uint8))
             for i, (h, w) in enumerate(grids)]
    res = []
    for qk in (1, 0):
        w = workloads.make_weights(desc, 38, std=1.43 / desc.d ** 0.5, random_affine=True)
        w["l0.w_qkv"][:2 * desc.d] *= qk
        w["l0.b_qkv"][:2 * desc.d] *= qk
        enc, pl, patches, hidden, out = run_gpu(workloads.Workload("equal_keys", desc, items, w))
        assert B.tcmv_op_attention_rows(B.TCMV_BF16, pl.cu_seqlens, desc.d, heads) == rows and B.tcmv_plan_key_norms(pl.handle, 0) == 0
        res.append(hidden)
    assert torch.equal(*res)


@pytest.mark.parametrize("grid,n,heads,rows", [((16, 16), 1, 4, 64), ((20, 35), 1, 4, 128), ((24, 24), 16, 8, 128)])
@pytest.mark.parametrize("border", [0.3, 0.8])
def test_softmax_reference_moves_between_keys(grid, n, heads, rows, border):
    """Pictures whose lower part is white under a black one: two kinds of tokens, whose scores differ by far more than 2^8
    in some heads, so the reference that scores start from moves when the first white keys arrive (or must not, where the
    black ones score higher).  The tokens of a kind are equal, so a rounded score moves all their probabilities alike and
    the outputs stay a mixture of two values: the scores (up to 17, 4 to 32 apart) may be larger than in the tests above."""
    h, w = grid
    desc = workloads.ModelDesc(layers=1, d=heads * 80, heads=heads, mlp=128, patch=14, tpatch=1, merge=1)
    items = []
    for _ in range(n):
        f = np.zeros((1, 14 * h, 14 * w, 3), np.uint8)
        f[:, 14 * int(h * border):] = 255
        items.append(workloads.Item(workloads.IMAGE, 1, 14 * h, 14 * w, 14 * h, 14 * w, f))
    wl = workloads.Workload("two_kinds", desc, items, workloads.make_weights(desc, 36, std=2.5 / desc.d ** 0.5, random_affine=True))
    ref = oracle.run(wl, workers=4)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert B.tcmv_op_attention_rows(B.TCMV_BF16, pl.cu_seqlens, heads * 80, heads) == rows and B.tcmv_plan_key_norms(pl.handle, 0) == 0
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, "two kinds of tokens")


def _first_attention(wl):
    """Queries, keys and values of the first layer and the weights of its softmax in log2 units, by the reference."""
    res = oracle.run(wl, stages=("preprocess",))
    d, dh, g = wl.desc.d, wl.desc.d // wl.desc.heads, lambda n: wl.weights["l0." + n].astype(np.float64)
    x = oe.norm(wl.desc, oe.embed(res["patches"], res["grids"], wl.desc, wl.weights), g("ln1_g"), g("ln1_b"))
    qkv = x @ g("w_qkv").T + g("b_qkv")
    q, k, v = (qkv[:, i * d:(i + 1) * d].reshape(-1, wl.desc.heads, dh).transpose(1, 0, 2) for i in range(3))
    return q @ k.transpose(0, 2, 1) * (np.log2(np.e) / dh ** 0.5), v


@pytest.mark.parametrize("heads,dh", [(4, 64), (4, 80), (2, 96)])
@pytest.mark.parametrize("row", [2, 6, 10, 14])
def test_softmax_reference_moves_inside_a_group_of_keys(row, heads, dh):
    """256 keys, a tile of 64 for each of four groups of waves, black above the given picture row and white below it: the border
    lies between the two blocks of 32 keys of one group, whose reference has to move there, with what it has summed by then;
    the groups behind it start from the reference of the black keys and move before they begin.  Where the white keys score
    higher, by more than the 8 that leave a reference alone, sums that do not move along would give the black keys of that
    group as much weight as the white ones: an error that this bar sees."""
    desc = workloads.ModelDesc(layers=1, d=heads * dh, heads=heads, mlp=128, patch=14, tpatch=1, merge=1)
    f = np.zeros((1, 224, 224, 3), np.uint8)
    f[:, 14 * row:] = 255
    wl = workloads.Workload("two_kinds", desc, [workloads.Item(workloads.IMAGE, 1, 224, 224, 224, 224, f)],
                            workloads.make_weights(desc, 36, std=2.5 / desc.d ** 0.5, random_affine=True))
    s, v = _first_attention(wl)
    b = 16 * row                                             # the first white key; black ones from b - 32 on share its tile
    rise = s[:, :, b:b + 32].max(2) - s[:, :, b - 32:b].max(2)
    moved = rise > 9
    assert b % 64 == 32 and moved.any() and (rise < -9).any()
    p = np.exp2(s - s.max(2, keepdims=True))
    right = (p / p.sum(2, keepdims=True)) @ v
    p[:, :, b - 32:b] = np.where(moved[:, :, None], 1.0, p[:, :, b - 32:b])
    wrong = (p / p.sum(2, keepdims=True)) @ v
    assert np.abs(wrong - right).max() > 0.1 * np.abs(right).max()
    ref = oracle.run(wl, workers=4)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert B.tcmv_op_attention_rows(B.TCMV_BF16, pl.cu_seqlens, heads * dh, heads) == 64
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, "two kinds of tokens in a tile")


# colours of a picture's patches: what the scores of its keys become in the first head
_PLAIN, _LIGHT, _MINUS_INF, _PLUS_INF = (0, 0, 0), (255, 255, 255), (0, 255, 0), (255, 0, 0)


def _infinite_scores_model(heads, dh):
    """One layer in which the key of a red patch has +inf in its first element, of a green one -inf, of a black or white one 0,
    and every query has a positive number there (first head; the others are ordinary).  Elements 0 and 1 of the
    embedding are the means of the red and green channels, the key element is 2^126 times their difference behind the norm."""
    desc = workloads.ModelDesc(layers=1, d=heads * dh, heads=heads, mlp=128, patch=14, tpatch=1, merge=1)
    w = workloads.make_weights(desc, 39, std=1.0 / desc.d ** 0.5, random_affine=True)
    w["w_pe"] = np.random.default_rng(7).normal(0, 0.01, w["w_pe"].shape).astype(np.float32)
    w["w_pe"] = workloads.snap_to_bf16_grid(w["w_pe"])
    channel = oracle.run(workloads.Workload("channels", desc, [workloads.Item(workloads.IMAGE, 1, 14, 14, 14, 14, np.array([[[255, 0, 0]]], np.uint8)
                         .repeat(14, 0).repeat(14, 1)[None])], w), stages=("preprocess",))["patches"][0][0]
    red = channel > 0
    green = oracle.run(workloads.Workload("channels", desc, [workloads.Item(workloads.IMAGE, 1, 14, 14, 14, 14, np.array([[[0, 255, 0]]], np.uint8)
                       .repeat(14, 0).repeat(14, 1)[None])], w), stages=("preprocess",))["patches"][0][0] > 0
    assert red.sum() == green.sum() == 196
    w["w_pe"][:2] = 0
    w["w_pe"][0, red] = w["w_pe"][1, green] = 2.0 ** -6
    w["b_pe"] = np.random.default_rng(8).normal(0, 1, desc.d).astype(np.float32)
    w["b_pe"][:2] = 0
    w["l0.ln1_g"][:2], w["l0.ln1_b"][:2] = 1, 0
    w["l0.w_qkv"][0] = 0                                     # first element of the first query: a bias
    w["l0.b_qkv"][0] = 1
    w["l0.w_qkv"][desc.d] = 0                                # of the first key
    w["l0.w_qkv"][desc.d, 0], w["l0.w_qkv"][desc.d, 1] = 2.0 ** 126, -2.0 ** 126
    w["l0.b_qkv"][desc.d] = 0
    return desc, w


def _picture(h, w, rng, *runs):
    """Patches black or white at random, then (first key, last key, colour) runs."""
    c = np.where(rng.integers(0, 2, (h * w, 1)) > 0, np.array(_LIGHT), np.array(_PLAIN)).astype(np.uint8)
    for a, b, colour in runs:
        c[a:b] = colour
    return workloads.Item(workloads.IMAGE, 1, 14 * h, 14 * w, 14 * h, 14 * w, c.reshape(h, w, 3).repeat(14, 0).repeat(14, 1)[None])


@pytest.mark.parametrize("heads,dh", [(2, 64), (4, 80)])
@pytest.mark.parametrize("rows,h,w,more", [(64, 16, 16, 0), (128, 20, 35, 0), (128, 24, 24, 12)])
def test_attention_with_infinite_scores(rows, h, w, more, heads, dh):
    """Keys that score -inf weigh nothing wherever they lie (the first keys, a whole tile, a whole group of waves' keys, all but
    one); where all keys score -inf, or one +inf, softmax has no value and the segment's rows are NaN.  The other
    segments of the launch are what they are without them."""
    desc, wts = _infinite_scores_model(heads, dh)
    rng = np.random.default_rng(rows + h)
    n, half = h * w, (h * w + 127) // 128 * 64                # keys of the first of two groups, in whole tiles
    items = [_picture(h, w, rng, (0, 40, _MINUS_INF)), _picture(h, w, rng, (0, 64, _MINUS_INF)), _picture(h, w, rng, (64, 128, _MINUS_INF)),
             _picture(h, w, rng, (0, half, _MINUS_INF)), _picture(h, w, rng, (half, n, _MINUS_INF)), _picture(h, w, rng, (0, 77, _MINUS_INF), (78, n, _MINUS_INF)),
             _picture(h, w, rng), _picture(h, w, rng, (0, n, _MINUS_INF)), _picture(h, w, rng, (5, 6, _PLUS_INF)), _picture(h, w, rng, (n - 1, n, _PLUS_INF))]
    items += [_picture(h, w, rng, (32 * i, 32 * i + 48, _MINUS_INF)) for i in range(more)]
    wl = workloads.Workload("infinities", desc, items, wts)
    ref = oracle.run(wl, workers=4)["hidden"]                 # 64-bit numbers hold what is infinite on the GPU
    pre = oracle.run(wl, stages=("preprocess",))
    x = oe.embed(pre["patches"], pre["grids"], desc, wts)
    ln = oe.layernorm(x, wts["l0.ln1_g"].astype(np.float64), wts["l0.ln1_b"].astype(np.float64), desc.ln_eps)[:, :2]
    # each of the two products is finite in 32 bits, their difference of a coloured patch is not
    assert np.all(np.abs(ln) < 3.9) and np.all((ln[:, 0] == ln[:, 1]) | (np.abs(ln[:, 0] - ln[:, 1]) > 4.1))
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert B.tcmv_op_attention_rows(B.TCMV_BF16, pl.cu_seqlens, heads * dh, heads) == rows and B.tcmv_plan_key_norms(pl.handle, 0) == 0
    got = hidden.cpu().numpy()
    for i, (a, b) in enumerate(zip(pl.cu_seqlens, pl.cu_seqlens[1:])):
        if 7 <= i <= 9:
            assert np.isnan(got[a:b]).all(), i
        else:
            assert_tokens_close(got[a:b], ref[a:b], 2e-2, 0.999, f"segment {i}")


@pytest.mark.parametrize("pos", ["rope2d", "none"])
def test_qkv_product_in_whole_rounds_and_the_rest(pos):
    """Rotary factors, transposed values and key norms of the rows behind the whole rounds, which a second kernel computes."""
    test_key_norms_from_the_write_out_of_every_kernel_that_computes_them(16, 80, (33, 33), 6, "256x320 persistent + 128x160", 0.36, pos)


@pytest.mark.parametrize("pos", ["sep2d", "learned1d"])
def test_patch_embedding_in_whole_rounds_and_the_rest(pos):
    """The serving batch's 16656 patches at full width: 13056 in whole rounds of tiles, the rest on another kernel that scatters
    its rows and reads its positions from where the first stopped.  No layers behind it: every row is the fp32 sum itself."""
    desc = workloads.ModelDesc(layers=0, d=1280, heads=16, mlp=128, patch=14, tpatch=2, merge=2 if pos == "sep2d" else 1, pos=pos, max_pos=4300)
    rng = np.random.default_rng(47)
    sizes = [(1, 56, 64), (2, 48, 44), (1, 60, 60), (1, 40, 66), (6, 28, 12), (1, 20, 28), (1, 4, 8)]    # frames / 2 for videos, patches
    items = []
    for t, h, w in sizes:
        n = 2 * t if t > 1 else 1
        items.append(workloads.Item(workloads.VIDEO if t > 1 else workloads.IMAGE, n, 14 * h, 14 * w, 14 * h, 14 * w, workloads.random_frames(rng, n, 14 * h, 14 * w)))
    wl = workloads.Workload("embedding", desc, items, workloads.make_weights(desc, 40, random_affine=True))
    ref = oracle.run(wl, workers=4)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert B.tcmv_plan_gemm_kernel(pl.handle, "embed_gemm") == "256x256 persistent + 128x160"
    assert np.abs(hidden.cpu().numpy() - ref["hidden"]).max() <= 1e-4 * max(1.0, np.abs(ref["hidden"]).max())


def test_rows_behind_whole_rounds_in_slices_of_k():
    """fc2 of 13440 rows: 13056 in whole rounds of tiles, the rest in four slices of k that wait in the buffer of the queries and
    keys; run twice, equal bit for bit."""
    desc = workloads.ModelDesc(layers=1, d=1600, heads=25, mlp=2304, patch=14, tpatch=1, merge=1)
    rng = np.random.default_rng(41)
    items = [workloads.Item(workloads.IMAGE, 1, 392, 336, 392, 336, workloads.random_frames(rng, 1, 392, 336)) for _ in range(20)]
    wl = workloads.Workload("rest_in_slices", desc, items, workloads.make_weights(desc, 35, random_affine=True))
    ref = oracle.run(wl, workers=4)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert B.tcmv_plan_gemm_kernel(pl.handle, "fc2_gemm", 0) == "256x320 persistent + 64x64 slices"
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, "slices behind whole rounds")
    again = enc.encode(pl, patches)
    torch.cuda.synchronize()
    assert torch.equal(hidden, again)


def test_attention_too_wide_for_the_pass_over_the_keys():
    """120 heads (of 8, padded to 32): 3840 columns of keys are more than the pass over the keys holds; 1156 keys per query
    would ask for it."""
    desc = workloads.ModelDesc(layers=2, d=960, heads=120, mlp=256, patch=14, tpatch=1, merge=1)
    rng = np.random.default_rng(120)
    items = [workloads.Item(workloads.IMAGE, 1, 476, 476, 476, 476, workloads.random_frames(rng, 1, 476, 476))]
    wl = workloads.Workload("wide", desc, items, workloads.make_weights(desc, 33, random_affine=True))
    ref = oracle.run(wl, workers=4)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert B.tcmv_plan_key_norms(pl.handle, 0) == 0
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, "wide attention")


@pytest.mark.parametrize("dh", [80, 64])
def test_windows_of_up_to_64_tokens_with_ragged_edges(dh):
    """Windows of 8 x 8 patches on grids that are not multiples of 8: window sizes 64, 48, 32, 24, 16, 8 ... in
    one batch, every layer windowed (the short-window attention kernel: second wave idle below 33 tokens, keys
    masked beyond the window), then with every second layer over the whole request."""
    rng = np.random.default_rng(31)
    sizes = [(168, 140), (196, 252), (224, 224), (112, 28), (28, 364)]      # patch grids 12x10, 14x18, 16x16, 8x2, 2x26
    items = [workloads.Item(workloads.IMAGE, 1, h, w, h, w, workloads.random_frames(rng, 1, h, w)) for h, w in sizes]
    items.insert(2, workloads.Item(workloads.VIDEO, 4, 140, 196, 140, 196, workloads.random_frames(rng, 4, 140, 196)))
    for full_every in (0, 2):
        desc = workloads.windowed_desc(layers=2, d=4 * dh, heads=4, mlp=640, out_dim=192, window=8, full_every=full_every)
        wl = workloads.Workload("ragged_windows", desc, items, workloads.make_weights(desc, 3100 + dh, random_affine=True))
        ref = oracle.run(wl)
        enc, pl, patches, hidden, out = run_gpu(wl)
        check_patches(wl, ref, patches)
        assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, f"ragged windows dh={dh} hidden")
        assert_tokens_close(out.float().cpu().numpy(), ref["out"], 2e-2, 0.999, f"ragged windows dh={dh} out")


def test_single_small_request_with_long_mlp_contraction():
    """One small request through a model whose fc2 contraction is long (mlp 2048 over 320 rows of tokens): the
    library computes that product in four slices of k and adds them in a fixed order.  Result within the usual
    bar, identical from run to run, and equal to what the same request gets inside a large batch (where the
    product is computed undivided) up to fp32 summation order."""
    rng = np.random.default_rng(41)
    desc = workloads.qwen_like_desc(layers=2, d=320, heads=4, mlp=2048, out_dim=192, max_grid=16)
    item = workloads.Item(workloads.IMAGE, 1, 224, 140, 224, 140, workloads.random_frames(rng, 1, 224, 140))
    wl = workloads.Workload("one_small_request", desc, [item], workloads.make_weights(desc, 4100, random_affine=True))
    ref = oracle.run(wl)
    enc, pl, patches, hidden, out = run_gpu(wl)
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, "single request hidden")
    assert_tokens_close(out.float().cpu().numpy(), ref["out"], 2e-2, 0.999, "single request out")
    again = enc.encode(pl, patches)
    torch.cuda.synchronize()
    assert torch.equal(hidden, again)
    # the same request as the first of a batch large enough for the undivided product
    others = [workloads.Item(workloads.IMAGE, 1, 224, 224, 224, 224, workloads.random_frames(rng, 1, 224, 224))
              for _ in range(40)]
    plb = enc.plan([item] + others)
    hb = enc.encode(plb, enc.preprocess(plb))
    torch.cuda.synchronize()
    n = hidden.shape[0]
    assert_tokens_close(hb[:n].cpu().numpy(), hidden.cpu().numpy().astype(np.float64), 2e-3, 0.99999, "batch vs alone")


@pytest.mark.parametrize("h,w,rms,final_ln", [(224, 224, 0, 0), (224, 224, 0, 1), (196, 252, 1, 0), (196, 252, 1, 1), (420, 504, 0, 1)])
def test_products_cut_along_k_and_added_by_the_norm(h, w, rms, final_ln):
    """One small image through full-width layers: the products that accumulate are computed in four slices of k, which
    the following norm (or, behind the last layer, a kernel of its own) adds to the residual stream; 256, 252 and 1080
    tokens (fc2 only), LayerNorm and RMSNorm, with and without a final norm."""
    import dataclasses
    if rms:
        desc = dataclasses.replace(workloads.windowed_desc(layers=2, d=1280, heads=16, mlp=5120, out_dim=0, window=8, full_every=2), merge=2)
    else:
        desc = workloads.qwen_like_desc(layers=2, d=1280, heads=16, mlp=5120, out_dim=0, max_grid=48)
    desc = dataclasses.replace(desc, final_ln=final_ln)
    rng = np.random.default_rng(h * w + rms + final_ln)
    items = [workloads.Item(workloads.IMAGE, 1, h, w, h, w, workloads.random_frames(rng, 1, h, w))]
    wl = workloads.Workload("slices", desc, items, workloads.make_weights(desc, 3, random_affine=True))
    for key, x in wl.weights.items():
        wl.weights[key] = workloads.snap_to_bf16_grid(x)
    ref = oracle.run(wl)
    _, pl, _, hidden, _ = run_gpu(wl)
    routes = [B.tcmv_plan_gemm_kernel(pl.handle, c, 0) for c in ("out_gemm", "fc2_gemm")]
    assert routes == (["64x64", "128x128 slices"] if h == 420 else ["64x64 slices"] * 2)
    assert_tokens_close(hidden.cpu().numpy(), ref["hidden"], 2e-2, 0.999, "hidden")
