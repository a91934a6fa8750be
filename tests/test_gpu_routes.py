"""GPU parity at the edges of the dispatch rules: the smallest and largest shapes of each kernel variant, ragged tiles,
workgroups that walk over several tiles and images.  Oracle, bar and protocol are those of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import test_gpu_block as block
import test_gpu_parity as base
from paper_2205_14756_amd import msla
from paper_2205_14756_amd import workloads as wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# long contractions: a workgroup walks two tiles that belong to different images (70 ragged tiles, 64 workgroups a channel
# block), 24 and 32 chunks of weights; one whose last head-branches are missing in some waves (33)
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(5, 512, 13, 33, 24, (5,)), (5, 512, 13, 33, 32, (5,)),
                                                  (2, 272, 9, 40, 11, (3, 5))])
def test_long_contraction_walks_tiles_of_several_images(dtype, B, C, H, W, heads, scales):
    print(f"routes: long contraction {dtype} {B}x{C}x{H}x{W} heads={heads}", flush=True)
    base.check_module(wk.random_module(41 + heads, dtype, B, C, H, W, heads, 16, scales), dtype, heads, 16, scales, stages=False)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
# H*W a multiple of 16 bytes' elements on no, on one and on every storage type; one partial tile, several tiles
@pytest.mark.parametrize("B,C,H,W", [(2, 32, 3, 5), (1, 48, 10, 10), (2, 80, 16, 9), (1, 64, 33, 67)])
def test_channel_planar_layout_equals_token_major_bit_for_bit(dtype, B, C, H, W):
    print(f"routes: planar {dtype} {B}x{C}x{H}x{W}", flush=True)
    t = wk.random_module(5 + H, dtype, B, C, H, W, C // 16, 16, (5,))
    x = base.dev(t["x"], dtype)
    wdw, wg = base.weights(t, dtype, (5,))
    w = (base.dev(t["w_qkv"], dtype), wdw, wg, base.dev(t["w_proj"], dtype))
    want = msla.msla_forward(x, *w, C // 16, 16, (5,))
    # (bytes around the planar result must stay as they are)
    room = torch.full((x.numel() + 64,), 7.0, dtype=x.dtype, device="cuda")
    out = room[32:32 + x.numel()].view(B, C, H, W)
    msla.msla_forward(x.permute(0, 3, 1, 2).contiguous(), *w, C // 16, 16, (5,), out=out, layout=msla.MSLA_NCHW)
    torch.cuda.synchronize()
    assert torch.equal(out.permute(0, 2, 3, 1), want)
    assert bool((room[:32] == 7.0).all()) and bool((room[32 + x.numel():] == 7.0).all())


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# heads of 32: few heads with many partial states each (their sum is split over waves), and one chunk only
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(1, 96, 45, 70, 3, (3, 5)), (1, 32, 4, 9, 1, (3,))])
def test_head_size_32_partial_state_sums(dtype, B, C, H, W, heads, scales):
    print(f"routes: head size 32 {dtype} {B}x{C}x{H}x{W}", flush=True)
    base.check_module(wk.random_module(61 + heads, dtype, B, C, H, W, heads, 32, scales), dtype, heads, 32, scales, stages=False)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
# 14 head-branches (the last quad half empty); one token; waves of several token groups, the last run shorter
@pytest.mark.parametrize("B,H,W,heads", [(1, 1, 1, 7), (3, 5, 7, 7), (2, 128, 129, 7)])
def test_core_writes_attention_rows(dtype, B, H, W, heads):
    print(f"routes: core {dtype} {B}x{H}x{W} heads={heads}", flush=True)
    t = wk.random_module(71 + H, dtype, B, 16 * heads, H, W, heads, 16, (3,))
    rng = np.random.default_rng(H)
    qkv = wk.round_to_dtype(rng.standard_normal((B, H, W, 48 * heads)), dtype)
    wdw, wg = base.weights(t, dtype, (3,))
    rows = B * H * W
    room = torch.full((rows + 1, 32 * heads), 7.0, dtype=base.TDT[dtype], device="cuda")
    msla.msla_core_forward(base.dev(qkv, dtype), wdw, wg, heads, 16, (3,), att=room[:rows].view(B, H, W, 32 * heads))
    torch.cuda.synchronize()
    assert bool((room[rows] == 7.0).all())
    # the states and the stored Q tokens the same call chain leaves, applied row by row in fp64 on the CPU: one rounding of
    # the result (unit roundoff u) on top of the 32-bit arithmetic of Eq. (3) and the state operands' 2^-16 (bf16 pairs)
    q_ms, kv = msla.msla_multiscale_state(base.dev(qkv, dtype), wdw, wg, heads, 16, (3,))
    q = np.maximum(base.host(q_ms).reshape(B, H * W, 2, heads, 16), 0.0)
    kv = base.host(kv)
    num = np.einsum("bnshe,bshef->bnshf", q, kv[..., :16])
    den = np.einsum("bnshe,bshe->bnsh", q, kv[..., 16])[..., None] + 1e-15
    ref = (num / den).reshape(rows, 32 * heads)
    u = {"f32": 2.0 ** -20, "f16": 2.0 ** -10.5, "bf16": 2.0 ** -7.9}[dtype]
    # Eq. (3) is a weighted mean of KV[e, :] / Ksum[e]: its rounding errors are relative to the largest of those
    hull = np.abs(kv[..., :16] / np.maximum(kv[..., 16:], 1e-30)).max(axis=(3, 4))
    bar = (u * np.broadcast_to(hull[:, None, :, :, None], num.shape)).reshape(rows, 32 * heads)
    assert (np.abs(base.host(room[:rows]) - ref) <= bar + 1e-12).all()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# in place, which the two launches take: blocks of 64 and of 128 tokens (as 4 x 32 and, the last, as 8 x 16), up to 128 and up to 256 output channels a workgroup; out
# of place, where one launch takes those of up to 256 channels, its blocks of 4 and of 8 rows; ragged columns and rows, channel
# groups past the output (48, 144), a hidden size that is no whole number of slabs, a narrow map, more than one group (272)
@pytest.mark.parametrize("B,C,H,W,hidden", [(1, 48, 5, 17, 80), (3, 48, 61, 130, 80), (2, 144, 7, 33, 144),
                                            (4, 144, 61, 113, 160), (2, 128, 50, 3, 128), (1, 272, 9, 18, 288),
                                            (6, 144, 61, 70, 64)])
def test_ffn_block_shapes(dtype, B, C, H, W, hidden):
    block.test_ffn(dtype, 1, B, C, H, W, hidden)
    block.test_ffn(dtype, 1, B, C, H, W, hidden, launches=2, in_place=True)


# fp32 projections and normalise-and-apply: 32, 64, 96, 128, 192 and 256 input channels (and the first beyond), 16 channels
# short of each; few and many tiles a workgroup, several images, 8, 16, 24, 32 and more head-branches, channel groups past
# the output
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(1, 16, 3, 5, 1, (5,)), (2, 48, 9, 33, 4, (3,)), (5, 64, 40, 41, 4, (5,)),
                                                  (2, 80, 7, 11, 8, (5,)), (3, 96, 30, 50, 6, (3, 5)), (1, 144, 6, 50, 9, (5,)),
                                                  (2, 208, 33, 47, 13, (5,)), (3, 256, 5, 21, 16, (5,)), (2, 272, 6, 21, 17, (5,))])
def test_fp32_weight_stationary_kernels(B, C, H, W, heads, scales):
    print(f"routes: fp32 {B}x{C}x{H}x{W} heads={heads}", flush=True)
    base.check_module(wk.random_module(91 + C, "f32", B, C, H, W, heads, 16, scales), "f32", heads, 16, scales)


def test_fp32_paired_heads_of_eight_keep_their_own_denominators():
    # two heads of 8 side by side in one state, keys of very different size: a denominator that mixed them would show
    t = wk.random_module(97, "f32", 2, 64, 12, 23, 8, 8, (3, 5))
    w = t["w_qkv"].reshape(8, 3, 8, 64).copy()
    w[1::2, 1] *= 100.0
    t["w_qkv"] = wk.round_to_dtype(w.reshape(192, 64), "f32")
    base.check_module(t, "f32", 8, 8, (3, 5), stages=False)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# a 3x3 and a 5x5 scale in one launch, image-head-chunk counts that are no multiple of 8, either order; with the copy of the raw Q
@pytest.mark.parametrize("B,H,W,heads,scales", [(1, 33, 40, 3, (3, 5)), (3, 20, 70, 5, (5, 3)), (1, 5, 4, 1, (3, 5))])
def test_paired_scales(dtype, B, H, W, heads, scales):
    base.test_multiscale_state_and_core(dtype, B, H, W, heads, scales)
    base.check_module(wk.random_module(17 + W, dtype, B, 16 * heads, H, W, heads, 16, scales), dtype, heads, 16, scales, stages=False)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# heads of 32, normalise-and-apply fused with the projection: 1, 2, 6, 12 and 16 head-branches (8 and 16 slots of weights),
# output channels that fill half a wave's pair of groups, a second channel group, tiles of several images in one workgroup;
# 18 head-branches: the separate kernels
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(1, 48, 3, 5, 1, ()), (3, 48, 5, 7, 1, (5,)), (5, 96, 40, 61, 3, (5,)),
                                                  (2, 272, 9, 40, 4, (3, 5)), (2, 512, 6, 11, 8, (5,)), (1, 192, 9, 10, 6, (3, 5))])
def test_head_size_32_fused_projection(dtype, B, C, H, W, heads, scales):
    print(f"routes: head size 32 fused {dtype} {B}x{C}x{H}x{W} heads={heads} scales={scales}", flush=True)
    base.check_module(wk.random_module(83 + C + H, dtype, B, C, H, W, heads, 32, scales), dtype, heads, 32, scales, stages=False)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
# the raw state of a map that holds Q, K and V side by side: three heads (one a workgroup), four, five (a second workgroup
# with one head), several chunks
@pytest.mark.parametrize("B,H,W,heads", [(2, 3, 7, 3), (1, 9, 11, 4), (2, 40, 33, 5)])
def test_raw_state_of_interleaved_heads(dtype, B, H, W, heads):
    base.test_multiscale_state_and_core(dtype, B, H, W, heads, ())


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# maps of few rows, many workgroups, in place: blocks of 4 x 32 tokens by up to 128 output channels; and by 256, one row short of a block
@pytest.mark.parametrize("B,C,H,W,hidden", [(40, 48, 3, 200, 80), (40, 144, 3, 200, 80)])
def test_ffn_blocks_of_flat_maps(dtype, B, C, H, W, hidden):
    block.test_ffn(dtype, 1, B, C, H, W, hidden)
    block.test_ffn(dtype, 1, B, C, H, W, hidden, launches=2, in_place=True)


# fp32 states: workgroups that walk 16 tiles of 8 x 32 tokens, and fewer, over a ragged map
@pytest.mark.parametrize("B,H,W,heads,scales", [(4, 64, 128, 64, (5,)), (6, 81, 100, 11, (3, 7))])
def test_fp32_states_take_one_rounding_a_tile(B, H, W, heads, scales):
    print(f"routes: fp32 states {B}x{H}x{W} heads={heads}", flush=True)
    t = wk.random_module(29 + H, "f32", 1, 16 * heads, 1, 1, heads, 16, scales)
    g = torch.Generator(device="cuda").manual_seed(H)
    qkv = torch.randn(B, H, W, 48 * heads, generator=g, device="cuda")
    wdw, wg = base.weights(t, "f32", scales)
    _, kv = msla.msla_multiscale_state(qkv, wdw, wg, heads, 16, scales)
    k, v = (qkv.view(B, H * W, heads, 3, 16)[:, :, :, i].double().permute(0, 2, 1, 3) for i in (1, 2))
    k = k.clamp(min=0)
    want = torch.cat([k.transpose(2, 3) @ v, k.sum(2).unsqueeze(3)], 3)
    d = kv[:, 0].double() - want
    err = float(d[..., :16].norm() / want[..., :16].norm())
    print(f"  relative error of the raw branch's KV {err:.2e}", flush=True)
    # Sums of n terms of either sign carry a relative error of about 0.6 u sqrt(n / 2), u = 2^-24: 16 matrix instructions a
    # tile and wave and up to 16 tiles, added separately, 0.6 u sqrt(8 + 8) = 1.4e-7; in one chain of 256, 4.0e-7 (of 176, 3.4e-7)
    assert err <= 2.0e-7
    assert float(d[..., 16].norm() / want[..., 16].norm()) <= 1.0e-7


# fp32 maps that fill the tiled forms' pieces: normalise-and-apply in pieces of 64 tokens (two images, ragged) and of 128, the
# Q/K/V projection tiled as well (all but the first)
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(3, 256, 61, 71, 16, ()), (1, 160, 127, 129, 10, (5,)), (2, 256, 127, 129, 16, ())])
def test_fp32_tiled_kernels_on_full_maps(B, C, H, W, heads, scales):
    print(f"routes: fp32 tiled {B}x{C}x{H}x{W} heads={heads}", flush=True)
    base.check_module(wk.random_module(101 + C, "f32", B, C, H, W, heads, 16, scales), "f32", heads, 16, scales, stages=False)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# long contractions beyond the few-token limit (more than 8 tile x channel-block pairs a compute unit), up to 384 channels: workgroups
# walk eight and more tiles over four images with ragged ends; 33, 48 and 64 head-branches (24, 24 and 32 chunks of weights)
@pytest.mark.parametrize("C,heads,scales", [(272, 11, (3, 5)), (384, 24, (5,)), (272, 32, (5,))])
def test_long_contraction_of_many_tokens(dtype, C, heads, scales):
    print(f"routes: long contraction, many tokens {dtype} 4x{C}x61x91 heads={heads}", flush=True)
    base.check_module(wk.random_module(51 + heads, dtype, 4, C, 61, 91, heads, 16, scales), dtype, heads, 16, scales, stages=False)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
# four heads a workgroup, which takes about a whole round of workgroups over the chip: 16 heads, 16 chunks; 11 heads (the
# last workgroup of an image's three one short), 12 chunks; ragged ends of both
@pytest.mark.parametrize("B,H,W,heads", [(4, 10, 101, 16), (7, 20, 37, 11)])
def test_raw_state_of_four_heads_a_workgroup(dtype, B, H, W, heads):
    base.test_multiscale_state_and_core(dtype, B, H, W, heads, ())


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# scales after the first, which have no raw branch, in launches of their own: matrix-core kernel (equal scales and a third one
# share no launch) and general kernel (7x7), on whole tiles and ragged ones
@pytest.mark.parametrize("B,H,W,heads,scales", [(1, 32, 64, 4, (5, 5)), (2, 21, 45, 3, (3, 3, 5)), (1, 32, 64, 4, (7, 7)),
                                                (2, 21, 45, 3, (5, 7, 7))])
def test_later_scales_in_launches_of_their_own(dtype, B, H, W, heads, scales):
    print(f"routes: later scales {dtype} {B}x{H}x{W} {scales}", flush=True)
    base.check_module(wk.random_module(23 + W, dtype, B, 16 * heads, H, W, heads, 16, scales), dtype, heads, 16, scales)


# fp32 products that fill the tiled form's pieces, whose contraction the weight-stationary form would pad; a ragged end
@pytest.mark.parametrize("n,c_in,c_out", [(16384, 160, 480), (16301, 144, 496)])
def test_fp32_linear_on_full_maps(n, c_in, c_out):
    base.test_linear("f32", n, c_in, c_out)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# one workgroup a tile of 8 x 32 tokens, Q, K and V computed there: 16, 48, 64, 80, 128, 144 and 192 input channels (the last step of
# 32 half empty in four of them), one and two scales in either order, several images, ragged tiles; one row of 33 tokens (fewer, as the one pixel,
# have no room for their partial states and keep the separate projection); with one scale 258 and 512 workgroups, the most there are, and 513; with
# two 256 and 258; then 208 channels (Q, K and V read)
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(1, 16, 1, 1, 1, (5,)), (1, 16, 1, 33, 1, (5,)), (1, 16, 1, 33, 1, (3, 5)),
                                                  (3, 48, 9, 33, 3, (3,)), (2, 64, 8, 32, 4, (3, 5)),
                                                  (1, 80, 17, 31, 5, (5, 3)), (7, 128, 23, 40, 6, (5,)), (2, 144, 7, 65, 9, (3,)),
                                                  (1, 192, 40, 60, 12, (3, 5)), (2, 208, 21, 45, 13, (3, 5)), (1, 128, 64, 128, 8, (5,)),
                                                  (4, 64, 64, 128, 4, (5,)), (1, 48, 149, 285, 3, (5,)),
                                                  (2, 64, 62, 127, 4, (3, 5)), (1, 48, 8, 32 * 43, 6, (3, 5)), (1, 48, 8, 32 * 43, 6, (5,))])
def test_small_maps(dtype, B, C, H, W, heads, scales):
    print(f"routes: small map {dtype} {B}x{C}x{H}x{W} heads={heads} scales={scales}", flush=True)
    base.check_module(wk.random_module(37 + C + H, dtype, B, C, H, W, heads, 16, scales), dtype, heads, 16, scales)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(2, 80, 19, 45, 5, (5,)), (1, 128, 33, 70, 8, (3, 5)), (3, 192, 9, 32, 4, (3,))])
def test_small_map_stages_equal_the_complete_call(dtype, B, C, H, W, heads, scales):
    # one stage after the other, on a workspace of other contents, and the last two on what a complete call left
    print(f"routes: small map, stages {dtype} {B}x{C}x{H}x{W}", flush=True)
    t = wk.random_module(3 + H, dtype, B, C, H, W, heads, 16, scales)
    wdw, wg = base.weights(t, dtype, scales)
    args = (base.dev(t["x"], dtype), base.dev(t["w_qkv"], dtype), wdw, wg, base.dev(t["w_proj"], dtype), heads, 16, scales)
    # (bytes around the result and behind the workspace must stay as they are)
    n = msla.msla_workspace_bytes(B, C, H, W, heads, 16, scales, base.TDT[dtype])
    ws = torch.full((n + 256,), 77, dtype=torch.uint8, device="cuda")
    room = torch.full((B * H * W + 2, C), 7.0, dtype=base.TDT[dtype], device="cuda")
    out = room[1:-1].view(B, H, W, C)
    msla.msla_forward(*args, out=out, workspace=ws[:n])
    want = out.clone()
    stages = (msla.MSLA_OPT_STAGE_PROJECT, msla.MSLA_OPT_STAGE_AGGREGATE, msla.MSLA_OPT_STAGE_FINALIZE, msla.MSLA_OPT_STAGE_APPLY)
    for left in (2, 0):
        out.fill_(0.0)
        if left == 0:
            ws[:n] = 99
        for s in stages[left:]:
            msla.msla_forward(*args, out=out, workspace=ws[:n], options=s)
        assert torch.equal(out, want), f"from stage {left} on"
    assert bool((room[0] == 7.0).all()) and bool((room[-1] == 7.0).all()) and bool((ws[n:] == 77).all())


# fp32 maps of one tile a workgroup: a tile as two workgroups (128 tile-heads and fewer, three of them ragged), as one of twelve waves
# (144 and 256, not with 7x7), and the first shape past that; several scales (later ones have no raw branch)
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(1, 16, 1, 1, 1, (7,)), (2, 48, 19, 45, 3, (3, 5)), (3, 32, 9, 33, 2, (5, 7)),
                                                  (1, 32, 64, 64, 8, (5,)), (1, 32, 61, 63, 9, (3, 5)), (1, 32, 64, 64, 9, (7,)),
                                                  (2, 16, 64, 61, 8, (5, 3)), (1, 32, 64, 64, 17, (5,))])
def test_fp32_small_maps(B, C, H, W, heads, scales):
    print(f"routes: fp32 small {B}x{C}x{H}x{W} heads={heads} scales={scales}", flush=True)
    base.check_module(wk.random_module(43 + W + heads, "f32", B, C, H, W, heads, 16, scales), "f32", heads, 16, scales)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# heads of 32, depthwise on the matrix cores: one token, tiles one short of and one past 16 x 32, workgroups that walk two tiles with a ragged
# end and an image count that leaves the last one empty, two scales in either order (the second without the raw branch); with a 7x7
# scale beside it (chunks counted for the other kernel, some of them without a tile)
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(1, 32, 1, 1, 1, (5,)), (2, 64, 15, 31, 2, (3,)), (1, 96, 17, 33, 3, (5,)),
                                                  (16, 64, 47, 95, 2, (5, 3)), (3, 160, 33, 64, 5, (3, 5)), (1, 32, 70, 100, 1, (3, 7)),
                                                  (2, 64, 16, 32, 2, (7, 5))])
def test_head_size_32_on_the_matrix_cores(dtype, B, C, H, W, heads, scales):
    print(f"routes: head size 32 {dtype} {B}x{C}x{H}x{W} heads={heads} scales={scales}", flush=True)
    base.check_module(wk.random_module(59 + C + H, dtype, B, C, H, W, heads, 32, scales), dtype, heads, 32, scales, stages=False)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# heads of 32, the state's operands in three parts (four 32-token tiles a workgroup and more, some of two images): 2 and 10 head-branches
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(3, 32, 100, 91, 1, (5,)), (3, 160, 100, 91, 5, (3,))])
def test_head_size_32_states_in_parts(dtype, B, C, H, W, heads, scales):
    print(f"routes: head size 32, states in parts {dtype} {B}x{C}x{H}x{W}", flush=True)
    base.check_module(wk.random_module(67 + C, dtype, B, C, H, W, heads, 32, scales), dtype, heads, 32, scales, stages=False)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# contractions of more than 1024 slots in parts of 768: 1040 and 1536 slots, 1600 (a third part of 64), 4096 (the last that takes it; a sixth
# part of 256) and 4112; ragged tiles of several images, channels past the output; workgroups that walk two tiles (70 of five images for 64 workgroups a
# channel block, 128 of one), and the first tile past that
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(2, 272, 5, 13, 65, ()), (3, 512, 7, 19, 32, (3, 5)), (1, 400, 6, 11, 25, (3, 5, 7)),
                                                  (1, 144, 3, 7, 128, (5,)), (1, 144, 3, 7, 257, ()), (5, 512, 13, 33, 66, ()),
                                                  (1, 448, 61, 67, 23, (3, 5)), (1, 448, 64, 64, 22, (3, 5)), (1, 448, 129, 32, 22, (3, 5))])
def test_long_contraction_in_parts(dtype, B, C, H, W, heads, scales):
    print(f"routes: long contraction in parts {dtype} {B}x{C}x{H}x{W} heads={heads} scales={scales}", flush=True)
    base.check_module(wk.random_module(73 + heads, dtype, B, C, H, W, heads, 16, scales), dtype, heads, 16, scales, stages=False)


# ... with the residual of the block: 1088 slots, one tile a workgroup; 1152, two.  The second in fp16 only: the block's bar is 5e-3 of its largest
# value, and in bf16 the two roundings of a value next to that, of x + module and of the result, are up to 2^-8 = 3.9e-3 of it each, so among a
# million values some miss it whatever the route (5.2e-3 with the tiled kernel too)
@pytest.mark.parametrize("dtype,B,C,H,W,heads,scales", [("f16", 1, 272, 9, 17, 34, (5,)), ("bf16", 1, 272, 9, 17, 34, (5,)),
                                                        ("f16", 5, 512, 13, 33, 24, (3, 5))])
def test_long_contraction_in_parts_of_a_block(dtype, B, C, H, W, heads, scales):
    block.test_block(dtype, B, C, H, W, heads, scales, C, 1)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# more than 128 channels on few tokens, in place: channel blocks of 128 (two, the second short; three; 256 blocks in all), and one block past a round
@pytest.mark.parametrize("B,C,H,W,hidden", [(1, 144, 5, 17, 80), (2, 272, 9, 18, 96), (2, 160, 32, 128, 64), (1, 144, 43, 192, 64)])
def test_ffn_channel_blocks_of_small_maps(dtype, B, C, H, W, hidden):
    block.test_ffn(dtype, 1, B, C, H, W, hidden)
    block.test_ffn(dtype, 1, B, C, H, W, hidden, launches=2, in_place=True)


def test_small_map_keeps_an_overflow_to_its_own_token():
    # one token's Q overflows fp16 in every head; its K and V stay small, so no other token's row may notice
    B, C, H, W, heads = 1, 64, 9, 33, 4
    t = wk.random_module(19, "f16", B, C, H, W, heads, 16, ())
    x, w = t["x"].copy(), t["w_qkv"].reshape(heads, 3, 16, C).copy()
    x[..., 0] = 0.0
    w[:, 0, :, 0], w[:, 1:, :, 0] = 8.0, 0.0
    rng = np.random.default_rng(5)
    dw = np.zeros((48 * heads, 5, 5))
    dw[:, 2, 2] = 1.0                                   # (the aggregated branch is the raw one: nothing spreads over the filter's taps)
    gp = rng.standard_normal((48 * heads, 16)) / 4.0
    w_proj = np.concatenate([rng.standard_normal((C, 16 * heads)) / 8.0, np.zeros((C, 16 * heads))], 1)      # ... and is left out
    dev = lambda a: base.dev(np.ascontiguousarray(a), "f16")
    def rows(big):
        x[0, 4, 7, 0] = big
        out = msla.msla_forward(dev(x), dev(w.reshape(48 * heads, C)), dev(dw.reshape(-1)), dev(gp[None]), dev(w_proj), heads, 16, (5,))
        return np.delete(base.host(out).reshape(H * W, C), 4 * W + 7, 0)

    want, got = rows(0.0), rows(6.0e4)
    assert np.isfinite(want).all() and np.array_equal(got, want)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# one token's Q overflows in every channel, in the middle of a tile of 16 x 32 and at the corner of four: tokens in a filter's reach get nothing from
# that branch (their aggregated Q is not a number, which the rectifier takes for 0), all others are bit for bit what they were
@pytest.mark.parametrize("scales,at", [((5,), (6, 9)), ((3,), (16, 31)), ((3, 5), (15, 32)), ((5, 3), (0, 0)), ((5,), (35, 44))])
def test_head_size_32_keeps_an_overflow_in_the_filters_reach(dtype, scales, at):
    B, C, H, W, heads, Ct = 2, 64, 36, 45, 2, 64
    print(f"routes: head size 32, overflow {dtype} {scales} {at}", flush=True)
    t = wk.random_module(31, dtype, B, C, H, W, heads, 32, scales)
    x, w = t["x"].copy(), t["w_qkv"].reshape(heads, 3, 32, C).copy()
    x[..., 0] = 0.0
    w[:, 0, :, 0], w[:, 1:, :, 0] = 8.0, 0.0
    wdw, wg = base.weights(t, dtype, scales)

    def rows(big, branches):
        x[1, at[0], at[1], 0] = big
        wp = t["w_proj"].reshape(C, 1 + len(scales), Ct).copy()
        wp[:, [b for b in range(1 + len(scales)) if b not in branches]] = 0.0
        args = [base.dev(np.ascontiguousarray(a), dtype) for a in (x, w.reshape(3 * Ct, C), wp.reshape(C, -1))]
        return base.host(msla.msla_forward(args[0], args[1], wdw, wg, args[2], heads, 32, scales)).reshape(B, H, W, C)

    got, every = rows(6.0e4 if dtype == "f16" else 3.0e38, range(1 + len(scales))), range(1 + len(scales))
    dy, dx = np.abs(np.arange(H) - at[0])[:, None], np.abs(np.arange(W) - at[1])[None]
    reached = np.stack([np.full((H, W), False)] + [np.maximum(dy, dx) <= k // 2 for k in scales])
    for some in set(map(tuple, reached.reshape(len(reached), -1).T)):
        here = (reached == np.array(some)[:, None, None]).all(0)
        here[at] = False                                # (its own raw Q is infinite)
        want = rows(0.0, [b for b in every if not some[b]])
        assert np.isfinite(got[1][here]).all() and np.array_equal(got[1][here], want[1][here]), f"branches reached: {some}"
    assert np.array_equal(got[0], rows(0.0, every)[0])


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# heads of 32, states in parts (2 and 10 head-branches): rows of the state 2^-13, 2^-24, 2^-27 and 2^-36 of the largest, each from one token, and queries
# that see one or two of them.  Such a query's attention is that token's V (or their mean by weight), so what is left is one rounding of
# it: half a unit of the storage type, 2^-11 or 2^-8 of the value, and 1 % of that for the fp32 sums
@pytest.mark.parametrize("heads", [1, 5])
def test_head_size_32_states_in_parts_of_wide_range(dtype, heads):
    print(f"routes: head size 32, states of wide range {dtype} heads={heads}", flush=True)
    B, H, W, C, Ct = 3, 100, 91, 96 * heads, 32 * heads
    N, rng = H * W, np.random.default_rng(heads)
    q, k = -np.abs(rng.standard_normal((B, N, heads, 32))), np.zeros((B, N, heads, 32))
    v = np.sign(rng.standard_normal((B, N, heads, 32))) * (1.0 + np.abs(rng.standard_normal((B, N, heads, 32))))
    k[..., :16] = 1024.0                                # Ksum 2^23.2
    lone = {16 + i: 2.0 ** s for i, s in enumerate((10, -1, -4, -13))}
    for i, (e, size) in enumerate(lone.items()):
        k[:, 700 * i + 33, :, e] = size
    seen = [(16,), (17,), (18,), (19,), (17, 18), (18, 19), (0, 3)]
    for i, es in enumerate(seen):
        q[:, i::len(seen) + 1][..., list(es)] = 1.0
    q[:, len(seen)::len(seen) + 1][..., ::3] *= -1.0
    q, k, v = (wk.round_to_dtype(a, dtype) for a in (q, k, v))
    x = np.stack([q, k, v], 3).reshape(B, H, W, C)
    dw = np.zeros((3 * Ct, 3, 3))
    dw[:, 1, 1] = 1.0                                   # (the aggregated branch is the raw one)
    w_proj = np.zeros((C, 2 * Ct))
    w_proj[:2 * Ct] = np.eye(2 * Ct)
    dev = lambda a: base.dev(np.ascontiguousarray(a), dtype)
    got = base.host(msla.msla_forward(dev(x), dev(np.eye(C)), dev(dw.reshape(-1)), dev(np.tile(np.eye(32), (3 * heads, 1))[None]), dev(w_proj),
                                      heads, 32, (3,), 1e-15)).reshape(B, N, C)[..., :2 * Ct].reshape(B, N, 2, heads, 32)
    r, ks = np.maximum(q, 0.0), k.sum(1)
    num = np.einsum("bnhe,bhef->bnhf", r, np.einsum("bnhe,bnhf->bhef", k, v))
    want = num / (np.einsum("bnhe,bhe->bnh", r, ks) + 1e-15)[..., None]
    tol = 1.01 * {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype]
    for branch in range(2):
        for i, es in enumerate(seen[:-1]):
            rows = slice(i, None, len(seen) + 1)
            err = np.abs(got[:, rows, branch] - want[:, rows]) / np.abs(want[:, rows])
            assert err.max() <= tol, f"branch {branch}, channels {es}: {err.max():.3e}"
        err = np.linalg.norm(got[:, :, branch] - want) / np.linalg.norm(want)
        assert err <= tol, f"branch {branch}: {err:.3e}"


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# the core with two scales: four heads and 64 tiles an image, the last that the small tiles take, and 65; one, two and three heads (two and three: in bf16)
@pytest.mark.parametrize("B,H,W,heads,scales", [(1, 64, 250, 4, (3, 5)), (1, 100, 160, 4, (5, 3)), (2, 19, 45, 1, (3, 5)), (3, 9, 70, 2, (5, 3)),
                                                (1, 40, 33, 3, (3, 5))])
def test_core_of_small_maps_with_two_scales(dtype, B, H, W, heads, scales):
    base.test_multiscale_state_and_core(dtype, B, H, W, heads, scales)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# heads of 32, an image whose map of two heads spans more than 2 GiB: 3x3 and 5x5 on the vector ALUs, each with the raw branch and without.  What the
# projection takes of the first head is compared with a module of that head alone, whose map has half the size: a value may differ by four roundings (of
# the aggregated maps, the attention and the result), and by more at one token in a thousand (Eq. (3) is ill-posed at some)
@pytest.mark.parametrize("scales", [(3, 5), (5, 3)])
def test_head_size_32_maps_beyond_2_gib(dtype, scales):
    H = W = 2600
    print(f"routes: head size 32, beyond 2 GiB {dtype} {scales}", flush=True)
    assert H * W * 96 * 2 * 2 > 2 ** 31 > H * W * 96 * 2
    t = wk.random_module(83, dtype, 1, 16, 8, 8, 2, 32, scales)
    x = torch.randn(1, H, W, 16, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda").to(base.TDT[dtype])
    wdw, wg = base.weights(t, dtype, scales)
    w_qkv, w_proj = base.dev(t["w_qkv"], dtype), base.dev(t["w_proj"], dtype).view(16, 3, 2, 32).clone()
    w_proj[:, :, 1] = 0.0
    both = msla.msla_forward(x, w_qkv, wdw, wg, w_proj.view(16, 192), 2, 32, scales)
    at, first = 0, []
    for k in scales:
        first.append(wdw.reshape(-1)[at:at + 96 * k * k])
        at += 192 * k * k
    one = msla.msla_forward(x, w_qkv[:96].contiguous(), torch.cat(first), wg[:, :96].contiguous(), w_proj[:, :, 0].reshape(16, 96).contiguous(), 1, 32,
                            scales)
    torch.cuda.synchronize()
    rms = float(one.float().square().mean().sqrt())
    off = (both.float() - one.float()).abs() > 4 * {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype] * one.float().abs().clamp(min=rms)
    share = float(off.any(-1).float().mean())
    print(f"  tokens further off: {share:.2e}", flush=True)
    assert bool(torch.isfinite(both).all()) and share <= 1e-3


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("act", [0, 1])
# the FFN in one launch: up to 128 channels and beyond, blocks of 64 and of 128 tokens (the last two of each); one, two and three
# slabs of hidden channels, half a slab at the end, blocks cut off on both sides, images of less than a block
@pytest.mark.parametrize("B,C,H,W,hidden", [
    (1, 128, 4, 16, 32), (2, 16, 1, 1, 48), (1, 112, 5, 17, 80), (3, 80, 9, 31, 16),
    (9, 112, 12, 150, 112), (17, 128, 8, 256, 32),
    (1, 256, 4, 16, 64), (1, 144, 7, 19, 16), (2, 208, 13, 5, 304), (11, 240, 19, 47, 336),
    (12, 160, 12, 150, 48), (16, 256, 9, 128, 32),
])
def test_ffn_in_one_launch(dtype, act, B, C, H, W, hidden):
    block.test_ffn(dtype, act, B, C, H, W, hidden, launches=1)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# more than 256 channels, which are two launches always: 64-token blocks of 256 output channels, 128-token ones as 8 x 16 and as 4 x 32, a second channel
# group of 16, hidden sizes that are no whole number of slabs
@pytest.mark.parametrize("B,C,H,W,hidden", [(6, 272, 13, 61, 80), (40, 272, 31, 7, 48), (40, 272, 3, 200, 112), (3, 272, 37, 70, 48)])
def test_ffn_of_more_than_256_channels(dtype, B, C, H, W, hidden):
    block.test_ffn(dtype, 1, B, C, H, W, hidden, launches=2)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("act", [0, 1])
# in place is two launches; out of place, in 16 bits, one: blocks of 4 and of 8 rows, up to 128 channels and beyond, half a slab at the end
@pytest.mark.parametrize("B,C,H,W,hidden", [(2, 48, 9, 31, 80), (9, 112, 12, 150, 112), (2, 208, 13, 5, 304), (12, 160, 12, 150, 48)])
def test_ffn_in_place_and_in_one_launch_agree_bit_for_bit(dtype, act, B, C, H, W, hidden):
    print(f"routes: ffn in place {dtype} act={act} {B}x{C}x{H}x{W} hidden={hidden}", flush=True)
    rng = np.random.default_rng(C)
    y = base.dev(rng.standard_normal((B, H, W, C)) * np.exp2(rng.integers(-24, 3, (B, H, W, 1))), dtype)      # (tokens of subnormal fp16 among them)
    y[0, H // 2, W // 2, 3], y[-1, 0, 0, 5] = float("inf"), float("nan")
    w = wk.ffn_weights(77, dtype, C, hidden)
    args = (base.dev(w["w1"], dtype), base.dev(w["w_ffn_dw"], dtype), base.dev(w["w2"], dtype), act)
    out = msla.msla_ffn_forward(y, *args)
    same = msla.msla_ffn_forward(y, *args, out=y)
    torch.cuda.synchronize()
    assert same.data_ptr() == y.data_ptr()
    bits = {"f32": torch.int32, "f16": torch.int16, "bf16": torch.int16}[dtype]
    nan = torch.isnan(out)
    assert torch.equal(nan, torch.isnan(y)) and bool(nan.any()) and not bool(nan.all())
    assert torch.equal(out.view(bits)[~nan], y.view(bits)[~nan])


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# the two-launch form where it is the faster one: rows and columns that leave most of a block empty, many slabs in few blocks (narrow and wide)
@pytest.mark.parametrize("B,C,H,W,hidden", [(8, 48, 1, 1040, 416), (600, 64, 3, 3, 272), (3, 128, 4, 16, 1040), (1, 208, 9, 17, 832)])
def test_ffn_in_two_launches(dtype, B, C, H, W, hidden):
    block.test_ffn(dtype, 1, B, C, H, W, hidden, launches=2)


# a channel-planar x read by the projection itself: planes shorter than a run of 8 (4) tokens and than a tile, of whole runs and odd ones,
# tiles that span several images, one and several channels a thread, channels that do not fill the last one; fp32 at both sides
# of the rules on channels and tokens
@pytest.mark.parametrize("dtype,B,C,H,W,heads,scales", [
    (dt, *shape) for dt in ("f16", "bf16", "f32") for shape in [
        (7, 32, 1, 3, 1, ()), (5, 48, 1, 7, 2, (5,)), (3, 16, 5, 8, 1, ()), (2, 112, 11, 13, 6, (7,)), (1, 128, 9, 16, 7, ())]
] + [("f16", 2, 208, 17, 19, 12, (3,)), ("bf16", 1, 256, 6, 11, 13, ()), ("f16", 9, 144, 77, 31, 5, (5,)),
     ("f32", 2, 96, 9, 31, 5, (5,)), ("f32", 1, 128, 64, 129, 5, (5,)), ("f32", 2, 144, 9, 31, 6, ())])
def test_channel_planar_input(dtype, B, C, H, W, heads, scales):
    base.test_forward_channel_planar_layout(dtype, B, C, H, W, heads, 16, scales)


# a channel-planar out written by the output projection itself: images shorter than a tile and than a run of 8 (4) tokens, of whole
# runs and odd ones, output channels that do not fill a wave's block; each contraction length of the kernels that keep their weights,
# more than 32 head-branches (one and several parts), and the tiled form, which leaves it to a transposition
@pytest.mark.parametrize("dtype,B,C,H,W,heads,scales", [
    (dt, *shape) for dt in ("f16", "bf16", "f32") for shape in [
        (5, 16, 1, 3, 1, ()), (2, 144, 5, 7, 9, ()), (3, 48, 3, 11, 9, (5,)), (2, 176, 13, 8, 12, (3,)), (2, 80, 9, 15, 14, (5,)),
        (1, 272, 7, 9, 16, (5,)), (2, 208, 17, 5, 13, (3, 5)), (3, 256, 32, 33, 16, (3,))]
] + [("f16", 2, 144, 9, 31, 23, (3, 5)), ("bf16", 1, 352, 7, 13, 22, (3, 5)), ("f16", 1, 512, 6, 7, 32, (3, 5)), ("bf16", 1, 288, 5, 9, 36, (3, 5)),
     ("f32", 1, 256, 129, 128, 16, (5,)),
     # only one of the two maps left to a transposition, by tiles of several small images, by 26 heads and by fp16's widest form on a large map of odd rows; and both
     ("bf16", 131, 144, 9, 7, 9, ()), ("f16", 2, 192, 45, 101, 26, ()), ("f16", 1, 256, 113, 115, 14, (5,)), ("f16", 3, 256, 65, 67, 26, ())])
def test_channel_planar_output(dtype, B, C, H, W, heads, scales):
    base.test_forward_channel_planar_layout(dtype, B, C, H, W, heads, 16, scales)
