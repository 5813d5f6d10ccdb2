"""Tiles of the direct-to-LDS engine, of the general filter gradient and the stem's kernels at their edges: ragged pixel and
column tiles, half a 64-channel chunk, split reductions, one patch and many.  Every case names the kernel it has to reach;
parity against the oracle (whole tensors) within the storage types' bounds, as in the other parity tests."""
import ctypes

import numpy as np
import pytest
import torch

import gpu_util as U
import oracle
from paper_1810_01993_amd import synth
from paper_1810_01993_amd.layers import ConvLayer
from test_gpu_conv import check_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_1810_01993_amd import api as _api
    return _api


def L(name, N, H, W, C, K, R, stride=1, dil=1):
    return ConvLayer(name, N, H, W, C, K, R, R, stride, dil * (R // 2), dil, 1)


FWD, DGRAD, WGRAD = range(3)
CASES = [
    # forward and data gradient: each tile, each order
    (L("64x32", 1, 9, 24, 152, 24, 3, 2), "f16", FWD, "cmajor<64,32>"),
    (L("64x64", 1, 34, 11, 32, 40, 1), "bf16", FWD, "cmajor<64,64>"),
    (L("64x64.k64", 1, 15, 26, 160, 72, 1, 2), "f16", FWD, "cmajor.k64<64,64>"),
    (L("128x64.k64", 2, 100, 111, 208, 8, 1), "bf16", FWD, "cmajor.k64<128,64>"),
    (L("128x128", 1, 95, 61, 32, 136, 1), "f16", FWD, "cmajor<128,128>"),
    (L("128x128.k64", 2, 226, 74, 232, 240, 1), "bf16", FWD, "cmajor.k64<128,128>"),
    (L("256x128.k64", 2, 91, 187, 512, 72, 1), "f16", FWD, "cmajor.k64<256,128>"),
    (L("256x256", 1, 257, 112, 32, 264, 3, 1, 2), "bf16", FWD, "cmajor<256,256>"),
    (L("bt.64x32", 1, 9, 21, 8, 256, 3), "f16", DGRAD, "bt<64,32>"),
    (L("bt.64x64", 2, 91, 15, 8, 32, 1), "bf16", DGRAD, "bt<64,64>"),
    (L("bt.64x64.k64", 1, 11, 13, 24, 224, 1), "f16", DGRAD, "bt.k64<64,64>"),
    (L("bt.128x64.k64", 2, 85, 120, 16, 160, 1), "bf16", DGRAD, "bt.k64<128,64>"),
    (L("bt.256x128.k64", 1, 139, 244, 80, 512, 1), "f16", DGRAD, "bt.k64<256,128>"),
    (L("bt.128x128.k64", 1, 252, 282, 80, 288, 1), "bf16", DGRAD, "bt.k64<128,128>"),
    (L("bt.batch.256x256", 1, 216, 142, 480, 32, 3, 2), "f16", DGRAD, "batch_kernel.bt<256,256>"),
    (L("bt.batch.64x32", 1, 9, 30, 16, 296, 3, 2), "bf16", DGRAD, "batch_kernel.bt<64,32>"),
    (L("bt.batch.128x128", 1, 62, 109, 264, 32, 3, 2), "f16", DGRAD, "batch_kernel.bt<128,128>"),
    # reductions in ranges of whole and of half chunks, with the ordered reduce
    (L("split.64x64", 1, 17, 9, 552, 8, 3, 2), "f16", FWD, "splitk_reduce"),
    (L("split.64x64.wide", 1, 28, 19, 232, 128, 3, 1, 2), "bf16", FWD, "splitk_reduce"),
    (L("split.128x64", 2, 41, 53, 392, 16, 3, 1, 2), "f16", FWD, "splitk_reduce"),
    (L("split.bt", 1, 9, 19, 8, 200, 5), "bf16", DGRAD, "splitk_reduce"),
    # filter gradient: each tile; maps narrower than a step, stride, dilation, one row of pixels
    (L("w.128x128", 1, 12, 11, 96, 368, 3, 2), "f16", WGRAD, "wgrad_dma_kernel<128,128>"),
    (L("w.128x256", 2, 13, 51, 704, 144, 5, 2), "bf16", WGRAD, "wgrad_dma_kernel<128,256>"),
    (L("w.128x64", 1, 16, 13, 64, 176, 1, 2), "f16", WGRAD, "wgrad_dma_kernel<128,64>"),
    (L("w.64x128", 1, 147, 77, 80, 32, 3), "bf16", WGRAD, "wgrad_dma_kernel<64,128>"),
    (L("w.64x64", 1, 109, 289, 136, 32, 1), "f16", WGRAD, "wgrad_dma_kernel<64,64>"),
    (L("w.256x256", 1, 249, 58, 440, 136, 5, 2), "bf16", WGRAD, "wgrad_dma_kernel<256,256>"),
    # the stem's kernels: one pixel, ragged patches, one and two halves of the output channels, 8 and 16 channels
    (L("stem.c16.k64", 2, 61, 77, 16, 64, 7, 2), "f16", FWD, "stem_fwd_kernel<16>"),
    (L("stem.c16.k24", 1, 64, 96, 16, 24, 7, 2), "bf16", FWD, "stem_fwd_kernel<16>"),
    (L("stem.c8.k40", 1, 33, 130, 8, 40, 7, 2), "f16", FWD, "stem_fwd_kernel<8>"),
    (L("stem.c8.k8.pixel", 1, 1, 1, 8, 8, 7, 2), "bf16", FWD, "stem_fwd_kernel<8>"),
    (L("stem.w.c16.k64", 2, 61, 77, 16, 64, 7, 2), "bf16", WGRAD, "wgrad_stem_kernel<16>"),
    (L("stem.w.c16.k24", 1, 64, 96, 16, 24, 7, 2), "f16", WGRAD, "wgrad_stem_kernel<16>"),
    (L("stem.w.c8.k40", 1, 33, 130, 8, 40, 7, 2), "bf16", WGRAD, "wgrad_stem_kernel<8>"),
    (L("stem.w.c8.k8.pixel", 1, 1, 1, 8, 8, 7, 2), "f16", WGRAD, "wgrad_stem_kernel<8>"),
    (L("stem.narrow.c16.k40", 290, 2, 31, 16, 40, 7, 2), "f16", FWD, "igemm_dma_kernel"),
    (L("stem.w.narrow.c16.k40", 188, 2, 56, 16, 40, 7, 2), "bf16", WGRAD, "wgrad_dma_kernel"),
    (L("stem.w.narrow.c8.k32", 130, 71, 1, 8, 32, 7, 2), "f16", WGRAD, "wgrad_dma_kernel"),
    (L("stem.w.many", 1, 400, 570, 16, 32, 7, 2), "f16", WGRAD, "wgrad_stem_kernel<16>"),
    # parity classes in one launch, tiles not a multiple of the eight XCDs: three taps or fewer each, one tile, two classes
    (L("bt.batch.64x64", 1, 41, 67, 40, 64, 3, 2), "bf16", DGRAD, "batch_kernel.bt<64,64>"),
    (L("bt.batch.128x64.k64", 1, 75, 250, 8, 64, 2, 2), "f16", DGRAD, "batch_kernel.bt.k64<128,64>"),
    (L("bt.batch.one-tile", 1, 5, 6, 40, 64, 3, 2), "f16", DGRAD, "batch_kernel.bt<64,64>"),
    (L("bt.batch.one-row", 1, 1, 131, 40, 64, 3, 2), "bf16", DGRAD, "batch_kernel.bt<64,64>"),
    # 11 G multiply-adds
    (L("bt.batch.large", 1, 185, 231, 256, 456, 3, 2), "f16", DGRAD, "batch_kernel.bt<"),
    # tap-major order (few channels): each tile, and a cut column range
    (L("tap.64x32", 1, 9, 13, 24, 24, 3), "f16", FWD, "tapmajor<64,32>"),
    (L("tap.64x64", 1, 25, 36, 40, 264, 1), "bf16", FWD, "tapmajor<64,64>"),
    (L("tap.128x64", 1, 198, 66, 24, 80, 3), "f16", FWD, "tapmajor<128,64>"),
    (L("tap.128x128", 1, 179, 98, 8, 72, 1), "bf16", FWD, "tapmajor<128,128>"),
    (L("tap.256x256", 2, 66, 261, 56, 136, 3), "f16", FWD, "tapmajor<256,256>"),
    (L("tap.cut", 1, 96, 170, 8, 576, 3), "f16", FWD, "tapmajor<128,128>[512]; igemm_dma_kernel.tapmajor<64,64>[255]"),
    # filter gradient: tiles of one shape with steps of the other depth, and read like dy (1x1, unit stride)
    (L("w.128x128.32-pixels", 1, 95, 13, 1952, 144, 3, 2), "f16", WGRAD, "wgrad_dma_kernel<128,128>["),
    (L("w.128x128.32-pixels.1x1", 1, 120, 285, 1328, 72, 1), "bf16", WGRAD, "wgrad_dma_kernel<128,128>.linear["),
    (L("w.128x128.1x1", 1, 6, 54, 1216, 256, 1), "f16", WGRAD, "wgrad_dma_kernel<128,128>.k64.linear["),
    (L("w.64x64.32-pixels", 2, 105, 2, 1048, 32, 3), "bf16", WGRAD, "wgrad_dma_kernel<64,64>["),
    (L("w.64x64.64-pixels", 1, 24, 58, 1584, 40, 7, 2), "f16", WGRAD, "wgrad_dma_kernel<64,64>.k64["),
    (L("w.128x256.1x1", 1, 158, 159, 672, 136, 1), "bf16", WGRAD, "wgrad_dma_kernel<128,256>.k64.linear["),
    (L("w.256x256.1x1", 1, 101, 299, 1368, 144, 1), "f16", WGRAD, "wgrad_dma_kernel<256,256>.linear["),
    # a stride-1 data gradient whose columns are cut: the offset into the reduction-major filter
    (L("bt.cut", 2, 89, 175, 264, 240, 1), "f16", DGRAD, "bt<128,128>[488]; igemm_dma_kernel.bt.k64<128,64>[244]"),
]


@pytest.mark.parametrize("layer,dtype,which,kernel", CASES, ids=[c[0].name for c in CASES])
def test_tiles_at_their_edges(api, layer, dtype, which, kernel):
    text = api.dl_conv_describe(api.desc_from_layer(layer, dtype), which)
    assert kernel in text, f"{layer.name}: {text}"
    name = ("fwd", "dgrad", "wgrad")[which]
    check_layer(api, layer, dtype, synth.seed_for(0, 2000 + [c[0].name for c in CASES].index(layer.name)), x_kind="normal", passes=(name,), full_passes=(name,))


@pytest.mark.parametrize("which,C,K,former", [(FWD, 352, 256, 4505600), (DGRAD, 256, 352, 9011200)], ids=["fwd", "dgrad"])
def test_many_small_maps_without_room_for_the_partial_sums(api, which, C, K, former):
    """260 maps of 3 x 3 (5x5, long reduction, split when there is room) in the workspace of the halo kernel that once took them, in
    the least and in the preferred one."""
    N, H = 260, 3
    desc = api.ConvDesc(N, H, H, C, K, 5, 5, 1, 1, 2, 2, 1, 1, api.DL_F16)
    least, best = api.dl_conv_least_workspace_bytes(desc, which), api.dl_conv_workspace_bytes(desc, which)
    assert "splitk_reduce" in api.dl_conv_describe(desc, which) and least <= former < best
    g = torch.Generator().manual_seed(2101)
    w = (torch.randn((K, 5, 5, C), generator=g) * 0.02).half()
    a = torch.randn((N, H, H, C if which == FWD else K), generator=g).half()
    nchw = lambda t: t.double().permute(0, 3, 1, 2)                                              # noqa: E731
    if which == FWD:
        ref, call = torch.nn.functional.conv2d(nchw(a), nchw(w), padding=2), api.conv2d_fwd
    else:
        ref, call = torch.nn.functional.conv_transpose2d(nchw(a), nchw(w), padding=2), api.conv2d_bwd_data
    ref = ref.permute(0, 2, 3, 1).numpy()
    for size in (max(least, 16), former, best):
        buf, ws = U.guarded_workspace(size)
        out = call(desc, a.cuda(), w.cuda(), workspace=ws)
        assert U.workspace_guards_intact(buf, size)
        assert U.rel_err(U.to_host_f64(out), ref) <= U.TOL["f16"], size


def test_split_forward_without_room_for_the_partial_sums(api):
    """A forward pass whose reduction is split when there is room runs unsplit, or in fewer ranges, when there is less."""
    layer = L("split.small-workspace", 1, 28, 19, 232, 128, 3, 1, 2)
    (x32, xb), (w32, wb), _ = U.conv_inputs(layer, "f16", synth.seed_for(0, 2100), "normal")
    desc = api.desc_from_layer(layer, "f16")
    best = api.dl_conv_workspace_bytes(desc, api.PASS_FWD)
    one = layer.N * layer.P * layer.Q * layer.K * 4
    assert best >= 2 * one and api.dl_conv_least_workspace_bytes(desc, api.PASS_FWD) == 0
    ref = oracle.conv_fwd(U.shape_of(layer), x32, w32)
    x, w = U.to_device(xb, "f16"), U.to_device(wb, "f16")
    for size in (best, 2 * one, 16):
        y = api.conv2d_fwd(desc, x, w, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
        assert U.rel_err(U.to_host_f64(y), ref) <= U.TOL["f16"]


@pytest.mark.parametrize("C", [8, 16])
def test_stem_keeps_infinities_to_their_windows(api, C):
    """An infinite input reaches the outputs whose window holds it and no other (the kernels' steps reach one tap further, and
    patches beyond the image's edge), in either pass; with zero gradients the other filter taps stay finite."""
    H, W, K = 45, 50, 64                                   # 23 x 25 outputs: ragged patches both ways
    desc = api.ConvDesc(1, H, W, C, K, 7, 7, 2, 2, 3, 3, 1, 1, api.DL_F16)
    P, Q = api.dl_conv_out_shape(desc)
    x = torch.zeros((1, H, W, C), dtype=torch.float16, device="cuda")
    h, w = 20, 49
    x[0, h, w, 3] = float("inf")
    y = api.conv2d_fwd(desc, x, torch.ones((K, 7, 7, C), dtype=torch.float16, device="cuda")).float().cpu().numpy()
    p, q = np.arange(P)[:, None], np.arange(Q)[None]
    hit = (abs(2 * p - h) <= 3) & (abs(2 * q - w) <= 3)
    assert np.isinf(y[0][hit]).all() and (y[0][~hit] == 0).all()
    dw = api.conv2d_bwd_filter(desc, x, torch.ones((1, P, Q, K), dtype=torch.float16, device="cuda")).float().cpu().numpy()
    r, s = np.arange(7)[:, None], np.arange(7)[None]
    # tap (r, s) meets the pixel where (h + 3 - r) / 2 and (w + 3 - s) / 2 are output positions
    met = ((h + 3 - r) % 2 == 0) & ((w + 3 - s) % 2 == 0) & ((h + 3 - r) // 2 < P) & ((w + 3 - s) // 2 < Q)
    assert np.isinf(dw[:, met][:, :, 3]).all() and (dw[:, ~met] == 0).all()
    assert (np.delete(dw, 3, axis=3) == 0).all()


# A stride far beyond the image leaves one output column (or row) per image: what a step of pixels advances in the input is then
# images or rows, and the step times the stride does not fit 32 bits.  2^25 and 2^26 are the first strides at which that is so
# for steps of 64 and 32 pixels.  (N, H, W, C, K, filter, strides, padding)
HUGE_STRIDES = [
    (4096, 1, 1, 64, 64, 1, (1, 40_000_000), 0),
    (700, 3, 2, 64, 40, 1, (1, 1 << 25), 0),
    (700, 3, 2, 64, 40, 1, (2_000_000_000, 1), 0),
    (500, 1, 5, 32, 136, 3, (2_000_000_000, 2_000_000_000), 1),
    (300, 2, 7, 136, 256, 3, (1, 1 << 26), 1),
    (2, 1, 3, 64, 32, 1, (1, 4_000_000), (0, 100_000_000)),          # 51 output columns, one of them inside
    (2, 1, 3, 64, 32, 1, (1, 40_000_000), (0, 1_000_000_000)),       # so wide that the kernel that counts output pixels takes it
]


@pytest.mark.parametrize("N,H,W,C,K,R,stride,pad", HUGE_STRIDES)
def test_filter_gradient_with_strides_beyond_the_image(api, N, H, W, C, K, R, stride, pad):
    ph, pw = pad if isinstance(pad, tuple) else (pad, pad)
    desc = api.ConvDesc(N, H, W, C, K, R, R, stride[0], stride[1], ph, pw, 1, 1, api.DL_F16, api.DL_F32)
    assert ("wgrad_dma_kernel" if pw < 1 << 28 else "wgrad_kernel") in api.dl_conv_describe(desc, api.PASS_BWD_FILTER)
    P, Q = api.dl_conv_out_shape(desc)
    g = torch.Generator().manual_seed(2200 + K)
    x, dy = torch.randn((N, H, W, C), generator=g).half(), torch.randn((N, P, Q, K), generator=g).half()
    # (the C entry: the wrapper would also size the data gradient's workspace, class by class of the stride)
    xd, dyd, dw = x.cuda(), dy.cuda(), torch.full((K, R, R, C), float("nan"), device="cuda")
    ws = torch.empty(api.dl_conv_workspace_bytes(desc, api.PASS_BWD_FILTER), dtype=torch.uint8, device="cuda")
    assert api._lib.conv2d_bwd_filter(ctypes.byref(desc.c_struct()), xd.data_ptr(), dyd.data_ptr(), dw.data_ptr(), ws.data_ptr(), ws.numel(),
                                      torch.cuda.current_stream().cuda_stream) == 0
    dw = dw.double().cpu()
    ref = torch.zeros((K, R, R, C), dtype=torch.float64)
    for p in range(P):
        for q in range(Q):
            for r in range(R):
                for s in range(R):
                    h, w = p * stride[0] - ph + r, q * stride[1] - pw + s
                    if 0 <= h < H and 0 <= w < W:
                        ref[:, r, s] += dy[:, p, q].double().t() @ x[:, h, w].double()
    # fp32 sums of exact fp16 products, as in the other parity tests with fp32 filter gradients
    assert float((dw - ref).norm()) <= 1e-5 * float(ref.norm())
