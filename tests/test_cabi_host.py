"""Host-only checks of the C boundary: the library loads without a GPU,
exports every symbol the header declares, and rejects bad arguments before
touching the device."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def api():
    from paper_1810_01993_amd import build
    if not os.path.exists(build.LIB):
        build.build_library()
    from paper_1810_01993_amd import api as _api
    return _api


def test_every_declared_symbol_is_exported(api):
    header = open(os.path.join(ROOT, "include", "dlconv.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(\w+)\s*\([^;{]*\)\s*;", header))
    assert {"conv2d_fwd", "conv2d_bwd_data", "conv2d_bwd_filter", "weighted_pixel_ce_fwd_bwd"} <= declared
    lib = ctypes.CDLL(api.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), f"{name} is declared in dlconv.h but not exported"
    assert declared == set(api.EXPORTS)
    # the measurement aids have a header of their own
    probe = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "dlprobe.h")).read(), flags=re.S)
    declared_probe = set(re.findall(r"\b(\w+)\s*\([^;{]*\)\s*;", probe))
    assert declared_probe == set(api.PROBE_EXPORTS)
    for name in declared_probe:
        assert hasattr(lib, name), f"{name} is declared in dlprobe.h but not exported"
    assert set(os.listdir(os.path.join(ROOT, "include"))) == {"dlconv.h", "dlprobe.h"}


def test_out_shape_and_workspace_queries(api):
    d = api.ConvDesc(2, 768, 1152, 16, 64, 7, 7, 2, 2, 3, 3, 1, 1, api.DL_BF16)
    assert api.dl_conv_out_shape(d) == (384, 576)
    assert api.dl_conv_workspace_bytes(d, api.PASS_FWD) == 0
    # data gradient: room for the re-laid-out filter (every tap lands in exactly one parity class)
    assert api.dl_conv_workspace_bytes(d, api.PASS_BWD_DATA) >= 64 * 7 * 7 * 16 * 2
    ws = api.dl_conv_workspace_bytes(d, api.PASS_BWD_FILTER)
    assert ws >= 64 * 7 * 7 * 16 * 4 and ws % (64 * 7 * 7 * 16 * 4) == 0
    assert api.dl_ce_workspace_bytes(0) >= 4
    assert api.dl_ce_workspace_bytes(2 * 768 * 1152) >= 4


def test_least_workspace(api):
    """Never more than the preferred size, one byte less is refused, and what the padded copies and the stem kernel add for
    channel counts that are not a multiple of 8 is not part of it."""
    lib = api._lib
    for C, K, R, st, H, W in ((300, 256, 3, 1, 768, 1152), (6, 64, 7, 2, 361, 577), (6, 40, 7, 2, 33, 45), (256, 256, 3, 2, 384, 576),
                              (2048, 256, 3, 1, 48, 72), (100, 3, 1, 1, 90, 100), (16, 64, 7, 2, 768, 1152), (24, 24, 5, 1, 100, 100)):
        d = api.ConvDesc(2, H, W, C, K, R, R, st, st, R // 2, R // 2, 1, 1, api.DL_F16)
        for which, fn in ((api.PASS_FWD, lib.conv2d_fwd), (api.PASS_BWD_DATA, lib.conv2d_bwd_data), (api.PASS_BWD_FILTER, lib.conv2d_bwd_filter)):
            least = api.dl_conv_least_workspace_bytes(d, which)
            assert least <= api.dl_conv_workspace_bytes(d, which)
            if least > 0:                                    # refused before anything is launched
                assert fn(ctypes.byref(d.c_struct()), 4096, 4096, 4096, 4096, least - 1, None) == 5
    big = api.ConvDesc(2, 768, 1152, 300, 256, 3, 3, 1, 1, 1, 1, 1, 1, api.DL_F16)
    for which, bound in ((api.PASS_FWD, 0), (api.PASS_BWD_FILTER, 80e6)):
        assert api.dl_conv_workspace_bytes(big, which) > 1e9 and api.dl_conv_least_workspace_bytes(big, which) <= bound
    assert lib.dl_conv_least_workspace_bytes(ctypes.byref(big.c_struct()), 0, None) == 1
    assert _code(api.dl_conv_least_workspace_bytes, big, 3) == 6
    assert _code(api.dl_conv_least_workspace_bytes, api.ConvDesc(1, 8, 8, 8, 8, 3, 3, 0), 0) == 2


# (N, H, W, C, K, filter, dilation), pass, bytes that were once the least of the pass: the filter copy of a halo kernel, the partial
# sums of a split with 256 x 256 tiles
FORMER_LEAST = [((260, 7, 7, 1024, 256, 3, 2), 0, 4718592), ((260, 7, 7, 256, 1024, 3, 2), 1, 9437184), ((300, 6, 8, 512, 256, 5, 1), 0, 6553600),
                ((300, 6, 8, 256, 512, 5, 1), 1, 13107200), ((46, 107, 2, 520, 256, 5, 1), 0, 6963200), ((2, 48, 72, 2048, 256, 3, 6), 0, 56623104)]


@pytest.mark.parametrize("shape,which,former", FORMER_LEAST)
def test_layers_with_long_reductions_need_no_partial_sums(api, shape, which, former):
    """The plain engine runs unsplit where there is no room for partial sums: a forward pass takes any workspace, a data gradient
    what its re-laid-out filter may take; sizes that were enough for a layer's former kernel still are."""
    N, H, W, C, K, R, dil = shape
    d = api.ConvDesc(N, H, W, C, K, R, R, 1, 1, dil * (R // 2), dil * (R // 2), dil, dil, api.DL_F16)
    least, best = api.dl_conv_least_workspace_bytes(d, which), api.dl_conv_workspace_bytes(d, which)
    assert least == (0 if which == 0 else 2 * R * R * C * K) and least < best
    assert least <= former


# Layers with few channels (tap-major order) and a column range behind a multiple of 256: one launch where a second one's start and
# end would cost more than its columns save (two took 1.5-1.7x the time), two where whole rounds of tiles are saved, or where
# the output exceeds the caches and the last of its widest tiles would be mostly empty
@pytest.mark.parametrize("N,H,W,C,K,R,launches", [(1, 24, 36, 40, 264, 1, 1), (1, 96, 144, 56, 384, 3, 1), (1, 45, 67, 104, 320, 1, 1),
                                                  (1, 1, 1, 8, 304, 1, 1), (1, 96, 170, 8, 576, 3, 2), (2, 400, 632, 24, 320, 1, 2),
                                                  (2, 400, 625, 24, 440, 1, 1)])
def test_tap_major_column_ranges(api, N, H, W, C, K, R, launches):
    text = api.dl_conv_describe(api.ConvDesc(N, H, W, C, K, R, R, 1, 1, R // 2, R // 2, 1, 1, api.DL_F16), api.PASS_FWD)
    assert text.count("igemm_dma_kernel.tapmajor") == launches and text.count("kernel") == launches, text


@pytest.mark.parametrize("N,H,W,C,K,R,stride,tiles", [(2, 50, 71, 120, 528, 7, 2, "<64,64>[261]"), (1, 42, 59, 120, 400, 7, 1, "<64,64>[273]"),
                                                      (1, 177, 192, 56, 64, 7, 1, "<128,64>[266]"), (1, 198, 66, 24, 80, 3, 1, "<128,64>[206]")])
def test_tap_major_tiles_a_little_beyond_a_round(api, N, H, W, C, K, R, stride, tiles):
    """260 tiles of 64 x 64 take 1.3 rounds' time, not 1.5: half as many larger ones are slower; 530 take 2.5."""
    text = api.dl_conv_describe(api.ConvDesc(N, H, W, C, K, R, R, stride, stride, R // 2, R // 2, 1, 1, api.DL_F16), api.PASS_FWD)
    assert text == "igemm_dma_kernel.tapmajor" + tiles, text


@pytest.mark.parametrize("N,H,W,C,K,R,dil,which", [(2, 141, 179, 96, 192, 5, 1, 0), (1, 230, 250, 32, 192, 3, 2, 0), (2, 147, 160, 256, 304, 5, 1, 0),
                                                   (1, 182, 263, 256, 128, 3, 2, 1), (223, 20, 22, 512, 320, 3, 3, 0)])
def test_dilated_and_5x5_layers_of_one_round_of_patches(api, N, H, W, C, K, R, dil, which):
    """200..256 patches of 16 x 16: on the ring kernels, without a filter copy."""
    text = api.dl_conv_describe(api.ConvDesc(N, H, W, C, K, R, R, 1, 1, dil * (R // 2), dil * (R // 2), dil, dil, api.DL_BF16), which)
    assert "igemm_dma_kernel" in text and "filter_block" not in text, text


def test_stem_filter_gradient_of_a_few_pixels(api):
    """Less than 64 output pixels, 16 channels and less than 32 outputs: the general kernel; from there on the stem's."""
    for N, H, W, C, K, kernel in ((1, 15, 15, 16, 24, "wgrad_stem"), (1, 14, 15, 16, 24, "wgrad_kernel"), (1, 8, 8, 16, 8, "wgrad_kernel"),
                                  (1, 8, 8, 16, 32, "wgrad_stem"), (1, 8, 8, 8, 8, "wgrad_stem")):
        assert kernel in api.dl_conv_describe(api.ConvDesc(N, H, W, C, K, 7, 7, 2, 2, 3, 3, 1, 1, api.DL_F16), api.PASS_BWD_FILTER)


def test_stem_kernels_leave_narrow_maps_to_the_general_ones(api):
    """Many images whose 16 x 16 patches lie mostly outside: the general kernels; filled patches, or one per compute unit: the stem's."""
    for N, H, W, C, K, fwd, wgrad in ((306, 1, 566, 16, 16, "igemm_dma", "wgrad_stem"), (188, 2, 56, 16, 40, "igemm_dma", "wgrad_dma"),
                                      (299, 256, 1, 8, 40, "igemm_dma", "wgrad_dma"), (60, 30, 30, 8, 64, "stem_fwd", "wgrad_stem"),
                                      (2, 768, 1152, 16, 64, "stem_fwd", "wgrad_stem"), (2, 361, 577, 8, 64, "stem_fwd", "wgrad_stem")):
        d = api.ConvDesc(N, H, W, C, K, 7, 7, 2, 2, 3, 3, 1, 1, api.DL_F16)
        assert fwd in api.dl_conv_describe(d, api.PASS_FWD) and wgrad in api.dl_conv_describe(d, api.PASS_BWD_FILTER)
        assert api.dl_conv_least_workspace_bytes(d, api.PASS_BWD_FILTER) <= api.dl_conv_workspace_bytes(d, api.PASS_BWD_FILTER)


def test_wrapper_takes_the_least_workspace_when_memory_is_short(api, monkeypatch):
    torch = api.torch
    big = api.ConvDesc(2, 768, 1152, 300, 256, 3, 3, 1, 1, 1, 1, 1, 1, api.DL_F16)
    room = [0]
    plain = torch.empty

    def short(n, **kw):
        if n > room[0]:
            raise torch.cuda.OutOfMemoryError("no room")
        return plain(n, **kw)
    monkeypatch.setattr(torch, "empty", short)
    ask = lambda which: api._conv_workspace(big, which, api.dl_conv_workspace_bytes(big, which), "meta", None)      # noqa: E731
    assert ask(api.PASS_FWD) == (None, 0)
    with pytest.raises(torch.cuda.OutOfMemoryError):
        ask(api.PASS_BWD_FILTER)
    room[0] = least = api.dl_conv_least_workspace_bytes(big, api.PASS_BWD_FILTER)
    assert ask(api.PASS_BWD_FILTER)[1] == least
    room[0] = 1 << 40
    assert ask(api.PASS_BWD_FILTER)[1] == api.dl_conv_workspace_bytes(big, api.PASS_BWD_FILTER)
    own = plain(64, dtype=torch.uint8)
    assert api._conv_workspace(big, api.PASS_FWD, 1 << 30, "meta", own) == (own, 64)


def _code(fn, *a):
    with pytest.raises(Exception) as e:
        fn(*a)
    return e.value.code


def test_descriptor_validation(api):
    ok = dict(N=1, H=8, W=8, C=8, K=8, R=3, S=3, stride_h=1, stride_w=1, pad_h=1, pad_w=1, dil_h=1, dil_w=1,
              dtype=api.DL_F16)
    assert api.dl_conv_out_shape(api.ConvDesc(**ok)) == (8, 8)
    for field, bad in [("N", 0), ("C", -1), ("K", 0), ("R", 0), ("stride_h", 0), ("dil_w", 0), ("pad_h", -1)]:
        assert _code(api.dl_conv_out_shape, api.ConvDesc(**{**ok, field: bad})) == 2, field
    assert _code(api.dl_conv_out_shape, api.ConvDesc(**{**ok, "H": 2, "pad_h": 0, "dil_h": 2})) == 2   # empty output
    assert _code(api.dl_conv_out_shape, api.ConvDesc(**{**ok, "dtype": api.DL_F32})) == 3
    assert _code(api.dl_conv_out_shape, api.ConvDesc(**{**ok, "dtype": api.DL_F16, "dw_dtype": api.DL_BF16})) == 3
    assert _code(api.dl_conv_out_shape, api.ConvDesc(**{**ok, "N": 4096, "H": 4096, "W": 4096})) == 2  # index overflow
    assert _code(api.dl_conv_workspace_bytes, api.ConvDesc(**ok), 7) == 6


def test_pointer_checks_happen_before_any_launch(api):
    lib = api._lib
    d = api.ConvDesc(1, 8, 8, 8, 8, 3, 3, 1, 1, 1, 1, 1, 1, api.DL_F16).c_struct()
    ref = ctypes.byref(d)
    for fn in (lib.conv2d_fwd, lib.conv2d_bwd_data, lib.conv2d_bwd_filter):
        assert fn(ref, None, None, None, None, 0, None) == 1           # null
        assert fn(None, 16, 16, 16, None, 0, None) == 1
        assert fn(ref, 16, 16, 24, None, 0, None) == 4                 # misaligned
    assert lib.conv2d_bwd_data(ref, 16, 16, 16, None, 0, None) == 5    # workspace missing
    assert lib.conv2d_bwd_filter(ref, 16, 16, 16, 32, 8, None) == 5    # workspace too small
    assert lib.weighted_pixel_ce_fwd_bwd(None, 0, None, None, 1.0, 8, None, None, None, 0, None) == 1
    assert lib.weighted_pixel_ce_fwd_bwd(16, 2, 16, 16, 1.0, 8, 16, 16, 16, 64, None) == 3
    assert lib.weighted_pixel_ce_fwd_bwd(16, 0, 16, 16, 1.0, -1, 16, 16, 16, 64, None) == 2
    assert lib.weighted_pixel_ce_fwd_bwd(16, 0, 16, 16, 1.0, 8, 16, 16, None, 0, None) == 5
    assert lib.weighted_pixel_ce_fwd_bwd(16, 0, 16, 16, 1.0, 8, 16, 24, 16, 64, None) == 4
    # the entry point without a workspace: same checks, plus its size limit, all before the first HIP call
    assert lib.weighted_pixel_ce_fwd_bwd_static(16, 0, 16, 16, 1.0, api.CE_STATIC_MAX_PIXELS + 1, 16, 16, None) == 2
    assert lib.weighted_pixel_ce_fwd_bwd_static(16, 0, 16, 16, 1.0, 8, None, 16, None) == 1
    assert lib.weighted_pixel_ce_map_fwd_bwd(16, 0, 16, None, 1.0, 8, 16, 16, 16, 64, None) == 1   # no weight map
    assert lib.weighted_pixel_ce_map_fwd_bwd(16, 0, 16, 24, 1.0, 8, 16, 16, 16, 64, None) == 4     # map misaligned
    assert lib.weighted_pixel_ce_map_fwd_bwd(16, 0, 16, 16, 1.0, 8, 16, 16, None, 0, None) == 5
    for fn in (lib.conv2d_transpose_fwd, lib.conv2d_transpose_bwd_data, lib.conv2d_transpose_bwd_filter):
        assert fn(ref, None, None, None, None, 0, None) == 1
        assert fn(ref, 16, 16, 24, None, 0, None) == 4
    assert lib.conv2d_fwd_bias_relu(ref, None, 16, None, 1, 16, None, 0, None) == 1
    assert lib.conv2d_fwd_bias_relu(ref, 16, 16, 18, 1, 16, None, 0, None) == 4                    # bias not 4-byte aligned
    assert lib.bias_relu_bwd(16, 16, 0, 8, 8, 1, 16, None, 16, 4096, None) == 1            # no dbias
    assert lib.bias_relu_bwd(16, None, 0, 8, 8, 1, 16, 16, 16, 4096, None) == 1            # ReLU needs y
    assert lib.bias_relu_bwd(16, 16, 2, 8, 8, 1, 16, 16, 16, 4096, None) == 3
    assert lib.bias_relu_bwd(16, 16, 0, 8, 0, 1, 16, 16, 16, 4096, None) == 2
    assert lib.bias_relu_bwd(16, 16, 0, 8, 8, 1, 16, 16, None, 0, None) == 5
    t = (api._LarcTensor * 2)(api._LarcTensor(16, 16, None, 8), api._LarcTensor(16, None, None, 8))
    tp = ctypes.cast(t, ctypes.c_void_p)
    f = ctypes.c_float
    assert lib.larc_sgd_step(tp, 2, 0, f(.1), f(.02), f(0), f(0), f(0), 1, None, 16, 1 << 20, None) == 1   # tensor 1 has no gradient
    assert lib.larc_sgd_step(tp, 1, 0, f(.1), f(.02), f(0), f(.9), f(0), 1, None, 16, 1 << 20, None) == 1  # momentum needs v
    assert lib.larc_sgd_step(tp, 1, 7, f(.1), f(.02), f(0), f(0), f(0), 1, None, 16, 1 << 20, None) == 3
    assert lib.larc_sgd_step(tp, 1, 0, f(.1), f(.02), f(0), f(0), f(0), 1, None, 16, 8, None) == 5
    assert lib.larc_sgd_step(None, 0, 0, f(.1), f(.02), f(0), f(0), f(0), 1, None, None, 0, None) == 0     # nothing to do
    assert lib.dl_status_string(0) == b"ok" and b"workspace" in lib.dl_status_string(5)
    flop = ctypes.c_double()
    assert lib.dl_probe_mfma(0, 0, 10, None, 16, ctypes.byref(flop), None) == 1
    assert lib.dl_probe_mfma(2, 0, 10, 16, 16, ctypes.byref(flop), None) == 2
    assert lib.dl_probe_stream(1, 16, None, 16, 3073, 16, None) == 2
    assert lib.dl_probe_stream(3, 16, None, 16, 3072, 16, None) == 1


_DISPATCH_PROBE = r"""
import sys
sys.path.insert(0, %r)
from paper_1810_01993_amd import api
out = []
shapes = [(2, 768, 1152, 256, 256, 3, 1, 1, 1),     # decoder 3x3: halo-tile kernel, fused-tap filter gradient
          (2, 48, 72, 2048, 256, 3, 1, 6, 6),       # ASPP 3x3: split reduction
          (2, 48, 72, 1024, 256, 1, 1, 0, 1),       # 1x1
          (2, 192, 288, 128, 128, 3, 2, 1, 1),      # stride 2: parity classes in one launch
          (2, 768, 1152, 16, 64, 7, 2, 3, 1),       # stem
          (2, 768, 1152, 208, 32, 5, 1, 2, 1)]      # 5x5 with 32 output channels
for (N, H, W, C, K, R, st, pad, dil) in shapes:
    d = api.ConvDesc(N, H, W, C, K, R, R, st, st, pad, pad, dil, dil, api.DL_F16)
    out.append([api.dl_conv_workspace_bytes(d, p) for p in (0, 1, 2)])
out.append(api.dl_ce_workspace_bytes(2 * 768 * 1152))
print(out)
"""


def test_dispatch_does_not_read_the_environment(api):
    """The library has no run-time knobs: the sweep variables of the tuning build change nothing (the
    workspace sizes follow the kernel choice, the split of reductions and the slice plans), no source
    file calls getenv outside the tuning build's helper, and the built library does not import it."""
    import subprocess
    import sys
    knobs = {"DLCONV_HALO": "0", "DLCONV_KSPLIT": "0", "DLCONV_WGRAD_CFG": "1", "DLCONV_WGRAD3X3": "0",
             "DLCONV_WGRAD5X5": "0", "DLCONV_NARROW": "0", "DLCONV_WIDE5X5": "0", "DLCONV_DGRAD_STEM": "0",
             "DLCONV_IGEMM_CFG": "103", "DLCONV_BATCH": "0", "DLCONV_BT": "0", "DLCONV_CE_BLOCKS": "7",
             "DLCONV_WGRAD_TARGET": "64", "DLCONV_C_OUTER": "0", "DLCONV_CFG128_MIN": "1", "DLCONV_REDUCE4": "0"}
    clean = {k: v for k, v in os.environ.items() if not k.startswith("DLCONV_")}
    code = _DISPATCH_PROBE % ROOT
    plain = subprocess.run([sys.executable, "-c", code], env=clean, capture_output=True, text=True, check=True).stdout
    steered = subprocess.run([sys.executable, "-c", code], env={**clean, **knobs}, capture_output=True, text=True,
                             check=True).stdout
    assert plain == steered and plain.strip().startswith("[[")
    csrc = os.path.join(ROOT, "paper_1810_01993_amd", "csrc")
    for name in os.listdir(csrc):
        if name.endswith(".hip"):
            assert "getenv" not in open(os.path.join(csrc, name)).read(), name
    syms = subprocess.run(["nm", "-D", "--undefined-only", api.LIB_PATH], capture_output=True, text=True, check=True).stdout
    assert "getenv" not in syms


def test_kept_descriptor_answers_follow_the_values(api):
    """The wrapper keeps the library's answers by the values of the descriptor: equal values share them, any other value
    gets its own, refused descriptors are refused every time and the store stays bounded."""
    base = dict(N=1, H=20, W=33, C=16, K=32, R=3, S=3, stride_h=1, stride_w=1, pad_h=1, pad_w=1, dil_h=1, dil_w=1)
    for change in ({}, {}, {"H": 40}, {"stride_w": 2}, {"dil_h": 2}, {"K": 8}, {"dtype": api.DL_BF16}, {"dw_dtype": api.DL_F32}):
        d = api.ConvDesc(**{**base, **change})
        for _ in range(2):
            _, P, Q, need = api._plan(d)
            assert (P, Q) == api.dl_conv_out_shape(d)
            assert list(need) == [api.dl_conv_workspace_bytes(d, w) for w in range(3)]
    for _ in range(2):
        assert _code(api._plan, api.ConvDesc(1, 8, 8, 8, 8, 3, 3, 0)) == 2
        with pytest.raises((TypeError, ctypes.ArgumentError)):
            api._plan(api.ConvDesc(**{**base, "N": 1.0}))
    for n in range(1100):
        api._plan(api.ConvDesc(1, 8, 8 + n, 8, 8, 1, 1))
    assert len(api._plans) <= 1024


# (N, H, W, C, K, R, stride, forward on channel-padded copies): timed both ways, us without / with the copies
PADDED_FORWARD = [
    ((2, 506, 512, 299, 1, 1, 2), False),       # 74 / 197: the copy moves four times the pixels that the layer reads
    ((2, 759, 884, 204, 12, 1, 2), False),      # 138 / 354
    ((1, 600, 900, 58, 96, 1, 2), False),
    ((1, 535, 1022, 58, 256, 1, 2), True),      # 85 / 46: the one-step kernel with enough columns
    ((2, 648, 1148, 189, 5, 1, 1), True),       # 596 / 456
    ((2, 224, 394, 27, 1, 1, 1), False),        # 16.2 / 20.8
    ((1, 60, 90, 17, 64, 1, 1), False),         # 9.1 / 9.9
    ((2, 730, 734, 1, 256, 7, 1), False),       # 372 / 856: seven of eight padded channels are zeros
    ((1, 328, 392, 1, 128, 5, 1), False),       # 24 / 49
    ((1, 304, 425, 6, 8, 3, 1), False),         # 16 / 24: a 32-channel chunk of the halo kernel for 8 outputs
    ((1, 397, 592, 7, 48, 3, 1), True),         # 32 / 29
    ((2, 402, 549, 5, 96, 3, 1), True),         # 83 / 58
    ((2, 475, 786, 9, 12, 2, 2), False),        # 21 / 28
    ((2, 361, 577, 6, 64, 7, 2), True),         # 56 / 28
    ((1, 60, 90, 100, 64, 3, 1), True),         # 92 / 14
]


@pytest.mark.parametrize("shape,padded", PADDED_FORWARD, ids=["x".join(map(str, s)) for s, _ in PADDED_FORWARD])
def test_forward_on_padded_copies_where_they_pay(api, shape, padded):
    N, H, W, C, K, R, st = shape
    d = api.ConvDesc(N, H, W, C, K, R, R, st, st, R // 2, R // 2, 1, 1, api.DL_F16)
    text = api.dl_conv_describe(d, api.PASS_FWD)
    assert text.startswith("pad_channels_kernel" if padded else "igemm_scalar_kernel"), text


def test_filter_gradient_on_padded_copies_where_they_pay(api):
    # (timed both ways, us without / with the copies: 244 / 325, 144 / 189, 389 / 312, 148 / 35)
    for (N, H, W, C, K, R, st), padded in (((2, 501, 962, 242, 64, 1, 2), False), ((1, 463, 801, 378, 32, 1, 2), False),
                                           ((2, 659, 1209, 141, 48, 1, 2), True), ((2, 361, 577, 6, 64, 7, 2), True)):
        d = api.ConvDesc(N, H, W, C, K, R, R, st, st, R // 2, R // 2, 1, 1, api.DL_F16)
        text = api.dl_conv_describe(d, api.PASS_BWD_FILTER)
        assert text.startswith("pad_channels_kernel" if padded else "wgrad_kernel"), text


def test_describe_names_the_kernels_of_the_decoder_layers(api):
    """dl_conv_describe runs the entry points' own dispatch with launches logged instead of issued
    (no GPU needed): the layers that carry 87 % of the FLOPs must reach the kernels built for them."""
    dec = api.ConvDesc(2, 768, 1152, 256, 256, 3, 3, 1, 1, 1, 1, 1, 1, api.DL_F16)
    assert "igemm_halo3x3_kernel<4>[6912]" in api.dl_conv_describe(dec, api.PASS_FWD)
    assert "igemm_halo3x3_kernel<4>[6912]" in api.dl_conv_describe(dec, api.PASS_BWD_DATA)
    assert api.dl_conv_describe(dec, api.PASS_BWD_FILTER).startswith("wgrad3x3_kernel[")
    dec304 = api.ConvDesc(2, 768, 1152, 304, 256, 3, 3, 1, 1, 1, 1, 1, 1, api.DL_BF16)
    assert "igemm_halo3x3_kernel<5>[6912]" in api.dl_conv_describe(dec304, api.PASS_BWD_DATA)
    stem = api.ConvDesc(2, 768, 1152, 16, 64, 7, 7, 2, 2, 3, 3, 1, 1, api.DL_F16)
    assert "dgrad_stem_kernel" in api.dl_conv_describe(stem, api.PASS_BWD_DATA)
    logits = api.ConvDesc(2, 768, 1152, 256, 3, 1, 1, 1, 1, 0, 0, 1, 1, api.DL_F16)
    assert api.dl_conv_describe(logits, api.PASS_FWD) == "thin_cols_kernel[2048]"
    assert "thin_rows_kernel" in api.dl_conv_describe(logits, api.PASS_BWD_DATA)
    assert "thin_wgrad_kernel" in api.dl_conv_describe(logits, api.PASS_BWD_FILTER)
    # filter gradient: large operands that every XCD would fetch for itself keep a slice on one XCD, small ones are dealt
    up = api.ConvDesc(2, 384, 576, 256, 256, 3, 3, 2, 2, 1, 1, 1, 1, api.DL_F16)
    assert api.dl_conv_describe(up, api.PASS_BWD_FILTER).startswith("wgrad_dma_kernel<256,256>[216]")
    # ... and so do large ones of which the XCDs fetch little twice: one row tile (76 us dealt, 108 us with slices on one XCD),
    # a number of column tiles that leaves every column on one XCD
    for shape, dealt in (((4, 130, 189, 1008, 80, 3, 2), 7 * 71), ((2, 114, 117, 984, 112, 3, 1), 7 * 70)):
        N, H, W, C, K, R, st = shape
        text = api.dl_conv_describe(api.ConvDesc(N, H, W, C, K, R, R, st, st, 1, 1, 1, 1, api.DL_F16), api.PASS_BWD_FILTER)
        assert text.startswith(f"wgrad_dma_kernel<128,128>[{dealt}]"), text
    # one-step reductions take their own kernel from 512 tiles of 128 x 128 on
    for H, name in ((256, "igemm_short_kernel["), (255, "igemm_dma_kernel")):
        assert api.dl_conv_describe(api.ConvDesc(1, H, 128, 64, 200, 1, 1), api.PASS_FWD).startswith(name)
    low = api.ConvDesc(2, 48, 72, 256, 256, 3, 3, 2, 2, 1, 1, 1, 1, api.DL_F16)
    assert api.dl_conv_describe(low, api.PASS_BWD_FILTER).startswith("wgrad_dma_kernel<128,128>")
    # the query leaves nothing behind: a call after it still validates and reports as before
    assert api._lib.conv2d_fwd(ctypes.byref(dec.c_struct()), None, None, None, None, 0, None) == 1
    assert _code(api.dl_conv_describe, api.ConvDesc(2, 8, 8, 8, 8, 3, 3, 1, 1, 1, 1, 1, 1, api.DL_F16), 5) == 6
