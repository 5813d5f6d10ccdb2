"""GPU parity of bias_relu_bwd (backward of the fused point-wise tail: ReLU mask
on dy and bias gradient in one pass) against the fp64 oracle."""
import sys

import numpy as np
import pytest
import torch

from oracle import epilogue as E
from paper_1810_01993_amd import synth

import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_1810_01993_amd import api as _api
    assert torch.cuda.is_available()
    return _api


def _run(api, n, K, dtype, seed, relu=True, alias=False, workspace=None):
    print(f"[case] bias_relu_bwd n={n} K={K} {dtype} relu={relu} alias={alias} seed={seed}", flush=True)
    sys.stdout.flush()
    dy32, dyb = synth.quantize(synth.normal(seed, (n, K)), dtype)
    # a forward output: about half of it cut to exactly zero (also -0 never appears after a ReLU)
    y32, yb = synth.quantize(np.maximum(synth.normal(seed + 1, (n, K)), 0.0), dtype)
    dyd, yd = U.to_device(dyb, dtype), U.to_device(yb, dtype)
    dz, db = api.bias_relu_bwd(dyd, yd if relu else None, relu, dz=dyd if (alias and relu) else None,
                               workspace=workspace)
    torch.cuda.synchronize()
    ref_dz, ref_db = E.bias_relu_bwd(dy32, y32, relu)
    got_dz = U.to_host_f64(dz)
    assert np.array_equal(got_dz, ref_dz)                       # masking copies bits: exact
    got_db = db.double().cpu().numpy()
    # fp32 running sums over up to n terms: error bounded by a few ulps of the sum of magnitudes
    bound = 1e-5 * np.abs(ref_dz).sum(axis=0) + 1e-30
    assert np.all(np.abs(got_db - ref_db) <= bound), float(np.max(np.abs(got_db - ref_db) / bound))
    return db


CASES = [(1, 8), (5, 8), (1000, 64), (777, 48), (4099, 256), (300, 304), (2500, 3), (911, 5), (64, 2048), (33, 4096),
         (70000, 16)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n,K", CASES, ids=[f"{n}x{K}" for n, K in CASES])
def test_mask_and_bias_gradient(api, n, K, dtype):
    _run(api, n, K, dtype, synth.seed_for(0, 1500 + (n * 7 + K) % 91))


# column blocks with a ragged last one (8-channel groups and odd counts), slabs that end inside the run of four pixels,
# and the limit of 1024 partial rows
EDGES = [(7, 264), (31, 520), (4097, 1024), (131, 257), (65, 511), (262145, 8), (131073, 24), (32801, 256)]


@pytest.mark.parametrize("n,K", EDGES, ids=[f"{n}x{K}" for n, K in EDGES])
def test_column_blocks_and_slab_edges(api, n, K):
    _run(api, n, K, "f16", synth.seed_for(0, 1540 + (n + K) % 37))


# either side of the change from four to eight pixels per thread (n * columns = 5 * 1024 * pixel lanes), where the number of
# partial rows falls: 1024 to 640 with 256 channels, 320 to 160 with 1024
SLABS = [(32737, 256), (40959, 256), (40960, 256), (10239, 1024), (10240, 1024)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n,K", SLABS, ids=[f"{n}x{K}" for n, K in SLABS])
def test_change_of_slab_length(api, n, K, dtype):
    _run(api, n, K, dtype, synth.seed_for(0, 1550 + (n + K) % 13), relu=n % 2 == 1)


# element-wise channel counts: workgroups of up to 256 channels below 4 M elements, interleaved columns of at most 64 from
# there on (last slab group short of eight, last column short), and a few channels with many pixel lanes
ELEMENTS = [(1, 1), (4097, 1), (9001, 2), (16383, 257), (16385, 257), (70001, 60), (33011, 129), (2800, 1501), (3, 300)]


@pytest.mark.parametrize("n,K", ELEMENTS, ids=[f"{n}x{K}" for n, K in ELEMENTS])
def test_element_wise_columns(api, n, K):
    _run(api, n, K, "f16" if n % 2 else "bf16", synth.seed_for(0, 1560 + (n + K) % 17))


@pytest.mark.parametrize("n", [32767, 32769])
def test_element_wise_columns_without_relu(api, n):
    _run(api, n, 257, "f16", synth.seed_for(0, 1585), relu=False)       # the line lies at 8 M elements here


# rows that are not whole 128-byte lines, from 16 M elements on: up to 512 channels in one column, wider ones interleaved
# (last slab group short of eight, last column short); below that and with whole lines columns of 256 channels
PIECES = [(33289, 504), (55190, 304), (32300, 520), (14503, 1160), (16289, 1032), (4100, 4104), (77, 328), (1000, 576)]


@pytest.mark.parametrize("n,K", PIECES, ids=[f"{n}x{K}" for n, K in PIECES])
def test_columns_of_16_byte_pieces(api, n, K):
    _run(api, n, K, "bf16" if n % 2 else "f16", synth.seed_for(0, 1570 + (n + K) % 17), relu=n != 16289)


def test_without_relu_in_place_and_repeatable(api):
    _run(api, 3001, 72, "f16", synth.seed_for(0, 1590), relu=False)
    a = _run(api, 3001, 72, "bf16", synth.seed_for(0, 1591), alias=True)
    b = _run(api, 3001, 72, "bf16", synth.seed_for(0, 1591), alias=True)
    assert torch.equal(a, b)


# (pixels, channels, partial rows): workspaces of the sizes that the query answered before slabs became shorter
SMALL_WORKSPACES = [(6912, 256, 27), (6912, 1024, 108), (3015, 256, 12), (11059, 64, 11), (5000, 12, 8), (2048, 264, 10)]


@pytest.mark.parametrize("n,K,rows", SMALL_WORKSPACES, ids=[f"{n}x{K}" for n, K, _ in SMALL_WORKSPACES])
def test_smaller_workspace(api, n, K, rows):
    """Fewer partial rows than the preferred number give the same sums, in nothing beyond the bytes given; less is refused."""
    buf, ws = U.guarded_workspace(rows * K * 4)
    _run(api, n, K, "bf16", synth.seed_for(0, 1580 + rows % 7), workspace=ws)
    assert U.workspace_guards_intact(buf, rows * K * 4)
    with pytest.raises(RuntimeError):
        _run(api, n, K, "bf16", synth.seed_for(0, 1580 + rows % 7), workspace=ws[:-16])


def test_decoder_sized_tensor(api):
    # one image of the full-resolution decoder output: 884 736 pixels x 256 channels
    _run(api, 768 * 1152, 256, "f16", synth.seed_for(0, 1595))


def test_tensor_beyond_the_last_level_cache(api):
    # 301 MB of dz: stored past the caches (299 MB, the other side of the line, is as test_decoder_sized_tensor)
    _run(api, 294001, 512, "bf16", synth.seed_for(0, 1596))


def test_empty(api):
    dy = torch.empty((0, 16), dtype=torch.float16, device="cuda")
    dz, db = api.bias_relu_bwd(dy, dy.clone(), True)
    torch.cuda.synchronize()
    assert dz.numel() == 0 and torch.count_nonzero(db).item() == 0
