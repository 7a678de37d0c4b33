"""Which tiles the bf16 contractions run on, as the library itself plans it (host code, no GPU)."""
import ctypes

import pytest

import paper_2410_13333_amd as mls

# Shapes that the GPU tests take through each tile size, with the plan they rely on: (leading columns on 256x256 tiles, rows,
# columns of the tiles behind them).  test_plan_of_the_tested_shapes fails when a change of the plan drops one.
GEMM_TILES = [  # NN and NT
    ((72, 136, 24), (0, 64, 64)), ((72, 136, 1032), (0, 64, 64)), ((1000, 2056, 1096), (0, 128, 64)), ((2040, 2040, 392), (0, 128, 128)),
    ((2000, 3000, 1032), (0, 256, 128)), ((4088, 4096, 192), (4096, 0, 0)), ((4096, 4360, 136), (4096, 64, 64)),
    ((4088, 5128, 192), (4096, 128, 64)), ((4088, 5064, 264), (4096, 128, 128)), ((4088, 5448, 64), (4096, 256, 128))]
TN_TILES = [
    ((72, 136, 136), (0, 64, 64)), ((4088, 456, 1096), (0, 128, 64)), ((3848, 968, 136), (0, 128, 128)), ((2040, 3912, 264), (0, 256, 128)),
    ((4088, 3720, 520), (3720, 0, 0)), ((4088, 4104, 776), (4096, 64, 64)), ((4088, 5128, 800), (4096, 128, 64)),
    ((3848, 4936, 776), (4096, 128, 128)), ((3848, 5832, 776), (4096, 256, 128))]
# hidden, q heads, kv heads, head dim, seq, micro-batch
ROPE_TILES = [
    ((264, 3, 1, 64, 129, 1), (0, 64, 128)), ((264, 3, 1, 128, 129, 1), (0, 64, 128)), ((264, 48, 16, 128, 129, 2), (0, 128, 128)),
    ((520, 48, 16, 64, 257, 2), (0, 128, 128)), ((264, 48, 16, 128, 257, 2), (0, 256, 128)), ((72, 32, 16, 64, 700, 2), (0, 256, 128)),
    ((328, 48, 16, 128, 999, 2), (8192, 128, 128)), ((328, 64, 16, 128, 999, 2), (8192, 256, 128))]
# hidden, ffn, tokens
SWIGLU_TILES = [
    ((136, 64, 72), (0, 64, 128)), ((520, 2720, 514), (0, 128, 128)), ((520, 4128, 700), (0, 256, 128)),
    ((264, 4128, 999), (8256, 0, 0)), ((136, 4128, 1998), (8192, 64, 128)), ((136, 2720, 4100), (3840, 256, 128))]
# hidden, q heads, kv heads, head dim, ffn, seq, micro-batch, micro-batches: one shared launch, stored or added to
WGRAD_TILES = [
    ((264, 1, 1, 64, 680, 129, 1, 1), (64, 64)), ((264, 1, 1, 64, 352, 129, 1, 1), (64, 64)),
    ((520, 8, 2, 64, 680, 300, 2, 3), (128, 64)), ((1032, 4, 2, 64, 352, 700, 2, 1), (128, 64)),
    ((1032, 8, 2, 64, 680, 129, 1, 2), (128, 128)), ((520, 2, 1, 64, 2048, 129, 1, 2), (128, 128)),
    ((2056, 4, 1, 128, 680, 129, 1, 3), (256, 128)), ((1032, 4, 1, 64, 2048, 129, 1, 3), (256, 128))]


def _cfg(hidden, nq, nkv, d, ffn, seq, mb, n, dtype=0):
    return mls.MlsConfig(hidden, nq, nkv, d, ffn, seq, mb, 1, n, 1e-5, 10000.0, dtype, 0)


def _k_tiles(n):
    return (n + 63) // 64 * 64


def test_plan_of_the_tested_shapes():
    for shape, plan in GEMM_TILES:
        assert mls.gemm_plan(0, *shape) == mls.gemm_plan(1, *shape) == plan, shape
    for shape, plan in TN_TILES:
        assert mls.gemm_plan(2, *shape) == plan, shape
    for (h, nq, nkv, d, seq, mb), plan in ROPE_TILES:
        assert mls.gemm_plan(4, seq * mb, (nq + 2 * nkv) * d, _k_tiles(h)) == plan, (h, nq, nkv, d, seq, mb)
    for (h, ffn, T), plan in SWIGLU_TILES:
        assert mls.gemm_plan(3, T, 2 * ffn, _k_tiles(h)) == plan, (h, ffn, T)
    for shape, tile in WGRAD_TILES:
        assert mls.wgrad_plan(_cfg(*shape), shape[-1]) == mls.wgrad_plan(_cfg(*shape), shape[-1], True) == tile, shape


# about a whole round or more of 256x256 tiles: the contraction length does not decide whether they are used
@pytest.mark.parametrize("mode,M,N,K", [(0, 8192, 8192, 8168), (1, 8192, 8192, 8168), (0, 4096, 11008, 1000), (1, 4096, 4096, 4104),
                                        (2, 11008, 4096, 2849 * 3), (2, 4096, 4096, 4095), (2, 4096, 22016, 2 * 4095)])
def test_large_products_of_any_depth_get_the_256_tiles(mode, M, N, K):
    big = mls.gemm_plan(mode, M, N, K)[0]
    assert big >= N // 2
    assert big == mls.gemm_plan(mode, M, N, (K + 63) // 64 * 64)[0]


def test_the_fused_forms_take_whole_k_tiles_there():
    assert mls.gemm_plan(3, 4096, 22016, 4096)[0] > 0 and mls.gemm_plan(4, 4096, 12288, 4096)[0] > 0
    assert mls.gemm_plan(3, 4096, 22016, 4072)[0] == 0 and mls.gemm_plan(4, 4096, 12288, 4072)[0] == 0


def test_refusals():
    for bad in [(5, 8, 8, 8), (-1, 8, 8, 8), (0, 0, 8, 8), (0, 8, 1 << 25, 8), (0, 8, 8, 0)]:
        with pytest.raises(mls.MlsError):
            mls.gemm_plan(*bad)


# hidden, q heads, kv heads, head dim, ffn, seq, micro-batch, micro-batches -> (shared, tile, weight with columns apart, from, tile there)
WGRAD_256 = [
    ((2048, 16, 16, 128, 5504, 700, 1, 3), (1, 256, 256, 1, 10752, 64, 64)),    # 776 tiles: three whole rounds, the gate/up weights' last columns apart
    ((2056, 16, 8, 128, 5512, 2049, 1, 1), (1, 256, 256, 0, 1792, 128, 64)),    # ragged rows, columns and pieces, a last gate/up group that is not full
    ((3072, 24, 8, 128, 8192, 1088, 2, 1), (1, 256, 256, -1, 0, 0, 0)),         # a last round that is kept
    ((2800, 43, 43, 64, 1344, 930, 1, 2), (0, 0, 0, -1, 0, 0, 0)),              # fewer than 32 k-tiles: launches apart
    ((1032, 8, 8, 128, 5688, 2285, 1, 2), (0, 0, 0, -1, 0, 0, 0))]              # fewer than 512 tiles


def test_how_the_weight_gradients_of_a_layer_run():
    for shape, launch in WGRAD_256:
        cfg = _cfg(*shape)
        assert mls.wgrad_launch(cfg, shape[-1]) == mls.wgrad_launch(cfg, shape[-1], True) == launch, shape
        assert mls.wgrad_plan(cfg, shape[-1]) == (0, 0)
    for shape, tile in WGRAD_TILES:
        assert mls.wgrad_launch(_cfg(*shape), shape[-1]) == (1, *tile, -1, 0, 0, 0), shape
    for n in (1, 4, 16, 40):
        assert mls.wgrad_launch(_cfg(4096, 32, 32, 128, 11008, 4096, 1, n), n) == (1, 256, 256, 1, 21760, 64, 64)
    # fp32 storage: 64x64 tiles from 320 on
    assert mls.wgrad_launch(_cfg(512, 8, 4, 64, 1376, 256, 2, 2, dtype=1), 2) == (1, 64, 64, -1, 0, 0, 0)
    assert mls.wgrad_launch(_cfg(256, 4, 4, 64, 688, 128, 2, 1, dtype=1), 1) == (1, 32, 32, -1, 0, 0, 0)
    for bad in ((0, False), (-1, True)):
        with pytest.raises(mls.MlsError):
            mls.wgrad_launch(_cfg(256, 4, 4, 64, 688, 128, 2, 1), *bad)


def test_weight_gradients_share_a_launch_of_smaller_tiles_on_small_layers_only():
    assert mls.wgrad_plan(_cfg(256, 4, 4, 64, 688, 128, 2, 1), 1) == (64, 64)
    for n in (1, 4, 16, 40):
        assert mls.wgrad_plan(_cfg(4096, 32, 32, 128, 11008, 4096, 1, n), n) == (0, 0)
    assert mls.wgrad_plan(_cfg(256, 4, 4, 64, 688, 128, 2, 1, dtype=1), 1) == (0, 0)
    with pytest.raises(mls.MlsError):
        mls.wgrad_plan(_cfg(256, 4, 4, 64, 688, 128, 2, 1), 0)


def test_short_contractions_into_fp32_results_take_small_tiles():
    """What such a product costs is the traffic of its result, which several workgroups on a CU overlap with the products."""
    assert mls.wgrad_plan(_cfg(1192, 32, 32, 64, 4120, 186, 1, 1), 1)[1] == 64
    assert mls.wgrad_plan(_cfg(2048, 32, 4, 128, 4872, 49, 1, 1), 1)[1] == 64
    assert mls.gemm_plan(2, 4120, 1192, 186)[0] == 0


# us measured with the tiles named here / with the 128x64 ones that the average CU speaks for: 260 to 324 of them, two on some CUs only
@pytest.mark.parametrize("M,N,K,us", [(1141, 2152, 5248, (36, 48)), (3350, 768, 2944, (23, 29)), (393, 4864, 23424, (138, 187)),
                                      (1650, 1280, 11840, (73, 96))])
def test_a_cu_with_a_workgroup_more_than_the_others_counts(M, N, K, us):
    for mode in (0, 1):
        assert mls.gemm_plan(mode, M, N, K) == (0, 128, 128), us


# fp32: 64x64 tiles where their rounds of whole chains are estimated shorter than those of the 32x32 ones (us, 32x32 / 64x64)
@pytest.mark.parametrize("M,N,K,large", [
    (768, 768, 64, True), (2120, 232, 24, True), (1536, 768, 128, True), (768, 768, 256, True), (768, 768, 400, True),  # 7.2 / 5.9, 7.2 / 5.8, 11.2 / 8.9, 9.2 / 8.1, 13.1 / 10.8
    (768, 768, 384, True), (768, 768, 512, True), (1152, 768, 4096, True), (1024, 704, 768, True),                    # 10.9 / 10.1, 12.3 / 12.0, 83 / 70, 19.4 / 17.2
    (2568, 264, 1064, True), (1016, 1024, 3080, True), (1000, 4096, 1024, True),                                      # 29.3 / 22.1, 67 / 55, 92 / 74
    (512, 1024, 256, False), (256, 256, 256, False), (512, 2752, 512, True), (512, 512, 2752, False),                 # 6.2 / 8.3, 5.8 / 7.9, 23.0 / 22.4, 16.9 / 47.6
    (1152, 1024, 768, False), (1024, 576, 768, False), (288, 4096, 4672, False), (624, 2048, 1984, False)])           # 24.7 / 29.0, 16.0 / 16.6, 120 / 156, 58 / 68
def test_fp32_tiles(M, N, K, large):
    f = mls.lib()._ZN3mls14gemm_f32_largeEiii
    f.restype = ctypes.c_bool
    assert f(M, N, K) is large
