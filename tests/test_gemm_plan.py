"""Which tiles the bf16 contractions run on, as the library itself plans it (host code, no GPU)."""
import pytest

import paper_2410_13333_amd as mls


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


def _cfg(hidden, nq, nkv, d, ffn, seq, mb, n, dtype=0):
    return mls.MlsConfig(hidden, nq, nkv, d, ffn, seq, mb, 1, n, 1e-5, 10000.0, dtype, 0)


def test_weight_gradients_share_a_launch_on_small_layers_only():
    assert mls.wgrad_plan(_cfg(256, 4, 4, 64, 688, 128, 2, 1), 1) == (64, 64)
    for n in (1, 4, 16, 40):
        assert mls.wgrad_plan(_cfg(4096, 32, 32, 128, 11008, 4096, 1, n), n) == (0, 0)
    assert mls.wgrad_plan(_cfg(256, 4, 4, 64, 688, 128, 2, 1, dtype=1), 1) == (0, 0)
    with pytest.raises(mls.MlsError):
        mls.wgrad_plan(_cfg(256, 4, 4, 64, 688, 128, 2, 1), 0)
