"""The stage's contraction kernel on its own, against fp64 matmul of the same bf16 operands."""
import numpy as np
import pytest

from tests.helpers import rel_err, to_host64, worst_block
from tests.test_gemm_plan import GEMM_TILES, TN_TILES

pytestmark = pytest.mark.gpu

SHAPES = [(256, 768, 256), (256, 1376, 256), (256, 256, 688), (392, 520, 328), (8, 8, 8), (1024, 2048, 512),
          (4096, 4096, 1024), (520, 4104, 264), (4096, 22016, 136),
          # tiling plans: whole rounds of 256x256 tiles + a 128x128 tail; 256x128 tiles only; an odd number of k-tiles
          (4096, 5120, 264), (2048, 4096, 200), (4096, 4096, 96)]


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_bf16_three_modes(M, N, K):
    import torch
    import paper_2410_13333_amd as mls
    g = torch.Generator(device="cpu").manual_seed(M * 7 + N * 3 + K)
    a = torch.randn(M, K, generator=g).to(torch.bfloat16).cuda()
    b = torch.randn(K, N, generator=g).to(torch.bfloat16).cuda()
    r = torch.randn(M, N, generator=g).to(torch.bfloat16).cuda()
    a64, b64, r64 = to_host64(a), to_host64(b), to_host64(r)
    c = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    mls.gemm(0, a, b, c)
    assert rel_err(to_host64(c), a64 @ b64) < 4e-3
    mls.gemm(0, a, b, c, r)
    assert rel_err(to_host64(c), a64 @ b64 + r64) < 4e-3
    mls.gemm(1, a, b.t().contiguous(), c)
    assert rel_err(to_host64(c), a64 @ b64) < 4e-3
    acc = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda")
    at = a.t().contiguous()
    mls.gemm(2, at, b, acc)
    mls.gemm(2, at, b, acc)
    torch.cuda.synchronize()
    assert rel_err(to_host64(acc), 0.5 + 2 * (a64 @ b64)) < 1e-5


@pytest.mark.parametrize("M,N,K", [(4096, 4096, 64), (4096, 4096, 128), (4096, 4096, 192), (4096, 4096, 320),
                                   (4000, 4104, 448), (4096, 4096, 32), (4088, 4096, 160)])
def test_bf16_16x16x32_kernel_at_awkward_depths(M, N, K):
    """At least 256 tiles of 256x256, so that the problem runs on the 16x16x32 kernel: contraction depths of one to a
    few k-tiles (prologue with nothing behind it, rings that do not come round, a k-tile count that is no multiple of
    the loop's period), ragged last tile rows, a column remainder beside it."""
    import torch
    import paper_2410_13333_amd as mls
    g = torch.Generator(device="cpu").manual_seed(M + 3 * N + 7 * K)
    a = torch.randn(M, K, generator=g).to(torch.bfloat16).cuda()
    b = torch.randn(K, N, generator=g).to(torch.bfloat16).cuda()
    r = torch.randn(M, N, generator=g).to(torch.bfloat16).cuda()
    ref = to_host64(a) @ to_host64(b)
    c = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    mls.gemm(0, a, b, c, r)
    assert rel_err(to_host64(c), ref + to_host64(r)) < 4e-3
    mls.gemm(1, a, b.t().contiguous(), c)
    assert rel_err(to_host64(c), ref) < 4e-3
    acc = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda")
    at = a.t().contiguous()
    mls.gemm(2, at, b, acc)
    mls.gemm(2, at, b, acc)
    torch.cuda.synchronize()
    assert rel_err(to_host64(acc), 0.5 + 2 * ref) < 1e-5


def _framed(r, c, g):
    """An r x c matrix of N(0, 1) in a buffer that is wider and longer, NaN around it: what lies behind the end of the
    contraction in memory (the rest of a row, the rows behind the last one) must not be looked at."""
    import torch
    buf = torch.full((r + 72, c + 72), float("nan"), dtype=torch.bfloat16, device="cuda")
    buf[:r, :c] = torch.randn(r, c, device="cuda", generator=g)
    return buf[:r, :c]


def _framed_product(mode, M, N, K):
    import torch
    import paper_2410_13333_amd as mls
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    a, b = _framed(K, M, g) if mode == 2 else _framed(M, K, g), _framed(N, K, g) if mode == 1 else _framed(K, N, g)
    ref = (a.double().t().contiguous() if mode == 2 else a.double()) @ (b.double().t().contiguous() if mode == 1 else b.double())
    if mode == 2:
        c = torch.full((M, N), 0.5, device="cuda")
        mls.gemm(2, a, b, c)
        # fp32 sums: a rounding of 6e-8 per step of the chain and the addition
        assert worst_block(c, 0.5 + ref) < 1e-5
        return
    c = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    mls.gemm(mode, a, b, c)
    assert worst_block(c, ref) < 4e-3  # one rounding to bf16
    if mode == 0:
        r = torch.randn(M, N, device="cuda", generator=g).to(torch.bfloat16)
        mls.gemm(0, a, b, c, r)
        assert worst_block(c, ref + r.double()) < 4e-3


# a depth that ends inside a k-tile in every way, on 256x256 tiles with a remainder beside them (NN, NT; TN from 1000 on)
@pytest.mark.parametrize("mode,K", [(m, K) for m in (0, 1) for K in (8, 40, 72, 104, 136, 200, 264, 328)] +
                         [(2, K) for K in (1000, 1032, 1096, 1544)])
def test_bf16_256_tiles_over_contractions_that_end_inside_a_tile(mode, K):
    import paper_2410_13333_amd as mls
    assert mls.gemm_plan(mode, 3848, 4360, K)[0] == 4096
    _framed_product(mode, 3848, 4360, K)


@pytest.mark.parametrize("mode,shape", [(m, s) for s, _ in GEMM_TILES for m in (0, 1)] + [(2, s) for s, _ in TN_TILES])
def test_bf16_every_plan(mode, shape):
    """Every tile size alone and behind whole 256x256 tiles, in each form (tests/test_gemm_plan.py holds the plans)."""
    _framed_product(mode, *shape)


def test_fp32_three_modes():
    import torch
    import paper_2410_13333_amd as mls
    M, N, K = 136, 200, 72
    g = torch.Generator(device="cpu").manual_seed(5)
    a, b = torch.randn(M, K, generator=g).cuda(), torch.randn(K, N, generator=g).cuda()
    ref = to_host64(a) @ to_host64(b)
    c = torch.empty(M, N, device="cuda")
    mls.gemm(0, a, b, c)
    assert rel_err(to_host64(c), ref) < 1e-6
    mls.gemm(1, a, b.t().contiguous(), c)
    assert rel_err(to_host64(c), ref) < 1e-6
    acc = torch.zeros(M, N, device="cuda")
    mls.gemm(2, a.t().contiguous(), b, acc)
    assert rel_err(to_host64(acc), ref) < 1e-6


@pytest.mark.parametrize("M,N,K", [(136, 200, 72), (8, 264, 520)])
def test_bf16_register_staged_kernel_for_operands_beyond_31_bit_offsets(M, N, K):
    """An operand whose rows lie 4 MiB apart spans more than 2 GiB, which the main kernel's 31-bit buffer offsets
    cannot address: the call runs on the register-staged kernel.  All three modes, ragged tiles."""
    import torch
    import paper_2410_13333_amd as mls
    LD = 1 << 21                                    # elements between rows: (rows + 512) * LD * 2 B >= 2^31
    g = torch.Generator(device="cpu").manual_seed(M + N + K)
    big = torch.zeros(max(M, N, K), LD, dtype=torch.bfloat16, device="cuda")

    def wide(t):                                    # t's values in the first columns of the wide buffer
        v = big[:t.shape[0], :t.shape[1]]
        v.copy_(t)
        return v
    a = torch.randn(M, K, generator=g).to(torch.bfloat16).cuda()
    b = torch.randn(K, N, generator=g).to(torch.bfloat16).cuda()
    bt = b.t().contiguous()
    r = torch.randn(M, N, generator=g).to(torch.bfloat16).cuda()
    a64, b64, r64 = to_host64(a), to_host64(b), to_host64(r)
    ref = a64 @ b64
    c = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    mls.gemm(0, wide(a), b, c, r)                   # NN, A wide
    torch.cuda.synchronize()
    assert rel_err(to_host64(c), ref + r64) <= 4e-3
    mls.gemm(1, wide(a), bt, c)                     # NT, A wide
    torch.cuda.synchronize()
    assert rel_err(to_host64(c), ref) <= 4e-3
    mls.gemm(1, a, wide(bt), c)                     # NT, B wide
    torch.cuda.synchronize()
    assert rel_err(to_host64(c), ref) <= 4e-3
    acc = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda")
    mls.gemm(2, wide(a.t().contiguous()), b, acc)   # TN, A wide, twice: it accumulates
    mls.gemm(2, wide(a.t().contiguous()), b, acc)
    torch.cuda.synchronize()
    assert rel_err(to_host64(acc), 0.5 + 2 * ref) <= 1e-5


def test_empty_contraction():
    """K = 0 (through the C ABI directly: the operands are valid pointers to nothing): C = R for the bf16 modes,
    C unchanged for the accumulating one."""
    import ctypes as C
    import torch
    import paper_2410_13333_amd as mls
    M, N = 264, 136
    buf = torch.ones(M, 8, dtype=torch.bfloat16, device="cuda")
    r = torch.randn(M, N, device="cuda").to(torch.bfloat16)
    c = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    acc = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda")
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    p = lambda t: C.c_void_p(t.data_ptr())
    L = mls.lib()
    assert L.mls_gemm(mls.MLS_BF16, 0, p(buf), 8, p(buf), N, p(c), N, p(r), M, N, 0, st) == 0
    torch.cuda.synchronize()
    assert torch.equal(c, r)
    assert L.mls_gemm(mls.MLS_BF16, 1, p(buf), 8, p(buf), 8, p(c), N, None, M, N, 0, st) == 0
    assert L.mls_gemm(mls.MLS_BF16, 2, p(buf), M, p(buf), N, p(acc), N, None, M, N, 0, st) == 0
    torch.cuda.synchronize()
    assert float(c.float().abs().max()) == 0.0 and float((acc - 0.5).abs().max()) == 0.0


# by the plan of gemm_bf16_dispatch.hip (NN and NT): 64x64 tiles; 128x64; 128x128; 256x128; 256x256 tiles with a 64x64 and a
# 128x64 tail.
# K: one k-tile that is not full, a last k-tile of one 16-byte chunk, more k-tiles than stages
@pytest.mark.parametrize("M,N,K", [(72, 136, 24), (72, 136, 1032), (1000, 2056, 1096), (2040, 2040, 392), (2000, 3000, 1032),
                                   (2048, 4096, 328), (4096, 4360, 136), (4088, 5128, 200)])
def test_bf16_every_tile_size(M, N, K):
    test_bf16_three_modes(M, N, K)


@pytest.mark.parametrize("M,N,K", [(72, 136, 77), (1000, 2056, 1091), (2040, 2040, 390), (2000, 3000, 1025), (8200, 4104, 1091),
                                   (4096, 4096, 45)])
def test_bf16_weight_gradient_over_any_token_count(M, N, K):
    """C += A^T B over K tokens, K no multiple of 8 (the C ABI's mls_gemm refuses such a K; a stage's weight gradients
    have it): through a one-layer stage's w_d, whose operands are captured."""
    import synth
    import torch
    import paper_2410_13333_amd as mls
    sh = synth.StageShape(hidden=N // 8 * 8, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=M // 8 * 8, seq=K, micro_batch=1,
                          layers=1, microbatches=2)
    st = mls.Stage.from_shape(sh, seed=1)
    x = torch.randn(2, 1, K, sh.hidden, device="cuda").to(torch.bfloat16)
    dy, dx, y = torch.randn_like(x), torch.empty_like(x), torch.empty_like(x[0])
    g = torch.full((st.grad_elems,), 0.5, device="cuda")
    ref = 0.5
    for i in range(2):
        st.forward(x[i], 1, y)
    z = [to_host64(st.debug_read("z", 0, i)) for i in range(2)]
    st.backward(dy, g, 2, dx)
    for i in range(2):  # two pieces in one contraction
        ref = ref + z[i].T @ to_host64(dy[i].reshape(K, -1))
    off, r, c = st.param_layout(0, "w_d")
    got = to_host64(g[off:off + r * c]).reshape(r, c)
    st.close()
    assert rel_err(got, ref) < 1e-5


@pytest.mark.parametrize("ldc", [(1 << 25) - 8, 1 << 25])
def test_fp32_results_in_very_wide_rows(ldc):
    """Row strides on either side of 2^25, up to which 16 rows lie within the 31 bits of a store's offset; nothing outside the
    result's columns changes."""
    import torch
    import paper_2410_13333_amd as mls
    g = torch.Generator(device="cpu").manual_seed(5)
    a = torch.randn(128, 40, generator=g).to(torch.bfloat16).cuda()
    b = torch.randn(128, 72, generator=g).to(torch.bfloat16).cuda()
    flat = torch.full((40 * ldc,), 0.25, dtype=torch.float32, device="cuda")
    c = flat.view(40, ldc)[:, 8:80]
    mls.gemm(2, a, b, c)
    assert rel_err(to_host64(c), 0.25 + to_host64(a).T @ to_host64(b)) < 1e-5
    c.fill_(0.25)
    assert bool((flat == 0.25).all())
