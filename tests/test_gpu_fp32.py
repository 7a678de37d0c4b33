"""The all-fp32 storage mode where its kernels change shape: head dimensions that do not fill their 32-column tiles,
sequences around the 32-row blocks and the four-way split of a workgroup, both tile sizes of the GEMM, causality with
non-finite values."""
import numpy as np
import pytest

import synth
from tests.helpers import gpu_step, grad_errors, oracle_step, rel_err, to_host64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,nkv,d,seq,mb", [(2, 1, 16, 1, 2), (4, 2, 48, 31, 1), (6, 2, 96, 33, 2), (4, 1, 112, 129, 1),
                                              (3, 3, 128, 257, 1), (8, 2, 32, 200, 2)])
def test_stage_fp32_against_the_exact_oracle(nq, nkv, d, seq, mb):
    sh = synth.StageShape(hidden=72, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=88, seq=seq, micro_batch=mb, layers=1,
                          microbatches=2, dtype="fp32")
    ys, dxs, g, st = gpu_step(sh, 1000, 2000, 3000, [1, 1])
    st.close()
    rys, rdxs, rg = oracle_step(sh, 1000, 2000, 3000, [1, 1])
    worst, _ = grad_errors(sh, g, rg, 1)
    # about sqrt(K) roundings of 6e-8 per contraction and a few contractions in a row: under 1e-5 at these widths
    for e in [rel_err(a, b) for a, b in zip(ys + dxs, rys + rdxs)] + [worst]:
        assert e <= 1e-5


# either side of the rule for 64x64 tiles that fill the chip at most once, and of a second round of them
@pytest.mark.parametrize("M,N,K,large", [(1024, 1024, 512, True), (512, 1376, 776, True), (1024, 720, 1376, True), (1024, 576, 1376, False),
                                         (1016, 1024, 3080, True), (1024, 512, 512, False), (1032, 1024, 512, False), (1032, 1024, 64, True)])
def test_gemm_fp32_on_one_round_of_large_tiles(M, N, K, large):
    import ctypes
    import paper_2410_13333_amd as mls
    f = mls.lib()._ZN3mls14gemm_f32_largeEiii
    f.restype = ctypes.c_bool
    assert f(M, N, K) is large
    test_gemm_fp32(M, N, K)


# the last one has 512 tiles of 64x64 and runs on them (with a ragged edge), the others on 32x32 tiles; K is not a
# multiple of a 32-deep piece, shorter than the four wavefronts' pieces, or one piece
@pytest.mark.parametrize("M,N,K", [(8, 8, 8), (32, 40, 32), (40, 96, 104), (256, 264, 136), (2040, 1016, 72)])
def test_gemm_fp32(M, N, K):
    import torch
    import paper_2410_13333_amd as mls
    g = torch.Generator(device="cpu").manual_seed(M + N + K)
    a, b, r = (torch.randn(s, generator=g).cuda() for s in ((M, K), (K, N), (M, N)))
    ref = to_host64(a) @ to_host64(b)
    c = torch.empty(M, N, device="cuda")
    mls.gemm(0, a, b, c, r)
    assert rel_err(to_host64(c), ref + to_host64(r)) < 1e-6
    mls.gemm(1, a, b.t().contiguous(), c)
    assert rel_err(to_host64(c), ref) < 1e-6
    acc = torch.full((M, N), 0.5, device="cuda")
    mls.gemm(2, a.t().contiguous(), b, acc)
    assert rel_err(to_host64(acc), 0.5 + ref) < 1e-6


@pytest.mark.parametrize("K", [8, 96, 136, 1000])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_both_tile_sizes_have_the_same_bits(mode, K):
    """480 tiles of 64x64 with ragged edges, against their upper left corner computed alone on 32x32 tiles; the stretch of a
    last piece that lies beyond K, and what it would read, hold no part of the result (NaN rows behind the operands)."""
    import torch
    import paper_2410_13333_amd as mls
    M, N, m, n = 1240, 1528, 264, 392
    g = torch.Generator(device="cpu").manual_seed(K)
    a, b = torch.randn(M, K, generator=g).cuda(), torch.randn(K, N, generator=g).cuda()
    ref = to_host64(a) @ to_host64(b)

    def framed(t):  # the tensor inside a wider and longer one of NaN
        big = torch.full((t.shape[0] + 64, t.shape[1] + 64), float("nan"), device="cuda")
        big[:t.shape[0], :t.shape[1]] = t
        return big[:t.shape[0], :t.shape[1]]
    at, bt = (a.t().contiguous() if mode == 2 else a), (b.t().contiguous() if mode == 1 else b)
    out = torch.zeros(M, N, device="cuda")
    mls.gemm(mode, framed(at), framed(bt), out)
    assert rel_err(to_host64(out), ref) < 1e-6
    part = torch.zeros(m, n, device="cuda")
    mls.gemm(mode, framed(at[:, :m] if mode == 2 else at[:m]), framed(bt[:n] if mode == 1 else bt[:, :n]), part)
    assert torch.equal(part, out[:m, :n])


def test_weight_gradients_over_an_odd_number_of_tokens_on_large_tiles():
    sh = synth.StageShape(hidden=776, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=1400, seq=333, micro_batch=1, layers=1,
                          microbatches=2, dtype="fp32")
    ys, dxs, g, st = gpu_step(sh, 1000, 2000, 3000, [1, 1])
    st.close()
    rys, rdxs, rg = oracle_step(sh, 1000, 2000, 3000, [1, 1])
    for e in [rel_err(a, b) for a, b in zip(ys + dxs, rys + rdxs)] + [grad_errors(sh, g, rg, 1)[0]]:
        assert e <= 1e-5


# one launch for the weight gradients of all micro-batches: 32x32 tiles, then 64x64 ones; pieces shorter than the four wavefronts' shares,
# of one token, not whole, whole; more micro-batches than a launch takes; a last call that adds to the first
@pytest.mark.parametrize("hidden,ffn,seq,n", [(72, 88, 1, 3), (72, 88, 40, 17), (72, 88, 96, 2), (264, 136, 133, 4), (520, 1400, 37, 3),
                                              (520, 1400, 64, 2)])
def test_weight_gradients_over_many_micro_batches(hidden, ffn, seq, n):
    sh = synth.StageShape(hidden=hidden, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=ffn, seq=seq, micro_batch=1, layers=1,
                          microbatches=n, dtype="fp32")
    for interleave in (False, True):
        ys, dxs, g, st = gpu_step(sh, 1000, 2000, 3000, [1] * n, interleave=interleave)
        st.close()
        rys, rdxs, rg = oracle_step(sh, 1000, 2000, 3000, [1] * n)
        for e in [rel_err(a, b) for a, b in zip(ys + dxs, rys + rdxs)] + [grad_errors(sh, g, rg, 1)[0]]:
            assert e <= 1e-5


# 32x32 tiles and 64x64 ones; tokens that are whole pieces of the four wavefronts or accumulators, and ones that are not
@pytest.mark.parametrize("hidden,nq,ffn,seq,n,tile", [(256, 4, 480, 222, 3, 32), (192, 3, 600, 384, 2, 32), (136, 2, 328, 37, 16, 32), (512, 8, 1376, 512, 2, 64),
                                                      (512, 4, 1400, 330, 4, 64), (520, 8, 1376, 45, 9, 64)])
def test_weight_gradients_of_one_call_are_as_exact_as_those_of_many(hidden, nq, ffn, seq, n, tile):
    """A call over n micro-batches adds up n sums, as n calls do: within 2 % as far from the exact gradients as those (64x64 tiles: the same
    bits), where one chain of additions through all of them was up to a quarter further."""
    import torch
    import paper_2410_13333_amd as mls
    st = mls.Stage(hidden, nq, nq, 64, ffn, seq, 1, 1, n, seed=1011, dtype="fp32")
    assert mls.wgrad_launch(st.cfg, n)[1] == tile
    gen = torch.Generator(device="cuda").manual_seed(seq)
    x, dy = (torch.randn(n, 1, seq, hidden, device="cuda", generator=gen) for _ in range(2))
    y, dx = torch.empty_like(x[0]), torch.empty_like(dy)
    one, many = (torch.empty(st.grad_elems, device="cuda") for _ in range(2))
    pairs = {"w_d": ("z", "dy"), "w_gu": ("b", "dgu"), "w_o": ("o", "dh"), "w_qkv": ("a", "dqkv")}
    ref = dict.fromkeys(pairs, 0.0)
    for i in range(n):
        st.forward(x[i], 1, y)
        left = {w: st.debug_read(a).double() for w, (a, _) in pairs.items()}
        st.backward(dy[i:i + 1], many, 1, dx[i:i + 1], overwrite=i == 0)
        for w, (_, b) in pairs.items():
            ref[w] = ref[w] + left[w].t().contiguous() @ st.debug_read(b).double()
    for i in range(n):
        st.forward(x[i], 1, y)
    st.backward(dy, one, n, dx, overwrite=True)
    for w in pairs:
        off, r, c = st.param_layout(0, w)
        e = [((g[off:off + r * c].view(r, c).double() - ref[w]).norm() / ref[w].norm()).item() for g in (one, many)]
        assert e[0] <= 1.02 * e[1], (w, e)
        assert tile == 32 or torch.equal(one[off:off + r * c], many[off:off + r * c]), w
    st.close()


# the backward in one launch, up to a number of blocks of 32 query rows that depends on the head width, the blocks of a sequence and the grouping,
# or apart; the query heads of a group apart, where their key blocks are few and long, or in one workgroup
@pytest.mark.parametrize("nq,nkv,d,seq,mb,together,apart", [
    (6, 2, 64, 33, 1, True, True), (6, 3, 80, 97, 3, True, True), (34, 17, 64, 481, 1, True, False), (34, 17, 64, 513, 1, False, False),
    (16, 15 + 1, 64, 200, 2, True, False), (32, 8, 16, 250, 2, True, True), (3, 1, 128, 160, 2, True, True), (46, 23, 128, 129, 3, False, False),
    (8, 4, 64, 32, 1, True, False), (45, 15, 16, 128, 1, True, True), (46, 23, 16, 128, 1, True, False), (64, 32, 32, 118, 2, False, False),
    (45, 45, 64, 128, 1, True, False), (46, 46, 64, 128, 1, False, False), (51, 51, 32, 160, 1, True, False), (48, 48, 48, 256, 1, True, False),
    (49, 49, 48, 256, 1, False, False), (32, 32, 80, 288, 1, True, False), (33, 33, 80, 288, 1, False, False), (57, 57, 96, 224, 1, True, False),
    (58, 58, 96, 224, 1, False, False), (45, 45, 112, 384, 1, True, False), (46, 46, 112, 384, 1, False, False), (41, 41, 112, 416, 1, False, False)])
def test_backward_launches_on_either_side_of_their_rules(nq, nkv, d, seq, mb, together, apart):
    import ctypes
    import paper_2410_13333_amd as mls
    f, w = mls.lib()._ZN3mls16bwd_f32_togetherEiiiii, mls.lib()._ZN3mls27attn_bwd_f32_scratch_floatsEiiiii
    f.restype, w.restype = ctypes.c_bool, ctypes.c_size_t
    assert f(mb, seq, nq, nkv, d) is together and (w(mb, seq, nq, nkv, d) > 0) is apart
    test_stage_fp32_against_the_exact_oracle(nq, nkv, d, seq, mb)


# rotary, SwiGLU and its backward as epilogues of the products: pairs of columns 8 to 64 apart and ffn apart, ending anywhere in a tile; 32x32
# tiles of one row to several, then 64x64 ones (q|k|v: 340 rows x 1536 columns and more; gate|up, its backward: 2 728, 2 720 columns)
@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,seq", [(72, 1, 1, 16, 8, 1), (72, 3, 1, 48, 24, 33), (64, 2, 2, 80, 40, 70), (40, 2, 1, 112, 1000, 5),
                                                     (264, 18, 3, 64, 1360, 1021), (136, 30, 10, 48, 2728, 517), (72, 5, 5, 128, 2720, 600)])
def test_epilogues_of_the_products(hidden, nq, nkv, d, ffn, seq):
    sh = synth.StageShape(hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=ffn, seq=seq, micro_batch=1, layers=1,
                          microbatches=1, dtype="fp32")
    ys, dxs, g, st = gpu_step(sh, 1000, 2000, 3000, [1])
    st.close()
    rys, rdxs, rg = oracle_step(sh, 1000, 2000, 3000, [1])
    for e in [rel_err(a, b) for a, b in zip(ys + dxs, rys + rdxs)] + [grad_errors(sh, g, rg, 1)[0]]:
        assert e <= 1e-5


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_a_non_finite_position_reaches_no_earlier_one(bad):
    import torch
    import paper_2410_13333_amd as mls
    sh = synth.StageShape(hidden=64, n_q_heads=2, n_kv_heads=1, head_dim=48, ffn=64, seq=70, micro_batch=1, layers=1,
                          microbatches=1, dtype="fp32")
    st = mls.Stage.from_shape(sh, seed=1000)
    x = synth.to_device(synth.make_x(sh, 2000, 0)[0], "fp32")
    y0, y1 = torch.empty_like(x), torch.empty_like(x)
    st.forward(x, 1, y0)
    st.reset()
    x[0, 45, 3] = bad
    st.forward(x, 1, y1)
    st.close()
    assert rel_err(to_host64(y1[0, :45]), to_host64(y0[0, :45])) < 1e-6
    assert not bool(torch.isfinite(y1[0, 45:]).all(dim=-1).any())
