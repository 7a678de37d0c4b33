"""GPU parity of the HIP decoder stage against the CPU oracle, through the C ABI (ctypes binding).

Tolerances (relative Frobenius error per tensor, fp64 metric):
  fp32 storage: 1e-4 for every output and gradient (validates the algorithm with no bf16 in the way);
  bf16 storage: 1e-2 for y, dX and the parameter gradients against the oracle fed the same bf16 inputs;
  weight-gradient contraction + fp32 accumulation given identical bf16 operands: 1e-4."""
import ctypes

import numpy as np
import pytest

import synth
from tests.helpers import (gpu_step, grad_errors, oracle_step, rel_err, round_bf16, storage_bits, to_device,
                           to_host64, worst_block)
from tests.test_gemm_plan import ROPE_TILES, SWIGLU_TILES, WGRAD_256, WGRAD_TILES

pytestmark = pytest.mark.gpu

TINY = synth.CONFIGS["tiny"]
# grouped KV heads, ragged everything: seq not a multiple of any tile, ffn = 8*41, 3 layers, 3 micro-batches
RAGGED = synth.StageShape(hidden=192, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=328, seq=200, micro_batch=2,
                          layers=3, microbatches=3)
# ffn a multiple of 32 (SwiGLU runs fused into the contractions around it), 2 ffn = 704 not a multiple of any tile
FUSED_RAGGED = synth.StageShape(hidden=192, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=352, seq=200, micro_batch=2,
                                layers=3, microbatches=3)
GQA128 = synth.StageShape(hidden=256, n_q_heads=4, n_kv_heads=1, head_dim=128, ffn=512, seq=328, micro_batch=1,
                          layers=1, microbatches=2)


def _check(sh, ks, tol, interleave=False):
    ys, dxs, g, st = gpu_step(sh, 1000, 2000, 3000, ks, interleave)
    assert st.inflight == 0
    st.close()
    refs = [("exact", tol, oracle_step(sh, 1000, 2000, 3000, ks))]     # the exact fp64 oracle is the only bar
    for kind, t, (rys, rdxs, rg) in refs:
        ey = max(rel_err(ys[mb], rys[mb]) for mb in range(len(ks)))
        ex = max(rel_err(dxs[mb], rdxs[mb]) for mb in range(len(ks)))
        worst, errs = grad_errors(sh, g, rg, max(ks) if ks else 0)
        print(f"[{sh.dtype} h={sh.hidden} S={sh.seq} ks={ks}] vs {kind} oracle: y {ey:.2e} dx {ex:.2e} grads {worst:.2e}")
        assert ey <= t and ex <= t, (kind, ey, ex)
        assert worst <= t, (kind, sorted(errs.items(), key=lambda kv: -kv[1])[:4])
    return ys, dxs, g


def test_weights_match_the_generator_bit_for_bit():
    import paper_2410_13333_amd as mls
    for dtype in ("bf16", "fp32"):
        sh = TINY.with_(dtype=dtype)
        st = mls.Stage.from_shape(sh, seed=1000)
        bits, _ = synth.make_params(sh, 1000)
        assert np.array_equal(storage_bits(st.get_params()), bits)
        off, r, c = st.param_layout(1, "w_gu")
        per = synth.layer_param_elems(sh)
        assert (off, r, c) == (per + 2 * 256 + 256 * 768 + 256 * 256, 256, 1376) and st.grad_elems == 2 * per
        st.close()


def test_tiny_fp32_matches_oracle_1e4():
    _check(TINY.with_(dtype="fp32"), [2], 1e-4)


def test_tiny_bf16_matches_oracle_1e2():
    _check(TINY, [2], 1e-2)


def test_ragged_gqa_fp32_and_bf16_multi_microbatch():
    _check(RAGGED.with_(dtype="fp32"), [3, 3, 3], 1e-4)
    _check(RAGGED, [3, 3, 3], 1e-2)


def test_ragged_shape_with_fused_swiglu():
    """w_gu, gu and dgu are in the interleaved gate/up column order inside the library; weights (generator and get/set), the
    captured gu / dgu operands and the w_gu gradient must still come out in the public order."""
    import paper_2410_13333_amd as mls
    sh = FUSED_RAGGED
    st = mls.Stage.from_shape(sh, seed=1000)
    bits, _ = synth.make_params(sh, 1000)
    assert np.array_equal(storage_bits(st.get_params()), bits)
    p = st.get_params()
    st.set_params(p.flip(0).contiguous())
    assert np.array_equal(storage_bits(st.get_params()), bits[::-1])
    st.close()
    _check(sh, [3, 3, 3], 1e-2)
    _check(sh, [1, 3, 2], 1e-2, interleave=True)


@pytest.mark.parametrize("ffn", [8, 24, 40, 1016])
def test_fused_swiglu_where_the_last_group_of_32_columns_is_not_full(ffn):
    """What fills it up is zero inside and never seen outside: weights, captured operands and gradients (the fill would lie in
    the next row of the w_gu gradient; the first overwriting call meets NaN there)."""
    import torch
    import paper_2410_13333_amd as mls
    sh = RAGGED.with_(ffn=ffn, layers=2)
    st = mls.Stage.from_shape(sh, seed=1000)
    bits, _ = synth.make_params(sh, 1000)
    assert np.array_equal(storage_bits(st.get_params()), bits)
    p = st.get_params()
    st.set_params(p.flip(0).contiguous())
    assert np.array_equal(storage_bits(st.get_params()), bits[::-1])
    st.set_params(p)
    x, dy = to_device(synth.make_x(sh, 2000, 0)[0], "bf16"), to_device(synth.make_dy(sh, 3000, 0)[0], "bf16")
    y, dx = torch.empty_like(x), torch.empty_like(dy)
    a, b = torch.full((st.grad_elems,), float("nan"), device="cuda"), torch.zeros(st.grad_elems, device="cuda")
    st.forward(x, 2, y)
    gu, z = st.debug_read("gu", 1).float(), st.debug_read("z", 1).float()
    ref = gu[:, :ffn] * torch.sigmoid(gu[:, :ffn]) * gu[:, ffn:]
    assert ((z - ref).norm() / ref.norm()).item() < 2.0 ** -7  # two roundings of the gate and the up, one of the product
    st.backward(dy.unsqueeze(0), a, 1, dx.unsqueeze(0), overwrite=True)
    st.forward(x, 2, y)
    st.backward(dy.unsqueeze(0), b, 1, dx.unsqueeze(0))
    assert torch.equal(a, b)
    st.close()
    _check(sh, [2, 1, 2], 1e-2)


def test_swiglu_as_a_kernel_of_its_own():
    """gate/up operands of 2 GiB (here dgu, with the slack the tiles ask for) leave the fused form: public column order, a SwiGLU
    kernel each way, the w_gu gradient and the data gradient on the register-staged kernel.  References in 64 bits from the
    captured operands; a result is rounded to bf16 once (below 2^-8), dgu comes from a rounded dz (2^-7), gradients are fp32 sums."""
    import torch
    import paper_2410_13333_amd as mls
    h, f, T = 64, 65536, 7700
    st = mls.Stage(h, 1, 1, 64, f, T, 1, 1, 1, seed=1000)
    assert mls.product_plan(st.cfg, 5) == (0, 1, 0, 0, 1)
    p = st.get_params()
    st.set_params(p.flip(0).contiguous())
    assert torch.equal(st.get_params(), p.flip(0))
    st.set_params(p)
    assert torch.equal(st.get_params(), p)
    gen = torch.Generator("cuda").manual_seed(3)
    x, dy = (torch.randn(1, T, h, device="cuda", generator=gen).bfloat16() for _ in range(2))
    y, dx = torch.empty_like(x), torch.empty_like(x)

    def weight(name):
        off, r, c = st.param_layout(0, name)
        return p[off:off + r * c].view(r, c).double()

    def err(got, ref):
        return ((got.double() - ref).norm() / ref.norm()).item()
    off, r, c = st.param_layout(0, "w_gu")
    for add in (False, True):
        st.forward(x, 1, y)
        b, gu, z, hid = (st.debug_read(n) for n in ("b", "gu", "z", "h"))
        g = torch.full((st.grad_elems,), 0.5 if add else float("nan"), device="cuda")
        st.backward(dy, g, 1, dx, overwrite=not add)
        dgu = st.debug_read("dgu")
        dw = torch.cat([b.double().t() @ dgu[:, i:i + f].double() for i in (0, f)], 1)
        assert err(g[off:off + r * c].view(r, c), dw + (0.5 if add else 0.0)) < 1e-5
    for i in (0, f):
        assert err(gu[:, i:i + f], b.double() @ weight("w_gu")[:, i:i + f]) < 2.0 ** -8
    gate, up = gu[:, :f].double(), gu[:, f:].double()
    s = torch.sigmoid(gate)
    assert err(z, gate * s * up) < 2.0 ** -8
    assert err(y.view(T, h), hid.double() + z.double() @ weight("w_d")) < 2.0 ** -8
    dz = dy.view(T, h).double() @ weight("w_d").t()
    assert err(dgu[:, :f], dz * up * s * (1 + gate * (1 - s))) < 2.0 ** -7
    assert err(dgu[:, f:], dz * gate * s) < 2.0 ** -7
    dn = sum(dgu[:, i:i + f].double() @ weight("w_gu")[:, i:i + f].t() for i in (0, f)) * weight("gamma2").view(-1)
    inv = (hid.double().square().mean(-1, keepdim=True) + 1e-5).rsqrt()
    n = hid.double() * inv
    assert err(st.debug_read("dh"), dy.view(T, h).double() + inv * (dn - n * (dn * n).mean(-1, keepdim=True))) < 2.0 ** -7
    st.close()


@pytest.mark.parametrize("hidden,tokens", [(72, 2047), (72, 2048), (512, 2051), (520, 2048), (1024, 2101), (1032, 2048)])
def test_norms_of_many_narrow_rows(hidden, tokens):
    """2048 rows of up to 1024 elements and more run by wavefronts: rows and columns that do not fill them, and the shapes next to
    the rule."""
    sh = synth.StageShape(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=64, seq=tokens, micro_batch=1, layers=1, microbatches=2)
    _check(sh, [1, 1], 1e-2)


def test_set_params_reaches_every_copy_of_the_weights():
    """The library keeps transposed copies of the weight matrices for its forward products: a stage whose parameters
    were replaced by another stage's must give that stage's output and input gradient bit for bit."""
    import torch
    import paper_2410_13333_amd as mls
    sh = FUSED_RAGGED
    a = mls.Stage.from_shape(sh, seed=1000)
    b = mls.Stage.from_shape(sh, seed=4321)
    x = to_device(synth.make_x(sh, 2000, 0)[0], "bf16")
    dy = to_device(synth.make_dy(sh, 3000, 0)[0], "bf16")
    out = []
    for st in (a, b):
        if st is b:
            st.set_params(a.get_params())
        y, dx = torch.empty_like(x), torch.empty_like(dy)
        g = torch.zeros(st.grad_elems, dtype=torch.float32, device="cuda")
        st.forward(x, sh.layers, y)
        st.backward(dy.unsqueeze(0), g, 1, dx.unsqueeze(0))
        torch.cuda.synchronize()
        out.append((y, dx, g))
    for u, v in zip(*out):
        assert torch.equal(u, v)
    a.close()
    b.close()


def test_head_dim_128_gqa_single_kv_head():
    _check(GQA128.with_(dtype="fp32"), [1, 1], 1e-4)
    _check(GQA128, [1, 1], 1e-2)


def test_uneven_layer_counts_and_interleaved_order_agree():
    """Entries forwarded with different layer counts (including zero) may be mixed; one-forward-one-backward
    order gives the same y and dX bit for bit as all forwards then one backward; the weight gradients differ only
    in fp32 summation order (one contraction over all micro-batches vs one per micro-batch)."""
    ks = [2, 0, 1]
    a = _check(TINY, ks, 1e-2)
    b = _check(TINY, ks, 1e-2, interleave=True)
    for u, v in zip(a[0] + a[1], b[0] + b[1]):
        assert np.array_equal(u, v)
    assert rel_err(a[2], b[2]) < 1e-6


def test_run_to_run_bitwise_determinism():
    a = gpu_step(RAGGED, 1000, 2000, 3000, [3, 2])
    b = gpu_step(RAGGED, 1000, 2000, 3000, [3, 2])
    for u, v in zip(a[0] + a[1], b[0] + b[1]):
        assert np.array_equal(u, v)
    assert np.array_equal(a[2], b[2])
    a[3].close()
    b[3].close()


def test_gradients_accumulate_and_are_never_zeroed():
    import torch
    import paper_2410_13333_amd as mls
    sh = TINY
    st = mls.Stage.from_shape(sh, seed=1000, max_inflight=2)
    x = to_device(synth.make_x(sh, 2000, 0)[0], "bf16")
    dy = to_device(synth.make_dy(sh, 3000, 0)[0], "bf16")[None]
    y, dx = torch.empty_like(x), torch.empty_like(dy)
    g1 = torch.zeros(st.grad_elems, dtype=torch.float32, device="cuda")
    st.forward(x, 2, y)
    st.backward(dy, g1, 1, dx)
    g2 = torch.full((st.grad_elems,), 7.0, dtype=torch.float32, device="cuda")
    st.forward(x, 2, y)
    st.forward(x, 2, y)
    st.backward(torch.cat([dy, dy]), g2, 2, torch.empty(2, *x.shape, dtype=x.dtype, device="cuda"))
    torch.cuda.synchronize()
    ref = 7.0 + 2.0 * to_host64(g1)
    assert rel_err(to_host64(g2), ref) < 1e-6
    st.close()


def test_zero_layers_zero_microbatches_and_errors():
    import torch
    import paper_2410_13333_amd as mls
    sh = TINY
    st = mls.Stage.from_shape(sh, seed=1, max_inflight=2)
    x = to_device(synth.make_x(sh, 2000, 0)[0], "bf16")
    y = torch.empty_like(x)
    g = torch.zeros(st.grad_elems, dtype=torch.float32, device="cuda")
    st.backward(None, None, 0, None)                      # n = 0: no-op even with null buffers
    st.forward(x, 0, y)                                   # k = 0: identity, still one stash entry
    assert st.inflight == 1
    dy = to_device(synth.make_dy(sh, 3000, 0)[0], "bf16")[None]
    dx = torch.empty_like(dy)
    st.backward(dy, g, 1, dx)
    torch.cuda.synchronize()
    assert torch.equal(y, x) and torch.equal(dx, dy) and not g.any()
    with pytest.raises(mls.MlsError) as e:
        st.backward(dy, g, 1, dx)                         # nothing stashed
    assert e.value.code == -4
    with pytest.raises(mls.MlsError) as e:
        st.forward(x, 3, y)                               # beyond max_layers
    assert e.value.code == -3
    st.forward(x, 1, y)
    st.forward(x, 1, y)
    with pytest.raises(mls.MlsError) as e:
        st.forward(x, 1, y)                               # stash full
    assert e.value.code == -4
    with pytest.raises(mls.MlsError) as e:
        st.forward(None, 1, y)
    assert e.value.code == -2
    st.reset()
    assert st.inflight == 0
    st.close()
    with pytest.raises(mls.MlsError) as e:
        mls.Stage(hidden=100, n_q_heads=4, n_kv_heads=3, head_dim=64, ffn=688, seq=8, micro_batch=1, max_layers=1,
                  max_inflight=1)
    assert e.value.code == -1


@pytest.mark.parametrize("batched", [0, 3, 17])
@pytest.mark.parametrize("base", ["ragged", "fused"])
def test_weight_gradient_contraction_given_identical_operands_1e4(base, batched):
    """The 1e-4 bar of the fp32-accumulated weight gradients: capture the bf16 operand pairs of every
    weight-gradient contraction of layer 0 and rebuild sum_mb X^T dY in fp64 from exactly those operands.
    batched = n > 0: n micro-batches go through ONE backward call (one contraction per weight over all of them, in a
    two-layer stage; 17 is one more than a launch's 16 segments, so every weight takes a second, accumulating launch);
    batched = 0: three micro-batches, one call per micro-batch accumulates into the same gradient vector."""
    import torch
    import paper_2410_13333_amd as mls
    sh = (RAGGED if base == "ragged" else FUSED_RAGGED).with_(layers=2 if batched else 1)
    n, K = batched or 3, sh.layers
    st = mls.Stage.from_shape(sh, seed=1000, max_inflight=n if batched else 1)
    g = torch.zeros(st.grad_elems, dtype=torch.float32, device="cuda")
    ref = {k: 0.0 for k in ("w_d", "w_gu", "w_o", "w_qkv")}
    pairs = (("w_d", "z", "dy"), ("w_gu", "b", "dgu"), ("w_o", "o", "dh"), ("w_qkv", "a", "dqkv"))
    xs = [to_device(synth.make_x(sh, 2000, mb)[0], "bf16") for mb in range(n)]
    dys = torch.stack([to_device(synth.make_dy(sh, 3000, mb)[0], "bf16") for mb in range(n)])
    y, dx = torch.empty_like(xs[0]), torch.empty_like(dys)
    if batched:
        for mb in range(n):
            st.forward(xs[mb], K, y)
        ops = [{k: to_host64(st.debug_read(k, 0, mb)) for _, k, _ in pairs} for mb in range(n)]
        st.backward(dys, g, n, dx)
        for mb in range(n):
            for w, a, b in pairs:
                ref[w] = ref[w] + ops[mb][a].T @ to_host64(st.debug_read(b, 0, mb))
        with pytest.raises(mls.MlsError):
            st.debug_read("dy", 0, n)  # beyond the micro-batches of that call
    else:
        for mb in range(n):
            st.forward(xs[mb], K, y)
            ops = {k: to_host64(st.debug_read(k)) for _, k, _ in pairs}
            st.backward(dys[mb:mb + 1], g, 1, dx[mb:mb + 1])
            for w, a, b in pairs:
                ref[w] = ref[w] + ops[a].T @ to_host64(st.debug_read(b))
    torch.cuda.synchronize()
    gh = to_host64(g)
    for name, r in ref.items():
        off, rows, cols = st.param_layout(0, name)
        e = rel_err(gh[off:off + rows * cols].reshape(rows, cols), r)
        assert e <= 1e-4, (name, e)
    st.close()


def test_wide_hidden_rows_span_many_chunks():
    """hidden above 4096 and above 8192 exercises the wider register tilings of the RMSNorm kernels."""
    for hidden in (4104, 8200):
        sh = synth.StageShape(hidden=hidden, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=64, seq=72, micro_batch=1,
                              layers=1, microbatches=2)
        _check(sh, [1, 1], 1e-2)
        _check(sh.with_(dtype="fp32"), [1], 1e-4)


@pytest.mark.parametrize("base", ["ragged", "fused", "fp32"])
def test_overwrite_mode_equals_zeroing_then_accumulating(base):
    """MLS_BWD_OVERWRITE: a gradient vector full of NaN goes in, exactly the gradients of zero-then-accumulate come
    out, layers no entry reached are zero, and a following plain call accumulates on top."""
    import torch
    import paper_2410_13333_amd as mls
    sh = {"ragged": RAGGED, "fused": FUSED_RAGGED, "fp32": RAGGED.with_(dtype="fp32")}[base].with_(layers=4)
    ks = [2, 3, 0, 1]
    ref = gpu_step(sh, 1000, 2000, 3000, ks)
    ref[3].close()
    st = mls.Stage.from_shape(sh, seed=1000, max_inflight=len(ks))
    shape = (sh.micro_batch, sh.seq, sh.hidden)
    xs = [to_device(synth.make_x(sh, 2000, mb)[0], sh.dtype) for mb in range(len(ks))]
    dy = torch.stack([to_device(synth.make_dy(sh, 3000, mb)[0], sh.dtype) for mb in range(len(ks))])
    ys = [torch.empty(shape, dtype=st.tdtype, device="cuda") for _ in ks]
    dx = torch.empty_like(dy)
    grads = torch.full((st.grad_elems,), float("nan"), dtype=torch.float32, device="cuda")
    for mb, k in enumerate(ks):
        st.forward(xs[mb], k, ys[mb])
    st.backward(dy, grads, len(ks), dx, overwrite=True)
    torch.cuda.synchronize()
    g = to_host64(grads)
    assert np.array_equal(g, ref[2])
    per = synth.layer_param_elems(sh)
    assert not g[3 * per:].any() and g[2 * per:3 * per].any()          # layer 3 untouched, layer 2 reached by one entry
    for u, v in zip(ref[1], dx):
        assert np.array_equal(u, to_host64(v))
    # a second, plain call adds the same gradients once more
    for mb, k in enumerate(ks):
        st.forward(xs[mb], k, ys[mb])
    st.backward(dy, grads, len(ks), dx)
    torch.cuda.synchronize()
    assert rel_err(to_host64(grads), 2 * ref[2]) < 1e-6
    st.backward(dy, grads, 0, dx, overwrite=True)                       # nothing to pop: everything zero
    torch.cuda.synchronize()
    assert not to_host64(grads).any()
    st.close()


@pytest.mark.parametrize("ffn", [328, 352])
def test_parameters_and_operands_reach_any_address(ffn):
    """The buffers of get_params and debug_read may begin at any element: nothing around them changes."""
    import torch
    import paper_2410_13333_amd as mls
    st = mls.Stage.from_shape(RAGGED.with_(ffn=ffn, layers=1), seed=1000)
    x = to_device(synth.make_x(RAGGED, 2000, 0)[0], "bf16")
    st.forward(x, 1, torch.empty_like(x))
    for ref, read in ((st.get_params(), lambda p: mls.lib().mls_stage_get_params(st._h, p)),
                      (st.debug_read("gu"), lambda p: mls.lib().mls_stage_debug_read(st._h, mls.T_IDS["gu"], 0, 0, p))):
        for shift in (1, 3):
            buf = torch.full((ref.numel() + 16,), 7.0, dtype=ref.dtype, device="cuda")
            assert read(ctypes.c_void_p(buf[shift:].data_ptr())) == 0
            assert torch.equal(buf[shift:shift + ref.numel()], ref.reshape(-1))
            assert bool((buf[:shift] == 7).all()) and bool((buf[shift + ref.numel():] == 7).all())
    st.close()


@pytest.mark.parametrize("seq,mb", [(37, 1), (1, 1), (3, 3), (65, 2)])
def test_token_counts_that_are_not_multiples_of_eight(seq, mb):
    """Tokens per micro-batch T = seq * micro_batch need not be a multiple of anything: T is the row count of
    every activation and the contraction length of the weight gradients (zero-filled beyond the last row).
    seq = 1: attention over a single position is the identity on v."""
    for ffn in (40, 64):  # a last group of 32 gate/up columns that is not full, and whole groups
        sh = synth.StageShape(hidden=72, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=ffn, seq=seq, micro_batch=mb,
                              layers=2, microbatches=2)
        _check(sh, [2, 1], 1e-2)
    _check(sh.with_(dtype="fp32", head_dim=16), [2, 1], 1e-4)


@pytest.mark.parametrize("nq,nkv,d,seq,mb", [(30, 2, 128, 4096, 1), (60, 4, 64, 4096, 1), (6, 2, 128, 1000, 3),
                                              (6, 2, 64, 1000, 3)])
def test_rotary_epilogue_of_the_qkv_projection(nq, nkv, d, seq, mb):
    """q|k|v after the rotary step, read back from the stash, against RMSNorm -> projection -> rotation in fp64 where
    only what the matrix unit needs is rounded to bf16: the normalised input before the projection and q|k|v once, after
    the rotation.  (30, 2, 128) and (60, 4, 64) at 4096 tokens give 17 column tiles of 256 = a full round of 256x256 tiles
    plus a launch of 64x128 tiles; 3000 tokens x 1280 / 640 columns run on 64x128 tiles with ragged rows.  The positions
    restart with every sequence of the micro-batch."""
    import paper_2410_13333_amd as mls
    import oracle.stage as O
    sh = synth.StageShape(hidden=256, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=64, seq=seq, micro_batch=mb,
                          layers=1, microbatches=1)
    st = mls.Stage.from_shape(sh, seed=1000)
    xbits, x = synth.make_x(sh, 2000, 0)
    xd = to_device(xbits, "bf16")
    import torch
    y = torch.empty_like(xd)
    st.forward(xd, 1, y)
    got = to_host64(st.debug_read("qkv"))
    st.close()
    _, p64 = synth.make_params(sh, 1000)
    w = synth.split_params(sh, p64, 0)
    a, _ = O.rmsnorm_fwd(x.reshape(seq * mb, sh.hidden), w["gamma1"], sh.rms_eps)
    pre = round_bf16(a) @ w["w_qkv"]
    qd, kvd = nq * d, nkv * d
    rot = O.rope_apply(pre[:, :qd + kvd].reshape(mb, seq, nq + nkv, d), O.rope_angles(seq, d, sh.rope_base))
    ref = round_bf16(np.concatenate([rot.reshape(seq * mb, qd + kvd), pre[:, qd + kvd:]], axis=1))
    # one rounding on each side; what is left are the elements whose fp32 and fp64 values round to different
    # neighbours (a bf16 step is 2^-8 of the value, and the normalised input already differs that way now and then)
    for name, lo, hi in (("q", 0, qd), ("k", qd, qd + kvd), ("v", qd + kvd, qd + 2 * kvd)):
        e = rel_err(got[:, lo:hi], ref[:, lo:hi])
        print(f"[rotary epilogue nq={nq} d={d}] {name}: {e:.2e}")
        assert e <= 2e-3, (name, e)
    # per-head check on the last head of k and the last rows: a wrong pairing or position would be O(1) there
    assert rel_err(got[-64:, qd + kvd - d:qd + kvd], ref[-64:, qd + kvd - d:qd + kvd]) <= 2e-3


@pytest.mark.parametrize("ffn", [328, 352])  # gate/up columns with a last group that is not full, and whole groups
@pytest.mark.parametrize("shift", [0, 1])    # a source at a 16-byte boundary (one pass) and off it (copies)
def test_set_params_from_any_address(ffn, shift):
    """Rows and columns that are no multiple of a 128 x 128 tile; both routes leave the same parameters and the same
    transposed copies (the forward reads those, the backward the parameters themselves)."""
    import torch
    import paper_2410_13333_amd as mls
    sh = RAGGED.with_(ffn=ffn, layers=2)
    a, b = mls.Stage.from_shape(sh, seed=1000), mls.Stage.from_shape(sh, seed=7)
    p = a.get_params()
    buf = torch.zeros(p.numel() + 8, dtype=p.dtype, device="cuda")
    buf[shift:shift + p.numel()] = p
    b.set_params(buf[shift:shift + p.numel()])
    assert torch.equal(b.get_params(), p)
    out = []
    for st in (a, b):
        x = to_device(synth.make_x(sh, 2000, 0)[0], sh.dtype)
        y, dx, g = torch.empty_like(x), torch.empty_like(x), torch.zeros(st.grad_elems, device="cuda")
        st.forward(x, 2, y)
        st.backward(x, g, 1, dx)
        out.append((y, dx, g))
        st.close()
    assert all(torch.equal(u, v) for u, v in zip(*out))


@pytest.mark.parametrize("nq,nkv,seq", [(56, 7, 4096), (2, 1, 72)])
def test_rotary_epilogue_with_an_odd_number_of_rotated_64_column_heads(nq, nkv, seq):
    """The last rotated head and the first head of v share a wavefront's 128 columns, on 256x256 tiles and on small ones."""
    test_rotary_epilogue_of_the_qkv_projection(nq, nkv, 64, seq, 1)


@pytest.mark.parametrize("nq,nkv,d,ffn,seq,mb", [(16, 16, 128, 544, 2048, 1), (33, 1, 64, 992, 700, 3), (12, 12, 128, 2048, 1500, 1)])
def test_fused_epilogues_on_mid_size_tiles(nq, nkv, d, ffn, seq, mb):
    """Rotary and SwiGLU epilogues on 256x256, 256x128 and 64x128 tiles: a whole layer against the exact oracle (every tile
    size of both: test_rotary_epilogue_on_every_plan, test_swiglu_epilogue_on_every_plan)."""
    sh = synth.StageShape(hidden=264, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=ffn, seq=seq, micro_batch=mb, layers=1,
                          microbatches=1)
    _check(sh, [1], 1e-2)


@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,seq,mb,n", [(264, 3, 1, 64, 680, 129, 1, 1), (1032, 16, 4, 64, 2728, 999, 2, 1),
                                                          (1544, 24, 8, 64, 4104, 700, 1, 2), (520, 4, 4, 128, 1056, 2050, 2, 2)])
def test_weight_gradients_of_a_layer_in_one_launch(hidden, nq, nkv, d, ffn, seq, mb, n):
    """Layers whose four weight gradients share a launch, with ragged edges: every matrix against fp64 on the captured operands,
    added to what the gradient vector held (each tile size: test_weight_gradients_on_every_shared_tile)."""
    import torch
    import paper_2410_13333_amd as mls
    st = mls.Stage(hidden, nq, nkv, d, ffn, seq, mb, 1, n, seed=1004)
    gen = torch.Generator(device="cuda").manual_seed(ffn)
    x, dy = (torch.randn(n, mb, seq, hidden, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    y, dx = torch.empty_like(x[0]), torch.empty_like(dy)
    g0 = torch.randn(st.grad_elems, device="cuda", generator=gen)
    g = g0.clone()
    for i in range(n):
        st.forward(x[i], 1, y)
    pairs = {"w_d": ("z", "dy"), "w_gu": ("b", "dgu"), "w_o": ("o", "dh"), "w_qkv": ("a", "dqkv")}
    left = {w: [st.debug_read(a, slot=i).double() for i in range(n)] for w, (a, _) in pairs.items()}
    st.backward(dy, g, n, dx)
    for w, (_, b) in pairs.items():
        off, r, c = st.param_layout(0, w)
        ref = sum(left[w][i].t().contiguous() @ st.debug_read(b, slot=i).double() for i in range(n))
        got = (g[off:off + r * c].double() - g0[off:off + r * c].double()).reshape(r, c)
        e = ((got - ref).norm() / ref.norm()).item()
        assert e <= 1e-5, (w, e)  # fp32 sums over at most 8200 products, fp32 rounding of the sum with g0
    st.close()


@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,seq,n,shared", [(256, 4, 4, 64, 688, 256, 2, True), (2048, 16, 16, 128, 5504, 2048, 2, True),
                                                              (1032, 8, 8, 128, 5688, 2285, 2, False), (64, 1, 1, 64, 64, 8, 17, True)])
def test_launch_counts_of_the_timing_classes(hidden, nq, nkv, d, ffn, seq, n, shared):
    """Weight gradients count once per layer (and 16 micro-batches) where they share a launch, four times where they do not."""
    import torch
    import paper_2410_13333_amd as mls
    layers = 2
    st = mls.Stage(hidden, nq, nkv, d, ffn, seq, 1, layers, n, seed=1)
    assert mls.wgrad_launch(st.cfg, n)[0] == shared
    x = torch.randn(n, 1, seq, hidden, device="cuda").to(torch.bfloat16)
    y, dx, g = torch.empty_like(x[0]), torch.empty_like(x), torch.zeros(st.grad_elems, device="cuda")
    st.timing(True)
    for i in range(n):
        st.forward(x[i], layers, y)
    st.backward(x, g, n, dx)
    torch.cuda.synchronize()
    launches = {k: v[1] for k, v in st.timing_read().items()}
    st.close()
    assert launches["gemm_wgrad"] == layers * -(-n // 16) * (1 if shared else 4)
    assert launches["gemm_fwd"] == launches["gemm_dgrad"] == 4 * layers * n


def _layer_matrix(st, name):
    off, r, c = st.param_layout(0, name)
    return st.get_params()[off:off + r * c].double().cuda().reshape(r, c)


@pytest.mark.parametrize("hidden,nq,nkv,d,seq,mb", [s for s, _ in ROPE_TILES])
def test_rotary_epilogue_on_every_plan(hidden, nq, nkv, d, seq, mb):
    """The q|k|v projection with its rotary epilogue on each tile size, alone and behind 256x256 tiles, against fp64 on the
    captured normalised input; blocks of 64 rows and columns one by one."""
    import torch
    import paper_2410_13333_amd as mls
    import oracle.stage as O
    st = mls.Stage(hidden, nq, nkv, d, 64, seq, mb, 1, 1, seed=1005)
    x = torch.randn(mb, seq, hidden, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seq)).to(torch.bfloat16)
    st.forward(x, 1, torch.empty_like(x))
    ref = st.debug_read("a").double().cuda() @ _layer_matrix(st, "w_qkv")
    got = st.debug_read("qkv").double().cuda()
    st.close()
    rot = (nq + nkv) * d
    u = ref[:, :rot].reshape(mb, seq, nq + nkv, d)
    ang = torch.from_numpy(np.ascontiguousarray(O.rope_angles(seq, d, 10000.0))).cuda().double()[None, :, None]
    u1, u2 = u[..., :d // 2], u[..., d // 2:]
    ref[:, :rot] = torch.cat([u1 * ang.cos() - u2 * ang.sin(), u1 * ang.sin() + u2 * ang.cos()], dim=-1).reshape(mb * seq, rot)
    assert worst_block(got, ref) <= 4e-3  # one rounding to bf16


@pytest.mark.parametrize("hidden,ffn,tokens", [s for s, _ in SWIGLU_TILES])
def test_swiglu_epilogue_on_every_plan(hidden, ffn, tokens):
    """The gate/up projection with the SwiGLU in its epilogue, the same way."""
    import torch
    import paper_2410_13333_amd as mls
    st = mls.Stage(hidden, 1, 1, 64, ffn, tokens, 1, 1, 1, seed=1006)
    x = torch.randn(1, tokens, hidden, device="cuda", generator=torch.Generator(device="cuda").manual_seed(ffn)).to(torch.bfloat16)
    st.forward(x, 1, torch.empty_like(x))
    ref = st.debug_read("b").double().cuda() @ _layer_matrix(st, "w_gu")
    gu, z = st.debug_read("gu").cuda(), st.debug_read("z").cuda()
    st.close()
    assert worst_block(gu, ref) <= 4e-3
    assert worst_block(z, torch.nn.functional.silu(ref[:, :ffn]) * ref[:, ffn:]) <= 4e-3  # formed in fp32, rounded once


@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,seq,mb,n", [s for s, _ in WGRAD_TILES])
def test_weight_gradients_on_every_shared_tile(hidden, nq, nkv, d, ffn, seq, mb, n):
    test_weight_gradients_of_a_layer_in_one_launch(hidden, nq, nkv, d, ffn, seq, mb, n)


@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,seq,mb,n", [
    (264, 4, 4, 128, 2048, 45, 1, 1), (520, 8, 2, 128, 2728, 45, 1, 1), (4096, 16, 8, 128, 2048, 45, 2, 1),
    (4096, 1, 1, 64, 2048, 129, 1, 2), (1544, 8, 2, 128, 4104, 999, 2, 1), (4096, 8, 8, 128, 2048, 129, 2, 3)])
def test_overwrite_equals_zeroing_where_the_two_run_on_different_tiles(hidden, nq, nkv, d, ffn, seq, mb, n):
    """Weight gradients that are stored and ones that are added to may be planned differently; the bits are the same."""
    import torch
    import paper_2410_13333_amd as mls
    st = mls.Stage(hidden, nq, nkv, d, ffn, seq, mb, 1, n, seed=1008)
    assert mls.wgrad_plan(st.cfg, n) != mls.wgrad_plan(st.cfg, n, True)
    gen = torch.Generator(device="cuda").manual_seed(seq)
    x, dy = (torch.randn(n, mb, seq, hidden, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    y, dx, got = torch.empty_like(x[0]), torch.empty_like(dy), []
    for over in (False, True):
        g = torch.full((st.grad_elems,), 3.0 if over else 0.0, device="cuda")
        for i in range(n):
            st.forward(x[i], 1, y)
        st.backward(dy, g, n, dx, overwrite=over)
        got.append(g)
    st.close()
    assert torch.equal(*got)


@pytest.mark.parametrize("shape", [s for s, _ in WGRAD_256])
def test_weight_gradients_on_256x256_tiles(shape):
    """In one launch, with and without a weight's last columns in another, and apart (test_how_the_weight_gradients_of_a_layer_run)."""
    test_weight_gradients_of_a_layer_in_one_launch(*shape)


# hidden, ffn, tokens -> (columns on 256x256 tiles, parts there, tile rows, columns, parts) of the down-projection's data gradient, and whether
# the SwiGLU backward is its epilogue
DSWIGLU_TILES = [
    ((72, 72, 65), (0, 1, 64, 64, 1), True), ((2056, 72, 65), (0, 1, 64, 64, 3), True), ((72, 1384, 2049), (0, 1, 128, 64, 1), True),
    ((4104, 680, 1000), (0, 1, 128, 64, 2), True), ((520, 1384, 2049), (0, 1, 128, 128, 1), True), ((4104, 8200, 65), (0, 1, 128, 128, 3), False),
    ((72, 2728, 2049), (0, 1, 256, 128, 1), True), ((72, 8200, 2049), (7168, 1, 64, 64, 1), False)]


@pytest.mark.parametrize("shape,plan,fused", DSWIGLU_TILES)
def test_swiglu_backward_on_every_plan(shape, plan, fused):
    """In the epilogue of the product on every smaller tile, the smallest ones shared out too; as a kernel of its own otherwise.
    The product is rounded to bf16, then the results: relative error below 2^-8 + 2^-8 in every element, a third of it in the norm."""
    import torch
    import paper_2410_13333_amd as mls
    h, f, T = shape
    st = mls.Stage(h, 2, 1, 64, f, T, 1, 1, 1, seed=1009)
    assert mls.product_plan(st.cfg, 4) == plan
    gen = torch.Generator(device="cuda").manual_seed(T)
    x, dy = (torch.randn(1, T, h, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    g, dx = torch.zeros(st.grad_elems, device="cuda"), torch.empty_like(dy)
    st.forward(x, 1, torch.empty_like(x))
    gu = st.debug_read("gu").double()
    st.timing(True)
    st.backward(dy, g, 1, dx)
    assert st.timing_read()["swiglu"][1] == (0 if fused else 1)
    dgu = st.debug_read("dgu").double()
    off, r, c = st.param_layout(0, "w_d")
    w_d = st.get_params()[off:off + r * c].double().reshape(r, c)
    dz = dy.double().reshape(T, h) @ w_d.t().contiguous()
    st.close()
    gate, up = gu[:, :f], gu[:, f:]
    s = torch.sigmoid(gate)
    assert worst_block(dgu[:, :f], dz * up * s * (1 + gate * (1 - s))) <= 6e-3
    assert worst_block(dgu[:, f:], dz * gate * s) <= 6e-3
