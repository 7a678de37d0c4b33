"""Products whose tiles are shared out over several workgroups, each over a share of the contraction: every tile size, the forms
with an epilogue, two to eight parts, ragged rows and contractions that end inside a k-tile."""
import pytest

import paper_2410_13333_amd as mls
import synth
from tests.helpers import gpu_step, grad_errors, oracle_step, rel_err

# hidden, q heads, kv heads, head dim, ffn, tokens; product (0 .. 3 q|k|v, o, gate|up, down, 4 .. 7 the data gradients of down,
# gate|up, o, q|k|v) -> its plan: (256x256 columns, parts there, tile rows, columns, parts)
SMALL = [
    ((72, 2, 1, 64, 16392, 65), {3: (0, 1, 64, 64, 8)}),
    ((72, 16, 8, 128, 64, 65), {1: (0, 1, 64, 64, 3), 7: (0, 1, 64, 64, 4)}),
    ((264, 2, 1, 64, 1376, 1000), {5: (0, 1, 64, 64, 2)}),
    ((2056, 2, 1, 64, 64, 65), {0: (0, 1, 64, 128, 3), 2: (0, 1, 64, 128, 3), 4: (0, 1, 64, 64, 3), 6: (0, 1, 64, 64, 3)}),
    ((8200, 2, 1, 64, 64, 65), {0: (0, 1, 64, 128, 6), 2: (0, 1, 64, 128, 6)}),
    ((264, 2, 1, 64, 8200, 1000), {5: (0, 1, 128, 64, 5)}),
    ((520, 2, 1, 64, 8200, 1000), {5: (0, 1, 128, 128, 6)}),
    ((8200, 16, 8, 128, 64, 257), {0: (0, 1, 128, 128, 2)}),
    ((8200, 2, 1, 64, 1376, 257), {2: (0, 1, 128, 128, 3)}),
]
# forward products on the two largest tiles
LARGE = [
    ((12288, 16, 8, 128, 352, 700), 0, (0, 1, 256, 128, 2)), ((12288, 32, 8, 128, 352, 700), 0, (6144, 2, 0, 0, 1)),
    ((12288, 2, 1, 64, 2048, 700), 2, (0, 1, 256, 128, 2)), ((12288, 2, 1, 64, 4096, 513), 2, (8192, 2, 0, 0, 1)),
    ((4104, 2, 1, 64, 16384, 700), 3, (0, 1, 256, 128, 2)), ((8200, 2, 1, 64, 16384, 513), 3, (8200, 2, 0, 0, 1))]

# leading columns on whole 256x256 tiles, the columns behind them shared out
BEHIND = [
    ((4456, 32, 32, 64, 80, 2710), 0, (5888, 1, 64, 128, 2)), ((7744, 16, 16, 128, 168, 2804), 0, (5888, 1, 128, 128, 5)),
    ((12976, 16, 16, 64, 88, 6310), 0, (2560, 1, 256, 128, 2)), ((7424, 32, 8, 128, 88, 2076), 1, (7168, 1, 128, 64, 3)),
    ((2776, 16, 4, 64, 16456, 318), 2, (32768, 1, 64, 128, 4)), ((4536, 4, 2, 64, 18416, 393), 2, (32768, 1, 128, 128, 2)),
    ((12024, 8, 2, 64, 20000, 430), 2, (32768, 1, 256, 128, 2)), ((13136, 8, 2, 64, 1776, 1070), 3, (13056, 1, 64, 64, 3)),
    ((3144, 2, 1, 64, 4376, 5080), 3, (3072, 1, 128, 64, 3)), ((7160, 2, 1, 128, 4768, 2345), 3, (6400, 1, 128, 128, 2)),
    ((4624, 4, 4, 64, 1104, 3389), 5, (4608, 1, 64, 64, 3)), ((3456, 4, 1, 128, 2168, 5214), 5, (3072, 1, 128, 128, 2)),
    ((5768, 4, 1, 128, 5888, 3238), 5, (4864, 1, 256, 128, 2))]


@pytest.fixture(autouse=True)
def _torch_first():
    """torch brings a HIP runtime of its own: loaded after the library, it would be a second one in the process, without a device."""
    import torch  # noqa: F401


def _cfg(hidden, nq, nkv, d, ffn, T):
    return mls.MlsConfig(hidden, nq, nkv, d, ffn, T, 1, 1, 1, 1e-5, 10000.0, 0, 0)


def test_plans_of_the_tested_shapes():
    for shape, plans in SMALL:
        for product, plan in plans.items():
            assert mls.product_plan(_cfg(*shape), product) == plan, (shape, product)
    for shape, product, plan in LARGE:
        assert mls.product_plan(_cfg(*shape), product) == plan, (shape, product)


def test_plan_refusals():
    cfg = _cfg(256, 4, 4, 64, 688, 256)
    for product in (-1, 8):
        with pytest.raises(mls.MlsError):
            mls.product_plan(cfg, product)
    cfg.dtype = 1
    with pytest.raises(mls.MlsError):
        mls.product_plan(cfg, 0)


def test_plans_of_the_remainders():
    for shape, product, plan in BEHIND:
        assert mls.product_plan(_cfg(*shape), product) == plan, (shape, product)


def test_operands_of_two_gib_run_on_no_tile_of_these():
    """dgu, the operand of the fifth product, on either side of the 31 bits that the tiles' offsets have."""
    assert mls.product_plan(_cfg(64, 1, 1, 64, 65536, 7700), 5) == (0, 1, 0, 0, 1)
    assert mls.product_plan(_cfg(64, 1, 1, 64, 65536, 7600), 5) == (0, 1, 128, 64, 8)


def test_a_stage_without_such_products_has_no_workspace_for_them():
    big, small = (mls.Stage.memory(synth.StageShape(h, 2, 1, 64, f, 65, 1, 1, 1))["workspace_bytes"] for h, f in ((72, 16392), (72, 64)))
    assert big > small + 4 * 8 * 64 * 64 * 4 and small < 1 << 18


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [s for s, _ in SMALL])
def test_layer_against_the_oracle(shape):
    """One layer; a second pass of the same stage has the same bits (which part of a tile comes last may differ)."""
    import numpy as np
    sh = synth.StageShape(*shape, micro_batch=1, layers=1, microbatches=1)
    ys, dxs, g, st = gpu_step(sh, 1000, 2000, 3000, [1])
    rys, rdxs, rg = oracle_step(sh, 1000, 2000, 3000, [1])
    assert rel_err(ys[0], rys[0]) <= 1e-2 and rel_err(dxs[0], rdxs[0]) <= 1e-2
    assert grad_errors(sh, g, rg, 1)[0] <= 1e-2
    for _ in range(3):
        ys2, dxs2, g2, _ = gpu_step(sh, 1000, 2000, 3000, [1], stage=st)
        assert np.array_equal(ys[0], ys2[0]) and np.array_equal(dxs[0], dxs2[0]) and np.array_equal(g, g2)
    st.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape,product", [(s, p) for s, p, _ in LARGE])
def test_large_tiles_on_captured_operands(shape, product):
    """The product in 64 bits from the operands the stage kept.  Results are rounded to bf16 once: relative error of a single
    rounding below 2^-8, 2^-8 / sqrt(3) in the mean."""
    import torch
    h, nq, nkv, d, f, T = shape
    st = mls.Stage(h, nq, nkv, d, f, T, 1, 1, 1, seed=7)
    x = torch.randn(1, T, h, device="cuda", generator=torch.Generator("cuda").manual_seed(3)).bfloat16()
    y = torch.empty_like(x)
    st.forward(x, 1, y)
    params = st.get_params()

    def weight(name):
        off, r, c = st.param_layout(0, name)
        return params[off:off + r * c].view(r, c).double()

    def err(got, ref):
        return ((got.double() - ref).norm() / ref.norm()).item()
    if product == 0:
        qkv = st.debug_read("a").double() @ weight("w_qkv")
        pos = torch.arange(T, dtype=torch.float64, device="cuda")
        ang = pos[:, None] * 10000.0 ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device="cuda") / d)
        cs, sn = ang.cos()[:, None], ang.sin()[:, None]
        rot = (nq + nkv) * d
        a, b = qkv[:, :rot].reshape(T, nq + nkv, d).chunk(2, dim=-1)
        ref = torch.cat([torch.cat([a * cs - b * sn, a * sn + b * cs], -1).reshape(T, rot), qkv[:, rot:]], 1)
        assert err(st.debug_read("qkv"), ref) < 2.0 ** -8
    elif product == 2:
        gu = st.debug_read("b").double() @ weight("w_gu")
        assert err(st.debug_read("gu"), gu) < 2.0 ** -8
        assert err(st.debug_read("z"), gu[:, :f] * torch.sigmoid(gu[:, :f]) * gu[:, f:]) < 2.0 ** -8
    else:
        ref = st.debug_read("h").double() + st.debug_read("z").double() @ weight("w_d")
        assert err(y.view(T, h), ref) < 2.0 ** -8
    for _ in range(3):
        st.reset()
        y2 = torch.empty_like(y)
        st.forward(x, 1, y2)
        assert torch.equal(y, y2)
    st.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape,product,plan", BEHIND)
def test_remainders_on_captured_operands(shape, product, plan):
    """The product in 64 bits from the operands the stage kept: all of it and the columns of the shared-out tiles alone.  A result
    is rounded to bf16 once (relative error below 2^-8); dh takes the rounded product and is rounded itself (2^-7)."""
    import torch
    h, nq, nkv, d, f, T = shape
    st = mls.Stage(h, nq, nkv, d, f, T, 1, 1, 1, seed=7)
    gen = torch.Generator("cuda").manual_seed(3)
    x, dy = (torch.randn(1, T, h, device="cuda", generator=gen).bfloat16() for _ in range(2))
    y, dx = torch.empty_like(x), torch.empty_like(x)
    grads = torch.empty(st.grad_elems, device="cuda") if product == 5 else None

    def once():
        st.reset()
        st.forward(x, 1, y)
        if product == 5:
            hid = st.debug_read("h").double()
            st.backward(dy, grads, 1, dx, overwrite=True)
            return [st.debug_read("dh"), hid]
        return [st.debug_read("qkv") if product == 0 else st.debug_read("h") if product == 1 else st.debug_read("gu") if product == 2 else y.view(T, h).clone()]
    got, *more = once()
    params = st.get_params()

    def weight(name):
        off, r, c = st.param_layout(0, name)
        return params[off:off + r * c].view(r, c).double()

    def check(a, ref, cols, tol=2.0 ** -8):
        for sel in (slice(None), cols):
            e = ((a.double()[:, sel] - ref[:, sel]).norm() / ref[:, sel].norm()).item()
            assert e < tol, (sel, e)
    behind = slice(plan[0], None)
    if product == 0:
        qkv = st.debug_read("a").double() @ weight("w_qkv")
        ang = torch.arange(T, dtype=torch.float64, device="cuda")[:, None] * 10000.0 ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device="cuda") / d)
        cs, sn = ang.cos()[:, None], ang.sin()[:, None]
        rot = (nq + nkv) * d
        a, b = qkv[:, :rot].reshape(T, nq + nkv, d).chunk(2, dim=-1)
        check(got, torch.cat([torch.cat([a * cs - b * sn, a * sn + b * cs], -1).reshape(T, rot), qkv[:, rot:]], 1), behind)
    elif product == 1:
        check(got, x.view(T, h).double() + st.debug_read("o").double() @ weight("w_o"), behind)
    elif product == 2:
        gu = st.debug_read("b").double() @ weight("w_gu")
        at = plan[0] // 2  # 32 gate and 32 up columns in turn
        for half in (gu[:, :f], got[:, :f]), (gu[:, f:], got[:, f:]):
            check(half[1], half[0], slice(at, None))
        check(st.debug_read("z"), gu[:, :f] * torch.sigmoid(gu[:, :f]) * gu[:, f:], slice(at, None))
    elif product == 3:
        check(got, st.debug_read("h").double() + st.debug_read("z").double() @ weight("w_d"), behind)
    else:
        hid = more[0]
        dn = st.debug_read("dgu").double() @ weight("w_gu").t() * weight("gamma2").view(-1)
        r = (hid.square().mean(-1, keepdim=True) + 1e-5).rsqrt()
        check(got, dy.view(T, h).double() + r * (dn - hid * r * (dn * hid * r).mean(-1, keepdim=True)), behind, 2.0 ** -7)
    for _ in range(2):
        assert torch.equal(once()[0], got)
    st.close()


@pytest.mark.gpu
def test_head_of_few_tokens():
    """The data gradient of the LM head contracts over the vocabulary: many parts per tile, in a workspace of the Ends handle."""
    import torch
    T, h, V = 72, 264, 8200
    en = mls.Ends(h, V, T, 1, 1, 1e-5, "bf16", seed=5)
    y = torch.randn(1, T, h, device="cuda", generator=torch.Generator("cuda").manual_seed(1)).bfloat16()
    tgt = torch.randint(0, V, (T,), device="cuda", dtype=torch.int32, generator=torch.Generator("cuda").manual_seed(2))
    out = []
    for _ in range(3):
        loss, g, dy = torch.zeros(1, device="cuda"), torch.zeros(en.grad_elems, device="cuda"), torch.empty_like(y)
        en.head_forward(y, tgt, 1.0, loss)
        dlog = en.debug_dlogits().double()
        en.head_backward(g, 1, dy)
        out.append((loss, g, dy))
    assert all(torch.equal(a, b) for o in out[1:] for a, b in zip(out[0], o))
    p = en.get_params().double()
    wlm = p[V * h + h:].view(h, V)
    gamma, t = p[V * h:V * h + h], y.double().view(T, h)
    dn = dlog @ wlm.t() * gamma
    r = (t.square().mean(-1, keepdim=True) + 1e-5).rsqrt()
    ref = r * (dn - t * r * (dn * t * r).mean(-1, keepdim=True))
    assert ((dy.double().view(T, h) - ref).norm() / ref.norm()).item() < 1e-2
    en.close()


@pytest.mark.gpu
def test_replays_from_a_graph():
    """The counters are zero again after every launch: replays, with eager steps in between, have the eager bits."""
    import torch
    h, nq, nkv, d, f, T = SMALL[3][0]
    side = torch.cuda.Stream()
    st = mls.Stage(h, nq, nkv, d, f, T, 1, 2, 1, seed=7, stream=side)
    gen = torch.Generator("cuda").manual_seed(3)
    x, dy = (torch.randn(1, T, h, device="cuda", generator=gen).bfloat16() for _ in range(2))
    y, dx, g = torch.empty_like(x), torch.empty_like(x), torch.zeros(st.grad_elems, device="cuda")

    def step():
        st.forward(x, 2, y)
        st.backward(dy, g, 1, dx, overwrite=True)
    torch.cuda.synchronize()

    def eager():
        with torch.cuda.stream(side):
            step()
        side.synchronize()
        return y.clone(), dx.clone(), g.clone()
    ref = eager()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for _ in range(3):
        for t in (y, dx, g):
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((y, dx, g), ref))
        assert all(torch.equal(a, b) for a, b in zip(eager(), ref))
    del graph
    st.close()
