"""The bf16 attention kernels on their own operands: q|k|v are read back from the stash, and o, the log-sum-exp and the
gradients w.r.t. q|k|v are compared with the same attention in fp64 on those values.  Sequences around the 32-row
sub-blocks, the 64-row blocks and the 128-row workgroups; scores of ordinary size and scores whose row maximum keeps
rising."""
import numpy as np
import pytest

import oracle.stage as O
import synth
from tests.helpers import rel_err, round_bf16, to_host64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gain", [1.0, 24.0])
@pytest.mark.parametrize("nq,nkv,d,seq,mb", [(2, 2, 128, 1, 2), (2, 1, 64, 33, 1), (2, 2, 128, 64, 1), (4, 2, 64, 65, 2),
                                             (2, 1, 128, 96, 1), (3, 1, 128, 129, 2), (2, 2, 64, 128, 1), (8, 1, 64, 200, 1),
                                             (4, 2, 128, 255, 1), (2, 2, 128, 321, 1), (6, 2, 64, 448, 1)])
def test_attention_against_fp64_on_the_same_operands(nq, nkv, d, seq, mb, gain):
    import torch
    import paper_2410_13333_amd as mls
    h = 128
    sh = synth.StageShape(hidden=h, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=64, seq=seq, micro_batch=mb, layers=1,
                          microbatches=1)
    st = mls.Stage.from_shape(sh, seed=1000)
    p = st.get_params()
    # a larger norm gain makes the scores large
    p[:h] *= gain
    st.set_params(p)
    x = torch.randn(mb, seq, h, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seq)).to(torch.bfloat16)
    dy = torch.randn(mb, seq, h, device="cuda", generator=torch.Generator(device="cuda").manual_seed(7)).to(torch.bfloat16)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    g = torch.zeros(st.grad_elems, device="cuda")
    st.forward(x, 1, y)
    qd, kvd, T = nq * d, nkv * d, mb * seq
    qkv, o, lse = (to_host64(st.debug_read(n)) for n in ("qkv", "o", "lse"))
    st.backward(dy, g, 1, dx)
    dh, dqkv = (to_host64(st.debug_read(n)) for n in ("dh", "dqkv"))
    off, r, c = st.param_layout(0, "w_o")
    w_o = to_host64(p[off:off + r * c]).reshape(r, c)
    st.close()
    q = qkv[:, :qd].reshape(mb, seq, nq, d)
    k = qkv[:, qd:qd + kvd].reshape(mb, seq, nkv, d)
    v = qkv[:, qd + kvd:].reshape(mb, seq, nkv, d)
    ro, pr = O.attention_fwd(q, k, v)
    # probabilities are rounded to bf16 (2^-9 relative each) before the product with v, o once more: about 3e-3
    assert rel_err(o, ro.reshape(T, qd)) <= 5e-3
    s = np.einsum("bind,bjnd->bnij", q, np.repeat(k, nq // nkv, axis=2)) / np.sqrt(d)
    s = np.where(np.tril(np.ones((seq, seq), dtype=bool)), s, -np.inf)
    top = s.max(axis=-1)
    rl = top + np.log(np.exp(s - top[..., None]).sum(axis=-1))
    if gain > 1 and seq >= 200:  # the case is what it claims: the running maximum of some row rises by more than 8 / log2(e)
        run = np.maximum.accumulate(s, axis=-1)
        assert (run[..., -1] - run[..., 31]).max() > 8
    assert np.abs(lse - rl).max() <= 2e-5 * max(1.0, np.abs(rl).max())
    # dO enters the kernels as dh w_o^T rounded to bf16; P and dS are rounded to bf16 as matrix operands
    do = round_bf16(dh @ w_o.T).reshape(mb, seq, nq, d)
    dq, dk, dv = O.attention_bwd(do, q, k, v, pr)
    ang = O.rope_angles(seq, d, sh.rope_base)
    ref = np.concatenate([O.rope_apply(dq, ang, sign=-1.0).reshape(T, qd), O.rope_apply(dk, ang, sign=-1.0).reshape(T, kvd),
                          dv.reshape(T, kvd)], axis=1)
    scale = np.linalg.norm(ref)
    for name, lo, hi in (("dq", 0, qd), ("dk", qd, qd + kvd), ("dv", qd + kvd, qd + 2 * kvd)):
        # (seq = 1: dq and dk vanish exactly, so the distance is taken relative to the whole gradient)
        e = np.linalg.norm(dqkv[:, lo:hi] - ref[:, lo:hi]) / max(np.linalg.norm(ref[:, lo:hi]), 0.05 * scale)
        print(f"[attention d={d} S={seq} gain={gain}] {name}: {e:.2e}")
        assert e <= 1.5e-2, (name, e)


# Which forward kernel a grid gets: pairs of wavefronts up to the number of workgroups where the other one wins, with exceptions for heads whose
# blocks lie on several XCDs and for more pairs than places.  Sequences around the blocks of either, at the last size of the one and the
# first of the other.
@pytest.mark.parametrize("nq,nkv,d,seq,mb,pairs", [
    (3, 1, 64, 383, 2, False), (3, 1, 64, 384, 2, True), (2, 1, 128, 385, 1, True), (4, 4, 128, 447, 1, True), (2, 2, 64, 449, 1, True),
    (2, 1, 64, 511, 1, True), (2, 1, 128, 577, 1, True), (32, 16, 64, 384, 4, True), (43, 43, 64, 384, 3, False), (20, 4, 128, 385, 4, False),
    (27, 9, 128, 385, 3, False), (16, 4, 128, 300, 3, False), (13, 13, 128, 448, 3, True), (41, 41, 128, 448, 1, False), (42, 14, 128, 448, 1, True),
    (32, 8, 128, 512, 2, True), (33, 11, 128, 512, 2, False), (32, 8, 128, 513, 2, True), (31, 31, 128, 513, 2, False), (43, 43, 128, 831, 1, False),
    (45, 15, 128, 832, 1, True), (97, 97, 64, 384, 1, False), (104, 26, 64, 384, 1, True), (66, 22, 64, 513, 1, True), (67, 67, 64, 513, 1, False),
    (70, 70, 64, 640, 1, True)])
def test_forward_kernels_on_either_side_of_their_rule(nq, nkv, d, seq, mb, pairs):
    import ctypes
    import paper_2410_13333_amd as mls
    f = mls.lib()._ZN3mls9fwd_pairsEiiii
    f.restype = ctypes.c_bool
    assert f(mb, seq, nq, d) is pairs
    test_attention_against_fp64_on_the_same_operands(nq, nkv, d, seq, mb, 8.0)


# How the backward's kernels are launched: dQ, dK and dV together up to a number of workgroups (fewer where every query head has KV heads of its
# own), dQ from the stored dS a little beyond it (heads of 128, 256 positions and more), else apart.
@pytest.mark.parametrize("nq,nkv,d,seq,mb,together,from_ds", [
    (3, 1, 64, 64, 2, True, False), (6, 2, 64, 193, 1, True, False), (16, 1, 128, 33, 8, True, False), (16, 4, 128, 128, 9, False, False),
    (43, 43, 128, 129, 3, False, False), (16, 8, 128, 161, 8, True, False), (22, 11, 128, 385, 3, False, True), (80, 16, 128, 260, 1, True, False),
    (24, 24, 64, 97, 32, False, False), (24, 8, 64, 97, 32, True, False), (24, 8, 64, 97, 33, False, False), (32, 16, 64, 129, 16, True, False),
    (32, 16, 64, 129, 17, False, False), (16, 16, 128, 33, 8, True, False), (43, 43, 128, 33, 3, False, False), (50, 50, 128, 200, 2, True, False),
    (51, 51, 128, 200, 2, False, False), (13, 13, 128, 256, 8, True, False), (83, 83, 128, 257, 1, True, False), (17, 17, 128, 257, 5, False, True),
    (45, 45, 64, 65, 8, True, False), (46, 46, 64, 65, 8, False, False), (57, 57, 64, 33, 9, True, False), (39, 39, 64, 33, 16, True, False),
    (69, 69, 64, 33, 9, False, False), (39, 39, 64, 33, 18, False, False), (42, 42, 64, 129, 5, True, False), (43, 43, 64, 129, 5, False, False),
    (60, 60, 64, 129, 5, True, False), (43, 43, 64, 129, 7, False, False),
    (19, 19, 64, 129, 16, True, False)])
def test_backward_launches_on_either_side_of_their_rules(nq, nkv, d, seq, mb, together, from_ds):
    import ctypes
    import paper_2410_13333_amd as mls
    for name, want in (("_ZN3mls12bwd_togetherEiiiii", together), ("_ZN3mls10dq_from_dsEiiiii", from_ds)):
        f = getattr(mls.lib(), name)
        f.restype = ctypes.c_bool
        assert f(mb, seq, nq, nkv, d) is want
    test_attention_against_fp64_on_the_same_operands(nq, nkv, d, seq, mb, 1.0)


@pytest.mark.parametrize("gain", [16.0, 40.0])
@pytest.mark.parametrize("nq,nkv,d,seq", [(4, 2, 64, 200), (4, 4, 128, 400)])
def test_the_largest_probability_of_a_row_is_not_rounded(nq, nkv, d, seq, gain):
    """Rows that look at few keys: the probability of the row's maximum is 1 before the division and exact in bf16, so an
    element of o is off by the rounding of the other terms and by its own, no more."""
    import torch
    import paper_2410_13333_amd as mls
    h = 128
    st = mls.Stage(h, nq, nkv, d, 64, seq, 1, 1, 1, seed=1000)
    p = st.get_params()
    p[:h] *= gain
    st.set_params(p)
    x = torch.randn(1, seq, h, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seq)).to(torch.bfloat16)
    st.forward(x, 1, torch.empty_like(x))
    qd, kvd = nq * d, nkv * d
    qkv, o = (to_host64(st.debug_read(n)) for n in ("qkv", "o"))
    st.close()
    q, k, v = qkv[:, :qd], qkv[:, qd:qd + kvd], qkv[:, qd + kvd:]
    dominant = 0
    for hq in range(nq):
        hk = slice(hq // (nq // nkv) * d, (hq // (nq // nkv) + 1) * d)
        s = np.where(np.tril(np.ones((seq, seq), dtype=bool)), q[:, hq * d:(hq + 1) * d] @ k[:, hk].T / np.sqrt(d), -np.inf)
        pr = np.exp(s - s.max(axis=1, keepdims=True))
        pr /= pr.sum(axis=1, keepdims=True)
        ref, mass = pr @ v[:, hk], pr @ np.abs(v[:, hk])
        top = pr.argmax(axis=1)
        others = mass - pr[np.arange(seq), top][:, None] * np.abs(v[top][:, hk])
        dominant += int((pr.max(axis=1) > 0.9).sum())
        # 2^-8: half a unit in the last of 8 bits; 1e-4: fp32 scores of up to some 100 (raw sums of up to 1e3 with errors of 1e-4), fp32 exponentials
        bound = 1.01 * 2.0 ** -8 * (np.abs(ref) + others) + 1e-4 * mass
        assert (np.abs(o[:, hq * d:(hq + 1) * d] - ref) <= bound).all()
    assert dominant > nq * seq // 20  # the case is what it claims


@pytest.mark.parametrize("nq,nkv,d,seq,mb", [(128, 128, 128, 1000, 1), (104, 104, 128, 1057, 1), (24, 24, 128, 2049, 3),
                                             (16, 2, 128, 1025, 1), (16, 1, 64, 1000, 2), (48, 4, 128, 40, 3),
                                             (128, 64, 128, 1000, 2), (96, 32, 128, 600, 2), (32, 16, 64, 200, 2)])
def test_dk_dv_kernel_forms(nq, nkv, d, seq, mb):
    """The forms of the dK / dV kernel on their own operands, against fp64: two key tiles per wavefront (many heads, long
    sequences; a last key block and a last query step that are partly or just filled), query heads of a group in several
    workgroups, several heads of a group one after the other in one."""
    import torch
    import paper_2410_13333_amd as mls
    h = 64
    st = mls.Stage(h, nq, nkv, d, 64, seq, mb, 1, 1, seed=1003)
    gen = torch.Generator(device="cuda").manual_seed(seq)
    x, dy = (torch.randn(mb, seq, h, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    y, dx, g = torch.empty_like(x), torch.empty_like(x), torch.zeros(st.grad_elems, device="cuda")
    st.forward(x, 1, y)
    qd, kvd, T = nq * d, nkv * d, mb * seq
    qkv = st.debug_read("qkv").double().cuda().reshape(mb, seq, -1)
    st.backward(dy, g, 1, dx)
    dh, dqkv = st.debug_read("dh").double().cuda(), st.debug_read("dqkv").double().cuda().reshape(mb, seq, -1)
    off, r, c = st.param_layout(0, "w_o")
    do = (dh.reshape(T, h) @ st.get_params()[off:off + r * c].double().cuda().reshape(r, c).t()).to(torch.bfloat16).double().reshape(mb, seq, qd)
    st.close()
    ang = torch.from_numpy(np.ascontiguousarray(O.rope_angles(seq, d, 10000.0))).cuda().double()
    hidden = torch.ones(seq, seq, dtype=torch.bool, device="cuda").triu(1)
    for b in range(mb):
        for hk in range(nkv):
            k, v = qkv[b, :, qd + hk * d:qd + (hk + 1) * d], qkv[b, :, qd + kvd + hk * d:qd + kvd + (hk + 1) * d]
            dk, dv = torch.zeros_like(k), torch.zeros_like(v)
            for hq in range(hk * (nq // nkv), (hk + 1) * (nq // nkv)):
                q, go = qkv[b, :, hq * d:(hq + 1) * d], do[b, :, hq * d:(hq + 1) * d]
                p = torch.softmax((q @ k.t() / d ** 0.5).masked_fill(hidden, -float("inf")), dim=-1)
                dp = go @ v.t()
                ds = p * (dp - (p * dp).sum(-1, keepdim=True)) / d ** 0.5
                dk += ds.t() @ q
                dv += p.t() @ go
            dk1, dk2 = dk[:, :d // 2], dk[:, d // 2:]
            dk = torch.cat([dk1 * ang.cos() + dk2 * ang.sin(), dk2 * ang.cos() - dk1 * ang.sin()], dim=1)
            for name, ref, lo in (("dk", dk, qd), ("dv", dv, qd + kvd)):
                got = dqkv[b, :, lo + hk * d:lo + (hk + 1) * d]
                e = ((got - ref).norm() / ref.norm()).item()
                # P, dS and the result are rounded to bf16 (2^-9 relative each), o and dO enter rounded
                assert e <= 1e-2, (name, b, hk, e)


@pytest.mark.parametrize("at", [0, 261])
@pytest.mark.parametrize("nq,nkv,d,seq,mb", [(128, 64, 128, 1000, 2), (96, 32, 128, 600, 2), (16, 2, 128, 1025, 1),
                                             (32, 16, 64, 400, 2)])
def test_a_non_finite_gradient_reaches_no_position_far_behind_it(nq, nkv, d, seq, mb, at):
    """dK and dV of a position sum over the queries from it on.  An infinity in the upstream gradient of an earlier position
    may touch the 64 rows of a product's tiles, no more: all others are bit for bit what they are without it."""
    import torch
    import paper_2410_13333_amd as mls
    st = mls.Stage(64, nq, nkv, d, 64, seq, mb, 1, 1, seed=1003)
    gen = torch.Generator(device="cuda").manual_seed(seq)
    x, dy = (torch.randn(mb, seq, 64, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    y, dx, g, got = torch.empty_like(x), torch.empty_like(x), torch.zeros(st.grad_elems, device="cuda"), []
    for value in (None, float("inf")):
        if value is not None:
            dy[0, at, 5] = value
        st.forward(x, 1, y)
        st.backward(dy, g, 1, dx)
        got.append(st.debug_read("dqkv").reshape(mb, seq, -1))
    st.close()
    clean, hit = got
    assert not bool(torch.isfinite(hit[0, at]).all())
    assert torch.equal(hit[0, at + 64:], clean[0, at + 64:])
    assert torch.equal(hit[1:], clean[1:])


# dQ from the dS in memory (128-column heads from 256 positions on, more workgroups than share a launch and at most 320), and the shapes next to
# it that form dS again; a last step, tile and workgroup that are partly filled; query heads of a group in several workgroups and one
# after the other
@pytest.mark.parametrize("nq,nkv,d,seq,mb,from_ds", [
    (2, 2, 128, 255, 1, False), (4, 2, 128, 256, 1, False), (2, 2, 128, 257, 2, False), (3, 1, 128, 287, 1, False), (2, 1, 128, 289, 2, False),
    (6, 6, 128, 385, 1, False), (16, 2, 128, 1025, 1, False), (32, 4, 128, 600, 2, True), (32, 32, 128, 1280, 1, True), (32, 32, 128, 1281, 1, False),
    (80, 80, 128, 500, 1, True), (10, 10, 128, 4000, 1, True), (4, 2, 64, 801, 2, False), (43, 43, 128, 255, 3, False), (43, 43, 128, 256, 3, True),
    (17, 17, 128, 257, 5, True), (29, 29, 128, 287, 3, True), (44, 22, 128, 289, 2, True)])
def test_dq_and_dkv_on_either_side_of_the_stored_ds(nq, nkv, d, seq, mb, from_ds):
    import ctypes
    import torch
    import paper_2410_13333_amd as mls
    f = mls.lib()._ZN3mls10dq_from_dsEiiiii
    f.restype = ctypes.c_bool
    assert f(mb, seq, nq, nkv, d) is from_ds
    h = 64
    st = mls.Stage(h, nq, nkv, d, 64, seq, mb, 1, 1, seed=1003)
    gen = torch.Generator(device="cuda").manual_seed(seq)
    x, dy = (torch.randn(mb, seq, h, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    y, dx, g = torch.empty_like(x), torch.empty_like(x), torch.zeros(st.grad_elems, device="cuda")
    out = []
    for _ in range(2):
        st.forward(x, 1, y)
        qkv = st.debug_read("qkv").double().reshape(mb, seq, nq + 2 * nkv, d)
        st.backward(dy, g, 1, dx)
        out.append(st.debug_read("dqkv"))
    assert torch.equal(*out)
    dqkv, dh = out[0].double().reshape(mb, seq, nq + 2 * nkv, d), st.debug_read("dh").double()
    off, r, c = st.param_layout(0, "w_o")
    do = (dh @ st.get_params()[off:off + r * c].double().reshape(r, c).t()).to(torch.bfloat16).double().reshape(mb, seq, nq, d)
    st.close()
    ang = torch.from_numpy(np.ascontiguousarray(O.rope_angles(seq, d, 10000.0))).cuda().double()
    back = lambda u: torch.cat([u[:, :d // 2] * ang.cos() + u[:, d // 2:] * ang.sin(), u[:, d // 2:] * ang.cos() - u[:, :d // 2] * ang.sin()], 1)  # noqa: E731
    hidden = torch.ones(seq, seq, dtype=torch.bool, device="cuda").triu(1)
    for b in range(mb):
        for hk in range(nkv):
            k, v = qkv[b, :, nq + hk], qkv[b, :, nq + nkv + hk]
            dk, dv = torch.zeros_like(k), torch.zeros_like(v)
            for hq in range(hk * (nq // nkv), (hk + 1) * (nq // nkv)):
                q, go = qkv[b, :, hq], do[b, :, hq]
                p = torch.softmax((q @ k.t() / d ** 0.5).masked_fill(hidden, -float("inf")), dim=-1)
                dp = go @ v.t()
                ds = p * (dp - (p * dp).sum(-1, keepdim=True)) / d ** 0.5
                dk += ds.t() @ q
                dv += p.t() @ go
                e = ((dqkv[b, :, hq] - back(ds @ k)).norm() / (ds @ k).norm()).item()
                # P, dS and the result are rounded to bf16 (2^-9 relative each), o and dO enter rounded
                assert e <= 1e-2, ("dq", b, hq, e)
            for name, ref, got in (("dk", back(dk), dqkv[b, :, nq + hk]), ("dv", dv, dqkv[b, :, nq + nkv + hk])):
                e = ((got - ref).norm() / ref.norm()).item()
                assert e <= 1e-2, (name, b, hk, e)
