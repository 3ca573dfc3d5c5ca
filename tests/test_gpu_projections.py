"""GPU parity of the projections either side of the attention (bf16 MFMA GEMMs with the head
split / head gather fused) against the float64 oracle, through the C ABI."""
import numpy as np
import pytest
import torch

from oracle import mate_oracle as orc
from paper_2109_04312_amd import synth
from tests import helpers as hp

pytestmark = pytest.mark.gpu
P = synth.TOK_PAD


def bf16(x):
    return synth.round_to_bf16(np.asarray(x, np.float32)).astype(np.float32)


def dev(x, dtype=torch.bfloat16):
    return torch.from_numpy(np.ascontiguousarray(x)).to(dtype).cuda()


def close(got, want, what):
    """bf16 output of an fp32-accumulated product: |err| <= 2e-2 + 2^-8 |ref| (a bf16 store alone
    costs |ref| 2^-9) and the bf16 path's mean-rel bound."""
    got = got.float().cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)), what
    err = np.abs(got - want)
    ratio = float((err / hp.bound("projection", want, "bf16")).max()) if err.size else 0.0
    mean_rel = float(err.mean() / (np.abs(want).mean() + 1e-3))
    print(f"   {what}: max-abs {float(err.max()):.2e} = {ratio:.2f} x bound, mean-rel {mean_rel:.2e}", flush=True)
    assert ratio <= 1.0 and mean_rel <= hp.TOL["bf16"]["mean_rel"], what


def make(seed, B, N, H, E, pad_tail=0, scattered_pads=True, bias=True):
    rng = np.random.default_rng(seed)
    x = bf16(rng.standard_normal((B, N, E)))
    w_qkv = bf16(rng.standard_normal((3 * H * 64, E)) / np.sqrt(E))
    w_o = bf16(rng.standard_normal((E, H * 64)) / np.sqrt(H * 64))
    b_qkv = rng.standard_normal(3 * H * 64).astype(np.float32) if bias else None
    b_o = rng.standard_normal(E).astype(np.float32) if bias else None
    flags = rng.choice([synth.TOK_LOCAL, synth.TOK_GLOBAL], size=(B, N)).astype(np.uint8)
    if scattered_pads:
        flags[rng.random((B, N)) < 0.1] = P
    if pad_tail:
        flags[:, N - pad_tail:] = P
    o = bf16(rng.standard_normal((B, H, N, 64)))
    return x, w_qkv, b_qkv, w_o, b_o, flags, o


def check(seed, B, N, H, E, **kw):
    from paper_2109_04312_amd import mate
    print(f"projections B={B} N={N} H={H} E={E} {kw}", flush=True)
    x, w_qkv, b_qkv, w_o, b_o, flags, o = make(seed, B, N, H, E, **kw)
    nan = lambda *shape: torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    fl = torch.from_numpy(flags).cuda()
    q, k, v = mate.qkv_project(dev(x), dev(w_qkv), None if b_qkv is None else dev(b_qkv, torch.float32), fl, H,
                               q=nan(B, H, N, 64), k=nan(B, H, N, 64), v=nan(B, H, N, 64))
    y = mate.out_project(dev(o), dev(w_o), None if b_o is None else dev(b_o, torch.float32), fl, y=nan(B, N, E))
    torch.cuda.synchronize()
    want = orc.project_qkv(x, w_qkv, b_qkv, flags, H)
    for name, g, r in zip("qkv", (q, k, v), want):
        close(g, r, name)
        assert bool((g.float().cpu().numpy()[np.broadcast_to((flags == P)[:, None, :, None], r.shape)] == 0).all())
    close(y, orc.project_out(o, w_o, b_o, flags), "y")
    assert bool((y.float().cpu().numpy()[flags == P] == 0).all())


@pytest.mark.parametrize("N", [1, 64, 127, 128, 129, 200, 333])
def test_small_ragged(N):
    check(N, 2, N, 2, 128)


def test_no_bias_and_tiles_of_padding_only():
    check(1, 3, 700, 4, 256, pad_tail=300, bias=False)
    check(2, 1, 512, 2, 128, pad_tail=512, scattered_pads=False)       # nothing but padding


def test_bert_base_shape():
    check(3, 4, 512, 12, 768, pad_tail=100)


def test_large_tiles_ragged_with_scattered_pads():
    # enough tiles for the 256 x 256 shape of the QKV kernel; N is not a multiple of 256
    check(5, 9, 1000, 12, 768, pad_tail=120)
    check(6, 3, 2500, 16, 1024, pad_tail=0)


def test_headline_shape():
    # configuration 4's layer: B=2, N=8192, 16 heads, model width 1024
    check(4, 2, 8192, 16, 1024, pad_tail=1700, scattered_pads=False)


def test_layer_forward_end_to_end():
    """x -> QKV projection -> segment build -> attention -> output projection, every step in the
    library, against the same chain in the oracle (which keeps float64 between the steps, so the
    bound is looser than a single step's: three roundings to bf16 on the way)."""
    from paper_2109_04312_amd import mate
    w = synth.make_config(2, tensors=False)
    st = w.structure
    B, N, H, E = st.B, st.N, 12, 768
    rng = np.random.default_rng(9)
    x = bf16(rng.standard_normal((B, N, E)))
    w_qkv = bf16(rng.standard_normal((3 * H * 64, E)) / np.sqrt(E))
    w_o = bf16(rng.standard_normal((E, H * 64)) / np.sqrt(H * 64))
    hk = synth.half_row_half_col(H)
    r, c, f = hp.dev_structure(st)
    q, k, v = mate.qkv_project(dev(x), dev(w_qkv), None, f, H)
    seg = mate.build_segments(r, c, f)
    o, _ = mate.attn_fwd(q, k, v, seg, hk, 0.125)
    y = mate.out_project(o, dev(w_o), None, f)
    torch.cuda.synchronize()
    for b in (0, 17):
        sl = slice(b, b + 1)
        qr, kr, vr = orc.project_qkv(x[sl], w_qkv, None, st.flags[sl], H)
        orf, _ = orc.attn_forward(qr, kr, vr, st.row_ids[sl], st.col_ids[sl], st.flags[sl], hk, 0.125)
        yr = orc.project_out(orf, w_o, None, st.flags[sl])
        got = y[sl].float().cpu().numpy().astype(np.float64)
        err = np.abs(got - yr)
        ratio = float((err / hp.bound("projection", yr, "bf16")).max())
        mean_rel = float(err.mean() / (np.abs(yr).mean() + 1e-3))
        print(f"   layer b={b}: max-abs {float(err.max()):.2e} = {ratio:.2f} x one step's bound, "
              f"mean-rel {mean_rel:.2e}", flush=True)
        assert ratio <= 1.5 and mean_rel <= 1.5e-2


def close_f32(got, want, what, k_len):
    """fp32 output of a bf16 x bf16 product accumulated in fp32 over k_len terms: the products are
    exact, so the only error is fp32 summation, bounded by k_len * 2^-24 * sum|terms|; held to
    1e-5 * (1 + |ref|) * sqrt(k_len), far above that and far below one bf16 ulp."""
    got = got.float().cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)), what
    err = np.abs(got - want)
    tol = 1e-5 * np.sqrt(k_len) * (1.0 + np.abs(want))
    print(f"   {what}: max-abs {float(err.max()):.2e} (|ref| up to {float(np.abs(want).max()):.1f}), "
          f"worst err/bound {float((err / tol).max()):.2f}", flush=True)
    assert (err <= tol).all(), what


def check_bwd(seed, B, N, H, E, **kw):
    from paper_2109_04312_amd import mate
    print(f"projection backward B={B} N={N} H={H} E={E} {kw}", flush=True)
    x, w_qkv, _, w_o, _, flags, o = make(seed, B, N, H, E, **kw)
    rng = np.random.default_rng(seed + 1000)
    dq, dk, dv = (bf16(rng.standard_normal((B, H, N, 64))) for _ in range(3))
    dy = bf16(rng.standard_normal((B, N, E)))
    fl = torch.from_numpy(flags).cuda()
    n_tok = max(1, int((flags != P).sum()))
    # --- QKV projection ---
    dx, dw, db = mate.qkv_project_bwd(dev(x), dev(w_qkv), fl, dev(dq), dev(dk), dev(dv))
    torch.cuda.synchronize()
    rx, rw, rb = orc.project_qkv_backward(x, w_qkv, flags, dq, dk, dv, H)
    close(dx, rx, "dx")
    assert bool((dx.float().cpu().numpy()[flags == P] == 0).all())
    close_f32(dw, rw, "dw_qkv", n_tok)
    close_f32(db, rb, "dbias_qkv", n_tok)
    # --- output projection ---
    d_o, dwo, dbo = mate.out_project_bwd(dev(o), dev(w_o), fl, dev(dy))
    torch.cuda.synchronize()
    ro, rwo, rbo = orc.project_out_backward(o, w_o, flags, dy)
    close(d_o, ro, "d_o")
    assert bool((d_o.float().cpu().numpy()[np.broadcast_to((flags == P)[:, None, :, None], ro.shape)] == 0).all())
    close_f32(dwo, rwo, "dw_o", n_tok)
    close_f32(dbo, rbo, "dbias_o", n_tok)


@pytest.mark.parametrize("N", [1, 63, 64, 65, 200, 333])
def test_backward_small_ragged(N):
    check_bwd(N, 2, N, 2, 128)


def test_backward_padding_only_blocks_and_scattered_pads():
    check_bwd(1, 3, 700, 4, 256, pad_tail=300)
    check_bwd(2, 1, 512, 2, 128, pad_tail=512, scattered_pads=False)       # nothing but padding: all zero


def test_backward_bert_base_and_large_shapes():
    check_bwd(3, 4, 512, 12, 768, pad_tail=100)
    check_bwd(5, 9, 1000, 12, 768, pad_tail=120)


def test_backward_headline_shape():
    check_bwd(4, 2, 8192, 16, 1024, pad_tail=1700, scattered_pads=False)


def test_backward_is_bit_reproducible_and_honours_null_outputs():
    from paper_2109_04312_amd import mate
    x, w_qkv, _, w_o, _, flags, o = make(7, 3, 900, 4, 256, pad_tail=77)
    rng = np.random.default_rng(77)
    dq, dk, dv = (dev(bf16(rng.standard_normal((3, 4, 900, 64)))) for _ in range(3))
    fl = torch.from_numpy(flags).cuda()
    a = mate.qkv_project_bwd(dev(x), dev(w_qkv), fl, dq, dk, dv)
    b = mate.qkv_project_bwd(dev(x), dev(w_qkv), fl, dq, dk, dv)
    only_dx = mate.qkv_project_bwd(dev(x), dev(w_qkv), fl, dq, dk, dv, want_dw=False, want_dbias=False)
    only_dw = mate.qkv_project_bwd(dev(x), dev(w_qkv), fl, dq, dk, dv, want_dx=False, want_dbias=False)
    torch.cuda.synchronize()
    for u, v in zip(a, b):
        assert torch.equal(u, v)
    assert torch.equal(only_dx[0], a[0]) and only_dx[1] is None and only_dx[2] is None
    assert only_dw[0] is None and torch.equal(only_dw[1], a[1])
    with pytest.raises(mate.MateError) as e:        # a bias gradient without the weight gradient
        mate.qkv_project_bwd(dev(x), dev(w_qkv), fl, dq, dk, dv, want_dw=False)
    assert e.value.status == mate.MATE_ERR_NULL


def test_layer_forward_backward_end_to_end():
    """x -> QKV projection -> attention -> output projection and all the way back (d y -> d o ->
    dq, dk, dv -> dx, plus the weight gradients), every step in the library, against the same
    chain in the oracle in float64.  Five bf16 roundings lie on the way to dx, so the bound is
    a multiple of a single step's."""
    from paper_2109_04312_amd import mate
    w = synth.make_config(2, tensors=False)
    st = w.structure
    B, N, H, E = st.B, st.N, 12, 768
    rng = np.random.default_rng(19)
    x = bf16(rng.standard_normal((B, N, E)))
    w_qkv = bf16(rng.standard_normal((3 * H * 64, E)) / np.sqrt(E))
    w_o = bf16(rng.standard_normal((E, H * 64)) / np.sqrt(H * 64))
    dy = bf16(rng.standard_normal((B, N, E)))
    hk = synth.half_row_half_col(H)
    r, c, f = hp.dev_structure(st)
    q, k, v = mate.qkv_project(dev(x), dev(w_qkv), None, f, H)
    seg = mate.build_segments(r, c, f)
    o, lse = mate.attn_fwd(q, k, v, seg, hk, 0.125)
    d_o, dwo, _ = mate.out_project_bwd(o, dev(w_o), f, dev(dy), want_dbias=False)
    dq, dk, dv = mate.attn_bwd(q, k, v, o, lse, d_o, seg, hk, 0.125)
    dx, dwq, _ = mate.qkv_project_bwd(dev(x), dev(w_qkv), f, dq, dk, dv, want_dbias=False)
    torch.cuda.synchronize()
    # the oracle chain on two sequences (weight gradients sum over the batch: compare dx per sequence,
    # and the weight gradients of a two-sequence batch computed separately below)
    for b in (0, 17):
        sl = slice(b, b + 1)
        qr, kr, vr = orc.project_qkv(x[sl], w_qkv, None, st.flags[sl], H)
        args = (st.row_ids[sl], st.col_ids[sl], st.flags[sl], hk, 0.125)
        orf, _ = orc.attn_forward(qr, kr, vr, *args)
        dor, _, _ = orc.project_out_backward(orf, w_o, st.flags[sl], dy[sl])
        dqr, dkr, dvr = orc.attn_backward(qr, kr, vr, dor, *args)
        dxr, _, _ = orc.project_qkv_backward(x[sl], w_qkv, st.flags[sl], dqr, dkr, dvr, H)
        got = dx[sl].float().cpu().numpy().astype(np.float64)
        err = np.abs(got - dxr)
        ratio = float((err / hp.bound("projection", dxr, "bf16")).max())
        mean_rel = float(err.mean() / (np.abs(dxr).mean() + 1e-3))
        print(f"   layer dx b={b}: max-abs {float(err.max()):.2e} = {ratio:.2f} x one step's bound, "
              f"mean-rel {mean_rel:.2e}", flush=True)
        assert ratio <= 2.0 and mean_rel <= 2e-2


def test_unsupported_arguments():
    from paper_2109_04312_amd import mate
    x, w_qkv, b_qkv, w_o, b_o, flags, o = make(0, 1, 64, 3, 128, bias=False)
    with pytest.raises(mate.MateError) as e:        # odd number of heads
        mate.qkv_project(dev(x), dev(w_qkv), None, torch.from_numpy(flags).cuda(), 3)
    assert e.value.status == mate.MATE_ERR_UNSUPPORTED
    x, w_qkv, b_qkv, w_o, b_o, flags, o = make(0, 1, 64, 2, 192, bias=False)
    with pytest.raises(mate.MateError) as e:        # width not a multiple of 128
        mate.out_project(dev(o), dev(w_o), None, torch.from_numpy(flags).cuda())
    assert e.value.status == mate.MATE_ERR_UNSUPPORTED


# every workgroup shape of the products, with a last feature tile that is not whole (1152 = 4.5 x 256 = 6 x
# 192) and token counts beside multiples of the token tiles; both tile sizes of the weight gradient; more
# token blocks than one list of them holds
@pytest.mark.parametrize("B,N,H,E", [(1, 65, 2, 128), (2, 1025, 6, 384), (1, 12001, 2, 1152), (5, 16384, 2, 128)])
def test_workgroup_shapes(B, N, H, E):
    check(N, B, N, H, E, pad_tail=N // 3)
    check_bwd(N, B, N, H, E, pad_tail=N // 3)


# contractions shared by two groups of wavefronts: one live token block (the other group has none), an odd
# number of them, tiles with and without a whole last one, and the eight wavefronts of one large tile in halves
@pytest.mark.parametrize("B,N,H,E", [(1, 63, 2, 128), (3, 129, 4, 256), (7, 577, 12, 768), (1, 4100, 16, 1024),
                                     (9, 10, 2, 128), (5, 40, 2, 128), (3, 70, 2, 128)])
def test_shared_contractions(B, N, H, E):
    check(N, B, N, H, E, pad_tail=N // 5)
    check_bwd(N, B, N, H, E, pad_tail=N // 5)


# few token tiles and many feature tiles, dealt to the XCDs by feature: heads or width large, feature tiles that are
# no multiple of eight, one token, several sequences
@pytest.mark.parametrize("B,N,H,E", [(1, 1, 36, 128), (1, 64, 36, 128), (1, 600, 12, 768), (2, 65, 2, 5120),
                                     (1, 130, 66, 256), (3, 100, 34, 128)])
def test_tiles_dealt_by_feature(B, N, H, E):
    check(N, B, N, H, E, pad_tail=N // 4)
    check_bwd(N, B, N, H, E, pad_tail=N // 4)


@pytest.mark.parametrize("B,N,H,E", [(5, 901, 12, 768), (1, 3999, 16, 1024), (2, 4225, 16, 1024)])
def test_one_round_of_eight_wavefronts(B, N, H, E):
    """192 x 256 and 256 x 192 both one round, the second with fewer tiles, which is taken: QKV of the first two sizes, the output
    of the last."""
    check(N, B, N, H, E, pad_tail=N // 7)
    check_bwd(N, B, N, H, E, pad_tail=N // 7)


@pytest.mark.parametrize("B,N,H,E", [(8, 442, 12, 768), (5, 700, 12, 768), (40, 250, 16, 1024), (12, 161, 16, 1024)])
def test_one_round_of_192_by_256(B, N, H, E):
    """Tiles of 192 x 256 in one round, fewer than of 256 x 192 or as many (180): QKV of the first two sizes (the last token tile
    186 and 188 rows), the output of the third (its last feature tile a third).  And 192 of them where 256 x 192 has 144: QKV of the last."""
    check(N, B, N, H, E, pad_tail=N // 7)


@pytest.mark.parametrize("B,N,H,E", [(8, 76, 32, 4096), (1, 1988, 20, 3456)])
def test_long_contractions(B, N, H, E):
    """More than 3271 terms and two 128 x 128 tiles a compute unit at most: QKV stays in those."""
    check(N, B, N, H, E, pad_tail=N // 8)


@pytest.mark.parametrize("B,N,H,E", [(12, 300, 12, 768), (13, 383, 12, 768), (1, 11000, 16, 1024), (2, 4225, 16, 1024)])
def test_one_round_of_256_by_192(B, N, H, E):
    """Tiles of 256 x 192 in one round, where 192 x 256 would be two or are not offered: QKV of the first two sizes (the last
    token tile 108 and 191 rows), the output of the third (56 rows), d_o of the last two (one row, by itself)."""
    from paper_2109_04312_amd import mate
    check(N, B, N, H, E, pad_tail=N // 7)
    x, _, _, w_o, _, flags, o = make(N, B, N, H, E, pad_tail=N // 7)
    dy = bf16(np.random.default_rng(N).standard_normal((B, N, E)))
    want, _, _ = orc.project_out_backward(o, w_o, flags, dy)
    args = (dev(o), dev(w_o), torch.from_numpy(flags).cuda(), dev(dy))
    got = mate.out_project_bwd(*args, want_dw=False, want_dbias=False)[0]
    close(got, want, "d_o")


def test_results_larger_than_the_caches():
    """QKV: the first tiles' results stay in the L2, the last 32 MB are written through it; dX and d_o: all stay (63 MB)."""
    check(7, 5, 16383, 6, 384, pad_tail=2000)
    check_bwd(7, 5, 16383, 6, 384, pad_tail=2000)


@pytest.mark.parametrize("B,N,H,E", [(1, 2690, 2, 128), (13, 100, 6, 384), (3, 1111, 4, 128)])
def test_last_token_tiles_dealt_one_by_one(B, N, H, E):
    """Token tiles that are no multiple of eight, of one sequence and of several: the last ones go to all XCDs."""
    check(N, B, N, H, E, pad_tail=N // 9)
    check_bwd(N, B, N, H, E, pad_tail=N // 9)


@pytest.mark.parametrize("B", [300_001, (1 << 21) + 3])
def test_very_many_sequences(B):
    """One token each: token tiles beyond what a grid's second dimension holds, and beyond 2^21, from where on a tile's sequence
    is found by whole division.  Products of 128 terms against fp32 ones of the same bf16 values."""
    from paper_2109_04312_amd import mate
    H, E = 2, 128
    gen = torch.Generator(device="cuda").manual_seed(B)
    normal = lambda *shape, scale=1.0: (torch.randn(shape, device="cuda", generator=gen) * scale).to(torch.bfloat16)
    x, o = normal(B, 1, E), normal(B, H, 1, 64)
    w_qkv, w_o = normal(3 * H * 64, E, scale=E ** -0.5), normal(E, H * 64, scale=(H * 64) ** -0.5)
    flags = torch.randint(0, 3, (B, 1), device="cuda", generator=gen, dtype=torch.uint8)
    live = (flags != P).float()

    def product_close(got, tokens, w, what):
        want = tokens.reshape(B, -1).float() @ w.float() * live
        err = (got.reshape(B, -1).float() - want).abs()
        print(f"   {what}: max-abs {float(err.max()):.2e}", flush=True)
        assert bool((err <= 2e-2 + 2.0 ** -8 * want.abs()).all()), what

    for name, got, i in zip("qkv", mate.qkv_project(x, w_qkv, None, flags, H), range(3)):
        product_close(got, x, w_qkv[128 * i:128 * (i + 1)].t(), name)
    product_close(mate.out_project(o, w_o, None, flags), o, w_o.t(), "y")
    product_close(mate.out_project_bwd(o, w_o, flags, x, want_dw=False, want_dbias=False)[0], x, w_o, "d_o")
    dx = mate.qkv_project_bwd(x, w_qkv, flags, o, o, o, want_dw=False, want_dbias=False)[0]
    product_close(dx, o.reshape(B, -1).repeat(1, 3), w_qkv, "dx")


# tiles of 192 x 128 that two groups of wavefronts share: 16 token tiles of two sequences with one row in the last
# (QKV), and 49 token tiles of one sequence (output)
@pytest.mark.parametrize("B,N,H,E", [(2, 897, 12, 768), (1, 6145, 12, 768)])
def test_one_round_of_shared_tiles(B, N, H, E):
    check(N, B, N, H, E, pad_tail=N // 5)


# both gradients in one launch: one token, several sequences with a shorter last block, all of one sequence's tail
# padding, the two tile shapes of the product, more dW tiles than products' tiles and fewer
@pytest.mark.parametrize("B,N,H,E", [(1, 1, 2, 128), (3, 65, 12, 768), (1, 1024, 16, 1024), (2, 130, 4, 1152), (9, 100, 24, 128)])
def test_both_gradients_in_one_launch(B, N, H, E):
    check_bwd(N, B, N, H, E, pad_tail=N // 2)


# ... and each alone, bit for bit, and both replayed from a graph (the words that ranges announce themselves with must be
# as good as new each time): dW whole and in ranges that are added in pairs, either tile shape
@pytest.mark.parametrize("B,N,H,E", [(1, 300, 12, 768), (1, 2048, 12, 768), (8, 512, 12, 768), (4, 1000, 8, 512), (4, 1024, 16, 1024)])
def test_each_gradient_alone_is_the_same(B, N, H, E):
    from paper_2109_04312_amd import mate
    x, w_qkv, _, w_o, _, flags, o = make(N, B, N, H, E, pad_tail=N // 7)
    x, w_qkv, w_o, o, fl = dev(x), dev(w_qkv), dev(w_o), dev(o), torch.from_numpy(flags).cuda()
    for call, want_x in ((lambda **kw: mate.qkv_project_bwd(x, w_qkv, fl, o, o, o, **kw), "want_dx"),
                         (lambda **kw: mate.out_project_bwd(o, w_o, fl, x, **kw), "want_do")):
        both, again = call(), call()
        no_w, no_x = call(want_dw=False, want_dbias=False), call(**{want_x: False})
        torch.cuda.synchronize()
        assert all(torch.equal(u, v) for u, v in zip(both, again))
        assert torch.equal(no_w[0], both[0]) and torch.equal(no_x[1], both[1]) and torch.equal(no_x[2], both[2])
        ws = torch.full((mate.mate_project_bwd_workspace_bytes(B, N, H, E) // 4 + 1,), float("nan"), device="cuda").view(torch.uint8)
        side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            captured = call(ws=ws)
        for replay in range(3):
            for y in captured:
                y.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(u, v) for u, v in zip(both, captured)), replay
            call(ws=ws)                                 # eager work on the same words


# dW without the other gradient: one token, tiles of 64 x 64 (one range, and several), 128 x 64 (the same) and 128 x 128, and
# more token blocks than the form shared with the product is for
@pytest.mark.parametrize("B,N,H,E", [(1, 1, 2, 128), (1, 2048, 4, 256), (3, 65, 12, 768), (2, 2047, 8, 512), (2, 200, 16, 1024),
                                     (9, 541, 6, 384)])
def test_weight_gradient_alone(B, N, H, E):
    from paper_2109_04312_amd import mate
    x, w_qkv, _, w_o, _, flags, o = make(N, B, N, H, E, pad_tail=N // 6)
    rng = np.random.default_rng(N)
    dq, dk, dv = (bf16(rng.standard_normal((B, H, N, 64))) for _ in range(3))
    dy = bf16(rng.standard_normal((B, N, E)))
    fl, n_tok = torch.from_numpy(flags).cuda(), max(1, int((flags != P).sum()))
    _, rw, rb = orc.project_qkv_backward(x, w_qkv, flags, dq, dk, dv, H)
    _, rwo, rbo = orc.project_out_backward(o, w_o, flags, dy)
    ws = torch.full((mate.mate_project_bwd_workspace_bytes(B, N, H, E) // 4 + 1,), float("nan"), device="cuda").view(torch.uint8)
    x, w_qkv, w_o, o, dq, dk, dv, dy = (dev(y) for y in (x, w_qkv, w_o, o, dq, dk, dv, dy))
    for call, want_x, want_w, want_b in ((lambda **kw: mate.qkv_project_bwd(x, w_qkv, fl, dq, dk, dv, ws=ws, **kw), "want_dx", rw, rb),
                                         (lambda **kw: mate.out_project_bwd(o, w_o, fl, dy, ws=ws, **kw), "want_do", rwo, rbo)):
        _, dw, db = call(**{want_x: False})
        both = call()
        torch.cuda.synchronize()
        close_f32(dw, want_w, "dw", n_tok)
        close_f32(db, want_b, "dbias", n_tok)
        if B * -(-N // 64) <= 64:
            assert torch.equal(dw, both[1]) and torch.equal(db, both[2])
        side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            _, dw2, db2 = call(**{want_x: False})
        for replay in range(3):
            dw2.fill_(float("nan")), db2.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(dw, dw2) and torch.equal(db, db2), replay
            call()                                      # eager work on the same words
