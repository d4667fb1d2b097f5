"""GPU parity at the edges of the kernels that take any shape: sizes that are no multiple of a tile, the
smallest and the largest of a range, and the borders between two kernels of a dispatch."""
import numpy as np
import pytest
import torch

import als_inputs as I
import paper_2401_09135_amd as A
from oracle import lm, run
from test_gpu_kernels import _attention_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def _model(**kw):
    w = I.workload("tiny")
    w.update(dict(L=1, d=64, h=2, ff=64, V=64, S=8, B=2, dtype="f32"), **kw)
    return w


def _loss_grad(w, tok, flags=0):
    theta0 = I.theta0(lm.param_layout(w), w["seed"])
    ctx = A.Context(A.Config.from_workload(w, flags=flags), theta0, n_streams=1)
    loss, g = ctx.worker_loss_grad(0, torch.from_numpy(tok).to(DEV))
    ctx.close()
    return theta0, loss, g


@pytest.mark.parametrize("V,B,S", [(2, 1, 3),           # one bit
                                   (256, 3, 40), (257, 3, 40),        # one digit of 8 bits, two
                                   (4095, 2, 70), (4096, 2, 70),      # V + 1 entries in one and in two blocks of 4096
                                   (65537, 1, 65),                    # three digits
                                   (300, 17, 1000)])                  # more than one tile of 16384 positions
def test_token_order_of_the_embedding_gradient(V, B, S):
    """dE sums dx over the sorted position list of every token: a position out of place or missing
    puts a whole row of dx into the wrong sum.  fp32 mode, so the bound is that of the sums."""
    w = _model(V=V, B=B, S=S)
    tok = I.TokenStream(1, 0, B, S, V).take(1)[0]
    theta0, loss, g = _loss_grad(w, tok)
    rloss, rg = lm.loss_and_grad(theta0, tok, w)
    assert abs(loss - rloss) < 1e-5 * abs(rloss)
    assert _rel(lm.views(g, w)["E"], lm.views(rg, w)["E"]) < 1e-5


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 31, 63), (32, 65, 65), (130, 70, 256),     # 32 x 32 tiles in natural order
                                   (31, 33, 257), (70, 40, 511), (31, 33, 513), (40, 96, 640),   # 4 and 8 shares of K
                                   (769, 1025, 65), (832, 960, 128),                # 64 x 64
                                   (2047, 2049, 33), (2048, 2048, 96)])             # 128 x 128, the least number of tiles
@pytest.mark.parametrize("al,bl", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_fp32_products(M, N, K, al, bl):
    """Every layout and epilogue at ragged and whole sizes, from operands that are not 16-byte aligned.  A sum of K fp32
    products in any order is off by at most K 2^-24 sum |a b|; the epilogue adds a few roundings."""
    gen = torch.Generator(device=DEV).manual_seed(M + N + K)
    r = lambda *s: torch.randn(*s, device=DEV, generator=gen)
    odd = lambda x: torch.cat([x.new_zeros(1), x.flatten()])[1:].view(x.shape)   # one element off the alignment
    a, b, res, u = r(M, K), r(K, N), r(M, N), r(M, N)
    ad, bd = odd(a if al == 0 else a.t().contiguous()), odd(b if bl == 0 else b.t().contiguous())
    ref, bound = a.double() @ b.double(), (K + 4) * 2.0 ** -24 * (a.abs().double() @ b.abs().double()) + 1e-7
    for epi, want, scale in ((0, ref, 1.0), (1, ref + res.double(), 1.0), (3, ref * u.double(), u.double().abs())):
        c = torch.full((M, N), float("nan"), device=DEV)
        A.step_gemm(ad, bd, c, M, N, K, al, bl, epi=epi, R=res if epi == 1 else None, U=u if epi == 3 else None)
        assert ((c.double() - want).abs() <= bound * scale + 2.0 ** -22 * want.abs()).all(), epi
    c, c2 = torch.full((M, N), float("nan"), device=DEV), torch.full((M, N), float("nan"), device=DEV)
    A.step_gemm(ad, bd, c, M, N, K, al, bl, epi=2, C2=c2)
    x = ref.requires_grad_()
    y = torch.nn.functional.gelu(x, approximate="tanh")
    y.sum().backward()
    assert ((c2.double() - y.detach()).abs() <= 1.2 * bound + 1e-6 * (1 + y.detach().abs())).all()
    assert ((c.double() - x.grad).abs() <= 1.2 * bound + 1e-5).all()


@pytest.mark.parametrize("M,N,K", [(128, 128, 512), (512, 256, 1024), (128, 384, 576),   # 32 x 32 tiles, whole slices and a last one of 64
                                   (1024, 896, 896), (640, 640, 640),               # 64 x 64
                                   (8192, 256, 512),                                # 128 x 64
                                   (512, 512, 448), (2048, 1280, 512),              # 128 x 128 kernels on both sides of the rule
                                   (2048, 2048, 64), (2304, 1792, 64)])             # 64 and 63 tiles of 256 x 256
@pytest.mark.parametrize("al,bl,epi", [(0, 0, 0), (0, 0, 1), (0, 0, 2), (0, 1, 0), (0, 1, 3), (1, 0, 0)])
def test_small_aligned_bf16_products(M, N, K, al, bl, epi):
    """Where the kernel is chosen by the number of tiles: fp32 results within K 2^-24 sum |a b| of float64, bf16 ones
    within one rounding (2^-9) more."""
    gen = torch.Generator(device=DEV).manual_seed(M + N + K)
    r = lambda *s: torch.randn(*s, device=DEV, generator=gen)
    a, b, res, u = r(M, K).bfloat16(), r(K, N).bfloat16(), r(M, N), r(M, N).bfloat16()
    ad, bd = a if al == 0 else a.t().contiguous(), b if bl == 0 else b.t().contiguous()
    out = torch.bfloat16 if epi >= 2 else torch.float32
    c, c2 = (torch.full((M, N), float("nan"), dtype=out, device=DEV) for _ in range(2))
    ws = torch.empty(2 * M * N, device=DEV)
    A.k_gemm_ex(ad, bd, c, M, N, K, al, bl, use_mfma=True, epi=epi, R=res if epi == 1 else None, C2=c2 if epi == 2 else None,
                U=u if epi == 3 else None, ws=ws)
    ref, bound = a.double() @ b.double(), (K + 4) * 2.0 ** -24 * (a.abs().double() @ b.abs().double()) + 1e-6
    if epi == 2:
        x = ref.requires_grad_()
        y = torch.nn.functional.gelu(x, approximate="tanh")
        y.sum().backward()
        assert ((c2.double() - y.detach()).abs() <= 1.2 * bound + 2.0 ** -8 * y.detach().abs()).all()
        assert ((c.double() - x.grad).abs() <= 1.2 * bound + 1e-5 + 2.0 ** -8 * x.grad.abs()).all()
    else:
        want, scale = (ref + res.double(), 1.0) if epi == 1 else (ref * u.double(), u.double().abs()) if epi == 3 else (ref, 1.0)
        assert ((c.double() - want).abs() <= bound * scale + (2.0 ** -8 if epi == 3 else 2.0 ** -22) * want.abs()).all()


@pytest.mark.parametrize("M,N,K", [(128, 128, 64), (256, 128, 256), (128, 256, 320), (256, 384, 448),   # 64 x 64 tiles: one slice, around the 5 in flight
                                   (2048, 1152, 192), (384, 896, 832),                                  # the most of them; K beyond the kernels that share K
                                   (2560, 1024, 192), (2560, 1024, 256), (1280, 2048, 320), (3840, 896, 448)])   # 128 x 128: around the 4 in flight
@pytest.mark.parametrize("al,bl,epi", [(0, 0, 0), (0, 0, 1), (0, 0, 2), (0, 1, 0), (0, 1, 3)])
def test_products_with_deep_prefetch(M, N, K, al, bl, epi):
    test_small_aligned_bf16_products(M, N, K, al, bl, epi)


@pytest.mark.parametrize("M,N,K", [(256, 256, 2112), (1024, 896, 8192), (8192, 256, 4160),
                                   (1024, 128, 8192), (128, 256, 8192)])           # 128 rows or columns: not split
def test_input_gradient_split_along_k(M, N, K):
    gen = torch.Generator(device=DEV).manual_seed(K)
    a, b = torch.randn(M, K, device=DEV, generator=gen).bfloat16(), torch.randn(N, K, device=DEV, generator=gen).bfloat16()
    for size in (2, 3, 16):   # as many partials as the workspace holds
        c = torch.full((M, N), float("nan"), device=DEV)
        A.k_gemm(a, b, c, M, N, K, 0, 1, use_mfma=True, ws=torch.empty(size * M * N, device=DEV))
        bound = (K + 4) * 2.0 ** -24 * (a.abs().double() @ b.abs().double().t())
        assert ((c.double() - a.double() @ b.double().t()).abs() <= bound).all()
    c = torch.full((M, N), float("nan"), device=DEV)
    A.k_gemm(a, b, c, M, N, K, 0, 1, use_mfma=True)
    assert ((c.double() - a.double() @ b.double().t()).abs() <= bound).all()


@pytest.mark.parametrize("kw", [dict(d=64, h=1, ff=192, V=201, S=33, B=3),          # nothing is a multiple of 128
                                dict(d=320, h=5, ff=1280, V=5003, S=200, B=3),
                                dict(d=128, h=2, ff=128, V=255, S=64, B=2),         # aligned blocks, a ragged head
                                dict(d=128, h=2, ff=128, V=256, S=65, B=1),         # ragged blocks, an aligned head
                                dict(d=64, h=1, ff=64, V=2050, S=683, B=3)])        # 17 x 17 tiles of 128 x 128 in the head
def test_ragged_bf16_models_match_the_generic_products(kw):
    """The same bf16 operands and roundings in both modes, other orders of fp32 sums: results differ by bf16 roundings that
    fall the other way (2^-9 each, a random few per sum), an order below the distance of either from fp32 (1e-2)."""
    w = _model(**kw)
    w["dtype"] = "bf16"
    tok = I.TokenStream(1, 0, w["B"], w["S"], w["V"]).take(1)[0]
    theta0, loss, g = _loss_grad(w, tok)
    _, gloss, gg = _loss_grad(w, tok, flags=1)
    assert abs(loss - gloss) < 2e-4 * abs(gloss)
    a, b = lm.views(g, w), lm.views(gg, w)
    for name in a:
        assert _rel(a[name], b[name]) < 5e-3, name
    _, rg = lm.loss_and_grad(theta0, tok, w)
    assert _rel(g, rg) < 1.1 * _rel(gg, rg)


@pytest.mark.parametrize("V,B,S", [(3, 1, 1), (1000, 1, 63), (4094, 3, 341),     # one wavefront; V + 1 entries in one run of 4096
                                   (4097, 16, 1000), (4096, 16, 1024),            # 16000 and 16384 positions, all of the tile
                                   (32767, 2, 512), (32768, 2, 512)])             # the largest vocabulary in LDS and the next
def test_token_order_in_lds(V, B, S):
    test_token_order_of_the_embedding_gradient(V, B, S)


# Small steps order their positions by counting: whole and partial groups of 64 positions and questions, the largest vocabulary, the most
# comparisons; and the sorts at the sizes that are left to them: just more comparisons (one bit, one digit and two, the largest vocabulary in
# LDS), a larger vocabulary (three digits), more of both.
@pytest.mark.parametrize("V,B,S", [(2, 1, 63), (63, 1, 64), (64, 5, 13), (131072, 1, 65), (13, 12, 1020),
                                   (14, 12, 1020), (256, 12, 1020), (257, 12, 1020), (32767, 5, 820), (32768, 5, 820), (131073, 1, 65), (65537, 4, 600)])
def test_token_order_by_counting_and_sorting(V, B, S):
    test_token_order_of_the_embedding_gradient(V, B, S)


@pytest.mark.parametrize("V,B,S,n,parts", [(256, 8, 32, 400, 2), (1000, 1, 63, 500, 4), (4094, 3, 341, 40, 8), (40000, 1, 65, 160, 8)])
def test_calls_of_many_steps_sort_their_tokens(V, B, S, n, parts):
    """Long calls sort the tokens of all their steps side by side where short ones count: the same order, so the same bits as the
    same steps in several calls."""
    assert A.token_order_route(B * S, V, n).startswith("sort") and A.token_order_route(B * S, V, n // parts) == "counting"
    w = _model(L=1, d=64, h=1, ff=64, V=V, S=S, B=B)
    cfg = A.Config.from_workload(w, max_local_steps=n)
    cfg.n_workers = 1
    tok = torch.from_numpy(I.TokenStream(1, 0, B, S, V).take(n)).to(DEV)
    out = []
    for m in (1, parts):
        ctx = A.Context(cfg, I.theta0(lm.param_layout(w), 3), n_streams=1)
        for i in range(m):
            ctx.worker_local_steps(0, tok[i * (n // m):(i + 1) * (n // m)], 1e-3)
        out.append([ctx.get_vector(v) for v in ("worker_theta", "adam_v", "grad")])
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("V", [64, 65, 71, 2048, 2049, 8192, 8193, 8200, 32767, 32768, 32769])   # whole and partial groups of 8; 256 and 1024 threads; three passes
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_cross_entropy_of_any_vocabulary(V, dtype):
    """Loss and the gradients that come straight from dlogits against the oracle: fp32 sums of V values (1e-5), bf16 logits and dlogits as
    in the other bf16 tests (their distance from fp32 is that of the roundings, 1e-2 of a gradient)."""
    w = _model(V=V, S=5, B=3)
    w["dtype"] = dtype
    tok = I.TokenStream(1, 0, 3, 5, V).take(1)[0]
    theta0, loss, g = _loss_grad(w, tok)
    rloss, rg = lm.loss_and_grad(theta0, tok, w)
    assert abs(loss - rloss) < (1e-5 if dtype == "f32" else 1e-3) * abs(rloss)
    assert _rel(lm.views(g, w)["Wout"], lm.views(rg, w)["Wout"]) < (1e-5 if dtype == "f32" else 2e-2)
    assert _rel(lm.views(g, w)["gf"], lm.views(rg, w)["gf"]) < (1e-5 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("d,S", [(512, 256), (576, 256), (1024, 128), (1024, 129)])    # T = 2 S: the last in one launch, the first in two
def test_embedding_gradient_of_wide_small_steps(d, S):
    """The same sums over a token's positions in either form: fp32 gradients against the oracle."""
    w = _model(d=d, h=d // 64, ff=64, V=300, S=S, B=2)
    assert A.embed_grad_route(2 * S, 300, d) == ("one launch" if S in (256, 128) and d != 576 else "two launches")
    tok = I.TokenStream(1, 0, 2, S, 300).take(1)[0]
    theta0, loss, g = _loss_grad(w, tok)
    rloss, rg = lm.loss_and_grad(theta0, tok, w)
    assert abs(loss - rloss) < 1e-5 * abs(rloss)
    for name in ("E", "Ppos", "g10", "gf"):
        assert _rel(lm.views(g, w)[name], lm.views(rg, w)[name]) < 1e-5, name


@pytest.mark.parametrize("dtype,kw", [("f32", dict(L=17, S=7, B=1)),                              # more products than one launch takes
                                      ("f32", dict(L=2, d=192, h=3, ff=320, V=333, S=31, B=2)),       # 32 x 32 tiles
                                      ("f32", dict(L=1, d=128, h=2, ff=192, V=130, S=103, B=5)),      # 8 shares
                                      ("f32", dict(L=2, d=512, h=8, ff=1024, V=70, S=33, B=1)),       # 64 x 64
                                      ("f32", dict(L=2, d=512, h=8, ff=2048, V=700, S=17, B=1)),      # 128 x 128
                                      ("bf16", dict(L=17, S=7, B=1)),
                                      ("bf16", dict(L=1, d=64, ff=192, V=131, S=31, B=3)),            # 32 x 32
                                      ("bf16", dict(L=1, d=256, h=4, ff=640, V=333, S=65, B=2)),      # 64 x 64
                                      ("bf16", dict(L=3, d=320, h=5, ff=1280, V=133, S=33, B=1)),     # 128 x 64
                                      ("bf16", dict(L=2, d=384, h=6, ff=1536, V=2048, S=64, B=3)),    # aligned, 92 tiles of 256 x 256
                                      ("bf16", dict(L=2, d=512, h=8, ff=2048, V=700, S=17, B=1))])    # 128 x 128
def test_weight_gradients_as_one_list(dtype, kw):
    """Flag bit 1 keeps one launch per product: the same operands, sums in the order of another tile at most, so fp32 gradients
    agree to a few roundings of their sums over the tokens (2^-24 sqrt(515) 4 < 1e-5)."""
    w = _model(**kw)
    w["dtype"] = dtype
    tok = I.TokenStream(1, 0, w["B"], w["S"], w["V"]).take(1)[0]
    _, loss, g = _loss_grad(w, tok)
    _, loss1, g1 = _loss_grad(w, tok, flags=2)
    assert loss == loss1
    a, b = lm.views(g, w), lm.views(g1, w)
    for name in a:
        assert _rel(a[name], b[name]) < 1e-5, name


@pytest.mark.parametrize("B,S,h,dh", [(33, 1, 2, 32), (33, 16, 2, 64), (33, 17, 2, 32),   # one tile, one and one row
                                      (1, 33, 1, 64), (1, 63, 1, 32), (2, 129, 3, 64),     # last tile of 1, 15, 1 rows; idle wavefronts
                                      (16, 272, 16, 32), (9, 1009, 8, 64),                 # two row blocks per wavefront
                                      (1, 70, 3, 40)])                                     # a width of the vector kernels
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_attention_in_fp32_arithmetic(B, S, h, dh, dt):
    """Sums of up to 1009 fp32 products in tile order: 2^-24 sqrt(1009) 4 < 1e-5; bf16 storage: one rounding (2^-9) of o and
    dqkv, and of the o that the row dots are formed from."""
    o, ro, lse, rlse, dq, rdq = _attention_case(B, S, h, dh, dt, 0, fwd=A.step_attention_fwd, bwd=A.step_attention_bwd)
    assert _rel(o, ro) < (1e-5 if dt == torch.float32 else 4e-3)
    np.testing.assert_allclose(lse, rlse, rtol=1e-5, atol=1e-5)
    if S > 1:
        assert _rel(dq, rdq) < (1e-5 if dt == torch.float32 else 8e-3)


@pytest.mark.parametrize("B,S,h,dh", [(1, 34, 1, 32), (1, 64, 3, 64), (2, 65, 1, 32),      # 3, 4 and 5 tiles for four wavefronts
                                      (1, 1023, 2, 64), (1, 1024, 2, 32), (16, 256, 16, 32),   # the longest chains; the most row blocks
                                      (37, 32, 2, 64), (65, 31, 1, 32)])                   # short rows: a row block per wavefront
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_attention_with_wavefronts_that_share_a_row_block(B, S, h, dh, dt):
    test_attention_in_fp32_arithmetic(B, S, h, dh, dt)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_attention_hides_what_a_query_does_not_see(bad):
    """Row 37 of v (k) is not finite: the output (dq) of every earlier position is what it is without it."""
    B, S, h, dh = 1, 70, 2, 64
    d = h * dh
    gen = torch.Generator(device=DEV).manual_seed(3)
    qkv = torch.randn(B * S, 3 * d, device=DEV, generator=gen)
    d_o = torch.randn(B * S, d, device=DEV, generator=gen)
    res = []
    for part in (None, 1, 2):
        x = qkv.clone()
        if part:
            x[37, part * d:(part + 1) * d] = bad
        o, lse, sc, dq = torch.empty(B * S, d, device=DEV), torch.empty(B * h * S, device=DEV), torch.empty(B * h * S, device=DEV), torch.empty_like(x)
        A.step_attention_fwd(x, o, lse, B, S, h, dh)
        A.step_attention_bwd(x, o, d_o, lse, sc, dq, B, S, h, dh)
        res.append((o.cpu(), dq.cpu()))
    for o, dq in res[1:]:
        assert torch.equal(o[:37], res[0][0][:37])
        assert torch.equal(dq[:37, :d], res[0][1][:37, :d])
    assert not torch.isfinite(res[2][0][37:]).any()


@pytest.mark.parametrize("B,S,h,dh", [(2, 33, 2, 32), (3, 200, 5, 64), (1, 1023, 1, 64),      # wavefronts that share a row block
                                      (33, 257, 16, 32), (33, 257, 16, 64),                # two row blocks per wavefront in both directions
                                      (65, 32, 1, 64)])                                    # one
def test_computed_operands_of_bf16_attention_stay_fp32(B, S, h, dh):
    """With whole fp32 probabilities and sums of up to 1024 products an output is within 2^-24 sqrt(1024) 4 of the exact one, less
    than a 500th of the spacing of bf16: all but 1 % of the outputs are the correctly rounded ones.  (Probabilities rounded to
    bf16 would move more than a tenth of them.)"""
    o, ro, lse, rlse, dq, rdq = _attention_case(B, S, h, dh, torch.bfloat16, 0, fwd=A.step_attention_fwd, bwd=A.step_attention_bwd)
    want = torch.from_numpy(ro).to(torch.bfloat16).float().numpy()
    assert (o != want).mean() < 0.01
    np.testing.assert_allclose(lse, rlse, rtol=1e-5, atol=1e-5)
    assert _rel(dq, rdq) < 8e-3


@pytest.mark.parametrize("B,S,h,dh", [(1, 70, 2, 64), (1, 70, 2, 32), (520, 33, 6, 64)])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_bf16_attention_hides_what_a_query_does_not_see(B, S, h, dh, bad):
    """Row 17 of v (k) of the first sample is not finite: the output (dq) of every earlier position and of every other sample is what it
    is without it, and an infinite v gives infinite outputs, not NaN, wherever it has a weight (parts of it that are 0 included)."""
    d = h * dh
    gen = torch.Generator(device=DEV).manual_seed(3)
    qkv = torch.randn(B * S, 3 * d, device=DEV, generator=gen).bfloat16()
    d_o = torch.randn(B * S, d, device=DEV, generator=gen).bfloat16()
    res = []
    for part in (None, 1, 2):
        x = qkv.clone()
        if part:
            x[17, part * d:(part + 1) * d] = bad
        o, lse, sc = torch.empty(B * S, d, device=DEV, dtype=torch.bfloat16), torch.empty(B * h * S, device=DEV), torch.empty(B * h * S, device=DEV)
        dq = torch.empty_like(x)
        A.step_attention_fwd(x, o, lse, B, S, h, dh)
        A.step_attention_bwd(x, o, d_o, lse, sc, dq, B, S, h, dh)
        res.append((o.cpu(), dq.cpu()))
    for o, dq in res[1:]:
        assert torch.equal(o[:17], res[0][0][:17]) and torch.equal(o[S:], res[0][0][S:])
        assert torch.equal(dq[:17, :d], res[0][1][:17, :d]) and torch.equal(dq[S:], res[0][1][S:])
    v_out = res[2][0][17:S].float()
    assert torch.isinf(v_out).all() if np.isinf(bad) else torch.isnan(v_out).all()


def test_a_gradient_does_not_depend_on_the_workers_beside_it():
    """8192 tokens of width 512: 64 tiles of 256 x 256 in the products of a layer, and a context of one and of four workers."""
    w = _model(d=512, h=8, ff=512, V=512, S=256, B=32)
    w["dtype"] = "bf16"
    tok = I.TokenStream(1, 0, w["B"], w["S"], w["V"]).take(1)[0]
    w["k"] = 1
    _, loss, g = _loss_grad(w, tok)
    w["k"] = 4
    _, loss4, g4 = _loss_grad(w, tok)
    assert loss == loss4 and np.array_equal(g, g4)


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_flag_bit_0_and_use_mfma_0_are_vector_code(dt):
    """The same bits from both, whatever the shape: one kernel, and not the matrix cores', whose fp32 sums run in another order."""
    gen = torch.Generator(device=DEV).manual_seed(11)
    r = lambda *s: torch.randn(*s, device=DEV, generator=gen).to(dt)
    M, N, K = 128, 192, 1024
    a, b = r(M, K), r(K, N)
    c = [torch.empty(M, N, device=DEV) for _ in range(3)]
    A.k_gemm(a, b, c[0], M, N, K)
    A.step_gemm(a, b, c[1], M, N, K, flags=1)
    A.step_gemm(a, b, c[2], M, N, K)
    assert torch.equal(c[0], c[1]) and not torch.equal(c[0], c[2])
    B, S, h, dh = 1, 200, 2, 64
    qkv, d_o = r(B * S, 3 * h * dh), r(B * S, h * dh)
    res = []
    for fwd, bwd, how in ((A.k_attention_fwd, A.k_attention_bwd, False), (A.step_attention_fwd, A.step_attention_bwd, 1),
                          (A.step_attention_fwd, A.step_attention_bwd, 0)):
        o, lse, sc, dq = torch.empty_like(d_o), torch.empty(B * h * S, device=DEV), torch.empty(B * h * S, device=DEV), torch.empty_like(qkv)
        fwd(qkv, o, lse, B, S, h, dh, how)
        bwd(qkv, o, d_o, lse, sc, dq, B, S, h, dh, how)
        res.append((o, lse, dq))
    assert all(torch.equal(x, y) for x, y in zip(res[0], res[1]))
    assert not all(torch.equal(x, y) for x, y in zip(res[0], res[2]))


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_a_product_of_more_than_2_22_small_tiles(dt):
    """131072 x 33001: element offsets beyond 2^32.  Rows and columns at the ends and across them against float64."""
    M, N, K = 131072, 33001, 40
    gen = torch.Generator(device=DEV).manual_seed(12)
    a, b = torch.randn(M, K, device=DEV, generator=gen).to(dt), torch.randn(K, N, device=DEV, generator=gen).to(dt)
    c = torch.full((M, N), float("nan"), dtype=dt, device=DEV)
    A.step_gemm(a, b, c, M, N, K)
    half = 2.0 ** -8 if dt == torch.bfloat16 else 2.0 ** -22
    for rows, cols in ((torch.arange(0, M, 4001), slice(None)), (torch.arange(M - 130, M), slice(None)), (slice(None), torch.arange(0, N, 3001)),
                       (slice(None), torch.arange(N - 3, N))):
        x, y = a[rows].double(), b[:, cols].double()
        bound = (K + 4) * 2.0 ** -24 * (x.abs() @ y.abs()) + half * (x @ y).abs()
        assert ((c[rows][:, cols] if isinstance(cols, slice) else c[:, cols]).double() - x @ y).abs().le(bound).all()


@pytest.mark.parametrize("out", [torch.float32, torch.bfloat16])
def test_both_outputs_of_gelu_are_written_for_any_output_type(out):
    M, N, K = 50, 70, 30
    gen = torch.Generator(device=DEV).manual_seed(13)
    a, b = torch.randn(M, K, device=DEV, generator=gen).bfloat16(), torch.randn(K, N, device=DEV, generator=gen).bfloat16()
    c, c2 = (torch.full((M, N), float("nan"), dtype=out, device=DEV) for _ in range(2))
    A.step_gemm(a, b, c, M, N, K, epi=2, C2=c2)
    x = (a.double() @ b.double()).requires_grad_()
    y = torch.nn.functional.gelu(x, approximate="tanh")
    y.sum().backward()
    half = 2.0 ** -8 if out == torch.bfloat16 else 1e-5   # one rounding; fp32 sums of 30 products and tanhf
    assert ((c2.double() - y.detach()).abs() <= half * (1 + y.detach().abs())).all()
    assert ((c.double() - x.grad).abs() <= half * (1 + x.grad.abs())).all()


@pytest.mark.parametrize("M,N,K", [(5, 3, 2), (64, 48, 200), (512, 512, 256), (100, 900, 255)])
@pytest.mark.parametrize("al,bl", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_fp32_products_of_few_tiles_have_the_bits_of_a_plain_loop(M, N, K, al, bl):
    """One fused multiply-add after the other, k ascending, whatever the number of tiles.  (A product of two fp32 numbers is exact in
    float64; its sum with the accumulator is rounded there first, which changes one result in 2^29.)"""
    gen = torch.Generator(device=DEV).manual_seed(M + N + K)
    a, b = torch.randn(M, K, device=DEV, generator=gen), torch.randn(K, N, device=DEV, generator=gen)
    c = torch.full((M, N), float("nan"), device=DEV)
    A.step_gemm(a if al == 0 else a.t().contiguous(), b if bl == 0 else b.t().contiguous(), c, M, N, K, al, bl)
    want = torch.zeros(M, N, device=DEV)
    for k in range(K):
        want = (a[:, k:k + 1].double() * b[k].double() + want.double()).float()
    assert (c != want).sum().item() <= 1 + M * N * K >> 26


@pytest.mark.parametrize("kw", [dict(ff=320, V=300, S=36), dict(d=128, h=4, V=300, S=33), dict(d=128, h=4, ff=384, V=511, S=60)])
def test_short_fp32_runs_are_as_near_to_float64_as_the_fp32_oracle(kw):
    """Models just past the smallest one, whose sums are longer than those in natural order: what fp32 mode holds there is the accuracy
    of an fp32 program (a quarter for the spread between two orders of sums), not its bits."""
    w = dict(I.workload("tiny"), N=1, **kw)
    theta0 = I.theta0(lm.param_layout(w), w["seed"])
    stream = lambda i: I.TokenStream(w["seed"], i, w["B"], w["S"], w["V"])
    rule = dict(poly_exponent=0.5)
    ref32, ref64 = (run.run_async(w, theta0, stream, rule=rule, dtype=t)["theta"] for t in (np.float32, np.float64))
    got = A.run_async(w, theta0, stream, rule=dict(rule))
    got["ctx"].close()
    assert _rel(got["theta"], ref64) < 1.25 * _rel(ref32, ref64)


def test_every_matrix_core_kernel_is_timed_on_request():
    """One entry per kernel with all of its flops, for products and for both lists of weight gradients."""
    dev = lambda m, n, dt: torch.zeros(m, n, dtype=dt, device=DEV)
    bf, f32 = torch.bfloat16, torch.float32
    cases = [((256, 128, 64), bf, "gemm_deep_kernel<64, 64, 0, STORE, float>"), ((2560, 1024, 64), bf, "gemm_deep_kernel<128, 128, 0, STORE, float>"),
             ((100, 100, 100), bf, "gemm_any_kernel<32, 32, 0, 0>"), ((2049, 2049, 33), bf, "gemm_any_kernel<128, 128, 0, 0>"),
             ((100, 100, 100), f32, "gemm_f32_kernel<32, 32 natural, 0, 0>"), ((100, 100, 300), f32, "gemm_f32_kernel<32, 32 / 4, 0, 0>"),
             ((1024, 768, 64), f32, "gemm_f32_kernel<64, 64, 0, 0>"), ((2048, 2048, 64), f32, "gemm_f32_kernel<128, 128, 0, 0>")]
    try:
        A.prof_enable(1)
        for (M, N, K), dt, name in cases:
            A.step_gemm(dev(M, K, dt), dev(K, N, dt), dev(M, N, f32), M, N, K)
            (got,) = A.prof_collect()
            assert got[0] == name and got[1] == 1 and got[2] > 0 and got[3] == 2.0 * M * N * K
        for dtype, name in (("f32", "gemm_f32_dw_list_kernel<32, 32 natural>"), ("bf16", "gemm_any_dw_list_kernel<64, 64>")):
            w = _model(L=17, S=7, B=1)
            w["dtype"] = dtype
            _loss_grad(w, I.TokenStream(1, 0, w["B"], w["S"], w["V"]).take(1)[0])
            got = {n: (l, f) for n, l, _, f in A.prof_collect()}
            d, T = w["d"], w["B"] * w["S"]
            assert got[name] == (2, 2.0 * T * d * (17 * (4 * d + 2 * w["ff"]) + w["V"]))   # 69 products, at most 64 in a launch
    finally:
        A.prof_enable(0)
        A.prof_collect()
