"""Kernels at the sizes where they can go wrong: edges of tiles, remainders, the smallest and largest of a
range, each against float64."""
import numpy as np
import pytest
import torch

from paper_2507_21276_amd import binding as Bd
from paper_2507_21276_amd import synth_inputs as S
from parity_util import TOL, assert_close, dev, host, out_rounding_bound
from test_gpu_stage import check_train, make_stage, run_train

pytestmark = pytest.mark.gpu
DT = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def q(x, name):
    """Values exactly representable in the storage type, as float64."""
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(DT[name]).to(torch.float64).numpy()


@pytest.mark.parametrize("name", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("T,N", [(1, 8), (63, 264), (64, 256), (65, 248), (1000, 24), (130, 7)])
def test_colsum_edges(name, T, N):
    """Row chunks of 64, column groups of 256, widths that are not multiples of eight (one column per thread).
    An element passes through fewer than 40 fp32 additions of partial sums below 6 sqrt(T): 1e-5 of the RMS."""
    x = q(S.normal(6, "x", (T, N)), name)
    for acc in (False, True):
        out = torch.full((N,), 3.0, dtype=torch.float32, device="cuda")
        Bd.lsk_colsum(dev(x, DT[name]), out, accumulate=acc)
        assert_close(host(out), x.sum(axis=0) + (3.0 if acc else 0.0), 2e-5, f"colsum {T}x{N}")


@pytest.mark.parametrize("name", ["bf16", "f16"])
@pytest.mark.parametrize("M,N,T", [(256, 264, 64), (264, 256, 65), (768, 768, 127), (520, 392, 130), (1000, 2304, 191), (256, 256, 1001),
                                   (4104, 2568, 64), (4104, 2568, 101), (4104, 2568, 192)])
def test_weight_gradient_of_any_token_count(name, M, N, T):
    """dW = dY^T X over T tokens: one k tile, whole tiles, a last tile of 1 .. 63 rows, fewer tiles than the ring
    holds, both tile sizes.  Operands are exact, sums fp32: T products of RMS 1 with T 2^-24 relative each."""
    dY, X = q(S.normal(2, "dY", (T, M)), name), q(S.normal(2, "X", (T, N)), name)
    dYd, Xd = dev(dY, DT[name]), dev(X, DT[name])
    ref = (torch.from_numpy(dY).cuda().t().contiguous() @ torch.from_numpy(X).cuda()).cpu().numpy()
    dW = torch.full((M, N), 7.0, dtype=torch.float32, device="cuda")
    for acc in (False, True):
        Bd.lsk_gemm(dYd, Xd, dW, M=M, N=N, K=T, a_kmajor=False, b_kmajor=False, lda=M, ldb=N, accumulate=acc)
        assert_close(host(dW), (1 + acc) * ref, 1e-5, f"dW T={T} acc={acc}")


@pytest.mark.parametrize("name", ["bf16", "f16"])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (129, 512, 2048), (200, 264, 128), (255, 4096, 4096), (255, 12800, 64)])
def test_products_of_64_to_255_rows(name, M, N, K):
    """One tile and two of 128 rows, split along k (>= 32 k tiles, few output tiles) and not, with and without the
    workspace, and the input-gradient layout.  Exact operands, fp32 sums: K 2^-24 of the RMS at the worst."""
    A, W = q(S.normal(3, "A", (M, K)), name), q(S.normal(3, "W", (N, K), 0.05), name)
    Ad, Wd = dev(A, DT[name]), dev(W, DT[name])
    A64, W64 = torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda()
    ref = (A64 @ W64.t().contiguous()).cpu().numpy()
    tol = max(1e-5, K * 2.0 ** -24)
    out = torch.empty(M, N, dtype=torch.float32, device="cuda")
    R = S.normal(3, "R", (M, N))
    ws = torch.empty(8 * M * N, dtype=torch.float32, device="cuda")
    Bd.lsk_gemm(Ad, Wd, out, M=M, N=N, K=K, resid=dev(R, torch.float32))
    assert_close(host(out), ref + R, tol, "forward")
    Bd.lsk_gemm_ws(Ad, Wd, out, ws, resid=dev(R, torch.float32))
    assert_close(host(out), ref + R, tol, "forward with a workspace")
    Bk = q(S.normal(3, "Bk", (K, N), 0.05), name)
    Bd.lsk_gemm(Ad, dev(Bk, DT[name]), out, M=M, N=N, K=K, a_kmajor=True, b_kmajor=False, lda=K, ldb=N)
    assert_close(host(out), (A64 @ torch.from_numpy(Bk).cuda()).cpu().numpy(), tol, "input gradient")


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (31, 33, 65), (128, 128, 128), (64, 256, 64), (130, 70, 129), (1030, 1025, 40), (1030, 1025, 16), (1030, 1025, 1)])
def test_fp32_products_of_both_tile_sizes(M, N, K):
    """32 x 32 and 64 x 64 tiles, k tiles of 64 and 16, all four layouts, remainders in each dimension.  Sums of K
    products in order: K 2^-24 of the largest partial sum at the worst, a few 1e-6 of the RMS here."""
    A, W = S.normal(5, "A", (M, K)), S.normal(5, "W", (N, K))
    ref = A.astype(np.float32).astype(np.float64) @ W.astype(np.float32).astype(np.float64).T
    for ak in (True, False):
        for bk in (True, False):
            out = torch.full((M, N), 2.0, dtype=torch.float32, device="cuda")
            Bd.lsk_gemm(dev(A if ak else A.T, torch.float32), dev(W if bk else W.T, torch.float32), out, M=M, N=N, K=K,
                        a_kmajor=ak, b_kmajor=bk, lda=K if ak else M, ldb=K if bk else N, accumulate=True)
            assert_close(host(out), ref + 2.0, max(4e-6, K * 2.0 ** -24), f"{M}x{N}x{K} {ak} {bk}", atol=1e-6)


@pytest.mark.parametrize("M,N,K", [(16, 16, 4), (17, 33, 15), (33, 128, 77), (1, 512, 128), (512, 528, 130), (528, 272, 193),
                                   (256, 250, 200), (40, 72, 385), (72, 40, 388), (1000, 1000, 49), (1000, 1000, 48)])
@pytest.mark.parametrize("offset", [0, 1])
def test_fp32_products_of_few_tiles(M, N, K, offset):
    """Both tile sizes and every number of wavefronts, shares of the contraction that are short or empty, all four layouts
    with everything the epilogue adds, operands that 16-byte loads can and cannot read.  K products summed in order: K 2^-24
    of the largest partial sum at the worst, 2e-6 of the RMS for the few of a split sum."""
    A, W, R, b = S.normal(6, "A", (M, K)), S.normal(6, "W", (N, K)), S.normal(6, "R", (M, N)), S.normal(6, "b", (N,))
    f64 = lambda x: x.astype(np.float32).astype(np.float64)  # noqa: E731
    ref = f64(A) @ f64(W).T + f64(b) + f64(R) + 2.0

    def at(x):   # the values, `offset` elements behind an aligned address
        buf = torch.empty(x.size + offset, dtype=torch.float32, device="cuda")
        buf[offset:] = dev(x, torch.float32).reshape(-1)
        return buf[offset:]
    for ak in (True, False):
        for bk in (True, False):
            out = torch.full((M, N), 2.0, dtype=torch.float32, device="cuda")
            Bd.lsk_gemm(at(A if ak else A.T), at(W if bk else W.T), out, M=M, N=N, K=K, a_kmajor=ak, b_kmajor=bk,
                        lda=K if ak else M, ldb=K if bk else N, bias=dev(b, torch.float32), resid=dev(R, torch.float32),
                        accumulate=True)
            assert_close(host(out), ref, max(2e-6, K * 2.0 ** -24), f"{M}x{N}x{K} {ak} {bk}")


@pytest.mark.parametrize("M,N", [(640, 1280), (800, 1000), (1000, 900)])   # 200, 208 and 240 tiles of 64 x 64
@pytest.mark.parametrize("K", [64, 65])
def test_fp32_products_of_short_contractions(M, N, K):
    """Both sides of the line between the kernels at contractions of one and two k tiles.  Bar and inputs as above."""
    test_fp32_products_of_few_tiles(M, N, K, 0)


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("T,d", [(1, 8), (9, 520), (1280, 512), (1281, 1024), (2049, 1032)])
@pytest.mark.parametrize("name,pname", [("f16", "f16"), ("bf16", "f32"), ("f32", "bf16")])
def test_norm_backward_over_rows_of_a_workgroup(kind, T, d, name, pname):
    """One and two rows per wavefront at the line between them, columns that end inside a wavefront's load, parameters of
    every type beside operands of another; with and without a residual gradient.  fp32 sums over d and over T rows."""
    x, dh, dres = S.normal(3, "x", (T, d)), q(S.normal(3, "dh", (T, d)), name), S.normal(3, "dres", (T, d))
    g = q(1.0 + S.normal(3, "g", (d,), 0.1), pname)
    mean, rstd = S.normal(3, "m", (T,), 0.1), 1.0 + 0.1 * np.abs(S.normal(3, "r", (T,)))
    f = lambda a: torch.from_numpy(np.asarray(a, np.float32)).cuda().double()  # noqa: E731
    xh = (f(x) - (f(mean)[:, None] if kind == 0 else 0.0)) * f(rstd)[:, None]
    dxh = f(dh) * f(g)
    ref = f(rstd)[:, None] * (dxh - (dxh.mean(1, keepdim=True) if kind == 0 else 0.0) - xh * (dxh * xh).mean(1, keepdim=True))
    dg, db = (torch.empty(d, dtype=torch.float32, device="cuda") for _ in range(2))
    dx, dx16 = torch.empty(T, d, dtype=torch.float32, device="cuda"), torch.empty(T, d, dtype=DT[name], device="cuda")
    for res in (dres, None):
        Bd.lsk_norm_bwd(kind, dev(dh, DT[name]), dev(x, torch.float32), dev(mean, torch.float32), dev(rstd, torch.float32),
                        dev(g, DT[pname]), None if res is None else dev(res, torch.float32), dx, dx16, dg,
                        db if kind == 0 else None, False)
        want = (ref if res is None else ref + f(res)).cpu().numpy()
        assert_close(host(dx), want, 1e-5, "dx", atol=1e-5)
        assert_close(host(dx16), want, 1e-5 + out_rounding_bound(want, name), "dx in the operand type", atol=1e-5)
        assert_close(host(dg), (f(dh) * xh).sum(0).cpu().numpy(), 1e-5, "dgamma")
        if kind == 0:
            assert_close(host(db), f(dh).sum(0).cpu().numpy(), 1e-5, "dbeta")


@pytest.mark.parametrize("name", ["f16", "bf16"])
@pytest.mark.parametrize("M,N,K", [(3000, 3848, 192),    # 16 x 16 tiles of 192 x 256, ragged on both sides
                                   (1915, 4104, 384),    # 15 x 17 of 128 x 256, six k tiles through three buffers
                                   (2000, 4000, 64), (2000, 4000, 128)])   # with something to add: 128 x 256, one and two k tiles
def test_products_of_192_and_128_row_tiles(name, M, N, K):
    """Every epilogue and both layouts of the 16x16x32 kernel's smaller tiles, every element against float64.  fp32 sums of K
    products of 16-bit operands; the SwiGLU epilogue bit for bit against the product followed by the element-wise kernel."""
    dt, dev_ = DT[name], "cuda"
    A, W, Bk = (S.normal_torch(31, n, shape, std, dtype=dt) for n, shape, std in
                (("A", (M, K), 1.0), ("W", (N, K), 0.05), ("Bk", (K, N), 0.05)))
    R, b = S.normal_torch(31, "R", (M, N), 1.0, dtype=torch.float32), S.normal_torch(31, "b", (N,), 1.0, dtype=torch.bfloat16)
    fwd, dgr = A.double() @ W.double().T.contiguous(), A.double() @ Bk.double()
    full = lambda d, v=0.0: torch.full((M, N), v, dtype=d, device=dev_)  # noqa: E731

    def check(got, ref, what):
        e = (got.double() - ref).abs().max().item() / ref.square().mean().sqrt().item()
        lim = 1e-5 + (0.0 if got.dtype == torch.float32 else out_rounding_bound(ref.cpu().numpy(), name))
        assert e <= lim, f"{what}: {e:.2e} > {lim:.2e}"
    for kmajor, ref, w, ld in ((True, fwd, W, K), (False, dgr, Bk, N)):
        kw = dict(M=M, N=N, K=K, a_kmajor=True, b_kmajor=kmajor, lda=K, ldb=ld)
        o16, o32, acc = full(dt), full(torch.float32), full(torch.float32, 2.0)
        Bd.lsk_gemm(A, w, o16, **kw)
        check(o16, ref, f"operand type {kmajor}")
        Bd.lsk_gemm(A, w, o32, **kw)
        check(o32, ref, f"fp32 {kmajor}")
        Bd.lsk_gemm(A, w, acc, accumulate=True, **kw)
        check(acc, ref + 2.0, f"accumulated {kmajor}")
        if kmajor:
            Bd.lsk_gemm(A, w, o32, bias=b, resid=R, **kw)
            check(o32, ref + b.double() + R.double(), "bias and residual")
            Bd.lsk_gemm(A, w, o16, bias=b, **kw)
            check(o16, ref + b.double(), "bias")
    pre = S.normal_torch(31, "pre", (M, 2 * N), 1.0, dtype=dt)
    one, two, da = torch.empty_like(pre), torch.empty_like(pre), full(dt)
    Bd.lsk_gemm_swiglu_bwd(A, Bk, pre, one, da)
    Bd.lsk_gemm(A, Bk, da, M=M, N=N, K=K, a_kmajor=True, b_kmajor=False, lda=K, ldb=N)
    Bd.lsk_swiglu_bwd(da, pre, two)
    assert torch.equal(one, two)


@pytest.mark.parametrize("name", ["f16", "bf16"])
@pytest.mark.parametrize("T,h", [(700, 32), (500, 32), (300, 32)])   # 192 x 256 tiles, 128 x 256, the rotary kernel
def test_rotary_embedding_behind_192_and_128_row_tiles(name, T, h):
    dt, d, half = DT[name], h * 128, 64
    x, w = S.normal_torch(32, "x", (T, d), 1.0, dtype=dt), S.normal_torch(32, "w", (3 * d, d), d ** -0.5, dtype=dt)
    pos = torch.as_tensor(S.uniform_ints(32, "pos", T, 0, 2047).astype(np.int32), device="cuda")
    ang = torch.arange(2048, device="cuda").double()[:, None] * 1e4 ** (-torch.arange(half, device="cuda").double() / half)
    table = torch.stack([ang.cos(), ang.sin()], -1).float().contiguous()
    qkv = torch.empty(T, 3 * d, dtype=dt, device="cuda")
    Bd.lsk_gemm_qkv_rope(x, w, qkv, h, 128, pos, table)
    ref = (x.double() @ w.double().T.contiguous()).reshape(T, 3, h, 128)
    c, s = ang.cos()[pos.long()][:, None], ang.sin()[pos.long()][:, None]
    for part in (0, 1):
        a, b = ref[:, part, :, :half].clone(), ref[:, part, :, half:].clone()
        ref[:, part, :, :half], ref[:, part, :, half:] = a * c - b * s, b * c + a * s
    ref = ref.reshape(T, 3 * d).cpu().numpy()
    # two 16-bit roundings where the rotary kernel follows the product
    assert_close(host(qkv), ref, 1e-5 + 2 * out_rounding_bound(ref, name), "qkv")


@pytest.mark.parametrize("name", ["f16", "bf16"])
@pytest.mark.parametrize("B,L,h", [(1, 1, 1), (2, 128, 3), (3, 160, 2), (2, 161, 2), (1, 257, 3), (1, 640, 2)])
def test_attention_backward_of_64_element_heads(name, B, L, h):
    """Four and eight wavefronts a workgroup at the line between them, sequences that end inside and at the edge of a tile of
    32, 64 and 128 rows.  16-bit probabilities and scores' gradients: the bar of the attention tests."""
    dh, dt, d = 64, DT[name], h * 64
    qkv, dO = S.normal_torch(51, "qkv", (B * L, 3 * d), 1.0, dtype=dt), S.normal_torch(51, "dO", (B * L, d), 1.0, dtype=dt)
    o, dqkv = torch.empty(B * L, d, dtype=dt, device="cuda"), torch.full((B * L, 3 * d), 7.0, dtype=dt, device="cuda")
    lse = torch.empty(B * L, h, dtype=torch.float32, device="cuda")
    Bd.lsk_attn_fwd(1, qkv, B, L, h, dh, o, lse)
    Bd.lsk_attn_bwd(1, qkv, o, dO, lse, B, L, h, dh, dqkv)
    x = qkv.double().reshape(B, L, 3, h, dh).permute(2, 0, 3, 1, 4).contiguous().requires_grad_()
    s = (x[0] @ x[1].transpose(-1, -2).contiguous()) / dh ** 0.5
    s = s.masked_fill(torch.ones(L, L, device="cuda").triu(1).bool(), float("-inf"))
    (torch.softmax(s, -1) @ x[2]).permute(0, 2, 1, 3).reshape(B * L, d).backward(dO.double())
    g = x.grad.permute(1, 3, 0, 2, 4).reshape(B * L, 3, d).cpu().numpy()
    for i, nm in enumerate(("dq", "dk", "dv")):
        r = g[:, i]
        assert_close(host(dqkv).reshape(B * L, 3, d)[:, i], r, 2e-2 + out_rounding_bound(r, name), nm, atol=1e-5 if L == 1 else 0.0)


@pytest.mark.parametrize("name,dh,P,h,ctx", [
    ("f16", 64, 16, 2, [0, 7, 15, 16, 31, 32, 33, 100]),              # groups of two pages; four wavefronts
    ("bf16", 64, 8, 3, [255, 256, 257, 140]),                          # four pages a group; sixteen
    ("f16", 64, 24, 2, [95, 96, 97, 500, 1]),                          # three loads a page; sixteen
    ("f16", 64, 64, 40, [63, 64, 200, 280, 5, 256, 17, 90]),           # half a page a group; 320 pairs: eight
    ("f16", 128, 16, 1, [1537, 40, 383]), ("bf16", 128, 64, 2, [1999, 64, 65]),   # split contexts, eight wavefronts
    ("f16", 128, 8, 64, [130, 1, 127, 128, 129, 1100, 31, 12]),        # 512 pairs in four parts; four
    ("f16", 128, 16, 128, [7000, 4095, 4096, 50]),                     # 512 pairs in four parts; eight
    ("f16", 128, 16, 128, [6200, 17, 4000, 90, 1, 333]),               # 768 pairs in three parts; sixteen
    ("bf16", 128, 16, 128, [1100, 1, 16, 900, 64, 5, 1023, 300]),      # 1024 pairs, whole contexts; sixteen
    ("f16", 128, 16, 128, [8193, 4095, 4096, 50, 8191, 1, 900, 64]),   # 1024 pairs, the chunks that the scratch holds
    ("bf16", 128, 16, 256, [300, 1, 16, 170, 64, 5, 299, 33]),         # 2048 pairs, short contexts; four
    ("f16", 64, 16, 256, [6200, 1023, 1024, 1025, 40, 2047, 2048, 12])])   # 2048 pairs in chunks of 1024 tokens
def test_decode_attention_plans(name, dh, P, h, ctx):
    """Pages smaller and larger than a group of loads, contexts that end at each edge, every number of wavefronts, with and
    without splits; the slots beyond the contexts hold NaN.  Softmax weights in fp32 and 16-bit results: 1e-5 beside the
    rounding of the result."""
    dt, T, d = DT[name], len(ctx), h * dh
    table, n_pages = S.page_tables(np.array(ctx), np.ones(T, np.int64), P, seed=4)
    bt = torch.as_tensor(table, dtype=torch.int32, device="cuda")
    kp, vp = (S.normal_torch(44, n, (n_pages, h, P, dh), 1.0, dtype=dt) for n in "KV")
    qkv = S.normal_torch(44, "qkv", (T, 3 * d), 1.0, dtype=dt)
    ref = torch.empty(T, d, dtype=torch.float64, device="cuda")
    for b, n in enumerate(ctx):
        pages = bt[b, :n // P + 1].long()
        K, V = (x[pages].transpose(1, 2).reshape(-1, h, dh)[:n + 1].double() for x in (kp, vp))
        w = torch.softmax((K * qkv[b, :d].double().reshape(h, dh)).sum(-1) / dh ** 0.5, 0)
        ref[b] = (w[..., None] * V).sum(0).reshape(d)
    for b, n in enumerate(ctx):
        kp[bt[b, n // P].long(), :, n % P + 1:] = float("nan")
        vp[bt[b, n // P].long(), :, n % P + 1:] = float("nan")
    o = torch.empty(T, d, dtype=dt, device="cuda")
    pos = torch.as_tensor(ctx, dtype=torch.int32, device="cuda")
    Bd.lsk_attn_paged(1, qkv, h, dh, pos, torch.arange(T, dtype=torch.int32, device="cuda"), kp, vp, bt, P, max(ctx) + 1, o)
    ref = ref.cpu().numpy()
    assert_close(host(o), ref, 1e-5 + out_rounding_bound(ref, name), "o")


@pytest.mark.parametrize("rows,h,n,parts", [
    (2, 32, 512, 1), (9, 32, 512, 1), (9, 32, 2048, 8), (12, 32, 4096, 6), (15, 32, 16384, 5), (31, 33, 1024, 1), (31, 33, 1040, 3),
    (32, 32, 6144, 1), (32, 32, 16384, 2), (64, 32, 6144, 1), (64, 32, 8192, 8), (64, 32, 9000, 8)])
def test_decode_attention_parts_of_long_contexts(rows, h, n, parts):
    """How many parts contexts of n tokens are cut into, and that no more of the scratch is written than was asked for.  The
    requests share their pages."""
    dh, P = 128, 16
    pool = torch.zeros(64, h, P, dh, dtype=torch.float16, device="cuda")
    bt = (torch.arange(rows * -(-n // P), device="cuda") % 64).to(torch.int32).view(rows, -1)
    qkv, o = torch.zeros(rows, 3 * h * dh, dtype=torch.float16, device="cuda"), torch.empty(rows, h * dh, dtype=torch.float16, device="cuda")
    pos, req = torch.full((rows,), n - 1, dtype=torch.int32, device="cuda"), torch.arange(rows, dtype=torch.int32, device="cuda")
    size = Bd.lib().lsk_attn_paged_scratch_floats(rows, h, dh, n, P)
    scratch = torch.full((size + 4096,), float("nan"), device="cuda")
    Bd._check(Bd.lib().lsk_attn_paged(1, qkv.data_ptr(), Bd.LS_F16, rows, h, dh, pos.data_ptr(), req.data_ptr(), pool.data_ptr(),
                                      pool.data_ptr(), bt.data_ptr(), bt.shape[1], P, n, o.data_ptr(), scratch.data_ptr(), None))
    written = int(scratch.isfinite().sum())
    assert written == (rows * h * parts * (dh + 2) if parts > 1 else 0)
    assert scratch[size:].isnan().all() and (o == 0).all()


@pytest.mark.parametrize("dh,h,ctx", [(64, 1, 511), (64, 40, 300), (128, 1, 1100), (128, 64, 700)])
def test_decode_attention_where_scores_overflow(dh, h, ctx):
    """bf16 queries and keys whose product overflows to -inf, one run of tokens after the other, so that every wavefront and
    every split has groups of nothing else first, later and throughout: weight 0, as in float64, where they are -1e40.
    Bar: that of the plans above."""
    P, d, T = 16, h * dh, 5
    table, n_pages = S.page_tables(np.full(T, ctx), np.ones(T, np.int64), P, seed=6)
    bt = torch.as_tensor(table, dtype=torch.int32, device="cuda")
    kp, vp = (S.normal_torch(45, n, (n_pages, h, P, dh), 1.0, dtype=torch.bfloat16) for n in "KV")
    qkv = S.normal_torch(45, "qkv", (T, 3 * d), 1.0, dtype=torch.bfloat16)
    qkv[:, :d].view(T, h, dh)[:, :, 0] = 1e20
    kp[..., 0] = 0.0
    ref = torch.empty(T, d, dtype=torch.float64, device="cuda")
    # a run of 64 tokens, every second one, the first half, the second half, all but one token
    n_pg = ctx // P + 1
    runs = [range(10, 14), [p for p in range(n_pg) if p // 4 % 2 == 0], range(n_pg // 2), range(n_pg // 2, n_pg), range(n_pg - 1)]
    for b, run in enumerate(runs):
        pages = bt[b, :n_pg].long()
        kp[pages[torch.as_tensor(list(run), device="cuda")], ..., 0] = -1e20
        K, V = (x[pages].transpose(1, 2).reshape(-1, h, dh)[:ctx + 1].double() for x in (kp, vp))
        w = torch.softmax((K * qkv[b, :d].double().reshape(h, dh)).sum(-1) / dh ** 0.5, 0)
        ref[b] = (w[..., None] * V).sum(0).reshape(d)
    o = torch.empty(T, d, dtype=torch.bfloat16, device="cuda")
    Bd.lsk_attn_paged(1, qkv, h, dh, torch.full((T,), ctx, dtype=torch.int32, device="cuda"),
                      torch.arange(T, dtype=torch.int32, device="cuda"), kp, vp, bt, P, ctx + 1, o)
    ref = ref.cpu().numpy()
    assert_close(host(o), ref, 1e-5 + out_rounding_bound(ref, "bf16"), "o")


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("L", [1, 15, 16, 17, 64, 65, 130])
def test_fp32_attention_over_batches_of_keys(dh, L):
    """Sequences that end inside a batch of 16 keys, at its edge, and leave wavefronts without a key; forward and backward
    against float64.  Sums of up to 130 terms and an exponential of arguments of a few units in fp32: below 1e-5 of the RMS."""
    B, h = 2, 3
    d = h * dh
    qkv, dO = (torch.from_numpy(S.normal(9, n, (B * L, w)).astype(np.float32)).cuda() for n, w in (("qkv", 3 * d), ("dO", d)))
    o, dqkv = torch.empty(B * L, d, device="cuda"), torch.empty(B * L, 3 * d, device="cuda")
    lse = torch.empty(B * L, h, device="cuda")
    Bd.lsk_attn_fwd(0, qkv, B, L, h, dh, o, lse)
    Bd.lsk_attn_bwd(0, qkv, o, dO, lse, B, L, h, dh, dqkv)
    x = qkv.double().reshape(B, L, 3, h, dh).permute(2, 0, 3, 1, 4).contiguous().requires_grad_()
    s = (x[0] @ x[1].transpose(-1, -2).contiguous()) / dh ** 0.5
    s = s.masked_fill(torch.ones(L, L, device="cuda").triu(1).bool(), float("-inf"))
    ref = (torch.softmax(s, -1) @ x[2]).permute(0, 2, 1, 3).reshape(B * L, d)
    ref.backward(dO.double())
    assert_close(host(o), ref.detach().cpu().numpy(), 1e-5, "o")
    assert_close(host(lse), torch.logsumexp(s, -1).permute(0, 2, 1).reshape(B * L, h).detach().cpu().numpy(), 1e-5, "lse")
    g = x.grad.permute(1, 3, 0, 2, 4).reshape(B * L, 3, d).cpu().numpy()
    for i, nm in enumerate(("dq", "dk", "dv")):
        assert_close(host(dqkv).reshape(B * L, 3, d)[:, i], g[:, i], 1e-5, nm, atol=1e-5 if L == 1 else 0.0)


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("dead", [(16, 32), (0, 16), (48, 80), (17, 130)])
def test_fp32_attention_where_scores_overflow(dh, dead):
    """Finite queries and keys whose product overflows to -inf, over a wavefront's first batch of 16 keys, its later ones and
    all of it: weight 0 for these keys, as in float64, where they are -1e40.  Contiguous and paged keys; rows that see no
    other key are left out.  Bar: that of the attention over batches of keys."""
    L, h, P = 130, 2, 16
    d = h * dh
    qkv = torch.from_numpy(S.normal(15, "qkv", (L, 3 * d)).astype(np.float32)).cuda()
    x = qkv.view(L, 3, h, dh)
    x[:, 0, :, 0], x[:, 1, :, 0] = 1e20, 0.0
    x[dead[0]:dead[1], 1, :, 0] = -1e20
    Q, K, V = x.double().permute(1, 2, 0, 3).contiguous()
    s = (Q @ K.transpose(-1, -2).contiguous()) / dh ** 0.5
    s = s.masked_fill(torch.ones(L, L, device="cuda").triu(1).bool(), float("-inf"))
    ref = host((torch.softmax(s, -1) @ V).permute(1, 0, 2).reshape(L, d))
    rows = slice(dead[1] if dead[0] == 0 else 0, L)
    o, lse = torch.empty(L, d, device="cuda"), torch.empty(L, h, device="cuda")
    Bd.lsk_attn_fwd(0, qkv, 1, L, h, dh, o, lse)
    assert_close(host(o)[rows], ref[rows], 1e-5, "o")
    assert_close(host(lse)[rows], host(torch.logsumexp(s, -1).T.contiguous())[rows], 1e-5, "lse")
    table, n_pages = S.page_tables(np.array([L]), np.ones(1, np.int64), P, seed=2)
    bt = torch.as_tensor(table, dtype=torch.int32, device="cuda")
    kp, vp = (torch.zeros(n_pages, h, P, dh, device="cuda") for _ in range(2))
    for j in range(L):
        kp[table[0, j // P], :, j % P], vp[table[0, j // P], :, j % P] = x[j, 1], x[j, 2]
    o.zero_()
    Bd.lsk_attn_paged(0, qkv, h, dh, torch.arange(L, dtype=torch.int32, device="cuda"),
                      torch.zeros(L, dtype=torch.int32, device="cuda"), kp, vp, bt, P, L, o)
    assert_close(host(o)[rows], ref[rows], 1e-5, "o over pages")


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("at", [0, 15, 16, 77])
def test_fp32_attention_where_the_last_row_is_infinite(dh, at):
    """An infinite element in a row of V is infinite in every output that sees the row, and one in a row of dO in dV of every
    key that the row sees: no NaN, and nothing else changes.  Contiguous and paged keys.  Bar: that of the attention over
    batches of keys."""
    L, h, P = at + 1, 2, 16
    d, inf = h * dh, float("inf")
    n = L + 5   # rows behind the infinite one, forward
    qkv = torch.from_numpy(S.normal(16, "qkv", (n, 3 * d)).astype(np.float32)).cuda()
    x = qkv.view(n, 3, h, dh)
    o, lse, plain = torch.empty(n, d, device="cuda"), torch.empty(n, h, device="cuda"), torch.empty(n, d, device="cuda")
    Bd.lsk_attn_fwd(0, qkv, 1, n, h, dh, plain, lse)
    v = x[at, 2, 1, 3].item()
    x[at, 2, 1, 3] = inf

    def check(got, ref, rows, what):
        assert (got[rows, dh + 3] == inf).all(), what
        got[rows, dh + 3] = ref[rows, dh + 3]
        assert_close(host(got), host(ref), 1e-5, what)

    Bd.lsk_attn_fwd(0, qkv, 1, n, h, dh, o, lse)
    check(o, plain, slice(at, n), "o")
    table, n_pages = S.page_tables(np.array([n]), np.ones(1, np.int64), P, seed=2)
    bt = torch.as_tensor(table, dtype=torch.int32, device="cuda")
    kp, vp = (torch.zeros(n_pages, h, P, dh, device="cuda") for _ in range(2))
    for j in range(n):
        kp[table[0, j // P], :, j % P], vp[table[0, j // P], :, j % P] = x[j, 1], x[j, 2]
    o.zero_()
    Bd.lsk_attn_paged(0, qkv, h, dh, torch.arange(n, dtype=torch.int32, device="cuda"),
                      torch.zeros(n, dtype=torch.int32, device="cuda"), kp, vp, bt, P, n, o)
    check(o, plain, slice(at, n), "o over pages")
    x[at, 2, 1, 3] = v
    part = qkv[:L].contiguous()
    dO = torch.from_numpy(S.normal(16, "dO", (L, d)).astype(np.float32)).cuda()
    ref, got = torch.empty_like(part), torch.empty_like(part)
    Bd.lsk_attn_bwd(0, part, plain[:L].contiguous(), dO, lse[:L].contiguous(), 1, L, h, dh, ref)
    dO[at, dh + 3] = inf
    Bd.lsk_attn_bwd(0, part, plain[:L].contiguous(), dO, lse[:L].contiguous(), 1, L, h, dh, got)
    check(got[:, 2 * d:], ref[:, 2 * d:], slice(0, L), "dV")


@pytest.mark.parametrize("name", ["bf16", "f16"])
@pytest.mark.parametrize("kind", [Bd.LS_ACT_GELU_TANH, Bd.LS_ACT_GELU_ERF])
@pytest.mark.parametrize("n", [8, 1000, 1003])
def test_gelu_of_16_bit_operands(name, kind, n):
    """Eight units per thread and one (n not a multiple of eight, an unaligned start), the tails and zero included.
    fp32 inside, so every value is off by half an ulp of the storage type and 1e-5 of itself (the erf form cancels in
    its tail: 1e-6 absolute), subnormals aside."""
    u = q(np.concatenate([S.normal(9, "u", (n,)) * 3.0])[:n], name)
    u[:8] = q(np.array([0.0, -0.0, 12.0, -12.0, -6.0, -9.0, 300.0, -300.0]), name)
    dg = q(S.normal(9, "dg", (n,)), name)
    x = torch.from_numpy(u).requires_grad_(True)
    y = torch.nn.functional.gelu(x, approximate="tanh" if kind == Bd.LS_ACT_GELU_TANH else "none")
    y.backward(torch.from_numpy(dg))
    half_ulp = 2.0 ** (-9 if name == "bf16" else -12) * 2
    for skip in (0, 1):
        buf = lambda v: torch.cat([torch.zeros(skip, dtype=DT[name], device="cuda"), dev(v, DT[name])])[skip:]  # noqa: E731
        ud, gd, out, dout = buf(u), buf(dg), buf(u), buf(u)
        Bd.lsk_gelu_fwd(ud, out, kind)
        Bd.lsk_gelu_bwd(gd, ud, dout, kind)
        for got, ref in ((host(out), y.detach().numpy()), (host(dout), x.grad.numpy())):
            assert (np.abs(got - ref) <= (half_ulp + 1e-5) * np.abs(ref) + 2e-6).all()


@pytest.mark.parametrize("name", ["bf16", "f16"])
@pytest.mark.parametrize("M,N,T,parts", [(256, 256, 1024, 4), (256, 264, 1025, 3), (520, 392, 1001, 4), (264, 256, 2049, 7),
                                         (2304, 768, 4096, 2), (768, 768, 999, 1), (72, 64, 63, 1)])
def test_weight_gradient_in_parts(name, M, N, T, parts):
    """Parts of equal and unequal k tiles, a last k tile of 1, 41 and 64 tokens, ragged tiles, the shapes that stay whole;
    the sum of the parts scaled and added to what is there; no workspace, and one that does not hold two parts.  Exact
    operands, fp32 sums of T products of RMS 1: the 1e-5 of the test of whole products above."""
    dY, X = q(S.normal(7, "dY", (T, M)), name), q(S.normal(7, "X", (T, N)), name)
    dYd, Xd = dev(dY, DT[name]), dev(X, DT[name])
    ref = (torch.from_numpy(dY).cuda().t().contiguous() @ torch.from_numpy(X).cuda()).cpu().numpy() / 8
    alpha = torch.full((1,), 0.125, dtype=torch.float32, device="cuda")
    ws = torch.full((8 * M * N,), float("nan"), dtype=torch.float32, device="cuda")
    for scratch, want in ((ws, parts), (ws[:2 * M * N - 4], 1), (None, 1)):
        dW = torch.full((M, N), 7.0, dtype=torch.float32, device="cuda")
        for acc in (False, True):
            assert Bd.lsk_gemm_wgrad(dYd, Xd, dW, scratch, alpha=alpha, accumulate=acc) == want
            assert_close(host(dW), (1 + acc) * ref, 1e-5, f"{M}x{N}x{T} in {want} acc={acc}")


@pytest.mark.parametrize("name", ["bf16", "f16"])
@pytest.mark.parametrize("T,N,K,parts", [(1025, 256, 1728, 5), (65, 72, 1024, 4), (129, 256, 4096, 8), (333, 768, 3072, 6),
                                         (999, 768, 768, 1), (63, 64, 512, 1)])
def test_input_gradient_in_parts(name, T, N, K, parts):
    """The same for the input gradient, whose result is stored in the operand type: its rounding and 1e-5 of the RMS."""
    dY, W = q(S.normal(8, "dY", (T, K)), name), q(S.normal(8, "W", (K, N), 0.05), name)
    dYd, Wd = dev(dY, DT[name]), dev(W, DT[name])
    ref = (torch.from_numpy(dY).cuda() @ torch.from_numpy(W).cuda()).cpu().numpy()
    ws = torch.full((8 * T * N,), float("nan"), dtype=torch.float32, device="cuda")
    for scratch, want in ((ws, parts), (ws[:2 * T * N - 4], 1), (None, 1)):
        dX = torch.full((T, N), 7.0, dtype=DT[name], device="cuda")
        assert Bd.lsk_gemm_dgrad(dYd, Wd, dX, scratch) == want
        assert_close(host(dX), ref, 1e-5 + out_rounding_bound(ref, name), f"{T}x{N}x{K} in {want}")


@pytest.mark.parametrize("name", ["bf16", "f16"])
@pytest.mark.parametrize("T,K,N,parts", [
    (999, 768, 3072, (1, 1)), (999, 3072, 768, (1, 2)), (333, 768, 768, (1, 1)), (65, 128, 72, (1, 1)), (64, 64, 64, (1, 1)),
    (1025, 256, 264, (4, 1)), (2049, 1728, 256, (4, 3)), (2049, 320, 200, (7, 1)), (129, 4096, 256, (1, 4)),
    (1000, 128, 1024, (4, 1)), (63, 768, 768, None), (300, 4096, 4096, None)])
def test_gradients_of_a_linear_map_in_one_launch(name, T, K, N, parts):
    """Either product first and in parts, a last k tile of 1, 39 and 64 tokens, ragged tiles, with and without a bias, added to
    what is there and scaled; a workspace that holds no parts.  Exact operands: 1e-5 of the RMS for fp32 sums of T or K
    products, the rounding of the input gradient beside it; sums of T values for the bias: 2e-6."""
    dt = DT[name]
    dO, x, w = (S.normal_torch(12, n, shape, std, dtype=dt) for n, shape, std in
                (("dO", (T, K), 1.0), ("x", (T, N), 1.0), ("w", (K, N), 0.05)))
    rx = (dO.double() @ w.double()).cpu().numpy()
    rw, rb = (dO.double().T.contiguous() @ x.double() / 8).cpu().numpy(), (dO.double().sum(0) / 8).cpu().numpy()
    alpha = torch.full((1,), 0.125, dtype=torch.float32, device="cuda")
    ws = torch.full((8 * (K * N + K) + 4 * T * N,), float("nan"), dtype=torch.float32, device="cuda")
    for scratch, want in ((ws, parts), (ws[:4], (1, 1))):
        for bias in (True, False):
            dx, dw = torch.full((T, N), 7.0, dtype=dt, device="cuda"), torch.full((K, N), 7.0, device="cuda")
            db = torch.full((K + 1,), 7.0, device="cuda")[1:] if bias else None   # not 16-byte aligned
            for acc in (False, True):
                got = Bd.lsk_gemm_grads(dO, w, x, dx, dw, db, scratch, alpha=alpha, accumulate=acc)
                if got is None:   # not covered, or better apart if each has to stay whole: nothing has been written
                    assert parts is None or want != parts
                    assert (dx == 7.0).all() and (dw == 7.0).all()
                    break
                assert got == want
                assert_close(host(dw), (1 + acc) * rw, 1e-5, "dW")
                assert_close(host(dx), rx, 1e-5 + out_rounding_bound(rx, name), "dIn")
                if bias:
                    assert_close(host(db), (1 + acc) * rb, 2e-6, "db")


@pytest.mark.parametrize("mma", ["f16", "bf16"])
@pytest.mark.parametrize("which", ["gpt", "llama"])
@pytest.mark.parametrize("B,L", [(5, 205), (3, 333), (1, 1024), (2, 255)])
def test_training_with_gradients_split_along_the_contraction(which, B, L, mma):
    """A block whose weight gradients are summed from three or four parts each and whose FFN-up input gradient from four
    or five, over token counts with a last k tile of 1, 39 and 64 rows, and one (510) whose weight gradients stay whole;
    gradients overwritten and accumulated.  Bars of the stage tests."""
    cfg = (S.scaled(S.CONFIGS["gpt2s_bf16"], n_layers=1, d_model=256, n_heads=4, d_ff=1536) if which == "gpt" else
           S.scaled(S.CONFIGS["llama7b_bf16"], n_layers=1, d_model=256, n_heads=2, d_ff=864))
    check_train(cfg, B, L, mma, dy_std=1.0 if which == "gpt" else 1e-2, io="f32",
                tol=TOL["bf16"] if mma == "f16" else "storage model")
    st, _, _ = make_stage(cfg, mma=mma, io="f32")
    X, dY = (S.make_activations(cfg, n, (B, L, cfg["d_model"])) for n in ("X", "dY"))
    _, _, once = run_train(st, cfg, X, dY, B, L)
    _, _, twice = run_train(st, cfg, X, dY, B, L, accumulate_twice=True)
    assert_close(twice, 2 * once, 1e-6, "accumulated gradients")
    st.close()


def test_norm_gradients_finished_together_or_one_by_one():
    """52 norms' pairs of column sums over 16384 rows are more than the 64 MB that are kept for one launch, so every norm is
    finished by itself; two micro-batches of half the rows are finished together, the second one accumulating.  The
    same gradients either way, within the fp32 stage's bar (sums of 16384 terms in another order)."""
    cfg = S.scaled(S.CONFIGS["tiny_gpt_f32"], n_layers=52, d_model=64, n_heads=2, d_ff=64)
    B, L, d = 32, 512, 64
    st = Bd.Stage(cfg, io_dtype="f32", mma_dtype="f32")
    st.ls_bind_params(S.make_params_torch(cfg, 3))
    X, dY = (S.normal_torch(3, n, (B, L, d), 1.0, dtype=torch.float32) for n in ("X", "dY"))

    def gradients(pieces):
        b = B // pieces
        grads = torch.full((st.ls_param_count(),), 7.0, dtype=torch.float32, device="cuda")
        saved, ws = st.new_saved(b, L), st.new_workspace(b * L)
        dX = torch.empty_like(X)
        for i in range(pieces):
            x, dy, dx = (t[i * b:(i + 1) * b] for t in (X, dY, dX))
            st.stage_train_fwd(x, b, L, torch.empty_like(x), saved, ws)
            st.stage_train_bwd(dy, b, L, saved, dx, grads, int(i > 0), ws)
        return host(grads), host(dX)

    (one, dx1), (two, dx2) = gradients(1), gradients(2)
    assert_close(two, one, 1e-4, "dParams")
    assert_close(dx2, dx1, 1e-4, "dX")
    st.close()


@pytest.mark.parametrize("T,K,N,calls", [(999, 768, 768, 1), (300, 4096, 4096, 0)])
def test_refused_gradient_launches_are_not_recorded(T, K, N, calls):
    """A shape that is left to separate launches adds nothing to the recording."""
    dO, x, w = (torch.zeros(s, dtype=torch.float16, device="cuda") for s in ((T, K), (T, N), (K, N)))
    dx, dw = torch.empty_like(x), torch.empty(K, N, device="cuda")
    scratch = torch.empty(2 * (K * N + K) + T * N, dtype=torch.float32, device="cuda")
    Bd.lsk_timing_begin()
    got = Bd.lsk_gemm_grads(dO, w, x, dx, dw, None, scratch)
    assert (got is not None) == (calls == 1)
    assert Bd.lsk_timing_end()["gemm"][1] == calls
