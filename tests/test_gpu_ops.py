"""Kernel-level parity: each HIP kernel against the oracle's matching operation, element by
element, on shapes that span several tiles and end in ragged tails."""
import numpy as np
import pytest
import torch

import paper_2209_02478_amd as mi
from oracle import model as om
from gpu_util import DEV, dev, host, quant, rel_l2, sync

pytestmark = pytest.mark.gpu

# elementwise bound of one rounding to the storage type (bf16: 8 significand bits)
EPS = {0: 1e-5, 1: 2.0 ** -8}


def close(got, ref, dtype, scale=None, k=1.0):
    ref = np.asarray(ref, dtype=np.float64)
    got = np.asarray(got, dtype=np.float64)
    scale = np.abs(ref).max() if scale is None else scale
    err = np.abs(got - ref)
    bound = k * EPS[dtype] * (np.abs(ref) + 0.1 * scale) + 1e-30
    assert np.all(err <= bound), f"max err {err.max():.3e} vs bound {bound.flat[err.argmax()]:.3e} at {np.unravel_index(err.argmax(), err.shape)}"


# ---------------------------------------------------------------- GEMM
GEMM_SHAPES = [(130, 70, 40), (257, 129, 96), (64, 64, 64), (1, 8, 8), (300, 200, 136), (128, 256, 520),
               (100, 72, 50), (257, 130, 77)]     # reduction lengths off the 8-element grid: general kernel


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("a_k,b_k", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_layouts(dtype, a_k, b_k, M, N, K):
    rng = np.random.default_rng(M * 7 + N * 3 + K + a_k * 2 + b_k)
    pad = 8
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((N, K)).astype(np.float32)
    ref = quant(A, dtype) @ quant(B, dtype).T
    # device layouts with a padded leading dimension
    def lay(X, kmajor):
        R, Kk = X.shape
        up = lambda v: (v + 7) // 8 * 8 + pad                  # bf16 needs leading dimensions in multiples of 8
        if kmajor:
            buf = np.zeros((R, up(Kk)), np.float32); buf[:, :Kk] = X
            return buf, up(Kk)
        buf = np.zeros((Kk, up(R)), np.float32); buf[:, :R] = X.T
        return buf, up(R)
    Ab, lda = lay(A, a_k)
    Bb, ldb = lay(B, b_k)
    dA, dB = dev(Ab, dtype), dev(Bb, dtype)
    ldc = N + 8
    C = torch.full((M, ldc), 7.0, dtype=dA.dtype, device=DEV)
    mi.mimose_op_gemm(dtype, dA, lda, a_k, dB, ldb, b_k, C, ldc, 0, M, N, K)
    sync()
    got = host(C)
    assert np.all(got[:, N:] == 7.0), "wrote outside the N columns"
    close(got[:, :N], ref, dtype, k=2.0)


@pytest.mark.parametrize("dtype", [0, 1])
def test_gemm_epilogues(dtype):
    rng = np.random.default_rng(5)
    M, N, K = 200, 136, 72
    A = rng.standard_normal((M, K)).astype(np.float32) * 0.5
    B = rng.standard_normal((N, K)).astype(np.float32) * 0.5
    bias = rng.standard_normal(N).astype(np.float32)
    resid = rng.standard_normal((M, N)).astype(np.float32)
    base = quant(A, dtype) @ quant(B, dtype).T
    dA, dB, dbias, dres = dev(A, dtype), dev(B, dtype), dev(bias, dtype), dev(resid, dtype)
    # bias + residual
    C = torch.zeros((M, N), dtype=dA.dtype, device=DEV)
    mi.mimose_op_gemm(dtype, dA, K, 1, dB, K, 1, C, N, 0, M, N, K, bias=dbias, resid=dres, ldr=N)
    sync()
    close(host(C), base + quant(bias, dtype) + quant(resid, dtype), dtype, k=2.0)
    # bias + GELU (both forms): C gets the pre-activation, gelu_out the activation
    for form in (1, 2):
        C = torch.zeros((M, N), dtype=dA.dtype, device=DEV)
        Gt = torch.zeros((M, N), dtype=dA.dtype, device=DEV)
        mi.mimose_op_gemm(dtype, dA, K, 1, dB, K, 1, C, N, 0, M, N, K, bias=dbias, gelu_out=Gt, gelu=form)
        sync()
        pre = base + quant(bias, dtype)
        close(host(C), pre, dtype, k=2.0)
        close(host(Gt), om.gelu_fwd(pre, form == 2), dtype, scale=np.abs(pre).max(), k=3.0)
    # weight-gradient form: fp32 output and row sums of the A operand
    T = 333
    dY = rng.standard_normal((T, M)).astype(np.float32)
    X = rng.standard_normal((T, N)).astype(np.float32)
    ddY, dX = dev(dY, dtype), dev(X, dtype)
    W = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    rs = torch.zeros(M, dtype=torch.float32, device=DEV)
    mi.mimose_op_gemm(dtype, ddY, M, 0, dX, N, 0, W, N, 1, M, N, T, a_rowsum=rs)
    sync()
    close(host(W), quant(dY, dtype).T @ quant(X, dtype), 0, k=20.0)
    close(host(rs), quant(dY, dtype).sum(0), 0, k=20.0)
    # the same product with the reduction cut in parts (long reduction, few output tiles)
    T = 2000
    dY = rng.standard_normal((T, M)).astype(np.float32)
    X = rng.standard_normal((T, N)).astype(np.float32)
    ddY, dX = dev(dY, dtype), dev(X, dtype)
    nws = mi.mimose_op_gemm_workspace_bytes(M, N)
    assert nws > 0                                             # ignored by the fp32 kernel
    ws = torch.zeros(max(nws, 16), dtype=torch.uint8, device=DEV)
    W.fill_(9.0); rs.fill_(9.0)
    mi.mimose_op_gemm(dtype, ddY, M, 0, dX, N, 0, W, N, 1, M, N, T, a_rowsum=rs, workspace=ws, workspace_bytes=nws)
    sync()
    close(host(W), quant(dY, dtype).T @ quant(X, dtype), 0, k=40.0)
    close(host(rs), quant(dY, dtype).sum(0), 0, k=40.0)


@pytest.mark.parametrize("a_k,b_k", [(1, 1), (1, 0), (0, 0), (0, 1)])
def test_gemm_many_tiles(a_k, b_k):
    """More output tiles than the chip has block slots (several rounds of the tile -> block map),
    ragged in every dimension, with bias, residual and A row sums."""
    dtype, M, N, K = 1, 5001, 4100, 104
    rng = np.random.default_rng(77 + 2 * a_k + b_k)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((N, K)).astype(np.float32)
    bias = rng.standard_normal(N).astype(np.float32)
    resid = rng.standard_normal((M, N)).astype(np.float32)
    up = lambda v: (v + 7) // 8 * 8
    def lay(X, kmajor):
        R, Kk = X.shape
        if kmajor:
            buf = np.zeros((R, up(Kk)), np.float32); buf[:, :Kk] = X
            return buf, up(Kk)
        buf = np.zeros((Kk, up(R)), np.float32); buf[:, :R] = X.T
        return buf, up(R)
    Ab, lda = lay(A, a_k)
    Bb, ldb = lay(B, b_k)
    dA, dB, dbias, dres = dev(Ab, dtype), dev(Bb, dtype), dev(bias, dtype), dev(resid, dtype)
    ldc = up(N) + 8
    C = torch.full((M, ldc), 7.0, dtype=dA.dtype, device=DEV)
    rs = torch.full((M,), 9.0, dtype=torch.float32, device=DEV)
    mi.mimose_op_gemm(dtype, dA, lda, a_k, dB, ldb, b_k, C, ldc, 0, M, N, K, bias=dbias, resid=dres, ldr=N,
                      a_rowsum=rs)
    sync()
    got = host(C)
    assert np.all(got[:, N:] == 7.0), "wrote outside the N columns"
    ref = quant(A, dtype).astype(np.float64) @ quant(B, dtype).astype(np.float64).T
    close(got[:, :N], ref + quant(bias, dtype) + quant(resid, dtype), dtype, k=2.0)
    close(host(rs), quant(A, dtype).astype(np.float64).sum(1), 0, k=20.0)
    # plain fp32 output
    Cf = torch.full((M, N), 7.0, dtype=torch.float32, device=DEV)
    mi.mimose_op_gemm(dtype, dA, lda, a_k, dB, ldb, b_k, Cf, N, 1, M, N, K)
    sync()
    close(host(Cf), ref, 0, k=20.0)


@pytest.mark.parametrize("a_k,b_k", [(1, 1), (1, 0), (0, 0), (0, 1)])
def test_gemm_large_tiles(a_k, b_k):
    """Shapes the dispatch gives to the kernel with 256 x 256 tiles (14 x 15 = 210 of 256 units in its
    one round; reduction 520 = 8 tiles of 64 and a tail of 8): ragged edges in both dimensions,
    bias + residual + GELU, row sums, fp32 output, and the same bits on a second run."""
    dtype, M, N, K = 1, 3500, 3800, 520
    rng = np.random.default_rng(170 + 2 * a_k + b_k)
    A = rng.standard_normal((M, K)).astype(np.float32) * 0.5
    B = rng.standard_normal((N, K)).astype(np.float32) * 0.5
    bias = rng.standard_normal(N).astype(np.float32)
    resid = rng.standard_normal((M, N)).astype(np.float32)
    up = lambda v: (v + 7) // 8 * 8
    def lay(X, kmajor):
        R, Kk = X.shape
        if kmajor:
            buf = np.zeros((R, up(Kk) + 8), np.float32); buf[:, :Kk] = X
            return buf, up(Kk) + 8
        buf = np.zeros((Kk, up(R)), np.float32); buf[:, :R] = X.T
        return buf, up(R)
    Ab, lda = lay(A, a_k)
    Bb, ldb = lay(B, b_k)
    dA, dB, dbias, dres = dev(Ab, dtype), dev(Bb, dtype), dev(bias, dtype), dev(resid, dtype)
    ref = quant(A, dtype) @ quant(B, dtype).T
    ldc = up(N) + 8
    C = torch.full((M, ldc), 7.0, dtype=dA.dtype, device=DEV)
    Gt = torch.full((M, ldc), 7.0, dtype=dA.dtype, device=DEV)
    mi.mimose_op_gemm(dtype, dA, lda, a_k, dB, ldb, b_k, C, ldc, 0, M, N, K, bias=dbias, gelu_out=Gt, gelu=1)
    sync()
    pre = ref + quant(bias, dtype)
    assert np.all(host(C)[:, N:] == 7.0) and np.all(host(Gt)[:, N:] == 7.0), "wrote outside the N columns"
    close(host(C)[:, :N], pre, dtype, k=2.0)
    close(host(Gt)[:, :N], om.gelu_fwd(pre, False), dtype, scale=np.abs(pre).max(), k=3.0)
    # fp32 output with residual; row sums when A is stored m-major (the weight-gradient form)
    Cf = torch.full((M, N), 7.0, dtype=torch.float32, device=DEV)
    rs = torch.full((M,), 9.0, dtype=torch.float32, device=DEV)
    mi.mimose_op_gemm(dtype, dA, lda, a_k, dB, ldb, b_k, Cf, N, 1, M, N, K, resid=dres, ldr=N, a_rowsum=rs)
    sync()
    first = host(Cf)
    close(first, ref + quant(resid, dtype), 0, k=20.0)
    close(host(rs), quant(A, dtype).astype(np.float64).sum(1), 0, k=20.0)
    Cf.fill_(3.0)
    mi.mimose_op_gemm(dtype, dA, lda, a_k, dB, ldb, b_k, Cf, N, 1, M, N, K, resid=dres, ldr=N, a_rowsum=rs)
    sync()
    assert np.array_equal(host(Cf), first)


@pytest.mark.parametrize("M,N,K", [(5000, 4872, 776),    # 400 tiles of 256 x 256 in two rounds, ragged in each dimension
                                   (4700, 4300, 520),    # 629 tiles of 128 x 256 in three rounds
                                   (25600, 768, 640),    # 600 of them, whole in each dimension
                                   (9000, 9736, 520),    # 1404 tiles of 256 x 256 in six rounds
                                   (9216, 9472, 576),    # 1332, whole in each dimension
                                   (17000, 256, 1032),   # row sums: one column tile, which is too few (266 units: past the ring's round)
                                   (11000, 300, 1096),   # two, the fewest (258 units)
                                   (3000, 300, 1096),    # 72 units: the ring
                                   (20000, 768, 584)])   # three, of the four that 256 rows take
@pytest.mark.parametrize("a_k,b_k", [(1, 1), (1, 0), (0, 0), (0, 1)])
def test_gemm_large_tiles_bits(M, N, K, a_k, b_k):
    """Blocks that take several tiles, in every form of the store: the bits are those of the same rows
    multiplied alone, which other kernels do (the sum of an element is one chain over k in all of them)."""
    g = torch.Generator(device=DEV).manual_seed(M + K + 2 * a_k + b_k)
    up = lambda v: (v + 7) // 8 * 8
    mk = lambda r, c: (torch.randn((r, c), generator=g, device=DEV) * 0.5).to(torch.bfloat16)
    A, B = mk(M, K) if a_k else mk(K, up(M)), mk(N, K) if b_k else mk(K, up(N))
    bias, resid = mk(1, N)[0], mk(M, up(N))
    rows = 256 if M > 4096 else 128                             # alone: 64 x 32 or 64 x 64 tiles
    forms = [dict(c_f32=1), dict(c_f32=1, bias=1, resid=1), dict(c_f32=0, bias=1), dict(c_f32=0, resid=1),
             dict(c_f32=0, bias=1, gelu=1), dict(c_f32=0, bias=1, gelu=2),
             dict(c_f32=0, bias=1, resid=1, gelu=1), dict(c_f32=0, resid=1, gelu=2)]
    if not a_k:
        forms = forms[:4] + [dict(c_f32=0, bias=1, rowsum=1), dict(c_f32=1, rowsum=1)] if b_k else [dict(c_f32=1, rowsum=1), dict(c_f32=1), dict(c_f32=0)]
    for form in forms:
        def product(r0, n_rows):
            kw = {}
            C = torch.full((n_rows, up(N)), 7.0, dtype=torch.float32 if form["c_f32"] else torch.bfloat16, device=DEV)
            G = torch.full_like(C, 7.0) if form.get("gelu") else None
            rs = torch.zeros(n_rows, device=DEV) if form.get("rowsum") else None
            if form.get("bias"): kw["bias"] = bias
            if form.get("resid"): kw.update(resid=resid[r0:], ldr=up(N))
            if G is not None: kw.update(gelu_out=G, gelu=form["gelu"])
            if rs is not None: kw["a_rowsum"] = rs
            mi.mimose_op_gemm(1, A[r0:] if a_k else A[:, r0:], K if a_k else up(M), a_k, B, K if b_k else up(N), b_k, C, up(N),
                              form["c_f32"], n_rows, N, K, **kw)
            sync()
            if rs is not None and b_k:                          # (the kernel with a few rows of this layout sums in another order)
                exact, bound = A[:, r0:r0 + n_rows].double().sum(0), K * 2.0**-24 * A[:, r0:r0 + n_rows].double().abs().sum(0)
                assert bool(((rs.double() - exact).abs() <= bound).all()), (form, r0)
                rs = None
            return [x for x in (C, G, rs) if x is not None]
        whole = product(0, M)
        assert bool((whole[0][:, N:] == 7.0).all()), "wrote outside the N columns"
        for r0 in (0, M // 2 // 8 * 8, (M - rows) // 8 * 8):
            for full, alone in zip(whole, product(r0, rows)):
                assert torch.equal(full[r0:r0 + rows], alone), (form, r0)


@pytest.mark.parametrize("M,N,K", [(3500, 3801, 520), (2304, 2306, 512)])   # 256 x 256 and 128 x 256 tiles
@pytest.mark.parametrize("a_k,b_k", [(1, 1), (1, 0), (0, 0), (0, 1)])
def test_gemm_large_tiles_off_16_bytes(M, N, K, a_k, b_k):
    """C, bias and residual wherever an element may lie: the bits are those of the aligned product."""
    g = torch.Generator(device=DEV).manual_seed(N + 2 * a_k + b_k)
    up = lambda v: (v + 7) // 8 * 8
    mk = lambda r, c: (torch.randn((r, c), generator=g, device=DEV) * 0.5).to(torch.bfloat16)
    A, B = mk(M, K) if a_k else mk(K, up(M)), mk(N, K) if b_k else mk(K, up(N))
    bias, resid = mk(1, up(N))[0], mk(M, up(N))
    def place(x, pitch):                                        # rows `pitch` apart, from the second element on
        out = torch.full((M * pitch + 8,), 7.0, dtype=x.dtype, device=DEV)[1:M * pitch + 1].view(M, pitch)
        out[:, :N] = x[:, :N]
        return out
    for dt, epilogue in ((torch.bfloat16, True), (torch.float32, True), (torch.bfloat16, False), (torch.float32, False)):
        if epilogue and not (a_k or b_k):
            continue
        def product(C, r, b):
            mi.mimose_op_gemm(1, A, K if a_k else up(M), a_k, B, K if b_k else up(N), b_k, C, C.stride(0), int(dt == torch.float32),
                              M, N, K, **(dict(bias=b, resid=r, ldr=r.stride(0)) if epilogue else {}))
            sync()
            return C
        blank = torch.full((M, up(N)), 7.0, dtype=dt, device=DEV)
        off = product(place(blank, N + 4), place(resid, N + 2), torch.cat([bias[:1], bias])[1:])
        assert torch.equal(off[:, :N], product(blank, resid, bias)[:, :N]), (dt, epilogue)
        assert bool((off[:, N:] == 7.0).all()), "wrote outside the N columns"


@pytest.mark.parametrize("M,N,K", [(3500, 3801, 520), (2304, 2306, 512)])   # 256 x 256 and 128 x 256 tiles
@pytest.mark.parametrize("form,resid", [(1, 0), (2, 0), (1, 1), (2, 1)])
def test_gemm_gelu_off_16_bytes(M, N, K, form, resid):
    """The C library's functions in every column: the bits are those of the same rows multiplied alone, which
    another kernel does."""
    g = torch.Generator(device=DEV).manual_seed(N + form)
    A, B, bias, r = ((torch.randn(s, generator=g, device=DEV) * k).to(torch.bfloat16)
                     for s, k in (((M, K), 0.5), ((N, K), 0.5), ((N,), 1.0), ((M, N), 4.0)))
    def product(r0, rows):
        C, G = (torch.full((rows * N + 1,), 7.0, dtype=torch.bfloat16, device=DEV)[1:].view(rows, N) for _ in range(2))
        kw = dict(resid=r[r0:], ldr=N) if resid else {}
        mi.mimose_op_gemm(1, A[r0:], K, 1, B, K, 1, C, N, 0, rows, N, K, bias=bias, gelu_out=G, gelu=form, **kw)
        sync()
        return C, G
    whole = product(0, M)
    for r0 in (0, 1000, M - 128):
        for full, alone in zip(whole, product(r0, 128)):
            assert torch.equal(full[r0:r0 + 128], alone), r0


@pytest.mark.parametrize("M,N,K", [(3500, 3800, 520), (2304, 2304, 512)])   # 256 x 256 and 128 x 256 tiles
@pytest.mark.parametrize("form", [1, 2])
def test_gemm_gelu_of_a_sum_with_residual(M, N, K, form):
    rng = np.random.default_rng(M + form)
    A, B = (rng.standard_normal(s).astype(np.float32) * 0.5 for s in ((M, K), (N, K)))
    bias, resid = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32) * 4
    C, G = (torch.zeros((M, N), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    mi.mimose_op_gemm(1, dev(A, 1), K, 1, dev(B, 1), K, 1, C, N, 0, M, N, K, bias=dev(bias, 1), resid=dev(resid, 1), ldr=N,
                      gelu_out=G, gelu=form)
    sync()
    pre = quant(A, 1) @ quant(B, 1).T + quant(bias, 1) + quant(resid, 1)
    close(host(C), pre, 1, k=2.0)
    close(host(G), om.gelu_fwd(pre, form == 2), 1, scale=np.abs(pre).max(), k=3.0)


def test_gemm_large_tiles_split_reduction():
    """Weight-gradient shape of the fused QKV projection with a ragged reduction length cut in
    parts, row sums included, and the same bits on a second run."""
    dtype, M, N, T = 1, 2304, 768, 2100
    rng = np.random.default_rng(171)
    dY = rng.standard_normal((T, M)).astype(np.float32)
    X = rng.standard_normal((T, N)).astype(np.float32)
    ddY, dX = dev(dY, dtype), dev(X, dtype)
    nws = mi.mimose_op_gemm_workspace_bytes(M, N)
    assert nws >= 2 * (M * N + M) * 4
    ws = torch.zeros(nws, dtype=torch.uint8, device=DEV)
    W = torch.full((M, N), 9.0, dtype=torch.float32, device=DEV)
    rs = torch.full((M,), 9.0, dtype=torch.float32, device=DEV)
    mi.mimose_op_gemm(dtype, ddY, M, 0, dX, N, 0, W, N, 1, M, N, T, a_rowsum=rs, workspace=ws, workspace_bytes=nws)
    sync()
    first = host(W)
    close(first, quant(dY, dtype).T @ quant(X, dtype), 0, k=40.0)
    close(host(rs), quant(dY, dtype).sum(0), 0, k=40.0)
    W.fill_(1.0)
    mi.mimose_op_gemm(dtype, ddY, M, 0, dX, N, 0, W, N, 1, M, N, T, a_rowsum=rs, workspace=ws, workspace_bytes=nws)
    sync()
    assert np.array_equal(host(W), first)


@pytest.mark.parametrize("a_k,M,K", [(0, 1000, 2000), (0, 520, 2089), (1, 600, 8320)])
@pytest.mark.parametrize("N", [1001, 1002, 1003])
def test_gemm_parts_of_odd_columns(a_k, M, K, N):
    """Parts whose rows do not lie on 16 bytes: the same bits as with the columns filled up."""
    g = torch.Generator(device=DEV).manual_seed(N + M)
    A = torch.randn((M, K) if a_k else (K, M), generator=g, device=DEV).to(torch.bfloat16)
    B = torch.randn((K, 1008), generator=g, device=DEV).to(torch.bfloat16)
    nws = mi.mimose_op_gemm_long_k_workspace_bytes(1008) if a_k else mi.mimose_op_gemm_workspace_bytes(M, 1008)
    assert nws >= 2 * (M * 1008 + M) * 4
    def product(n):
        C, rs = torch.full((M, 1008), 7.0, device=DEV), torch.full((M,), 7.0, device=DEV)
        ws = torch.zeros(nws, dtype=torch.uint8, device=DEV)
        mi.mimose_op_gemm(1, A, K if a_k else M, a_k, B, 1008, 0, C, 1008, 1, M, n, K, a_rowsum=None if a_k else rs,
                          workspace=ws, workspace_bytes=nws)
        sync()
        return C, rs
    (C, rs), (whole, rs_whole) = product(N), product(1008)
    assert torch.equal(C[:, :N], whole[:, :N]) and torch.equal(rs, rs_whole)
    assert bool((C[:, N:] == 7.0).all()), "wrote outside the N columns"


@pytest.mark.parametrize("c_f32", [0, 1])
def test_gemm_long_reduction_in_parts(c_f32):
    """Data-gradient layout with a very long reduction and few output tiles (the shape class of the
    head's data gradient): with the scratch it runs on the large tiles in parts; bf16 and fp32
    output, ragged rows, the same bits twice, and the same values as without the scratch."""
    dtype, M, N, K = 1, 600, 768, 8320
    rng = np.random.default_rng(181 + c_f32)
    A = (rng.standard_normal((M, K)) * 0.1).astype(np.float32)
    B = rng.standard_normal((N, K)).astype(np.float32)
    dA = dev(A, dtype)
    dB = dev(np.ascontiguousarray(B.T), dtype)                      # m-major: [K][N]
    ref = quant(A, dtype) @ quant(B, dtype).T
    nws = mi.mimose_op_gemm_long_k_workspace_bytes(N)
    assert nws >= 8 * M * N * 4
    ws = torch.zeros(nws, dtype=torch.uint8, device=DEV)
    odt = torch.float32 if c_f32 else dA.dtype
    C = torch.full((M, N), 7.0, dtype=odt, device=DEV)
    mi.mimose_op_gemm(dtype, dA, K, 1, dB, N, 0, C, N, c_f32, M, N, K, workspace=ws, workspace_bytes=nws)
    sync()
    first = host(C)
    close(first, ref, 0 if c_f32 else dtype, k=40.0 if c_f32 else 2.0)
    C.fill_(3.0)
    mi.mimose_op_gemm(dtype, dA, K, 1, dB, N, 0, C, N, c_f32, M, N, K, workspace=ws, workspace_bytes=nws)
    sync()
    assert np.array_equal(host(C), first)
    C.fill_(3.0)
    mi.mimose_op_gemm(dtype, dA, K, 1, dB, N, 0, C, N, c_f32, M, N, K)      # no scratch: one part
    sync()
    close(host(C), ref, 0 if c_f32 else dtype, k=40.0 if c_f32 else 2.0)


# products that one round of small tiles covers: each tile size of the ring kernel, whole and ragged
# rows, columns and reduction lengths (one, an odd and an even count of 64-deep stages)
@pytest.mark.parametrize("a_k,b_k", [(1, 1), (1, 0), (0, 0)])
@pytest.mark.parametrize("M,N,K", [(70, 96, 64), (33, 8, 200), (130, 4104, 136), (640, 776, 192), (1700, 768, 72),
                                   (1536, 1600, 320), (2500, 776, 264), (300, 600, 1096)])
def test_gemm_ring_tiles(a_k, b_k, M, N, K):
    dtype = 1
    rng = np.random.default_rng(M + N + K)
    up = lambda v: (v + 7) // 8 * 8
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((N, K)).astype(np.float32)
    bias, resid = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    def lay(X, kmajor):
        if kmajor:
            return np.ascontiguousarray(X), X.shape[1]
        buf = np.zeros((X.shape[1], up(X.shape[0])), np.float32)
        buf[:, :X.shape[0]] = X.T
        return buf, up(X.shape[0])
    (Ab, lda), (Bb, ldb) = lay(A, a_k), lay(B, b_k)
    dA, dB, dbias, dres = dev(Ab, dtype), dev(Bb, dtype), dev(bias, dtype), dev(resid, dtype)
    base = quant(A, dtype) @ quant(B, dtype).T
    C = torch.full((M, N + 8), 7.0, dtype=dA.dtype, device=DEV)
    mi.mimose_op_gemm(dtype, dA, lda, a_k, dB, ldb, b_k, C, N + 8, 0, M, N, K, bias=dbias, resid=dres, ldr=N)
    sync()
    assert np.all(host(C)[:, N:] == 7.0), "wrote outside the N columns"
    close(host(C)[:, :N], base + quant(bias, dtype) + quant(resid, dtype), dtype, k=2.0)
    G = torch.zeros((M, N + 8), dtype=dA.dtype, device=DEV)
    mi.mimose_op_gemm(dtype, dA, lda, a_k, dB, ldb, b_k, C, N + 8, 0, M, N, K, bias=dbias, gelu_out=G, gelu=1)
    sync()
    pre = base + quant(bias, dtype)
    close(host(G)[:, :N], om.gelu_fwd(pre, False), dtype, scale=np.abs(pre).max(), k=3.0)


# weight gradients on the ring: parts with an odd and an even count of stages, a ragged last part; a round of
# units and a few
@pytest.mark.parametrize("M,N", [(1024, 1024), (300, 600), (8, 40)])
@pytest.mark.parametrize("T", [1024, 1100, 2000, 2089])
def test_gemm_ring_weight_gradient(T, M, N):
    dtype, ld = 1, lambda v: (v + 7) // 8 * 8
    rng = np.random.default_rng(T)
    dY, X = rng.standard_normal((T, M)).astype(np.float32), rng.standard_normal((T, N)).astype(np.float32)
    nws = mi.mimose_op_gemm_workspace_bytes(M, N)
    ws = torch.zeros(nws, dtype=torch.uint8, device=DEV)
    W = torch.full((M, N), 9.0, dtype=torch.float32, device=DEV)
    rs = torch.full((M,), 9.0, dtype=torch.float32, device=DEV)
    pad = lambda X: np.ascontiguousarray(np.pad(X, ((0, 0), (0, ld(X.shape[1]) - X.shape[1]))))
    mi.mimose_op_gemm(dtype, dev(pad(dY), dtype), ld(M), 0, dev(pad(X), dtype), ld(N), 0, W, N, 1, M, N, T, a_rowsum=rs, workspace=ws,
                      workspace_bytes=nws)
    sync()
    close(host(W), quant(dY, dtype).T @ quant(X, dtype), 0, k=40.0)
    close(host(rs), quant(dY, dtype).sum(0), 0, k=40.0)


def test_gemm_rejects_misaligned_bf16():
    a = torch.zeros(64 * 20, dtype=torch.bfloat16, device=DEV)
    with pytest.raises(mi.MimoseError):
        mi.mimose_op_gemm(1, a, 12, 1, a, 12, 1, a, 16, 0, 4, 4, 12)


# ---------------------------------------------------------------- LayerNorm
@pytest.mark.parametrize("dtype,x_f32,dy_f32", [(0, 0, 0), (1, 0, 0), (1, 1, 1), (1, 1, 0), (1, 0, 1)])
@pytest.mark.parametrize("T,H", [(37, 64), (130, 768), (5, 1024), (64, 24)])
def test_layernorm_fwd_bwd(dtype, x_f32, dy_f32, T, H):
    """x_f32 / dy_f32: in a bf16 configuration the input rows / incoming gradients are fp32
    (unrounded residual sums and the fp32 gradient carrier of the residual stream)."""
    rng = np.random.default_rng(T + H)
    x = (rng.standard_normal((T, H)) * 2 + 0.5).astype(np.float32)
    g = (1 + 0.2 * rng.standard_normal(H)).astype(np.float32)
    b = (0.1 * rng.standard_normal(H)).astype(np.float32)
    dy = rng.standard_normal((T, H)).astype(np.float32)
    add = rng.standard_normal((T, H)).astype(np.float32)
    xq = quant(x, 0 if x_f32 else dtype)
    dyq = quant(dy, 0 if dy_f32 else dtype)
    gq, bq, addq = (quant(v, dtype) for v in (g, b, add))
    y_ref, saved = om.layernorm_fwd(xq, gq, bq, 1e-5)
    dx_ref, dg_ref, db_ref = om.layernorm_bwd(dyq, saved, gq)
    dx_ = dev(x, 0 if x_f32 else dtype)
    ddy = dev(dy, 0 if dy_f32 else dtype)
    dg_, db_, dadd = dev(g, dtype), dev(b, dtype), dev(add, dtype)
    y = torch.zeros((T, H), dtype=dg_.dtype, device=DEV)
    mi.mimose_op_layernorm_fwd(dtype, dx_, x_f32, dg_, db_, y, T, H, 1e-5)
    sync()
    close(host(y), y_ref, dtype, k=2.0)
    P = mi.mimose_op_partial_rows(T)
    partial = torch.zeros(P * 2 * H, dtype=torch.float32, device=DEV)
    dgam = torch.zeros(H, dtype=torch.float32, device=DEV)
    dbet = torch.zeros(H, dtype=torch.float32, device=DEV)
    out = torch.zeros_like(y)
    mi.mimose_op_layernorm_bwd(dtype, ddy, dy_f32, dx_, x_f32, dg_, out, dadd, dgam, dbet, partial, T, H, 1e-5)
    sync()
    close(host(out), dx_ref + addq, dtype, k=3.0)
    close(host(dgam), dg_ref, 0, k=50.0)
    close(host(dbet), db_ref, 0, k=50.0)
    if not (dtype == 1 and dy_f32):
        # in place, no residual input
        mi.mimose_op_layernorm_bwd(dtype, ddy, dy_f32, dx_, x_f32, dg_, ddy, None, dgam, dbet, partial, T, H, 1e-5)
        sync()
        close(host(ddy), dx_ref, dtype, k=3.0)
    else:
        with pytest.raises(mi.MimoseError):                  # fp32 gradient in, bf16 out cannot alias
            mi.mimose_op_layernorm_bwd(dtype, ddy, dy_f32, dx_, x_f32, dg_, ddy, None, dgam, dbet, partial, T, H, 1e-5)


# 256 blocks of 16 rows have a wave for each row, 257 four waves with four rows' elements at a time, 513 with two;
# 768 and 1024 columns are three and four chunks a lane in fp32.  All add in the same order.
@pytest.mark.parametrize("dtype,wide", [(0, 0), (1, 0), (1, 1)])
@pytest.mark.parametrize("H", [8, 768, 1024])
def test_layernorm_bwd_waves_of_a_block(dtype, wide, H):
    few, sizes = 4088, (4104, 8200)                          # the last block half full
    g = torch.Generator(device=DEV).manual_seed(H)
    storage = torch.bfloat16 if dtype else torch.float32
    x = (torch.randn(sizes[-1], H, generator=g, device=DEV) * 2 + 0.5).to(torch.float32 if wide else storage)
    dy = torch.randn(sizes[-1], H, generator=g, device=DEV).to(x.dtype)
    dy[few:] = 0.0                                           # what the larger ones add to the sums
    gamma = torch.randn(H, generator=g, device=DEV).to(storage)
    add = torch.randn(sizes[-1], H, generator=g, device=DEV).to(storage)

    def run(T, residual, form):
        dx, masked = (torch.zeros(T, H, dtype=storage, device=DEV) for _ in range(2))
        d = dy[:T]
        if form == "in place":                               # later rows are loaded after earlier ones are stored
            d = dx = dy[:T].clone()
        partial = torch.zeros(mi.mimose_op_partial_rows(T) * 2 * H, device=DEV)
        dgam, dbet = torch.zeros(H, device=DEV), torch.zeros(H, device=DEV)
        a = add if residual else None
        if form == "masked":
            mi.mimose_op_layernorm_bwd_dropout(dtype, d, wide, x, wide, gamma, dx, a, masked, dgam, dbet, partial, T, H, 1e-5,
                                               0.2, 0xA5A5A5A5DEADBEEF, 14, 77)
        else:
            mi.mimose_op_layernorm_bwd(dtype, d, wide, x, wide, gamma, dx, a, dgam, dbet, partial, T, H, 1e-5)
        sync()
        return dx[:few], masked[:few], partial[:256 * 2 * H], dgam, dbet

    first = None
    for residual in (0, 1):
        for form in ("plain", "masked") + (() if wide else ("in place",)):
            a = run(few, residual, form)
            first = first or a
            for T in sizes:
                b = run(T, residual, form)
                assert all(torch.equal(a[i], b[i]) for i in range(3)), (residual, form, T)
            assert torch.equal(a[2], first[2])               # the sums are those of the plain form
            if residual:
                continue
            assert torch.equal(a[0], first[0])
    _, saved = om.layernorm_fwd(host(x[:few]), host(gamma), host(gamma), 1e-5)
    dx_ref, dg_ref, db_ref = om.layernorm_bwd(host(dy[:few]), saved, host(gamma))
    close(host(first[0]), dx_ref, dtype, k=3.0)
    close(host(a[0]), dx_ref + host(add[:few]), dtype, k=3.0)
    close(host(first[3]), dg_ref, 0, k=50.0)
    close(host(first[4]), db_ref, 0, k=50.0)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("form", [0, 1])
def test_gelu_bwd(dtype, form):
    rng = np.random.default_rng(9)
    n = 8 * 1000 + 5
    pre = (rng.standard_normal(n) * 2).astype(np.float32)
    d = rng.standard_normal(n).astype(np.float32)
    ref = quant(d, dtype) * om.gelu_grad(quant(pre, dtype), form)
    dd, dp = dev(d, dtype), dev(pre, dtype)
    mi.mimose_op_gelu_bwd(dtype, dd, dp, n, form)
    sync()
    close(host(dd), ref, dtype, k=2.0)


@pytest.mark.parametrize("n", [1, 4, 1023, 1027])
def test_gelu_bwd_fp32_off_16_bytes(n):
    """Operands that do not lie on 16 bytes give the bits of those that do."""
    g = torch.Generator(device=DEV).manual_seed(n)
    pre, d = (torch.randn(n, generator=g, device=DEV) * 2 for _ in range(2))
    for form in (0, 1):
        out = []
        for shift in (0, 1):
            buf, p = torch.full((2, n + 8), 9.0, device=DEV)
            buf[shift:shift + n], p[shift:shift + n] = d, pre
            mi.mimose_op_gelu_bwd(0, buf[shift:], p[shift:], n, form)
            sync()
            assert bool((buf[shift + n:] == 9.0).all()) and bool((buf[:shift] == 9.0).all())
            out.append(buf[shift:shift + n].clone())
        assert torch.equal(out[0], out[1])
        close(host(out[0]), host(d) * om.gelu_grad(host(pre), form), 0, k=2.0)


# ---------------------------------------------------------------- attention
def attention_case(dtype, B, L, nh, d, causal, seed, lengths=None, p_drop=0.0):
    rng = np.random.default_rng(seed)
    keep, kw = None, {}
    if p_drop:
        from oracle import philox as ph
        kw = dict(p_drop=float(np.float32(p_drop)), seed=0xABCDEF0123456789, site=4 * 3, step=77)
        keep = ph.keep_scale(ph.attn_index(B, nh, L), kw["p_drop"], kw["seed"], kw["site"], kw["step"])
    lens_dev = None if lengths is None else torch.tensor(lengths, dtype=torch.int32, device=DEV)
    H = nh * d
    qkv = rng.standard_normal((B * L, 3 * H)).astype(np.float32)
    dctx = rng.standard_normal((B * L, H)).astype(np.float32)
    qq = quant(qkv, dtype)
    q, k, v = (om.split_heads(qq[:, i * H:(i + 1) * H], B, L, nh) for i in range(3))
    o, p = om.attention_fwd(q, k, v, causal, lengths=lengths, keep=keep)
    ctx_ref = om.merge_heads(o)
    s = (q @ k.transpose(0, 1, 3, 2)) / np.sqrt(d)
    if causal:
        s = np.where(np.triu(np.ones((L, L), bool), 1), -np.inf, s)
    if lengths is not None:                                  # padded keys carry no weight
        s = np.where(np.arange(L)[None, None, None, :] >= np.asarray(lengths)[:, None, None, None], -np.inf, s)
    lse_ref = np.log(np.exp(s - s.max(-1, keepdims=True)).sum(-1)) + s.max(-1)
    dqkv_dev = dev(qkv, dtype)
    ctx = torch.zeros((B * L, H), dtype=dqkv_dev.dtype, device=DEV)
    lse = torch.zeros(B * nh * L, dtype=torch.float32, device=DEV)
    mi.mimose_op_attention_fwd(dtype, dqkv_dev, ctx, lse, B, L, nh, d, causal, lengths=lens_dev, **kw)
    sync()
    if dtype == 0:
        close(host(ctx), ctx_ref, dtype, k=3.0)
    else:
        # bf16 path: probabilities are rounded to bf16 before the P V product, so the output error
        # is a sum of many independent roundings: bound it in norm and in the largest element
        assert rel_l2(host(ctx), ctx_ref) < 6e-3
        assert np.abs(host(ctx) - ctx_ref).max() < 4 * EPS[1] * np.abs(ctx_ref).max()
    assert np.abs(host(lse).reshape(B, nh, L) - lse_ref).max() < (1e-4 if dtype == 0 else 2e-2)
    # backward consumes the stored (rounded) forward output, like the training step does
    ctx_q = host(ctx)
    do = om.split_heads(quant(dctx, dtype), B, L, nh)
    dq, dk, dv = om.attention_bwd(do, q, k, v, p, keep)
    ref = np.concatenate([om.merge_heads(dq), om.merge_heads(dk), om.merge_heads(dv)], axis=1)
    ddctx = dev(dctx, dtype)
    delta = torch.zeros(B * nh * L, dtype=torch.float32, device=DEV)
    out = torch.zeros_like(dqkv_dev)
    mi.mimose_op_attention_bwd(dtype, dqkv_dev, ctx, ddctx, lse, delta, out, B, L, nh, d, causal, lengths=lens_dev, **kw)
    sync()
    got = host(out)
    if lengths is not None:                                  # dK, dV of padded keys: exact zeros
        pad = (np.arange(L)[None, :] >= np.asarray(lengths)[:, None]).reshape(-1)
        assert not got[pad, H:].any()
    floor = 1e-2 * np.linalg.norm(ref)                      # dQ and dK vanish identically when L = 1
    for i, name in enumerate("qkv"):
        part = ref[:, i * H:(i + 1) * H]
        e = np.linalg.norm(got[:, i * H:(i + 1) * H] - part) / max(np.linalg.norm(part), floor)
        assert e < (2e-5 if dtype == 0 else 1.5e-2), (name, e)
    assert ctx_q.shape == ctx_ref.shape


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("B,L,nh,d", [(2, 70, 2, 32), (1, 200, 3, 64), (3, 1, 2, 64), (2, 17, 1, 32), (1, 129, 2, 64), (2, 333, 2, 64)])
def test_attention(dtype, causal, B, L, nh, d):
    attention_case(dtype, B, L, nh, d, causal, seed=B * 100 + L)


# samples padded to the batch's longest: a sample of one token, padding that starts inside a key
# tile, whole key blocks of padding, no padding at all
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("L,nh,d,lengths", [(70, 2, 32, [70, 1, 33]), (200, 3, 64, [200, 64, 65]),
                                            (333, 2, 64, [5, 333, 128, 129]), (17, 1, 64, [17, 16])])
def test_attention_padded(dtype, causal, L, nh, d, lengths):
    attention_case(dtype, len(lengths), L, nh, d, causal, seed=L + 7, lengths=lengths)


# pairs of sample and head that do not fill the 8 XCDs, tiles of 64 keys and blocks of 128 queries
# whole, one row short and one row over, several row blocks of which a causal tile misses some waves
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("L,nh,lengths", [(63, 1, None), (64, 3, [64, 1, 31]), (65, 2, None), (127, 3, [33, 127, 95]),
                                          (256, 1, [256] * 8 + [97]), (257, 5, [257, 64, 256])])
def test_attention_tile_edges(causal, L, nh, lengths):
    attention_case(1, len(lengths) if lengths else 3, L, nh, 64, causal, seed=L + 3, lengths=lengths)


# fp32 MFMAs: four waves take the tiles of 32 in turn, some of them none, or none that a query may see
@pytest.mark.parametrize("dtype,d", [(0, 64), (0, 32), (1, 32)])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("L,lengths,p_drop", [(32, None, 0.0), (65, [1, 32, 33, 65], 0.0), (128, [97, 128], 0.2),
                                              (161, [31, 129, 160, 161], 0.0)])
def test_attention_fp32_waves(dtype, d, causal, L, lengths, p_drop):
    attention_case(dtype, len(lengths) if lengths else 2, L, 3, d, causal, seed=L + 5, lengths=lengths, p_drop=p_drop)


# Waves of a block by tiles of 32 rows and by blocks of the batch (samples x heads x tiles): one, two, twice two or four
@pytest.mark.parametrize("dtype,d", [(0, 64), (0, 32), (1, 32)])
@pytest.mark.parametrize("B,L,nh,causal,p_drop", [(3, 31, 3, 0, 0.2), (5, 32, 2, 1, 0.0),        # one tile: one wave
                                                  (127, 64, 3, 0, 0.0), (128, 64, 3, 1, 0.0),    # 762, 768 blocks of two: two, one
                                                  (129, 33, 3, 0, 0.2),                          # 774, the last of one row
                                                  (170, 96, 3, 0, 0.0), (171, 70, 3, 0, 0.2),    # 1530, 1539 of three: two, one
                                                  (52, 129, 3, 1, 0.2),                          # 780 of five: two
                                                  (171, 97, 3, 0, 0.0),                          # 2052 of four: two
                                                  (42, 64, 3, 0, 0.2), (43, 64, 3, 0, 0.2),      # 252, 258 of two: two, twice two
                                                  (85, 33, 3, 1, 0.0), (86, 50, 3, 0, 0.0),      # 510, 516: twice two, two
                                                  (256, 64, 3, 0, 0.2)])                         # 1536: one, with d = 32 twice two
def test_attention_waves_of_a_block(dtype, d, B, L, nh, causal, p_drop):
    lengths = [(1, L, max(1, L - 1), min(L, 32), min(L, 33), max(1, L // 2))[b % 6] for b in range(B)]
    attention_case(dtype, B, L, nh, d, causal, seed=L + B, lengths=lengths, p_drop=p_drop)


@pytest.mark.parametrize("dtype,d", [(0, 64), (0, 32), (1, 32)])
def test_attention_groups_of_a_block_bits(dtype, d):
    """Two groups of waves in a block (258 blocks of 32 rows) give every sample the bits that one gives it (252)."""
    B, L, nh = 43, 60, 3
    st = torch.bfloat16 if dtype else torch.float32
    g = torch.Generator(device=DEV).manual_seed(d + dtype)
    H = nh * d
    qkv, dctx = torch.randn(B * L, 3 * H, generator=g, device=DEV).to(st), torch.randn(B * L, H, generator=g, device=DEV).to(st)
    lengths = torch.tensor([(60, 32, 33, 1, 59)[b % 5] for b in range(B)], dtype=torch.int32, device=DEV)
    for causal in (0, 1):
        out = []
        for n in (B, B - 1):
            ctx, dq = torch.zeros(n * L, H, dtype=st, device=DEV), torch.zeros(n * L, 3 * H, dtype=st, device=DEV)
            lse, delta = torch.zeros(n * nh * L, device=DEV), torch.zeros(n * nh * L, device=DEV)
            mi.mimose_op_attention_fwd(dtype, qkv, ctx, lse, n, L, nh, d, causal, lengths=lengths)
            mi.mimose_op_attention_bwd(dtype, qkv, ctx, dctx, lse, delta, dq, n, L, nh, d, causal, lengths=lengths)
            sync()
            out.append((ctx, lse, delta, dq))
        assert all(torch.equal(a[:len(b)], b) for a, b in zip(*out))


# dropout of the probabilities: the kept set is the oracle's (integer comparisons of generator
# words), so the usual tolerances apply; lengths off the 4-key grid, several key tiles, padding
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("B,L,nh,d,lengths", [(2, 70, 2, 32, None), (1, 200, 3, 64, None), (2, 333, 2, 64, None),
                                              (3, 5, 1, 64, None), (2, 130, 2, 64, [130, 61])])
def test_attention_dropout(dtype, causal, B, L, nh, d, lengths):
    attention_case(dtype, B, L, nh, d, causal, seed=L + 11, lengths=lengths, p_drop=0.2)


# ---------------------------------------------------------------- softmax cross-entropy
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("T,V", [(50, 1000), (9, 37), (20, 30522)])
def test_softmax_xent(dtype, T, V):
    rng = np.random.default_rng(V)
    ld = (V + 63) // 64 * 64
    logits = (rng.standard_normal((T, V)) * 3).astype(np.float32)
    labels = rng.integers(0, V, T).astype(np.int32)
    labels[1] = -1
    n_valid = int((labels >= 0).sum())
    loss_ref, d_ref = om.cross_entropy(quant(logits, dtype), labels)
    buf = np.full((T, ld), 3.0, np.float32)
    buf[:, :V] = logits
    dl = dev(buf, dtype)
    row_loss = torch.zeros(T, dtype=torch.float32, device=DEV)
    loss = torch.zeros(1, dtype=torch.float32, device=DEV)
    mi.mimose_op_softmax_xent(dtype, dl, ld, torch.tensor(labels, device=DEV), row_loss, loss, T, V, n_valid)
    sync()
    got = host(dl)
    assert np.all(got[:, V:] == 0.0)
    assert abs(float(loss.item()) - loss_ref) <= 2e-6 * abs(loss_ref) * (1 if dtype == 0 else 10)
    close(got[:, :V], d_ref, dtype, scale=np.abs(d_ref).max(), k=3.0)
    assert np.all(got[1] == 0.0)


# ---------------------------------------------------------------- embedding
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("has_ln", [0, 1])
def test_embedding_fwd_bwd(dtype, has_ln):
    rng = np.random.default_rng(3)
    B, L, H, V, max_seq = 3, 21, 192, 50, 32
    tok = rng.standard_normal((V, H)).astype(np.float32)
    pos = rng.standard_normal((max_seq, H)).astype(np.float32)
    g = (1 + 0.1 * rng.standard_normal(H)).astype(np.float32)
    b = (0.1 * rng.standard_normal(H)).astype(np.float32)
    ids = rng.integers(0, V, B * L).astype(np.int32)
    p = np.tile(np.arange(L), B)
    s_ref = quant(quant(tok, dtype)[ids] + quant(pos, dtype)[p], dtype)
    y_ref = om.layernorm_fwd(s_ref, quant(g, dtype), quant(b, dtype), 1e-5)[0] if has_ln else s_ref
    dtok, dpos, dg, db_ = dev(tok, dtype), dev(pos, dtype), dev(g, dtype), dev(b, dtype)
    dids = torch.tensor(ids, device=DEV)
    ssum = torch.zeros((B * L, H), dtype=dtok.dtype, device=DEV)
    y = torch.zeros_like(ssum)
    mi.mimose_op_embed_fwd(dtype, dids, dtok, dpos, dg, db_, ssum, y, B, L, H, 1e-5, has_ln)
    sync()
    assert np.array_equal(host(ssum), s_ref)
    close(host(y), y_ref, dtype, k=2.0)
    # backward: deterministic scatter-add
    d = rng.standard_normal((B * L, H)).astype(np.float32)
    order = np.argsort(ids, kind="stable").astype(np.int32)
    sorted_ids = ids[order]
    starts = np.flatnonzero(np.r_[True, sorted_ids[1:] != sorted_ids[:-1]]).astype(np.int32)
    seg = np.r_[starts, B * L].astype(np.int32)
    gtok = torch.ones((V, H), dtype=torch.float32, device=DEV)
    gpos = torch.full((max_seq, H), 5.0, dtype=torch.float32, device=DEV)
    mi.mimose_op_embed_bwd(dtype, dev(d, dtype), dids, torch.tensor(order, device=DEV), torch.tensor(seg, device=DEV),
                           len(starts), gtok, gpos, B, L, H, max_seq)
    sync()
    ref_tok = np.ones((V, H)); np.add.at(ref_tok, ids, quant(d, dtype))
    ref_pos = np.zeros((max_seq, H)); np.add.at(ref_pos, p, quant(d, dtype))
    close(host(gtok), ref_tok, 0, k=20.0)
    close(host(gpos), ref_pos, 0, k=20.0)


# runs of one id around the length a single wave still sums, and far beyond it; widths whose last
# column group is partial, and one that takes the scalar accesses
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("H", [64, 264, 1024, 70])
def test_embedding_bwd_frequent_ids(dtype, H):
    rng = np.random.default_rng(4)
    runs = [1, 63, 64, 65, 7, 128, 129, 700, 1, 9, 8, 1, 2, 3, 5, 6, 7, 11, 1023]
    ids = rng.permutation(np.repeat(np.arange(3, 3 + len(runs)), runs)).astype(np.int32)
    B, L, V, max_seq = 2, len(ids) // 2, 40, len(ids)
    ids = ids[:B * L]
    d = rng.standard_normal((B * L, H)).astype(np.float32)
    order = np.argsort(ids, kind="stable").astype(np.int32)
    si = ids[order]
    starts = np.flatnonzero(np.r_[True, si[1:] != si[:-1]]).astype(np.int32)
    gtok = torch.ones((V, H), dtype=torch.float32, device=DEV)
    gpos = torch.zeros((max_seq, H), dtype=torch.float32, device=DEV)
    mi.mimose_op_embed_bwd(dtype, dev(d, dtype), torch.tensor(ids, device=DEV), torch.tensor(order, device=DEV),
                           torch.tensor(np.r_[starts, B * L].astype(np.int32), device=DEV), len(starts), gtok, gpos, B, L, H,
                           max_seq)
    sync()
    ref = np.ones((V, H)); np.add.at(ref, ids, quant(d, dtype))
    close(host(gtok), ref, 0, k=200.0)


# ---------------------------------------------------------------- dropout (counter-based masks)
@pytest.mark.parametrize("dtype,io_f32", [(0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("n", [4096 + 3, 5, 1 << 18])
@pytest.mark.parametrize("with_resid", [0, 1])
def test_dropout_op(dtype, io_f32, n, with_resid):
    """The kept set must be the oracle's bit for bit (an integer comparison of generator words);
    the values are one multiplication and one addition in fp32."""
    from oracle import philox as ph
    rng = np.random.default_rng(n + dtype)
    p = float(np.float32(0.3))
    seed, site, step = 0x9E3779B97F4A7C15, 4 * 7 + 1, 123456
    src = rng.standard_normal(n).astype(np.float32)
    resid = rng.standard_normal(n).astype(np.float32)
    io_dtype = 0 if io_f32 else dtype
    d_src = dev(src, io_dtype)
    d_res = dev(resid, dtype) if with_resid else None
    out = torch.full_like(d_src, 9.0)
    mi.mimose_op_dropout(dtype, out, d_src, io_f32, d_res, n, p, seed, site, step)
    inplace = d_src.clone()
    mi.mimose_op_dropout(dtype, inplace, inplace, io_f32, d_res, n, p, seed, site, step)
    sync()
    keep = ph.keep_scale(np.arange(n, dtype=np.uint64), p, seed, site, step)
    base = quant(resid, dtype).astype(np.float64) if with_resid else np.zeros(n)
    ref = base + keep * quant(src, io_dtype)
    got = host(out)
    if not with_resid:
        assert np.array_equal(got != 0, (keep != 0) & (quant(src, io_dtype) != 0))      # the same elements survive
    close(got, ref, io_dtype, k=1.5)
    assert np.array_equal(host(inplace), got)
    assert 0.25 < (keep == 0).mean() < 0.35 or n < 100


# H % 8 and H % 4, and `shift`: elements by which every row operand starts off a 16-byte boundary,
# decide between the one-pass kernels and separate passes
@pytest.mark.parametrize("dtype,wide", [(0, 0), (1, 0), (1, 1)])
@pytest.mark.parametrize("T,H,shift", [(37, 64, 0), (130, 768, 0), (5, 1024, 0), (18, 24, 0), (18, 20, 0), (18, 70, 0),
                                       (18, 64, 1), (33, 768, 4)])
def test_dropout_inside_layernorm(dtype, wide, T, H, shift):
    """x = resid + dropout(x), y = LayerNorm(x), and LayerNorm's backward with a masked copy of dx: the
    kept set and the sum are those of the element-wise pass bit for bit, the rest the oracle's."""
    from oracle import philox as ph
    rng = np.random.default_rng(T * H + shift)
    p, seed, site, step = float(np.float32(0.2)), 0xA5A5A5A5DEADBEEF, 4 * 3 + 2, 77
    io = 0 if wide else dtype

    def at(a, dt):                                    # a copy that starts `shift` elements into its buffer
        buf = torch.zeros(a.size + shift, dtype=dev(a, dt).dtype, device=DEV)
        buf[shift:] = dev(a, dt).reshape(-1)
        return buf[shift:].view(T, H)

    x, resid, dy, add = (rng.standard_normal((T, H)).astype(np.float32) for _ in range(4))
    g = (1 + 0.2 * rng.standard_normal(H)).astype(np.float32)
    b = (0.1 * rng.standard_normal(H)).astype(np.float32)
    dg_, db_, dres, dadd = dev(g, dtype), dev(b, dtype), at(resid, dtype), at(add, dtype)
    keep = ph.keep_scale(np.arange(T * H, dtype=np.uint64), p, seed, site, step).reshape(T, H)

    separate = at(x, io)
    mi.mimose_op_dropout(dtype, separate, separate, wide, dres, T * H, p, seed, site, step)
    xs, y = at(x, io), at(np.full((T, H), 9.0, np.float32), dtype)
    mi.mimose_op_dropout_layernorm_fwd(dtype, xs, wide, dres, dg_, db_, y, T, H, 1e-5, p, seed, site, step)
    alone = at(x, io)
    mi.mimose_op_dropout_layernorm_fwd(dtype, alone, wide, dres, dg_, db_, None, T, H, 1e-5, p, seed, site, step)
    sync()
    assert torch.equal(xs, separate) and torch.equal(alone, separate)
    close(host(xs), quant(resid, dtype) + keep * quant(x, io), io, k=1.5)
    y_ref, saved = om.layernorm_fwd(host(xs), quant(g, dtype), quant(b, dtype), 1e-5)
    close(host(y), y_ref, dtype, k=2.0)

    ddy = at(dy, io)
    out, masked = (at(np.full((T, H), 9.0, np.float32), dtype) for _ in range(2))
    dgam, dbet = (torch.zeros(H, dtype=torch.float32, device=DEV) for _ in range(2))
    partial = torch.zeros(mi.mimose_op_partial_rows(T) * 2 * H, dtype=torch.float32, device=DEV)
    mi.mimose_op_layernorm_bwd_dropout(dtype, ddy, wide, xs, wide, dg_, out, dadd, masked, dgam, dbet, partial, T, H, 1e-5,
                                       p, seed, site, step)
    want = at(np.zeros((T, H), np.float32), dtype)
    mi.mimose_op_dropout(dtype, want, out, 0, None, T * H, p, seed, site, step)
    sync()
    dx_ref, dg_ref, db_ref = om.layernorm_bwd(quant(dy, io), saved, quant(g, dtype))
    close(host(out), dx_ref + quant(add, dtype), dtype, k=3.0)
    close(host(dgam), dg_ref, 0, k=50.0)
    close(host(dbet), db_ref, 0, k=50.0)
    assert torch.equal(masked, want) and (host(masked) != 9.0).all()
    assert np.array_equal(host(masked) != 0, (keep != 0) & (host(out) != 0))
    for alias in (out, ddy):
        with pytest.raises(mi.MimoseError):
            mi.mimose_op_layernorm_bwd_dropout(dtype, ddy, wide, xs, wide, dg_, out, dadd, alias, dgam, dbet, partial, T, H,
                                               1e-5, p, seed, site, step)


@pytest.mark.parametrize("rows,N,K", [(1, 8, 1536), (74, 768, 1544), (300, 776, 3072),          # 32 x 32 tiles: one, a tail, ragged
                                      (700, 1000, 1600), (640, 1024, 1656),                     # 64 x 64 (k-major B): a stage half full, a tail in its first half
                                      (1500, 1032, 1664), (1441, 1024, 1736),                   # 96 x 64
                                      (2000, 1032, 1536), (2048, 1000, 1592)])                  # 128 x 64 (k-major B)
@pytest.mark.parametrize("b_k", [1, 0])
def test_gemm_long_reductions_bits(rows, N, K, b_k):
    """Few rows behind a long reduction: the bits are those of the same rows in a product of more,
    which other kernels do, in every form of the store."""
    g = torch.Generator(device=DEV).manual_seed(rows + K + b_k)
    up = lambda v: (v + 7) // 8 * 8
    mk = lambda r, c: (torch.randn((r, c), generator=g, device=DEV) * 0.5).to(torch.bfloat16)
    M = rows + 6000
    A, B, bias, resid = mk(M, K), mk(N, K) if b_k else mk(K, up(N)), mk(1, up(N))[0], mk(M, up(N))
    forms = [dict(c_f32=1), dict(c_f32=1, bias=1, resid=1), dict(c_f32=0, resid=1), dict(c_f32=0, bias=1),
             dict(c_f32=0, bias=1, gelu=1), dict(c_f32=0, bias=1, resid=1, gelu=2)]
    for form in forms:
        for pitch in (up(N) + 8, N + 3):                        # rows of C on 16 bytes, and not
            if form.get("gelu") and pitch != up(N) + 8:         # (off 16 bytes GELU is the C library's in every kernel but the store of 8 columns)
                continue
            def product(r0, n_rows):
                C = torch.full((n_rows, pitch), 7.0, dtype=torch.float32 if form["c_f32"] else torch.bfloat16, device=DEV)
                G = torch.full_like(C, 7.0) if form.get("gelu") else None
                kw = {}
                if form.get("bias"): kw["bias"] = bias
                if form.get("resid"): kw.update(resid=resid[r0:], ldr=up(N))
                if G is not None: kw.update(gelu_out=G, gelu=form["gelu"])
                mi.mimose_op_gemm(1, A[r0:], K, 1, B, K if b_k else up(N), b_k, C, pitch, form["c_f32"], n_rows, N, K, **kw)
                sync()
                return [x for x in (C, G) if x is not None]
            for full, alone in zip(product(0, M), product(0, rows)):
                assert bool((alone[:, N:] == 7.0).all()), "wrote outside the N columns"
                assert torch.equal(full[:rows, :N], alone[:, :N]), form
