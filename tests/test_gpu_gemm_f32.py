"""fp32 products, whose operands are split in three bf16 parts, against 64-bit products: every block
tile and number of ways the launcher chooses, with the reduction's end alone and with the pipelined loop before
it, at ragged ends, in every layout."""
import os
import re

import numpy as np
import pytest
import torch

import paper_2209_02478_amd as mi
from oracle import model as om
from gpu_util import DEV, host, sync

pytestmark = pytest.mark.gpu

U = 2.0 ** -24                        # unit roundoff of fp32

# block tile, ways and slices requested ahead of the launcher's variants
TILES = [(128, 128, 1, 1), (64, 64, 1, 2), (64, 64, 2, 2), (32, 32, 2, 3), (32, 32, 4, 2), (96, 64, 1, 2), (128, 64, 1, 2)]


def variant(M, N, K):
    """The variant `estimate` picks, by the constants in the source."""
    src = open(os.path.join(os.path.dirname(mi.__file__), "csrc", "gemm_f32.hip")).read()
    table = {k: [int(x) for x in v.split(",")] for k, v in re.findall(r"(k\w+)\[kVariants\] = \{([-0-9, ]+)\}", src)}
    assert [t[:2] for t in TILES] == list(zip(table["kM"], table["kN"]))

    def estimate(w):
        rounds = -(-(-(-M // table["kM"][w]) * -(-N // table["kN"][w])) // 256)
        slices = -(-K // 32)
        return (table["kAlone"][w] + slices * table["kAloneSlice"][w] if rounds == 1 else
                rounds * (table["kMany"][w] + slices * table["kManySlice"][w]))
    return min(range(len(TILES)), key=estimate)


SUMS = [1, 2, 2, 2, 4, 2, 2]          # that share an element's reduction: the ways, or a single way's two slices of a turn


# (M, N, K) -> variant it gets; remainders of tiles, of slices and of ways' turns
SHAPES = {(1, 1, 1): 4, (33, 65, 31): 4, (130, 129, 100): 4, (130, 70, 515): 4,        # 32 x 32, four ways
          (130, 2300, 250): 3, (130, 1867, 99): 3,                                     # 32 x 32, two
          (260, 2300, 99): 2, (520, 1030, 1000): 2,                                    # 64 x 64, two
          (129, 2305, 32): 1, (900, 900, 70): 1, (1410, 3000, 130): 1,                 # 64 x 64, one
          (1100, 1030, 260): 5, (1409, 770, 515): 5,                                   # 96 x 64
          (700, 2300, 300): 6, (2305, 750, 515): 6,                                    # 128 x 64
          (1500, 1500, 70): 0, (1345, 2300, 99): 0}                                    # 128 x 128
# every variant with a reduction that its pipelined loop takes several turns of, and a ragged end
LONG = {(227, 130, 1300): 4, (130, 1736, 1030): 3, (325, 1474, 850): 2, (906, 2129, 515): 1, (325, 2784, 515): 5,
        (615, 2391, 515): 6, (712, 2784, 303): 0}


def test_shapes_reach_every_variant():
    for shapes in (SHAPES, LONG):
        assert set(shapes.values()) == set(range(len(TILES)))
        for shape, which in shapes.items():
            assert variant(*shape) == which, shape
    for (M, N, K), which in LONG.items():
        ways, ahead = TILES[which][2:]
        for way in range(ways):
            whole = (K // 32 - way + ways - 1) // ways          # slices of the way that lie inside K
            assert whole > 2 * ahead + 2 * ahead and K % 32, (M, N, K)


def put(X, kmajor, pad):
    """X [rows, K] as the operand lies on the device, and its leading dimension (pad 3: no 16-byte rows)."""
    Y = X if kmajor else X.T
    buf = np.full((Y.shape[0], (Y.shape[1] + 3) // 4 * 4 + pad), np.nan, np.float32)    # the padding is not read
    buf[:, :Y.shape[1]] = Y
    return torch.from_numpy(buf).to(DEV), buf.shape[1]


@pytest.mark.parametrize("a_k,b_k", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_split_products(M, N, K, a_k, b_k):
    rng = np.random.default_rng(M + 3 * N + 5 * K + a_k + 2 * b_k)
    A, B = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    bias, resid = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    a64, b64 = A.astype(np.float64), B.astype(np.float64)
    prod, mag = a64 @ b64.T, np.abs(a64) @ np.abs(b64).T
    # three left-out products of 2^-27, a rounding or a few for the 32 products of a slice (at most half the
    # largest sum each, on average far less), the ways' sums, bias and residual
    bound = (K / 32 + 16) * U * (mag + np.abs(bias) + np.abs(resid)) + 1e-30
    for pad in (0, 3):
        dA, lda = put(A, a_k, pad)
        dB, ldb = put(B, b_k, pad)
        C = torch.full((M, N + 5), 7.0, device=DEV)
        G = torch.full((M, N + 5), 7.0, device=DEV)
        rs = torch.full((M + 1,), 9.0, device=DEV)
        mi.mimose_op_gemm(0, dA, lda, a_k, dB, ldb, b_k, C, N + 5, 0, M, N, K, bias=torch.from_numpy(bias).to(DEV),
                          resid=torch.from_numpy(resid).to(DEV), ldr=N, gelu_out=G, gelu=1, a_rowsum=rs)
        sync()
        got = host(C)
        pre = prod + bias + resid
        assert np.all(np.abs(got[:, :N] - pre) <= bound)
        assert np.all(got[:, N:] == 7.0) and np.all(host(G)[:, N:] == 7.0), "wrote outside the N columns"
        # GELU's slope is at most 1.13; its own evaluation a few roundings
        assert np.all(np.abs(host(G)[:, :N] - om.gelu_fwd(pre, False)) <= 1.13 * bound + 16 * U * (1 + np.abs(pre)))
        s = host(rs)
        assert np.all(np.abs(s[:M] - a64.sum(1)) <= (K / 4 + 16) * U * np.abs(a64).sum(1)) and s[M] == 9.0
        # aligned rows of C: the same bits through 8-byte stores
        C2 = torch.full((M, (N + 3) // 4 * 4), 7.0, device=DEV)
        mi.mimose_op_gemm(0, dA, lda, a_k, dB, ldb, b_k, C2, C2.shape[1], 0, M, N, K, bias=torch.from_numpy(bias).to(DEV))
        C3 = torch.full((M, N + 5), 7.0, device=DEV)
        mi.mimose_op_gemm(0, dA, lda, a_k, dB, ldb, b_k, C3, N + 5, 0, M, N, K, bias=torch.from_numpy(bias).to(DEV))
        sync()
        assert torch.equal(C2[:, :N], C3[:, :N])


@pytest.mark.parametrize("a_k,b_k", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("M,N,K", LONG)
def test_pipelined_loop(M, N, K, a_k, b_k):
    """Aligned operands, without row sums as forward and data gradients have them, and with the row sums of weight
    gradients (both operands m-major); values of both signs, and of one (a rounding that always goes one way adds up)."""
    rng = np.random.default_rng(M + 3 * N + 5 * K + a_k + 2 * b_k)
    for one_sign in (False, True):
        A, B = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
        if one_sign:
            A, B = np.abs(A), np.abs(B)
        a64, b64 = A.astype(np.float64), B.astype(np.float64)
        prod, mag = a64 @ b64.T, np.abs(a64) @ np.abs(b64).T
        dA, lda = put(A, a_k, 0)
        dB, ldb = put(B, b_k, 0)
        C = torch.full((M, (N + 3) // 4 * 4), 7.0, device=DEV)
        rs = torch.zeros(M, device=DEV) if not a_k and not b_k else None
        mi.mimose_op_gemm(0, dA, lda, a_k, dB, ldb, b_k, C, C.shape[1], 0, M, N, K, a_rowsum=rs)
        sync()
        if rs is not None:
            assert np.all(np.abs(host(rs) - a64.sum(1)) <= (K / 4 + 16) * U * np.abs(a64).sum(1))
        err = host(C)[:, :N] - prod
        assert np.all(np.abs(err) <= (K / 32 + 16) * U * mag) and bool((C[:, N:] == 7.0).all())
        if one_sign:
            # Independent errors of at most that size have a mean of its 1 / sqrt(M N) (four times that here), and the last rounding
            # of a sum may lean to one side by a quarter; one that went down in each of K / 32 slices would be K / 64 roundings.
            assert abs((err / mag).mean()) <= U / 4 + 4 * (K / 32 + 16) * U / np.sqrt(M * N)
            # 2-norm: s sums of mag / s each, that grow evenly in K / (8 s) roundings (the matrix core rounds for eight indices), each
            # off by at most 0.5 of a roundoff (rms; 0.42 on average), and two or three roundings of the whole
            s = SUMS[LONG[M, N, K]]
            assert np.linalg.norm(err) <= 0.5 * U * np.sqrt(K / (24 * s * s) + 2) * np.linalg.norm(prod)


@pytest.mark.parametrize("a_k,b_k", [(1, 1), (1, 0), (0, 0)])
@pytest.mark.parametrize("M,N,K", [(130, 129, 100), (130, 2300, 250), (260, 2300, 99), (900, 900, 70), (1409, 770, 515),
                                   (700, 2300, 300), (1500, 1500, 70)])
def test_infinities_and_nan(M, N, K, a_k, b_k):
    """Values the split cannot carry come out as fp32 arithmetic has them, and disturb no other output."""
    rng = np.random.default_rng(K)
    A, B = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    A[3, 5] = np.inf
    A[70, 9] = np.nan
    B[11, 2] = -np.inf
    B[20, 5] = 0.0                                                 # inf * 0
    A[100, 7] = np.finfo(np.float32).max                           # rounds to infinity as bf16
    B[:, 7] *= 0.125
    with np.errstate(invalid="ignore", over="ignore"):
        ref = A.astype(np.float64) @ B.astype(np.float64).T
        want = ref.astype(np.float32)
    dA, lda = put(A, a_k, 0)
    dB, ldb = put(B, b_k, 0)
    C = torch.zeros((M, N), device=DEV)
    mi.mimose_op_gemm(0, dA, lda, a_k, dB, ldb, b_k, C, N, 0, M, N, K)
    sync()
    got = C.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf])
    fin = np.isfinite(want)
    with np.errstate(invalid="ignore", over="ignore"):
        mag = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64)).T
    # the tiles taken again round for every two indices
    assert np.all(np.abs(got[fin] - ref[fin]) <= (K / 2 + 16) * U * mag[fin])


# A's and B's values around 2^ea and 2^eb: where parts of a value would be bf16 denormals or vanish (below 2^-109),
# fp32 denormals; and operands above 2^112 and sums above 2^96, which the split's scale takes out of fp32's range
@pytest.mark.parametrize("ea,eb", [(-112, 0), (-116, 90), (60, -124), (-133, 100), (-145, 100), (90, -149), (-60, -60), (50, 50), (-20, 114)])
@pytest.mark.parametrize("M,N,K,a_k,b_k", [(33, 65, 131, 1, 1), (260, 2300, 99, 0, 0), (1410, 1300, 200, 1, 0), (1409, 770, 515, 1, 1)])
def test_small_and_large_operands(M, N, K, a_k, b_k, ea, eb):
    rng = np.random.default_rng(M + K + 1000 * (ea + 200) + eb + 200)
    A, B = rng.standard_normal((M, K)), rng.standard_normal((N, K))
    A, B = (A * 2.0 ** ea).astype(np.float32), (B * 2.0 ** eb).astype(np.float32)
    # every fourth column of B sees the small or large values alone, its others stand beside common ones
    A[:, : K // 2] = rng.standard_normal((M, K // 2))
    B[:, : K // 2] = rng.standard_normal((N, K // 2)) * 2.0 ** min(0, ea + eb)
    B[::4, : K // 2] = 0.0
    a64, b64 = A.astype(np.float64), B.astype(np.float64)
    ref, mag = a64 @ b64.T, np.abs(a64) @ np.abs(b64).T
    dA, lda = put(A, a_k, 0)
    dB, ldb = put(B, b_k, 0)
    C = torch.zeros((M, N), device=DEV)
    mi.mimose_op_gemm(0, dA, lda, a_k, dB, ldb, b_k, C, N, 0, M, N, K)
    sync()
    # as above, or one rounding for every two indices where a tile is taken again; sums below 2^-126 round to 2^-149
    per = 2 if ea + eb > 80 or max(ea, eb) > 105 else 32
    bound = (K / per + 16) * U * mag + 2.0 ** -149 * K
    err = np.abs(host(C).astype(np.float64) - ref)
    assert np.all(err <= bound), (err / np.maximum(mag, 1e-300)).max()
