"""Kernel-by-kernel parity of the HIP path against the fp64 oracle, through the C-ABI.
Sizes span several tiles and a ragged tail; the oracle finishes each in well under a second."""
import numpy as np
import pytest
import torch

from oracle import stage_fp64 as O
from paper_2510_05186_amd import binding as B
from gpu_util import TOL, dev, host, ok, q, rel_err, rms_err, stream

pytestmark = pytest.mark.gpu
RNG = np.random.default_rng(42)
FP32, BF16 = 0, 1


def lib():
    return B.lib()


# ------------------------------------------------------------------ GEMM
@pytest.mark.parametrize("dtype,M,N,K", [
    (BF16, 520, 776, 328),        # 128x128 tiles, ragged in M, N and K
    (BF16, 2824, 3080, 264),      # 256x256 tiles (12 x 13), ragged
    (BF16, 2824, 3080, 320),      # same, K a multiple of 64: direct global->LDS tile loads, ragged M and N
    (BF16, 4096, 2048, 64),       # direct path, a single k-tile
    (BF16, 3000, 4096, 128),      # direct path, two k-tiles
    (BF16, 2824, 3080, 192),      # direct path: 3, 6, 7 and 11 k-tiles walk the ring of five LDS slots through every
    (BF16, 2824, 3080, 384),      # alignment of a tile's two slots, with and without a wrap inside the tile
    (BF16, 2824, 3080, 448),
    (BF16, 2824, 3080, 704),
    (BF16, 256, 256, 64),
    (BF16, 8, 8, 8),
    (FP32, 130, 77, 50),
    (FP32, 128, 256, 1024),
])
def test_gemm_nt_store_and_residual(dtype, M, N, K):
    a = q(RNG.standard_normal((M, K)), dtype)
    w = q(0.05 * RNG.standard_normal((N, K)), dtype)
    r = q(RNG.standard_normal((M, N)), dtype)
    A, W, R = dev(a, dtype), dev(w, dtype), dev(r, dtype)
    C = torch.empty_like(R)
    ok(lib().optstage_op_gemm(dtype, B.GEMM_NT, B.EPI_STORE, A.data_ptr(), W.data_ptr(), C.data_ptr(), 0, M, N, K, K, K, N, stream()))
    torch.cuda.synchronize()
    assert rel_err(host(C), O.linear_fwd(a, w)) < TOL[dtype]
    ok(lib().optstage_op_gemm(dtype, B.GEMM_NT, B.EPI_RESID, A.data_ptr(), W.data_ptr(), C.data_ptr(), R.data_ptr(), M, N, K, K, K, N, stream()))
    torch.cuda.synchronize()
    assert rel_err(host(C), r + O.linear_fwd(a, w)) < TOL[dtype]


@pytest.mark.parametrize("dtype,M,N,K", [
    (BF16, 520, 776, 333),        # K (tokens) need not be a multiple of anything
    (BF16, 2824, 3080, 200),
    (BF16, 2824, 3080, 64),       # direct path (whole 64-token k-tiles, 156 tiles): 1, 2, 5, 7 and 11 k-tiles
    (BF16, 2824, 3080, 128),
    (BF16, 2824, 3080, 320),
    (BF16, 2824, 3080, 448),
    (BF16, 2824, 3080, 704),
    (BF16, 8, 16, 1),
    (FP32, 130, 76, 50),
])
def test_gemm_tn_accumulate(dtype, M, N, K):
    # dW[M,N] += dY^T X with dY [K,M], X [K,N]
    dy = q(RNG.standard_normal((K, M)), dtype)
    x = q(RNG.standard_normal((K, N)), dtype)
    c0 = RNG.standard_normal((M, N)).astype(np.float32)
    DY, X = dev(dy, dtype), dev(x, dtype)
    C = torch.from_numpy(c0.copy()).cuda()
    for rep in range(2):
        ok(lib().optstage_op_gemm(dtype, B.GEMM_TN, B.EPI_ACCUM, DY.data_ptr(), X.data_ptr(), C.data_ptr(), 0, M, N, K, M, N, N, stream()))
    torch.cuda.synchronize()
    ref = c0.astype(np.float64) + 2 * O.linear_bwd_weight(dy, x)
    assert rel_err(host(C), ref) < (1e-5 if dtype == FP32 else 1e-4)    # fp32 accumulators: no bf16 rounding of C


# Products below the 256 x 256 kernels and the edges between the kernels: one k-chunk, one k-tile, K with a tail that is no multiple
# of 64 (NT: 16-byte chunks fetched out of range, TN: any K), tiles of 64 and 128 cut in both directions, 1 to 14 k-tiles
# for the four waves that share a contraction, one tile more and less than a threshold, and the direct kernel with a K tail.
# The absolute bound is the fp32 sum's plus, for bf16 results, one rounding (2^-9 of the value).
@pytest.mark.parametrize("M,N,K", [(1, 4, 8), (63, 60, 64), (64, 64, 72), (65, 68, 200), (130, 516, 448), (127, 64, 896), (320, 1000, 264),
                                   (1160, 2440, 136), (1160, 2304, 520), (2056, 2056, 72), (2824, 3080, 72), (4096, 2048, 8),
                                   # between 256 tiles of 128 and 128 of 256: little work in many cut tiles, whole and cut columns, rows off 128 bytes
                                   (1053, 3664, 128), (2048, 2304, 64), (2056, 2056, 1024), (2056, 2056, 1016), (2056, 2056, 2048),
                                   # 256 and 257 tiles of 64 and the contraction that four waves share from K = 768 on, 480 and 486, 512 and 513
                                   (1024, 1024, 760), (1024, 1024, 768), (64, 16448, 768), (960, 2048, 1024), (1152, 1728, 1024), (1152, 1728, 64),
                                   (2048, 1024, 200), (1216, 1728, 200)])
def test_gemm_tiles_of_every_size_nt(M, N, K):
    a, w, r = (q(RNG.standard_normal(s), BF16) for s in ((M, K), (N, K), (M, N)))
    A, W, R = dev(a, BF16), dev(w, BF16), dev(r, BF16)
    ref, mag = a @ w.T, np.abs(a) @ np.abs(w).T
    for epi, want, start in ((B.EPI_STORE, ref, None), (B.EPI_RESID, ref + r, None), (B.EPI_ACCUM, ref + 3.0, 3.0)):
        C = torch.full((M + 1, N + 4), 7.0 if start is None else start, dtype=torch.bfloat16 if start is None else torch.float32, device="cuda")
        keep = C.clone()
        Rp = torch.full((M + 1, N + 4), 9.0, dtype=torch.bfloat16, device="cuda")
        Rp[:M, :N] = R
        ok(lib().optstage_op_gemm(BF16, B.GEMM_NT, epi, A.data_ptr(), W.data_ptr(), C.data_ptr(), Rp.data_ptr(), M, N, K, K, K, N + 4, stream()))
        torch.cuda.synchronize()
        bound = K * 2.0 ** -24 * (mag + 3.0) + (2.0 ** -8 * np.abs(want) if start is None else 0.0) + 1e-6
        assert np.all(np.abs(host(C)[:M, :N] - want) <= bound), (epi, np.max(np.abs(host(C)[:M, :N] - want) / bound))
        assert torch.equal(C[M:], keep[M:]) and torch.equal(C[:, N:], keep[:, N:])          # nothing past the edges


@pytest.mark.parametrize("M,N,K", [(8, 8, 1), (64, 64, 63), (72, 56, 65), (136, 520, 449), (264, 1000, 130), (1160, 3080, 67), (1800, 2048, 321),
                                   (2056, 2056, 71), (2824, 3080, 129), (1048, 3664, 128), (2048, 2304, 65), (2056, 2056, 255), (2056, 2056, 256), (2048, 1024, 161),
                                   (1216, 1728, 161), (1600, 1792, 160), (1600, 1800, 160)])
def test_gemm_tiles_of_every_size_tn(M, N, K):
    dy, x = q(RNG.standard_normal((K, M)), BF16), q(RNG.standard_normal((K, N)), BF16)
    DY, X = dev(dy, BF16), dev(x, BF16)
    ref, mag = dy.T @ x, np.abs(dy).T @ np.abs(x)
    for epi, want in ((B.EPI_ACCUM, ref + 3.0), (3, ref), (B.EPI_STORE, ref)):
        C = torch.full((M + 1, N + 4), 3.0, dtype=torch.bfloat16 if epi == B.EPI_STORE else torch.float32, device="cuda")
        ok(lib().optstage_op_gemm(BF16, B.GEMM_TN, epi, DY.data_ptr(), X.data_ptr(), C.data_ptr(), 0, M, N, K, M, N, N + 4, stream()))
        torch.cuda.synchronize()
        bound = K * 2.0 ** -24 * (mag + 3.0) + (2.0 ** -8 * np.abs(want) if epi == B.EPI_STORE else 0.0) + 1e-6
        assert np.all(np.abs(host(C)[:M, :N] - want) <= bound), (epi, np.max(np.abs(host(C)[:M, :N] - want) / bound))
        assert float((C[M:] - 3.0).abs().max()) == 0.0 and float((C[:, N:] - 3.0).abs().max()) == 0.0


# fp32 products on every tile shape that the least estimated time picks (64 x 64, 64 x 32, 32 x 32, 16 x 32, 16 x 16), both layouts, cut tiles, contractions
# that are no multiple of a step of 16, of four steps, or of the steps a wave keeps in flight, and fewer steps than waves.  Bound: partial
# sums of K rounded products, each rounding 2^-24 of a sum that grows as a random walk: sqrt(K) 2^-24 RMS-relative is never reached.
@pytest.mark.parametrize("M,N,K", [(1000, 1004, 1000), (1023, 1021, 999), (508, 1020, 1040), (510, 1023, 1043), (1020, 252, 132), (1021, 251, 133),
                                   (124, 764, 260), (123, 763, 261), (60, 44, 1028), (61, 43, 1029), (20, 36, 12), (33, 17, 67), (256, 512, 320), (512, 512, 52),
                                   # short contractions of many tiles, some of them in the plain kernel
                                   (1004, 1024, 16), (1004, 1024, 20), (4100, 4096, 32), (4100, 4096, 36), (1761, 1262, 12), (1761, 1262, 13), (1761, 1262, 24), (1761, 1262, 25),
                                   (2052, 4096, 16), (1761, 1263, 16), (4101, 4095, 99)])
def test_gemm_fp32_tile_shapes_and_remainders(M, N, K):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)
    A, Bt = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    ref = A.double() @ Bt.double().t()
    C = torch.full((M, N), float("nan"), device="cuda")
    ok(lib().optstage_op_gemm(FP32, B.GEMM_NT, B.EPI_STORE, A.data_ptr(), Bt.data_ptr(), C.data_ptr(), 0, M, N, K, K, K, N, stream()))
    At, Btt, C2 = A.t().contiguous(), Bt.t().contiguous(), torch.full((M, N), 2.0, device="cuda")
    ok(lib().optstage_op_gemm(FP32, B.GEMM_TN, B.EPI_ACCUM, At.data_ptr(), Btt.data_ptr(), C2.data_ptr(), 0, M, N, K, M, N, N, stream()))
    torch.cuda.synchronize()
    for got in (C.double(), C2.double() - 2.0):
        assert ((got - ref).norm() / ref.norm()).item() < K ** 0.5 * 2.0 ** -24 + 2.0 ** -24


# fp32 products on tiles of 16, 32 and 64, cut in both directions, with 16-byte loads (all extents multiples of 4) and without,
# fewer steps of 16 k than waves and a ragged last step, and leading dimensions past 32-bit offsets (the plain kernel).
# Bound: K + 1 roundings of 2^-24 on sums of magnitudes.
@pytest.mark.parametrize("M,N,K,pad", [(1, 1, 1, 0), (16, 16, 4, 0), (17, 20, 15, 3), (130, 36, 68, 4), (200, 500, 200, 0), (201, 499, 77, 1),
                                       (1000, 1100, 132, 0), (1001, 1023, 67, 2), (8, 8, 16, 1 << 24),
                                       # contractions of a few steps on many tiles, 16-byte rows and others
                                       (2048, 2040, 32, 0), (2048, 2040, 36, 0), (4052, 2048, 76, 0), (4052, 2048, 80, 0), (1760, 1262, 60, 0),
                                       (1760, 1262, 61, 0), (1760, 1262, 64, 0), (1760, 1262, 130, 0), (1760, 1262, 131, 0), (1001, 1023, 20, 0), (1001, 1023, 33, 0),
                                       (301, 499, 16, 0), (301, 499, 17, 0)])
def test_gemm_fp32_tiles_of_every_size(M, N, K, pad):
    nt = q(RNG.standard_normal((M, K)), FP32), q(RNG.standard_normal((N, K)), FP32)
    r = q(RNG.standard_normal((M, N)), FP32)
    ldc = N + min(pad, 5)
    for layout in (B.GEMM_NT, B.GEMM_TN):
        ops, lds = [], []
        for x in nt:
            x = x if layout == B.GEMM_NT else np.ascontiguousarray(x.T)
            t = torch.full((x.shape[0], x.shape[1] + pad), float("nan"), dtype=torch.float32, device="cuda")   # what lies between rows is never used
            t[:, :x.shape[1]] = dev(x, FP32)
            ops.append(t)
            lds.append(t.shape[1])
        ref, mag = nt[0] @ nt[1].T, np.abs(nt[0]) @ np.abs(nt[1]).T
        for epi, add in ((B.EPI_STORE, 0.0), (B.EPI_RESID, r), (B.EPI_ACCUM, 3.0), (3, 0.0)):
            C = torch.full((M + 1, ldc), 3.0, dtype=torch.float32, device="cuda")
            R = torch.full((M + 1, ldc), 9.0, dtype=torch.float32, device="cuda")
            R[:M, :N] = dev(r, FP32)
            ok(lib().optstage_op_gemm(FP32, layout, epi, ops[0].data_ptr(), ops[1].data_ptr(), C.data_ptr(), R.data_ptr(), M, N, K, lds[0], lds[1], ldc, stream()))
            torch.cuda.synchronize()
            bound = (K + 1) * 2.0 ** -24 * (mag + 3.0 + np.abs(r))
            assert np.all(np.abs(host(C)[:M, :N] - (ref + add)) <= bound), (layout, epi)
            assert float((C[M:] - 3.0).abs().max()) == 0.0 and (ldc == N or float((C[:, N:] - 3.0).abs().max()) == 0.0)
        del ops


# Operands that are the leading rows of larger tensors, NaN behind them as far as any prefetch goes: TN contractions whose last step of 16 and
# whose loads ahead lie past the operand (up to 576 rows), NT rows past it, on every tile shape.
@pytest.mark.parametrize("M,N,K", [(1000, 1004, 1001), (508, 1020, 1037), (1020, 252, 133), (124, 764, 259), (60, 44, 1027), (20, 36, 13), (64, 64, 1), (1004, 1000, 17)])
def test_gemm_fp32_reads_nothing_behind_its_operands(M, N, K):
    a, w = q(RNG.standard_normal((K, M)), FP32), q(RNG.standard_normal((K, N)), FP32)
    ref, bound = a.T @ w, (K + 1) * 2.0 ** -24 * (np.abs(a).T @ np.abs(w))
    for layout, x, y in ((B.GEMM_TN, a, w), (B.GEMM_NT, a.T, w.T)):
        ops = []
        for part in (x, y):
            t = torch.full((part.shape[0] + 640, part.shape[1]), float("nan"), dtype=torch.float32, device="cuda")
            t[:part.shape[0]] = dev(part, FP32)
            ops.append(t)
        C = torch.full((M, N), 3.0, dtype=torch.float32, device="cuda")
        ok(lib().optstage_op_gemm(FP32, layout, 3, ops[0].data_ptr(), ops[1].data_ptr(), C.data_ptr(), 0, M, N, K, ops[0].shape[1], ops[1].shape[1], N, stream()))
        torch.cuda.synchronize()
        assert np.all(np.abs(host(C) - ref) <= bound), layout


def test_gemm_with_rows_further_apart_than_a_tile_can_address():
    """Leading dimensions of 2^23 elements: the kernel that stages its tiles through registers."""
    ld, n, k = 1 << 23, 16, 72
    a, w = q(RNG.standard_normal((n, k)), BF16), q(RNG.standard_normal((n, k)), BF16)
    A = torch.zeros(n, ld, dtype=torch.bfloat16, device="cuda")
    A[:, :k] = dev(a, BF16)
    W, C = dev(w, BF16), torch.zeros(n, n, dtype=torch.bfloat16, device="cuda")
    ok(lib().optstage_op_gemm(BF16, B.GEMM_NT, B.EPI_STORE, A.data_ptr(), W.data_ptr(), C.data_ptr(), 0, n, n, k, ld, k, n, stream()))
    torch.cuda.synchronize()
    assert rel_err(host(C), a @ w.T) < TOL[BF16] / 4
    X, D = dev(w[:, :16].copy(), BF16), torch.zeros(k, 16, dtype=torch.float32, device="cuda")     # A as [16 tokens][ld], 72 columns used
    ok(lib().optstage_op_gemm(BF16, B.GEMM_TN, 3, A.data_ptr(), X.data_ptr(), D.data_ptr(), 0, k, 16, n, ld, 16, 16, stream()))
    torch.cuda.synchronize()
    assert rel_err(host(D), a.T @ w[:, :16]) < 1e-5


def test_gemm_grouped_equals_one_by_one_and_the_oracle():
    """The weight-gradient products of a W op in one launch (shapes of the Llama stage's four linears at a
    shorter token count, including a ragged 200-row edge tile): bitwise the same as launching each on its
    own, and within tolerance of dY^T X from the oracle on sampled rows."""
    import ctypes as C
    K = 768
    shapes = [(1024, 2752), (5504, 1024), (1024, 1024), (3072, 1024), (200, 1024)]
    probs = (B.GemmProblem * len(shapes))()
    keep = []
    for i, (M, N) in enumerate(shapes):
        dy = q(RNG.standard_normal((K, M)), BF16)
        x = q(RNG.standard_normal((K, N)), BF16)
        c0 = torch.from_numpy(RNG.standard_normal((M, N)).astype(np.float32)).cuda()
        DY, X = dev(dy, BF16), dev(x, BF16)
        grouped, single = c0.clone(), c0.clone()
        ok(lib().optstage_op_gemm(BF16, B.GEMM_TN, B.EPI_ACCUM, DY.data_ptr(), X.data_ptr(), single.data_ptr(), 0, M, N, K, M, N, N, stream()))
        probs[i].A, probs[i].B, probs[i].C, probs[i].R = DY.data_ptr(), X.data_ptr(), grouped.data_ptr(), 0
        probs[i].M, probs[i].N, probs[i].lda, probs[i].ldb, probs[i].ldc = M, N, M, N, N
        keep.append((dy, x, c0, DY, X, grouped, single))
    ok(lib().optstage_op_gemm_grouped(B.GEMM_TN, B.EPI_ACCUM, len(shapes), C.cast(probs, C.c_void_p), K, stream()))
    torch.cuda.synchronize()
    for dy, x, c0, DY, X, grouped, single in keep:
        assert torch.equal(grouped, single)
        rows = RNG.choice(dy.shape[1], size=min(16, dy.shape[1]), replace=False)
        ref = host(c0)[rows] + dy[:, rows].T.astype(np.float64) @ x.astype(np.float64)
        assert rel_err(host(grouped)[rows], ref) < 1e-4
    # a set that does not qualify (K not a multiple of 64) is refused and nothing runs
    assert lib().optstage_op_gemm_grouped(B.GEMM_TN, B.EPI_ACCUM, len(shapes), C.cast(probs, C.c_void_p), 72, stream()) == B.E_ARG


@pytest.mark.parametrize("shapes,K,left", [([(4096, 4200)], 64, 16), ([(4096, 4096), (1024, 1032)], 128, 20),
                                           ([(2048, 8192), (512, 1000), (8192, 264)], 64, 72),     # too many to cut
                                           ([(4096, 3840), (512, 4872)], 64, 24),                  # the cheapest cut is in the second product
                                           ([(4096, 4096), (2048, 1032)], 1024, 40),               # a tail of 656 tiles of 64: on tiles of 128
                                           ([(4096, 4096), (4096, 1024)], 1024, 64),               # the most that is cut
                                           ([(4096, 4096), (1280, 3320)], 1024, 65),               # one more: uncut
                                           ([(4096, 4096), (2048, 1024)], 960, 32),    # the most with a short contraction
                                           ([(4096, 4096), (256, 8400)], 960, 33)])                # one more: uncut
def test_gemm_grouped_with_a_short_last_round(shapes, K, left):
    """Sets of one round of 256 tiles and a few more, whose last columns go to the small kernels: bitwise each product
    on its own, for every epilogue, ragged last column included."""
    import ctypes as C
    assert sum(-(-M // 256) * -(-N // 256) for M, N in shapes) % 256 == left
    for epi, dt in ((B.EPI_ACCUM, torch.float32), (3, torch.float32), (B.EPI_STORE, torch.bfloat16)):
        probs, keep = (B.GemmProblem * len(shapes))(), []
        for i, (M, N) in enumerate(shapes):
            g = torch.Generator(device="cuda")
            g.manual_seed(17 * i + K)
            DY, X = (torch.randn((K, x), generator=g, device="cuda").bfloat16() for x in (M, N))
            grouped = torch.full((M, N + 8), 2.0, dtype=dt, device="cuda")
            single = grouped.clone()
            ok(lib().optstage_op_gemm(BF16, B.GEMM_TN, epi, DY.data_ptr(), X.data_ptr(), single.data_ptr(), 0, M, N, K, M, N, N + 8, stream()))
            probs[i].A, probs[i].B, probs[i].C, probs[i].R = DY.data_ptr(), X.data_ptr(), grouped.data_ptr(), 0
            probs[i].M, probs[i].N, probs[i].lda, probs[i].ldb, probs[i].ldc = M, N, M, N, N + 8
            keep.append((DY, X, grouped, single))
        ok(lib().optstage_op_gemm_grouped(B.GEMM_TN, epi, len(shapes), C.cast(probs, C.c_void_p), K, stream()))
        torch.cuda.synchronize()
        for DY, X, grouped, single in keep:
            assert torch.equal(grouped, single), epi
            rows = [0, 255, grouped.shape[0] - 1]
            ref = host(DY)[:, rows].T @ host(X) + (2.0 if epi == B.EPI_ACCUM else 0.0)
            assert rel_err(host(grouped)[rows, : X.shape[1]], ref) < (TOL[BF16] / 4 if epi == B.EPI_STORE else 1e-5)
            assert float((grouped[:, X.shape[1]:].float() - 2.0).abs().max()) == 0.0


def slabs_of(w):
    """[N, K] -> the slab layout of layout code 2: slab (n // 256, k // 64) holds rows 256 x columns 64, row-major,
    slabs ordered by (n // 256, k // 64); rows padded to a multiple of 256."""
    n, k = w.shape
    n_pad = (n + 255) // 256 * 256
    wp = np.zeros((n_pad, k), dtype=w.dtype)
    wp[:n] = w
    return np.ascontiguousarray(wp.reshape(n_pad // 256, 256, k // 64, 64).transpose(0, 2, 1, 3))


@pytest.mark.parametrize("M,N,K,epi", [(2816, 3072, 192, B.EPI_STORE), (2817, 3000, 256, B.EPI_RESID), (4096, 2048, 64, B.EPI_STORE)])
def test_gemm_with_b_in_slabs(M, N, K, epi):
    """The layout the stage keeps its weight copies in: bitwise the row-major product, and the oracle's on
    sampled rows (ragged edges in both directions)."""
    a = q(RNG.standard_normal((M, K)), BF16)
    w = q(RNG.standard_normal((N, K)), BF16)
    r = q(RNG.standard_normal((M, N)), BF16)
    A, W, WS, R = dev(a, BF16), dev(w, BF16), dev(slabs_of(w), BF16), dev(r, BF16)
    rp = R.data_ptr() if epi == B.EPI_RESID else 0
    C0 = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    C1 = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    ok(lib().optstage_op_gemm(BF16, B.GEMM_NT, epi, A.data_ptr(), W.data_ptr(), C0.data_ptr(), rp, M, N, K, K, K, N, stream()))
    ok(lib().optstage_op_gemm(BF16, B.GEMM_NT_SLAB, epi, A.data_ptr(), WS.data_ptr(), C1.data_ptr(), rp, M, N, K, K, 0, N, stream()))
    torch.cuda.synchronize()
    assert torch.equal(C0, C1)
    rows = RNG.choice(M, size=24, replace=False)
    ref = a[rows].astype(np.float64) @ w.astype(np.float64).T + (r[rows] if epi == B.EPI_RESID else 0.0)
    assert rel_err(host(C1)[rows], ref) < TOL[BF16]
    # too few tiles for the kernel that reads slabs, a contraction that is not whole slabs, fp32: refused
    f = lib().optstage_op_gemm
    assert f(BF16, B.GEMM_NT_SLAB, epi, A.data_ptr(), WS.data_ptr(), C1.data_ptr(), rp, 512, 512, K, K, 0, N, stream()) == B.E_ARG
    assert f(BF16, B.GEMM_NT_SLAB, epi, A.data_ptr(), WS.data_ptr(), C1.data_ptr(), rp, M, N, K - 8, K, 0, N, stream()) == B.E_ARG
    assert f(FP32, B.GEMM_NT_SLAB, epi, A.data_ptr(), WS.data_ptr(), C1.data_ptr(), rp, M, N, K, K, 0, N, stream()) == B.E_ARG
    assert f(BF16, B.GEMM_NT_SLAB, B.EPI_ACCUM, A.data_ptr(), WS.data_ptr(), C1.data_ptr(), 0, M, N, K, K, 0, N, stream()) == B.E_ARG


@pytest.mark.parametrize("N,K", [(512, 128), (300, 64), (1000, 448)])
def test_weight_slabs_match_the_host_layout(N, K):
    w = q(RNG.standard_normal((N, K)), BF16)
    want = torch.from_numpy(slabs_of(w).astype(np.float32)).bfloat16().reshape(-1)
    n_pad = (N + 255) // 256 * 256
    for transposed, src in ((0, w), (1, np.ascontiguousarray(w.T))):
        S = dev(src, BF16)
        D = torch.full((n_pad * K,), 3.0, dtype=torch.bfloat16, device="cuda")
        ok(lib().optstage_op_weight_slabs(S.data_ptr(), D.data_ptr(), N, K, transposed, stream()))
        torch.cuda.synchronize()
        assert torch.equal(D.cpu(), want), transposed
    assert lib().optstage_op_weight_slabs(S.data_ptr(), D.data_ptr(), N, K + 8, 0, stream()) == B.E_ARG


@pytest.mark.parametrize("N,K,shift", [(256, 64, 0), (264, 128, 0), (256, 64, 1), (264, 128, 1)])
def test_weight_slabs_with_and_without_16_byte_rows(N, K, shift):
    """All three codes, from sources that start on 16 bytes and from ones that do not (shift, in elements)."""
    w = q(RNG.standard_normal((N, K)), BF16)
    n_pad = (N + 255) // 256 * 256
    f = N // 2
    rows = [qq * f + 128 * t + 64 * half + o for t in range(N // 256) for half in range(2) for qq in range(2) for o in range(64)]
    cases = [(0, w, slabs_of(w)), (1, np.ascontiguousarray(w.T), slabs_of(w))] + ([(2, w, slabs_of(w[rows]))] if N % 256 == 0 else [])
    for code, src, want in cases:
        S = torch.zeros(src.size + 8, dtype=torch.bfloat16, device="cuda")
        S[shift:shift + src.size] = dev(src, BF16).reshape(-1)
        D = torch.full((n_pad * K + 8,), 3.0, dtype=torch.bfloat16, device="cuda")
        ok(lib().optstage_op_weight_slabs(S[shift:].data_ptr(), D.data_ptr(), N, K, code, stream()))
        torch.cuda.synchronize()
        assert torch.equal(D[: n_pad * K].cpu(), torch.from_numpy(want.astype(np.float32)).bfloat16().reshape(-1)), code
        assert float((D[n_pad * K:] - 3.0).abs().max()) == 0.0


def test_gemm_rejects_bad_shapes():
    A = torch.zeros(64, 64, dtype=torch.bfloat16, device="cuda")
    f = lib().optstage_op_gemm
    assert f(BF16, 0, 0, A.data_ptr(), A.data_ptr(), A.data_ptr(), 0, 64, 64, 60, 60, 60, 64, stream()) == B.E_ARG   # K % 8
    assert f(BF16, 0, 0, A.data_ptr(), A.data_ptr(), A.data_ptr(), 0, 64, 62, 64, 64, 64, 62, stream()) == B.E_ARG   # N % 4
    assert f(BF16, 0, 0, 0, A.data_ptr(), A.data_ptr(), 0, 64, 64, 64, 64, 64, 64, stream()) == B.E_ARG              # null
    assert f(BF16, 0, 1, A.data_ptr(), A.data_ptr(), A.data_ptr(), 0, 64, 64, 64, 64, 64, 64, stream()) == B.E_ARG   # residual missing
    assert f(BF16, 0, 0, A.data_ptr(), A.data_ptr(), A.data_ptr(), 0, 64, 64, 64, 32, 64, 64, stream()) == B.E_ARG   # lda < K
    assert f(BF16, 1, 2, A.data_ptr(), A.data_ptr(), A.data_ptr(), 0, 60, 64, 64, 64, 64, 64, stream()) == B.E_ARG   # TN: M % 8
    torch.cuda.synchronize()


# ------------------------------------------------------------------ norms
@pytest.mark.parametrize("dtype,family,rows,h", [
    (BF16, O.LLAMA, 300, 4096), (BF16, O.LLAMA, 37, 520), (BF16, O.GPT, 64, 1024), (BF16, O.LLAMA, 700, 8192),
    (FP32, O.GPT, 128, 256), (FP32, O.LLAMA, 130, 1000), (BF16, O.GPT, 2100, 2048), (FP32, O.GPT, 8200, 256), (BF16, O.LLAMA, 2500, 1024),
])
def test_norm_fwd_bwd(dtype, family, rows, h):
    eps = 1e-5
    x = q(2.0 * RNG.standard_normal((rows, h)) + 0.3, dtype)
    g = q(1 + 0.1 * RNG.standard_normal(h), dtype)
    b = q(0.1 * RNG.standard_normal(h), dtype)
    dn = q(RNG.standard_normal((rows, h)), dtype)
    dres = q(RNG.standard_normal((rows, h)), dtype)
    X, G, Bt, DN, DR = (dev(a, dtype) for a in (x, g, b, dn, dres))
    OUT = torch.empty_like(X)
    nst = 1 if family == O.LLAMA else 2
    ST = torch.empty(rows * nst, dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_norm_fwd(dtype, family, X.data_ptr(), G.data_ptr(), Bt.data_ptr(), OUT.data_ptr(), ST.data_ptr(), rows, h, eps, stream()))
    DX = torch.empty_like(X)
    part = torch.empty(2 * min(rows, 512) * h, dtype=torch.float32, device="cuda")
    dg0 = RNG.standard_normal(h).astype(np.float32)
    DG, DB = torch.from_numpy(dg0.copy()).cuda(), torch.zeros(h, dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_norm_bwd(dtype, family, DN.data_ptr(), X.data_ptr(), ST.data_ptr(), G.data_ptr(), DR.data_ptr(), DX.data_ptr(), part.data_ptr(), DG.data_ptr(), DB.data_ptr(), rows, h, stream()))
    torch.cuda.synchronize()
    if family == O.LLAMA:
        n, r = O.rmsnorm_fwd(x, g, eps)
        dx, dgam = O.rmsnorm_bwd(dn, x, r, g)
        assert rel_err(host(ST), r[:, 0]) < 1e-5
    else:
        n, mu, r = O.layernorm_fwd(x, g, b, eps)
        dx, dgam, dbeta = O.layernorm_bwd(dn, x, mu, r, g)
        st = host(ST).reshape(rows, 2)
        assert rel_err(st[:, 0], mu[:, 0]) < 1e-5 and rel_err(st[:, 1], r[:, 0]) < 1e-5
        assert rel_err(host(DB), dbeta) < 1e-5
    assert rel_err(host(OUT), n) < TOL[dtype]
    assert rel_err(host(DX), dres + dx) < TOL[dtype]
    assert rel_err(host(DG), dg0 + dgam) < 1e-5      # fp32 accumulation of exactly representable inputs


# ------------------------------------------------------------------ activations
@pytest.mark.parametrize("dtype,family,rows,f", [(BF16, O.LLAMA, 333, 1376), (BF16, O.GPT, 50, 1024),
                                                  (FP32, O.GPT, 128, 1024), (FP32, O.LLAMA, 17, 100)])
def test_activation_fwd_bwd(dtype, family, rows, f):
    w = 2 * f if family == O.LLAMA else f
    gu = q(1.5 * RNG.standard_normal((rows, w)), dtype)
    da = q(RNG.standard_normal((rows, f)), dtype)
    GU, DA = dev(gu, dtype), dev(da, dtype)
    A = torch.empty(rows, f, dtype=GU.dtype, device="cuda")
    ok(lib().optstage_op_act_fwd(dtype, family, GU.data_ptr(), A.data_ptr(), rows, f, stream()))
    ok(lib().optstage_op_act_bwd(dtype, family, DA.data_ptr(), GU.data_ptr(), GU.data_ptr(), rows, f, stream()))   # in place
    torch.cuda.synchronize()
    if family == O.LLAMA:
        a, dgu = O.swiglu_fwd(gu), O.swiglu_bwd(da, gu)
    else:
        a, dgu = O.gelu_fwd(gu), O.gelu_bwd(da, gu)
    assert rel_err(host(A), a) < TOL[dtype]
    assert rel_err(host(GU), dgu) < TOL[dtype]


# ------------------------------------------------------------------ rotary
@pytest.mark.parametrize("dtype,seq,batch,nq,nkv,d", [(BF16, 300, 1, 4, 2, 128), (FP32, 70, 2, 3, 3, 64), (BF16, 4096, 1, 2, 1, 128),
                                                       (BF16, 333, 2, 6, 2, 128), (FP32, 70, 1, 2, 2, 64)])   # q + k heads a multiple of 4
def test_rotary(dtype, seq, batch, nq, nkv, d):
    base = 10000.0
    rows = seq * batch
    w = (nq + 2 * nkv) * d
    qkv = q(RNG.standard_normal((rows, w)), dtype)
    table = torch.empty(seq * d, dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_rope_table(table.data_ptr(), seq, d, base, stream()))
    SRC = dev(qkv, dtype)
    DST = torch.zeros_like(SRC)
    ok(lib().optstage_op_rope(dtype, SRC.data_ptr(), DST.data_ptr(), table.data_ptr(), rows, seq, nq, nkv, d, 1, stream()))   # backward, out of place
    ok(lib().optstage_op_rope(dtype, SRC.data_ptr(), SRC.data_ptr(), table.data_ptr(), rows, seq, nq, nkv, d, 0, stream()))   # forward, in place
    torch.cuda.synchronize()
    # table against fp64
    k = np.arange(d // 2)
    ang = np.arange(seq)[:, None] * base ** (-2.0 * k / d)[None, :]
    tb = host(table).reshape(seq, d // 2, 2)
    assert np.max(np.abs(tb[..., 0] - np.cos(ang))) < 1e-7 and np.max(np.abs(tb[..., 1] - np.sin(ang))) < 1e-7

    def ref(sign):
        out = qkv.copy().reshape(batch, seq, w)
        for b in range(batch):
            qq = out[b, :, : nq * d].reshape(seq, nq, d)
            kk = out[b, :, nq * d: (nq + nkv) * d].reshape(seq, nkv, d)
            out[b, :, : nq * d] = O.rope_apply(qq, base, sign).reshape(seq, -1)
            out[b, :, nq * d: (nq + nkv) * d] = O.rope_apply(kk, base, sign).reshape(seq, -1)
        return out.reshape(rows, w)
    assert rel_err(host(SRC), ref(1.0)) < TOL[dtype]
    assert rel_err(host(DST), ref(-1.0)) < TOL[dtype]


# ------------------------------------------------------------------ attention
@pytest.mark.parametrize("dtype,seq,batch,nq,nkv,d", [
    (FP32, 128, 1, 4, 4, 64), (FP32, 67, 2, 4, 2, 64), (BF16, 200, 1, 4, 2, 128), (BF16, 130, 1, 2, 2, 64),
    (BF16, 512, 1, 8, 2, 128), (BF16, 1, 1, 2, 1, 128), (BF16, 384, 2, 2, 2, 128), (BF16, 1000, 1, 4, 1, 128),
    (BF16, 65, 1, 1, 1, 128), (BF16, 129, 3, 2, 2, 128),
    # heads of 64, short sequences (the general kernels): both sides of each limit
    (BF16, 4, 3, 4, 2, 64), (BF16, 4, 64, 4, 2, 64), (BF16, 5, 64, 4, 2, 64), (BF16, 8, 2, 2, 2, 64), (BF16, 9, 2, 2, 2, 64),
    (BF16, 8, 1, 2, 1, 64), (BF16, 9, 1, 2, 1, 64),
])
def test_attention_fwd_bwd(dtype, seq, batch, nq, nkv, d):
    rows = seq * batch
    w = (nq + 2 * nkv) * d
    qkv = q(RNG.standard_normal((rows, w)), dtype)
    do = q(RNG.standard_normal((rows, nq * d)), dtype)
    QKV, DO = dev(qkv, dtype), dev(do, dtype)
    Ot = torch.empty(rows, nq * d, dtype=QKV.dtype, device="cuda")
    LSE = torch.empty(batch * nq * seq, dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_attn_fwd(dtype, QKV.data_ptr(), Ot.data_ptr(), LSE.data_ptr(), seq, batch, nq, nkv, d, stream()))
    DQKV = torch.zeros_like(QKV)
    nws = lib().optstage_op_attn_bwd_ws_floats(seq, batch, nq, nkv, d)
    WS = torch.empty(max(1, nws), dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_attn_bwd(dtype, QKV.data_ptr(), Ot.data_ptr(), DO.data_ptr(), LSE.data_ptr(), DQKV.data_ptr(), WS.data_ptr(), seq, batch, nq, nkv, d, stream()))
    torch.cuda.synchronize()
    o_g, lse_g, dq_g = host(Ot), host(LSE).reshape(batch, nq, seq), host(DQKV)
    for b in range(batch):
        sl = slice(b * seq, (b + 1) * seq)
        qq = qkv[sl, : nq * d].reshape(seq, nq, d)
        kk = qkv[sl, nq * d: (nq + nkv) * d].reshape(seq, nkv, d)
        vv = qkv[sl, (nq + nkv) * d:].reshape(seq, nkv, d)
        o, lse = O.attention_fwd(qq, kk, vv)
        assert rel_err(o_g[sl], o.reshape(seq, -1)) < TOL[dtype]
        assert np.max(np.abs(lse_g[b] - lse)) < (1e-4 if dtype == FP32 else 2e-2)
        # backward is fed the GPU's own (stored-precision) o, as in the stage
        dq, dk, dv = O.attention_bwd(qq, kk, vv, o_g[sl].reshape(seq, nq, d), do[sl].reshape(seq, nq, d))
        ref = np.concatenate([dq.reshape(seq, -1), dk.reshape(seq, -1), dv.reshape(seq, -1)], axis=1)
        for lo, hi in ((0, nq * d), (nq * d, (nq + nkv) * d), ((nq + nkv) * d, w)):
            assert rel_err(dq_g[sl, lo:hi], ref[:, lo:hi]) < TOL[dtype], (lo, hi)


# Heads of 128 from a workgroup or two to several per compute unit: ragged ends, grouped heads (partials of several workgroups per kv
# head), several sequences.
@pytest.mark.parametrize("seq,batch,nq,nkv", [(127, 1, 2, 2), (129, 2, 4, 1), (257, 1, 256, 256), (257, 1, 64, 8), (33, 5, 64, 64), (257, 3, 128, 128)])
def test_attention_of_few_and_of_many_workgroups(seq, batch, nq, nkv):
    d, rows, w = 128, seq * batch, (nq + 2 * nkv) * 128
    g = torch.Generator(device="cuda")
    g.manual_seed(seq)
    QKV = torch.randn((rows, w), generator=g, device="cuda").bfloat16()
    DO = torch.randn((rows, nq * d), generator=g, device="cuda").bfloat16()
    Ot, DQKV = torch.empty_like(DO), torch.full_like(QKV, float("nan"))
    LSE = torch.empty(batch * nq * seq, dtype=torch.float32, device="cuda")
    WS = torch.empty(lib().optstage_op_attn_bwd_ws_floats(seq, batch, nq, nkv, d), dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_attn_fwd(BF16, QKV.data_ptr(), Ot.data_ptr(), LSE.data_ptr(), seq, batch, nq, nkv, d, stream()))
    ok(lib().optstage_op_attn_bwd(BF16, QKV.data_ptr(), Ot.data_ptr(), DO.data_ptr(), LSE.data_ptr(), DQKV.data_ptr(), WS.data_ptr(), seq, batch, nq, nkv, d, stream()))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(DQKV).all()) and bool(torch.isfinite(Ot).all())
    qkv, o_g, do, dq_g = host(QKV), host(Ot), host(DO), host(DQKV)
    rep = nq // nkv
    for b, kvh in ((0, 0), (batch - 1, nkv - 1)):          # a whole group of the first and of the last sequence
        sl, hs = slice(b * seq, (b + 1) * seq), slice(kvh * rep * d, (kvh + 1) * rep * d)
        ks, vs = (slice((nq + x * nkv + kvh) * d, (nq + x * nkv + kvh + 1) * d) for x in (0, 1))
        qq, kk, vv = qkv[sl, hs].reshape(seq, rep, d), qkv[sl, ks].reshape(seq, 1, d), qkv[sl, vs].reshape(seq, 1, d)
        o, _ = O.attention_fwd(qq, kk, vv)
        assert rms_err(o_g[sl, hs], o.reshape(seq, -1)) < TOL[BF16] / 4
        dq, dk, dv = O.attention_bwd(qq, kk, vv, o_g[sl, hs].reshape(seq, rep, d), do[sl, hs].reshape(seq, rep, d))
        for got, ref in ((dq_g[sl, hs], dq), (dq_g[sl, ks], dk), (dq_g[sl, vs], dv)):
            assert rms_err(got, ref.reshape(seq, -1)) < TOL[BF16] / 4


# Every division of the rows among workgroups and waves (two, four or eight waves, one or two groups that share a block of keys or queries) on
# both sides of the lines between them, ragged ends and grouped heads, and scores whose largest key lies in either half of a block,
# so that each group's softmax reference is the higher one for some rows.  Bounds: rounding of the results and of the probabilities
# (heads of 128) to 8 bits, as in the tests above.
@pytest.mark.parametrize("seq,batch,nq,nkv,d", [
    (91, 1, 3, 1, 128), (129, 1, 2, 1, 128), (193, 1, 2, 2, 128), (449, 1, 8, 2, 128), (321, 3, 32, 16, 128), (705, 3, 16, 16, 128),
    (1601, 1, 36, 36, 128), (1601, 1, 36, 12, 128), (2561, 1, 16, 8, 128), (577, 1, 104, 52, 128), (257, 4, 64, 64, 128), (385, 1, 256, 128, 128),
    (63, 1, 2, 2, 64), (129, 1, 4, 1, 64), (391, 2, 8, 8, 64), (705, 3, 16, 16, 64), (300, 1, 128, 32, 64), (129, 2, 256, 256, 64)])
def test_attention_divisions_of_the_rows(seq, batch, nq, nkv, d):
    rows, w, rep = seq * batch, (nq + 2 * nkv) * d, nq // nkv
    g = torch.Generator(device="cuda")
    g.manual_seed(seq)
    QKV = torch.randn((rows, w), generator=g, device="cuda")
    QKV[:, nq * d:(nq + nkv) * d] *= 1.0 + 2.0 * ((torch.arange(rows, device="cuda") // 37) % 3 == 1).float()[:, None]   # keys of unequal weight
    QKV = QKV.bfloat16()
    DO = torch.randn((rows, nq * d), generator=g, device="cuda").bfloat16()
    Ot, DQKV = torch.full_like(DO, float("nan")), torch.full_like(QKV, float("nan"))
    LSE = torch.full((batch, nq, seq), float("nan"), dtype=torch.float32, device="cuda")
    WS = torch.empty(lib().optstage_op_attn_bwd_ws_floats(seq, batch, nq, nkv, d), dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_attn_fwd(BF16, QKV.data_ptr(), Ot.data_ptr(), LSE.data_ptr(), seq, batch, nq, nkv, d, stream()))
    ok(lib().optstage_op_attn_bwd(BF16, QKV.data_ptr(), Ot.data_ptr(), DO.data_ptr(), LSE.data_ptr(), DQKV.data_ptr(), WS.data_ptr(), seq, batch, nq, nkv, d, stream()))
    torch.cuda.synchronize()
    assert all(bool(torch.isfinite(t).all()) for t in (DQKV, Ot, LSE))
    mask = torch.ones((seq, seq), dtype=torch.bool, device="cuda").triu(1)
    rms = lambda got, ref: ((got.double() - ref).norm() / ref.norm()).item()  # noqa: E731
    for b, kvh in ((0, 0), (batch - 1, nkv - 1)):
        sl = slice(b * seq, (b + 1) * seq)
        k, v = (QKV[sl, (nq + x * nkv + kvh) * d:(nq + x * nkv + kvh + 1) * d].double() for x in (0, 1))
        dk, dv = torch.zeros_like(k), torch.zeros_like(v)
        for a in range(kvh * rep, (kvh + 1) * rep):
            cols = slice(a * d, (a + 1) * d)
            q_, do = QKV[sl, cols].double(), DO[sl, cols].double()
            s = ((q_ @ k.t()) / d ** 0.5).masked_fill(mask, float("-inf"))
            p = torch.softmax(s, -1)
            assert (LSE[b, a].double() - torch.logsumexp(s, -1)).abs().max().item() < 2e-5 * max(1.0, s.abs()[~mask].max().item())
            assert rms(Ot[sl, cols], p @ v) < TOL[BF16] / 4
            dp = do @ v.t()
            ds = p * (dp - (do * Ot[sl, cols].double()).sum(-1, keepdim=True)) / d ** 0.5      # the kernels' row term: the stored o
            assert rms(DQKV[sl, cols], ds @ k) < TOL[BF16] / 4
            dk += ds.t() @ q_
            dv += p.t() @ do
        for x, ref in ((0, dk), (1, dv)):
            assert rms(DQKV[sl, (nq + x * nkv + kvh) * d:(nq + x * nkv + kvh + 1) * d], ref) < TOL[BF16] / 4


# Heads of 64: edges of the 32- and 64-wide tiles and of the 256 rows of a workgroup, one row, grouped heads, several sequences,
# peaked and flat scores, and operands that are not 16-byte aligned (shift, in elements: the general kernels).  The second
# products multiply probabilities of 16 significant bits (two bf16 numbers; the general kernels 24), so what is left is the
# rounding of the results to 8 bits: an error spread evenly over +- 2^-8 of the power of two below a value, at most 2^-8 / sqrt(3) RMS-relative, and all but
# the values within about 2^-16 of a tie, 2^-7 of them and a few more where a sum cancels, equal the correctly rounded
# ones (below 6 %; probabilities of 8 bits miss a third).
@pytest.mark.parametrize("seq,batch,nq,nkv,gain,shift", [(1, 2, 2, 1, 1.0, 0), (31, 1, 2, 2, 1.0, 0), (33, 1, 1, 1, 1.0, 0), (64, 2, 2, 1, 1.0, 0),
                                                         (65, 1, 4, 1, 1.0, 0), (255, 1, 2, 2, 1.0, 0), (257, 2, 2, 1, 1.0, 0), (700, 1, 8, 2, 4.0, 0),
                                                         (600, 1, 2, 2, 0.05, 0), (130, 1, 2, 1, 1.0, 1)])
def test_attention_of_64_wide_heads_rounds_only_its_results(seq, batch, nq, nkv, gain, shift):
    d, rows, w = 64, seq * batch, (nq + 2 * nkv) * 64
    qkv = RNG.standard_normal((rows, w))
    qkv[:, : (nq + nkv) * d] *= gain
    qkv, do = q(qkv, BF16), q(RNG.standard_normal((rows, nq * d)), BF16)

    def place(a):
        flat = torch.zeros(a.size + 8, dtype=torch.bfloat16, device="cuda")
        flat[shift:shift + a.size] = dev(a, BF16).reshape(-1)
        return flat[shift:shift + a.size].view(a.shape)
    QKV, DO, Ot, DQKV = place(qkv), place(do), place(np.zeros((rows, nq * d))), place(np.zeros((rows, w)))
    LSE = torch.empty(batch * nq * seq, dtype=torch.float32, device="cuda")
    WS = torch.empty(lib().optstage_op_attn_bwd_ws_floats(seq, batch, nq, nkv, d), dtype=torch.float32, device="cuda")
    assert WS.numel() == batch * nq * seq
    ok(lib().optstage_op_attn_fwd(BF16, QKV.data_ptr(), Ot.data_ptr(), LSE.data_ptr(), seq, batch, nq, nkv, d, stream()))
    ok(lib().optstage_op_attn_bwd(BF16, QKV.data_ptr(), Ot.data_ptr(), DO.data_ptr(), LSE.data_ptr(), DQKV.data_ptr(), WS.data_ptr(), seq, batch, nq, nkv, d, stream()))
    torch.cuda.synchronize()
    o_g, lse_g, dq_g = host(Ot), host(LSE).reshape(batch, nq, seq), host(DQKV)
    refs = []
    for b in range(batch):
        sl = slice(b * seq, (b + 1) * seq)
        qq, kk, vv = (x.reshape(seq, -1, d) for x in (qkv[sl, : nq * d], qkv[sl, nq * d: (nq + nkv) * d], qkv[sl, (nq + nkv) * d:]))
        o, lse = O.attention_fwd(qq, kk, vv)
        assert np.max(np.abs(lse_g[b] - lse) / np.maximum(1.0, np.abs(lse))) < 1e-5
        dq, dk, dv = O.attention_bwd(qq, kk, vv, o_g[sl].reshape(seq, nq, d), do[sl].reshape(seq, nq, d))
        refs.append((o.reshape(seq, -1), np.concatenate([x.reshape(seq, -1) for x in (dq, dk, dv)], axis=1)))
    ref_o, ref_d = (np.concatenate(x) for x in zip(*refs))
    for got, ref in ((o_g, ref_o), *((dq_g[:, lo:hi], ref_d[:, lo:hi]) for lo, hi in ((0, nq * d), (nq * d, (nq + nkv) * d), ((nq + nkv) * d, w)))):
        assert np.isfinite(got).all()
        if np.sqrt(np.mean(ref ** 2)) < 1e-3:      # a single row: its scores have no gradient, dQ and dK are what the rounding of O leaves
            continue
        assert rms_err(got, ref) < 1.05 * 2.0 ** -8 / np.sqrt(3.0)
        # scores of order one only: at gain 4 they reach +- 60, whose fp32 rounding is 2^-18 of a probability, and dP - D cancels
        # to the rounding of dP in most elements
        assert gain > 1.0 or np.mean(got != q(ref, BF16)) < 0.06


# fp32 attention on tiles of 16 rows shared by four waves: one row, a cut tile, more waves than tiles, both head sizes, grouped heads,
# several sequences, peaked scores, and operands that are not 16-byte aligned (shift, in elements: the general kernels).  Bound:
# fp32 sums of up to a few hundred products, 2^-24 each, in softmax and both products; 1e-5 of the largest value.
@pytest.mark.parametrize("seq,batch,nq,nkv,d,gain,shift", [(1, 1, 1, 1, 64, 1.0, 0), (15, 2, 2, 1, 128, 1.0, 0), (16, 1, 2, 2, 64, 1.0, 0),
                                                           (17, 1, 4, 2, 64, 1.0, 0), (100, 2, 4, 1, 128, 1.0, 0), (257, 1, 2, 2, 64, 4.0, 0),
                                                           (200, 1, 3, 3, 128, 0.05, 0), (65, 1, 2, 1, 64, 1.0, 1),
                                                           # short sequences (the general kernels): both sides of each limit
                                                           (4, 65, 2, 2, 64, 1.0, 0), (5, 65, 2, 2, 64, 1.0, 0), (8, 1, 2, 1, 128, 1.0, 0),
                                                           (9, 1, 2, 2, 128, 1.0, 0), (12, 2, 2, 2, 64, 1.0, 0), (13, 2, 2, 2, 64, 1.0, 0)])
def test_attention_fp32(seq, batch, nq, nkv, d, gain, shift):
    rows, w = seq * batch, (nq + 2 * nkv) * d
    qkv = RNG.standard_normal((rows, w))
    qkv[:, : (nq + nkv) * d] *= gain
    qkv, do = q(qkv, FP32), q(RNG.standard_normal((rows, nq * d)), FP32)

    def place(a):
        flat = torch.zeros(a.size + 8, dtype=torch.float32, device="cuda")
        flat[shift:shift + a.size] = dev(a, FP32).reshape(-1)
        return flat[shift:shift + a.size].view(a.shape)
    QKV, DO, Ot, DQKV = place(qkv), place(do), place(np.zeros((rows, nq * d))), place(np.zeros((rows, w)))
    LSE = torch.empty(batch * nq * seq, dtype=torch.float32, device="cuda")
    WS = torch.empty(lib().optstage_op_attn_bwd_ws_floats(seq, batch, nq, nkv, d), dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_attn_fwd(FP32, QKV.data_ptr(), Ot.data_ptr(), LSE.data_ptr(), seq, batch, nq, nkv, d, stream()))
    ok(lib().optstage_op_attn_bwd(FP32, QKV.data_ptr(), Ot.data_ptr(), DO.data_ptr(), LSE.data_ptr(), DQKV.data_ptr(), WS.data_ptr(), seq, batch, nq, nkv, d, stream()))
    torch.cuda.synchronize()
    o_g, lse_g, dq_g = host(Ot), host(LSE).reshape(batch, nq, seq), host(DQKV)
    for b in range(batch):
        sl = slice(b * seq, (b + 1) * seq)
        qq, kk, vv = (x.reshape(seq, -1, d) for x in (qkv[sl, : nq * d], qkv[sl, nq * d: (nq + nkv) * d], qkv[sl, (nq + nkv) * d:]))
        o, lse = O.attention_fwd(qq, kk, vv)
        assert np.max(np.abs(o_g[sl] - o.reshape(seq, -1))) < 1e-5 * np.max(np.abs(o))
        assert np.max(np.abs(lse_g[b] - lse) / np.maximum(1.0, np.abs(lse))) < 1e-5
        dq, dk, dv = O.attention_bwd(qq, kk, vv, o_g[sl].reshape(seq, nq, d), do[sl].reshape(seq, nq, d))
        ref = np.concatenate([x.reshape(seq, -1) for x in (dq, dk, dv)], axis=1)
        assert np.max(np.abs(dq_g[sl] - ref)) < 1e-5 * np.max(np.abs(ref)) * max(1.0, gain * gain)


# lse of 64-wide heads is held to its own rounding: at most 2^-24 / sqrt(3) of the value, RMS, and a third of 2^-24 for the
# exponentials, their sum and its logarithm (scores of order one, whose own rounding does not show).
@pytest.mark.parametrize("seq,batch,nq,nkv", [(700, 2, 4, 2), (1024, 1, 8, 8)])
def test_lse_of_64_wide_heads_is_rounded_once(seq, batch, nq, nkv):
    d, rows = 64, seq * batch
    qkv = q(RNG.standard_normal((rows, (nq + 2 * nkv) * d)), BF16)
    QKV = dev(qkv, BF16)
    Ot = torch.empty(rows, nq * d, dtype=torch.bfloat16, device="cuda")
    LSE = torch.empty(batch * nq * seq, dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_attn_fwd(BF16, QKV.data_ptr(), Ot.data_ptr(), LSE.data_ptr(), seq, batch, nq, nkv, d, stream()))
    torch.cuda.synchronize()
    want = []
    for b in range(batch):
        x = qkv[b * seq:(b + 1) * seq]
        want.append(O.attention_fwd(*(v.reshape(seq, -1, d) for v in (x[:, : nq * d], x[:, nq * d: (nq + nkv) * d], x[:, (nq + nkv) * d:])))[1])
    assert rms_err(host(LSE).reshape(batch, nq, seq), np.stack(want)) < 2.0 ** -24 * np.sqrt(1 / 3 + 1 / 9)


def attention_by_rows(qkv, do, seq, nq, nkv, d):
    """fp64 attention of one sequence in which a row multiplies the keys up to its own and nothing else, so that a value that is
    not finite reaches exactly the rows that depend on it: o, lse, dqkv, and dqkv from the o that is passed."""
    qkv, do = torch.from_numpy(qkv), torch.from_numpy(do)
    head = lambda i: qkv[:, i * d:(i + 1) * d]  # noqa: E731
    o, lse, dqkv = torch.zeros(seq, nq * d, dtype=torch.float64), torch.zeros(nq, seq, dtype=torch.float64), torch.zeros_like(qkv)
    for a in range(nq):
        g = a * nkv // nq
        Q, K, V, dO = head(a), head(nq + g), head(nq + nkv + g), do[:, a * d:(a + 1) * d]
        dk, dv = (dqkv[:, (nq + x * nkv + g) * d:(nq + x * nkv + g + 1) * d] for x in (0, 1))
        for t in range(seq):
            s = (K[:t + 1] * Q[t]).sum(1) / np.sqrt(d)
            m = s[~s.isnan()].max() if bool((~s.isnan()).any()) else s.max()
            e = torch.exp(s - m)
            p = e / e.sum()
            row = (p[:, None] * V[:t + 1]).sum(0)
            o[t, a * d:(a + 1) * d], lse[a, t] = row, m + torch.log(e.sum())
            ds = p * ((V[:t + 1] * dO[t]).sum(1) - (row * dO[t]).sum()) / np.sqrt(d)
            dqkv[t, a * d:(a + 1) * d] = (ds[:, None] * K[:t + 1]).sum(0)
            dk[:t + 1] += ds[:, None] * Q[t]
            dv[:t + 1] += p[:, None] * dO[t]
    return o.numpy(), lse.numpy(), dqkv.numpy()


# A value that is not finite stays with the rows that depend on it: a later token's with the later rows (forward, dQ), an earlier
# one's with the earlier keys (dK, dV).  The poisoned token sits inside a tile of 16 and of 32 rows, and at the end of a cut
# one, whose last row stands in for the rows past it; 300 tokens are divided over two groups of waves (bf16), of which either may have
# it.  Infinity and NaN themselves only have to be where the reference has either.
@pytest.mark.parametrize("dtype,d,seq", [(BF16, 64, 75), (BF16, 64, 300), (FP32, 64, 75), (FP32, 128, 75)])
@pytest.mark.parametrize("what", ["q", "k", "v", "do"])
def test_attention_keeps_what_is_not_finite_to_the_rows_that_depend_on_it(dtype, d, seq, what):
    nq, nkv = 2, 1
    w, tol = (nq + 2 * nkv) * d, {BF16: 2.0 ** -7, FP32: 1e-5}[dtype]
    clean, do0 = q(RNG.standard_normal((seq, w)), dtype), q(RNG.standard_normal((seq, nq * d)), dtype)
    for row, value in ((36, np.inf), (36, np.nan), (seq - 1, np.inf), (seq // 2 - 5, np.inf)):
        qkv, do = clean.copy(), do0.copy()
        if what == "do":
            do[row, 5] = value
        else:
            qkv[row, {"q": 0, "k": nq * d, "v": (nq + nkv) * d}[what] + 5] = value
        QKV, DO = dev(qkv, dtype), dev(do, dtype)
        Ot, DQKV = torch.zeros_like(DO), torch.zeros_like(QKV)
        LSE = torch.zeros(nq * seq, dtype=torch.float32, device="cuda")
        WS = torch.empty(lib().optstage_op_attn_bwd_ws_floats(seq, 1, nq, nkv, d), dtype=torch.float32, device="cuda")
        ok(lib().optstage_op_attn_fwd(dtype, QKV.data_ptr(), Ot.data_ptr(), LSE.data_ptr(), seq, 1, nq, nkv, d, stream()))
        ok(lib().optstage_op_attn_bwd(dtype, QKV.data_ptr(), Ot.data_ptr(), DO.data_ptr(), LSE.data_ptr(), DQKV.data_ptr(), WS.data_ptr(), seq, 1, nq, nkv, d, stream()))
        torch.cuda.synchronize()
        for got, want in zip((host(Ot), host(LSE).reshape(nq, seq), host(DQKV)), attention_by_rows(qkv, do, seq, nq, nkv, d)):
            fine = np.isfinite(want)
            assert np.array_equal(np.isfinite(got), fine), (what, row, value)
            assert np.max(np.abs(got[fine] - want[fine])) <= tol * np.max(np.abs(want[fine])), (what, row, value)


@pytest.mark.parametrize("which", ["qkv", "o", "do", "dqkv"])
def test_attention_of_128_wide_heads_off_16_bytes(which):
    """An operand that does not start on 16 bytes takes the general kernels: 16-byte accesses would not be aligned."""
    seq, nq, nkv, d = 130, 2, 1, 128
    w = (nq + 2 * nkv) * d
    qkv, do = q(RNG.standard_normal((seq, w)), BF16), q(RNG.standard_normal((seq, nq * d)), BF16)

    def place(a, name):
        flat = torch.zeros(a.size + 8, dtype=torch.bfloat16, device="cuda")
        at = 1 if name == which else 0
        flat[at:at + a.size] = dev(a, BF16).reshape(-1)
        return flat[at:at + a.size].view(a.shape)
    QKV, DO, Ot, DQKV = place(qkv, "qkv"), place(do, "do"), place(0 * do, "o"), place(0 * qkv, "dqkv")
    LSE = torch.empty(nq * seq, dtype=torch.float32, device="cuda")
    WS = torch.empty(lib().optstage_op_attn_bwd_ws_floats(seq, 1, nq, nkv, d), dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_attn_fwd(BF16, QKV.data_ptr(), Ot.data_ptr(), LSE.data_ptr(), seq, 1, nq, nkv, d, stream()))
    ok(lib().optstage_op_attn_bwd(BF16, QKV.data_ptr(), Ot.data_ptr(), DO.data_ptr(), LSE.data_ptr(), DQKV.data_ptr(), WS.data_ptr(), seq, 1, nq, nkv, d, stream()))
    torch.cuda.synchronize()
    qq, kk, vv = (x.reshape(seq, -1, d) for x in (qkv[:, : nq * d], qkv[:, nq * d: (nq + nkv) * d], qkv[:, (nq + nkv) * d:]))
    o, lse = O.attention_fwd(qq, kk, vv)
    assert rms_err(host(Ot), o.reshape(seq, -1)) < TOL[BF16] / 4 and np.max(np.abs(host(LSE).reshape(nq, seq) - lse)) < 1e-4
    ref = O.attention_bwd(qq, kk, vv, host(Ot).reshape(seq, nq, d), do.reshape(seq, nq, d))
    assert rms_err(host(DQKV), np.concatenate([x.reshape(seq, -1) for x in ref], axis=1)) < TOL[BF16] / 4


@pytest.mark.parametrize("gain", [6.0, 0.05])
def test_attention_forward_with_peaked_and_flat_scores(gain):
    """Scores far larger than usual (the softmax reference has to be raised again and again, and most
    probabilities underflow) and far smaller (the reference is set once and never raised)."""
    seq, nq, nkv, d = 700, 2, 1, 128
    w = (nq + 2 * nkv) * d
    qkv = RNG.standard_normal((seq, w))
    qkv[:, : (nq + nkv) * d] *= gain
    qkv = q(qkv, BF16)
    QKV = dev(qkv, BF16)
    Ot = torch.empty(seq, nq * d, dtype=QKV.dtype, device="cuda")
    LSE = torch.empty(nq * seq, dtype=torch.float32, device="cuda")
    ok(lib().optstage_op_attn_fwd(BF16, QKV.data_ptr(), Ot.data_ptr(), LSE.data_ptr(), seq, 1, nq, nkv, d, stream()))
    torch.cuda.synchronize()
    qq = qkv[:, : nq * d].reshape(seq, nq, d)
    kk = qkv[:, nq * d: (nq + nkv) * d].reshape(seq, nkv, d)
    vv = qkv[:, (nq + nkv) * d:].reshape(seq, nkv, d)
    o, lse = O.attention_fwd(qq, kk, vv)
    assert np.isfinite(host(Ot)).all() and np.isfinite(host(LSE)).all()
    assert rel_err(host(Ot), o.reshape(seq, -1)) < TOL[BF16]
    assert np.max(np.abs(host(LSE).reshape(nq, seq) - lse) / np.maximum(1.0, np.abs(lse))) < 2e-2


# ------------------------------------------------------------------ checksum
def test_checksum_matches_host_arithmetic():
    for n in (0, 8, 4096, 1 << 20, (1 << 20) + 8):
        a = RNG.integers(0, 2**63, size=max(1, n // 8), dtype=np.uint64)[: n // 8]
        t = torch.from_numpy(a.view(np.int64).copy()).cuda() if n else torch.zeros(1, dtype=torch.int64, device="cuda")
        out = torch.zeros(2, dtype=torch.int64, device="cuda")
        ok(lib().optstage_op_checksum(t.data_ptr(), n, out.data_ptr(), stream()))
        torch.cuda.synchronize()
        got = out.cpu().numpy().view(np.uint64)
        s = int(np.sum(a, dtype=np.uint64)) if n else 0
        x = int(np.bitwise_xor.reduce(a)) if n else 0
        assert int(got[0]) == s and int(got[1]) == x


def test_empty_inputs_are_refused_not_launched():
    """A zero extent anywhere is an argument error of the call (nothing is launched, nothing is written)."""
    L_ = lib()
    a = torch.zeros(4096, dtype=torch.bfloat16, device="cuda")
    f = torch.zeros(4096, dtype=torch.float32, device="cuda")
    p, q = a.data_ptr(), f.data_ptr()
    for M, N, K in ((0, 64, 64), (64, 0, 64), (64, 64, 0)):
        assert L_.optstage_op_gemm(BF16, B.GEMM_NT, B.EPI_STORE, p, p, p, 0, M, N, K, 64, 64, 64, stream()) == B.E_ARG
        assert L_.optstage_op_gemm(BF16, B.GEMM_TN, B.EPI_ACCUM, p, p, q, 0, M, N, K, 64, 64, 64, stream()) == B.E_ARG
    assert L_.optstage_op_norm_fwd(BF16, O.LLAMA, p, p, 0, p, q, 0, 64, 1e-5, stream()) == B.E_ARG
    assert L_.optstage_op_norm_fwd(BF16, O.LLAMA, p, p, 0, p, q, 8, 0, 1e-5, stream()) == B.E_ARG
    assert L_.optstage_op_norm_bwd(BF16, O.LLAMA, p, p, q, p, 0, p, q, q, 0, 0, 64, stream()) == B.E_ARG
    assert L_.optstage_op_act_fwd(BF16, O.LLAMA, p, p, 0, 64, stream()) == B.E_ARG
    assert L_.optstage_op_act_bwd(BF16, O.LLAMA, p, p, p, 8, 0, stream()) == B.E_ARG
    assert L_.optstage_op_rope(BF16, p, p, q, 0, 8, 2, 2, 128, 0, stream()) == B.E_ARG
    assert L_.optstage_op_attn_fwd(BF16, p, p, q, 0, 1, 2, 2, 128, stream()) == B.E_ARG
    assert L_.optstage_op_attn_bwd(BF16, p, p, p, q, q, q, 0, 1, 2, 2, 128, stream()) == B.E_ARG
    assert L_.optstage_op_weight_slabs(p, q, 0, 64, 0, stream()) == B.E_ARG
    torch.cuda.synchronize()
    assert float(a.float().abs().sum()) == 0.0 and float(f.abs().sum()) == 0.0


# ------------------------------------------------------------------ projections with a fused epilogue
@pytest.mark.parametrize("layout,M,N,K,seq,rot", [(B.GEMM_NT, 2000, 4096, 256, 500, 3072), (2, 2048, 4096, 192, 2048, 4096),
                                                  (B.GEMM_NT, 4096, 2048, 128, 1024, 1024)])
def test_gemm_with_rotary_in_the_epilogue(layout, M, N, K, seq, rot):
    d = 128
    a = q(RNG.standard_normal((M, K)), BF16)
    w = q(0.1 * RNG.standard_normal((N, K)), BF16)
    A, W = dev(a, BF16), dev(w, BF16)
    L_ = lib()
    Wop = W
    if layout == 2:
        Wop = torch.empty((N + 255) // 256 * 256 * K, dtype=torch.bfloat16, device="cuda")
        ok(L_.optstage_op_weight_slabs(W.data_ptr(), Wop.data_ptr(), N, K, 0, stream()))
    table = torch.empty(seq * (d // 2) * 2, dtype=torch.float32, device="cuda")
    ok(L_.optstage_op_rope_table(table.data_ptr(), seq, d, 10000.0, stream()))
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ok(L_.optstage_op_gemm_rope(layout, A.data_ptr(), Wop.data_ptr(), C.data_ptr(), M, N, K, K, K, N, table.data_ptr(), seq, rot, stream()))
    # the unfused pair of kernels on the same operands
    C2 = torch.empty_like(C)
    ok(L_.optstage_op_gemm(BF16, B.GEMM_NT, B.EPI_STORE, A.data_ptr(), W.data_ptr(), C2.data_ptr(), 0, M, N, K, K, K, N, stream()))
    packed = (N // d) % 4 == 0 and rot == N // 4 * 3          # a packed qkv row: n_q = 2 n_kv query heads, n_kv key and value heads
    if packed:
        ok(L_.optstage_op_rope(BF16, C2.data_ptr(), C2.data_ptr(), table.data_ptr(), M, seq, N // d // 2, N // d // 4, d, 0, stream()))
    torch.cuda.synchronize()
    ref = a @ w.T
    heads = ref.reshape(M, N // d, d).copy()
    for s0 in range(0, M, seq):
        s1 = min(M, s0 + seq)
        heads[s0:s1, : rot // d] = O.rope_apply(heads[s0:s1, : rot // d], 10000.0)[: s1 - s0]
    ref = heads.reshape(M, N)
    assert rel_err(host(C), ref) < TOL[BF16] / 4 and rms_err(host(C), ref) < TOL[BF16] / 8
    if packed:            # against the two separate kernels: the same numbers up to the one extra rounding those make
        assert rms_err(host(C), host(C2)) < TOL[BF16] / 8
    # a shape the direct kernel does not serve, a head split by a tile, a missing table: refused, nothing written
    Z = torch.zeros(64, 256, dtype=torch.bfloat16, device="cuda")
    assert L_.optstage_op_gemm_rope(0, A.data_ptr(), W.data_ptr(), Z.data_ptr(), 64, 256, K, K, K, 256, table.data_ptr(), seq, 256, stream()) == B.E_ARG
    assert L_.optstage_op_gemm_rope(0, A.data_ptr(), W.data_ptr(), C.data_ptr(), M, N, K, K, K, N, table.data_ptr(), seq, 192, stream()) == B.E_ARG
    assert L_.optstage_op_gemm_rope(0, A.data_ptr(), W.data_ptr(), C.data_ptr(), M, N, K, K, K, N, 0, seq, rot, stream()) == B.E_ARG
    torch.cuda.synchronize()
    assert float(Z.float().abs().sum()) == 0.0


@pytest.mark.parametrize("M,f,K", [(2000, 2048, 192), (4096, 1024, 256), (2048, 2304, 64)])
def test_gate_up_projection_with_the_activation_in_the_epilogue(M, f, K):
    a = q(RNG.standard_normal((M, K)), BF16)
    w = q(0.15 * RNG.standard_normal((2 * f, K)), BF16)
    A, W = dev(a, BF16), dev(w, BF16)
    L_ = lib()
    Wp = torch.empty(2 * f * K, dtype=torch.bfloat16, device="cuda")
    ok(L_.optstage_op_weight_slabs(W.data_ptr(), Wp.data_ptr(), 2 * f, K, 2, stream()))
    GU = torch.full((M, 2 * f), float("nan"), dtype=torch.bfloat16, device="cuda")
    ACT = torch.full((M, f), float("nan"), dtype=torch.bfloat16, device="cuda")
    ok(L_.optstage_op_gemm_swiglu(A.data_ptr(), Wp.data_ptr(), GU.data_ptr(), ACT.data_ptr(), M, f, K, K, stream()))
    torch.cuda.synchronize()
    gu = a @ w.T
    assert rel_err(host(GU), gu) < TOL[BF16] / 4 and rms_err(host(GU), gu) < TOL[BF16] / 8       # plain [gate | up] layout
    act = O.swiglu_fwd(gu)
    assert rel_err(host(ACT), act) < TOL[BF16] / 4 and rms_err(host(ACT), act) < TOL[BF16] / 8
    # the stored gate / up tensor is what the separate projection stores, bit for bit
    GU2 = torch.empty_like(GU)
    ok(L_.optstage_op_gemm(BF16, B.GEMM_NT, B.EPI_STORE, A.data_ptr(), W.data_ptr(), GU2.data_ptr(), 0, M, 2 * f, K, K, K, 2 * f, stream()))
    torch.cuda.synchronize()
    assert torch.equal(GU, GU2)
    assert L_.optstage_op_gemm_swiglu(A.data_ptr(), Wp.data_ptr(), GU.data_ptr(), ACT.data_ptr(), M, f + 64, K, K, stream()) == B.E_ARG
    assert L_.optstage_op_gemm_swiglu(A.data_ptr(), Wp.data_ptr(), GU.data_ptr(), 0, M, f, K, K, stream()) == B.E_ARG
    assert L_.optstage_op_weight_slabs(W.data_ptr(), Wp.data_ptr(), 2 * f - 128, K, 2, stream()) == B.E_ARG
