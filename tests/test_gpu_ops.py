"""Per-kernel parity: each HIP kernel, called through the C boundary, against the CPU
oracle's function for the same operation on the same seeded inputs."""
import ctypes as C
import math

import numpy as np
import pytest

from oracle import ouro_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def L():
    import paper_1909_06695_amd as P
    return P.lib()


def stream():
    return C.c_void_p(torch.cuda.current_stream().cuda_stream)


def dev(a, dtype):
    """numpy -> device tensor of the op's element type (dtype 0 fp32, 1 bf16)."""
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    return t.to(torch.bfloat16).contiguous() if dtype == 1 else t


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


def p(t):
    return None if t is None else C.c_void_p(t.data_ptr())


def rel_err(a, b):
    # the floor keeps exactly-zero references (a single visible key has zero score gradient)
    # from turning rounding noise into an infinite ratio
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-2 * math.sqrt(b.size)))


def ok(rc):
    assert rc == 0, L().ouro_last_error()


TOL = {0: 2e-5, 1: 1e-2}


# ------------------------------------------------------------------------------- GEMM
# force: 0 automatic, 1 plain kernel, 10..16 one MFMA tile configuration each
@pytest.mark.parametrize("dtype,force", [(0, 0), (1, 1), (1, 0), (1, 10), (1, 11), (1, 12), (1, 13), (1, 14), (1, 15), (1, 16)])
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(200, 136, 328), (128, 256, 64), (72, 40, 1000), (384, 520, 96), (136, 264, 512),
                                   (392, 136, 192), (520, 392, 1024)])
def test_gemm_forms(dtype, force, tA, tB, M, N, K):
    rng = np.random.default_rng(M + 7 * N + 13 * K + tA * 2 + tB)
    A = rng.standard_normal((K, M) if tA else (M, K)).astype(np.float32)
    B = rng.standard_normal((N, K) if tB else (K, N)).astype(np.float32)
    dA, dB = dev(A, dtype), dev(B, dtype)
    out = torch.empty((M, N), dtype=torch.float32, device="cuda")
    ok(L().ouro_op_gemm(stream(), dtype, tA, tB, M, N, K, 1.0, p(dA), dA.shape[1], p(dB), dB.shape[1], p(out), N,
                        1, 0, None, None, 0, 0, None, 0, force))
    torch.cuda.synchronize()
    a64, b64 = host(dA), host(dB)
    ref = (a64.T if tA else a64) @ (b64.T if tB else b64)
    assert rel_err(host(out), ref) < 2e-6
    if dtype == 1 and force != 1:
        assert L().ouro_op_gemm_uses_mfma(dtype, tA, tB, M, N, K, p(dA), dA.shape[1], p(dB), dB.shape[1]) == 1


def test_gemm_row_tail():
    """A product on 256x256 tiles whose tile rows end a little past a full round of workgroups:
    the rows of the last partial round come from a second, split-K launch.  Rows on both sides
    of the seam and the last rows against fp64."""
    M, N, K = 16384 + 520, 1024, 4096
    rng = np.random.default_rng(77)
    dA = dev(rng.standard_normal((K, M)).astype(np.float32), 1)
    dB = dev(rng.standard_normal((K, N)).astype(np.float32), 1)
    out = torch.full((M, N), 7.0, dtype=torch.float32, device="cuda")
    ok(L().ouro_op_gemm(stream(), 1, 1, 0, M, N, K, 1.0, p(dA), M, p(dB), N, p(out), N, 1, 0, None, None, 0, 0, None, 0, 0))
    torch.cuda.synchronize()
    rows = np.r_[0:4, 8190:8194, 16376:16392, 16640:16644, M - 9:M]
    a64, b64 = host(dA), host(dB)
    ref = a64[:, rows].T @ b64
    assert rel_err(host(out)[rows], ref) < 2e-6


@pytest.mark.parametrize("dtype,tA,tB,M,N,K,by,bz,second,acc", [
    (1, 0, 0, 200, 64, 128, 3, 2, True, 0),      # one launch of the MFMA kernel over the grid, two grids, ragged M
    (1, 0, 1, 136, 72, 192, 2, 1, False, 0),
    (1, 1, 0, 128, 64, 2048, 3, 1, False, 1),    # split K with atomic adds inside a grid of products
    (1, 0, 0, 20, 64, 64, 2, 2, True, 0),        # fewer rows than an MFMA tile: one launch per product
    (1, 0, 0, 72, 40, 40, 2, 3, False, 0),       # K off the tile grid: one launch per product
    (1, 0, 1, 200, 136, 256, 3, 2, False, 2),    # added to C in the epilogue, one launch
    (1, 0, 1, 72, 40, 40, 2, 1, False, 2),       # ... one launch per product
    (0, 0, 1, 33, 17, 29, 2, 2, False, 2),       # ... fp32
    (0, 0, 1, 33, 17, 29, 2, 2, True, 0)])       # fp32
def test_gemm_batched(dtype, tA, tB, M, N, K, by, bz, second, acc):
    """Grids of equal products (operands laid out back to back, batch y fastest), optionally two
    grids in one call, against the fp64 product of the rounded operands."""
    rng = np.random.default_rng(1000 * M + 10 * K + by + bz)
    nb = by * bz
    shA, shB = ((K, M) if tA else (M, K)), ((N, K) if tB else (K, N))
    grids = 2 if second else 1
    A = rng.standard_normal((grids, nb) + shA).astype(np.float32)
    B = rng.standard_normal((grids, nb) + shB).astype(np.float32)
    dA, dB = dev(A, dtype), dev(B, dtype)
    init = rng.standard_normal((grids, nb, M, N)).astype(np.float32) if acc else np.zeros((grids, nb, M, N), np.float32)
    out = torch.from_numpy(init.copy()).cuda()
    nA, nB, nC = shA[0] * shA[1], shB[0] * shB[1], M * N
    at = lambda t, g: C.c_void_p(t.data_ptr() + g * nb * (t.numel() // (grids * nb)) * t.element_size())
    ok(L().ouro_op_gemm_batched(stream(), dtype, tA, tB, M, N, K, 0.5, at(dA, 0), shA[1], at(dB, 0), shB[1], at(out, 0), N,
                                1, acc, by, bz, nA, by * nA, nB, by * nB, nC, by * nC,
                                at(dA, 1) if second else None, at(dB, 1) if second else None, at(out, 1) if second else None, -2.0, 0))
    torch.cuda.synchronize()
    a64, b64, got = host(dA), host(dB), host(out)
    for g in range(grids):
        alpha = -2.0 if g else 0.5
        for i in range(nb):
            a, b = a64[g, i], b64[g, i]
            ref = init[g, i] + alpha * ((a.T if tA else a) @ (b.T if tB else b))
            assert rel_err(got[g, i], ref) < 2e-6, (g, i)


@pytest.mark.parametrize("force", [0, 11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("M,N,K", [(136, 72, 33), (128, 264, 63), (264, 128, 65), (40, 40, 127), (96, 320, 705), (768, 384, 2331)])
def test_gemm_ragged_contraction(force, M, N, K):
    """A^T B over a contraction that is no whole number of K-tiles (weight gradients of any token count): the
    direct-load kernels read k-rows past the end as zero.  What lies behind the operands here is NaN.  Overwriting
    and accumulating (split-K) forms; bound as in test_gemm_forms."""
    rng = np.random.default_rng(M + N + K + force)
    def operand(cols):
        x = torch.full((K + 64, cols), float("nan"), dtype=torch.bfloat16, device="cuda")
        x[:K] = torch.from_numpy(rng.standard_normal((K, cols)).astype(np.float32)).cuda()
        return x
    dA, dB = operand(M), operand(N)
    ref = host(dA[:K]).T @ host(dB[:K])
    for acc in (0, 1):
        out = torch.ones((M, N), dtype=torch.float32, device="cuda")
        ok(L().ouro_op_gemm(stream(), 1, 1, 0, M, N, K, 1.0, p(dA), M, p(dB), N, p(out), N, 1, acc, None, None, 0, 0, None, 0, force))
        torch.cuda.synchronize()
        assert rel_err(host(out), ref + acc) < 2e-6 + 1e-6 * acc


@pytest.mark.parametrize("dtype,force", [(0, 21), (0, 22), (1, 10), (1, 11), (1, 12), (1, 13), (1, 14), (1, 15), (1, 16)])
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(200, 72, 64), (136, 264, 128)])
def test_gemm_column_blocks(dtype, force, tA, tB, M, N, K):
    """Operands that are the last columns of a matrix twice as wide, the other half NaN: tiles reach past the operand on
    every side; bound as in test_gemm_forms."""
    rng = np.random.default_rng(M + N + K + force)
    def operand(rows, cols):
        x = torch.full((rows, 2 * cols), float("nan"), dtype=torch.bfloat16 if dtype else torch.float32, device="cuda")
        x[:, cols:] = torch.from_numpy(rng.standard_normal((rows, cols)).astype(np.float32)).cuda()
        return x, x[:, cols:]
    wA, A = operand(*((K, M) if tA else (M, K)))
    wB, B = operand(*((N, K) if tB else (K, N)))
    out = torch.empty((M, N), dtype=torch.float32, device="cuda")
    ok(L().ouro_op_gemm(stream(), dtype, tA, tB, M, N, K, 1.0, p(A), wA.shape[1], p(B), wB.shape[1], p(out), N, 1, 0, None, None, 0, 0, None, 0, force))
    torch.cuda.synchronize()
    ref = (host(A).T if tA else host(A)) @ (host(B).T if tB else host(B))
    assert rel_err(host(out), ref) < 2e-6


@pytest.mark.parametrize("dtype,shapes", [
    (1, [(256, 128, 2048), (128, 384, 2048), (136, 72, 1024), (128, 128, 512)]),     # all in one launch, ragged tiles
    (1, [(256, 128, 1024), (72, 40, 1000), (128, 256, 4096), (64, 64, 320)]),        # two of them go by themselves
    (1, [(128, 128, 1024)]),
    (0, [(33, 17, 29), (40, 24, 64)])])                                              # fp32: one by one
def test_gemm_group(dtype, shapes):
    """Several accumulating products C_i += alpha A_i^T B_i in one call against fp64."""
    rng = np.random.default_rng(sum(m + n + k for m, n, k in shapes))
    n = len(shapes)
    dA = [dev(rng.standard_normal((k, m)).astype(np.float32), dtype) for m, nn, k in shapes]
    dB = [dev(rng.standard_normal((k, nn)).astype(np.float32), dtype) for m, nn, k in shapes]
    init = [rng.standard_normal((m, nn)).astype(np.float32) for m, nn, k in shapes]
    out = [torch.from_numpy(x.copy()).cuda() for x in init]
    ia = lambda v: (C.c_int * n)(*v)
    pa = lambda ts: (C.c_void_p * n)(*[t.data_ptr() for t in ts])
    ok(L().ouro_op_gemm_group(stream(), dtype, n, ia([s[0] for s in shapes]), ia([s[1] for s in shapes]), ia([s[2] for s in shapes]),
                              pa(dA), ia([s[0] for s in shapes]), pa(dB), ia([s[1] for s in shapes]), pa(out), ia([s[1] for s in shapes]), 0.25))
    torch.cuda.synchronize()
    for i in range(n):
        ref = init[i] + 0.25 * (host(dA[i]).T @ host(dB[i]))
        assert rel_err(host(out[i]), ref) < 2e-6, i


@pytest.mark.parametrize("dtype,M,N,K", [(1, 256, 128, 512), (1, 1024, 512, 256), (1, 136, 72, 40), (0, 64, 64, 128), (0, 640, 1024, 32)])
def test_products_onto_one_output(dtype, M, N, K):
    """Accumulating products that share their output: six of them in one grouped call, then six calls on three streams.
    Integer operands, so that every order of additions gives the same sum and a lost one shows."""
    rng = np.random.default_rng(M + N + K)
    A = [dev(rng.integers(-2, 3, (K, M)), dtype) for _ in range(6)]
    B = [dev(rng.integers(-2, 3, (K, N)), dtype) for _ in range(6)]
    ref = 1.0 + sum(host(a).T @ host(b) for a, b in zip(A, B))
    ia = lambda v: (C.c_int * 6)(*[v] * 6)
    pa = lambda ts: (C.c_void_p * 6)(*[t.data_ptr() for t in ts])
    out = torch.ones((M, N), dtype=torch.float32, device="cuda")
    ok(L().ouro_op_gemm_group(stream(), dtype, 6, ia(M), ia(N), ia(K), pa(A), ia(M), pa(B), ia(N), pa([out] * 6), ia(N), 1.0))
    torch.cuda.synchronize()
    assert np.array_equal(host(out), ref)
    out = torch.ones((M, N), dtype=torch.float32, device="cuda")
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    for i in range(6):
        ok(L().ouro_op_gemm(C.c_void_p(streams[i % 3].cuda_stream), dtype, 1, 0, M, N, K, 1.0, p(A[i]), M, p(B[i]), N, p(out), N, 1, 1, None, None, 0, 0, None, 0, 0))
    torch.cuda.synchronize()
    assert np.array_equal(host(out), ref)


@pytest.mark.parametrize("cleared", [0, 1])
@pytest.mark.parametrize("shapes", [
    [(64, 64, 128), (64, 256, 128), (36, 100, 97), (1, 4, 33)],           # 32x32 tiles, one range; edges and a ragged contraction
    [(64, 64, 4096), (96, 32, 1000), (68, 40, 2050)],                      # 32x32 tiles, split contractions
    [(1024, 1024, 70), (520, 1024, 40)],                                   # 64x64 tiles
    [(64, 64, 128), (33, 64, 128), (64, 64, 8)],                           # beside products that go by themselves (unaligned rows)
])
def test_gemm_f32_group(shapes, cleared):
    """Weight gradients of an fp32 layer in one launch: fp32 sums of K products."""
    rng = np.random.default_rng(len(shapes) + cleared)
    n = len(shapes)
    A = [dev(rng.standard_normal((k, m)), 0) for m, _, k in shapes]; B = [dev(rng.standard_normal((k, w)) / math.sqrt(k), 0) for _, w, k in shapes]
    C_ = [torch.full((m, w), float(1 - cleared), device="cuda") for m, w, _ in shapes]
    ints = lambda i: (C.c_int * n)(*[s[i] for s in shapes])
    ptrs = lambda t: (C.c_void_p * n)(*[x.data_ptr() for x in t])
    ok(L().ouro_op_gemm_group_as(stream(), 0, n, ints(0), ints(1), ints(2), ptrs(A), ints(0), ptrs(B), ints(1), ptrs(C_), ints(1), 0.5, cleared, 0, 0))
    torch.cuda.synchronize()
    for a, b, c in zip(A, B, C_):
        assert rel_err(host(c), 1 - cleared + 0.5 * host(a).T @ host(b)) < TOL[0]


@pytest.mark.parametrize("tile,kchunk", [(128, 0), (256, 0), (128, 512), (256, 512)])
@pytest.mark.parametrize("cleared", [0, 1])
@pytest.mark.parametrize("shapes", [
    [(1024, 1024, 2331), (1032, 776, 2331)],                      # K range whole or split, ragged K-tile and edges of tiles
    [(264, 520, 8256), (512, 256, 8256)],
    [(1024, 2048, 1088), (512, 1024, 96), (256, 256, 40)],        # contractions of one and two K-tiles beside a long one
    [(72, 40, 33), (136, 264, 705)]])
def test_gemm_group_large_tiles(shapes, cleared, tile, kchunk):
    """Both kernels of the grouped launch by name, whatever the rule would choose: K ranges whole (stored where the caller
    cleared the output, added atomically otherwise) and split; outputs off the tiles; NaN behind the operands; same bound as
    test_gemm_group, plus the rounding of the atomic adds."""
    rng = np.random.default_rng(sum(m + n + k for m, n, k in shapes))
    n = len(shapes)
    def operand(k, cols):
        x = torch.full((k + 64, cols), float("nan"), dtype=torch.bfloat16, device="cuda")
        x[:k] = torch.from_numpy(rng.standard_normal((k, cols)).astype(np.float32)).cuda()
        return x
    dA = [operand(k, m) for m, nn, k in shapes]
    dB = [operand(k, nn) for m, nn, k in shapes]
    init = [np.zeros((m, nn), np.float32) if cleared else rng.standard_normal((m, nn)).astype(np.float32) for m, nn, k in shapes]
    out = [torch.full((m + 1, nn + 8), -7.0, device="cuda") for m, nn, k in shapes]
    for o, x in zip(out, init):
        o[:-1, :-8] = torch.from_numpy(x)
    ia = lambda v: (C.c_int * n)(*v)
    pa = lambda ts: (C.c_void_p * n)(*[t.data_ptr() for t in ts])
    ok(L().ouro_op_gemm_group_as(stream(), 1, n, ia([s[0] for s in shapes]), ia([s[1] for s in shapes]), ia([s[2] for s in shapes]), pa(dA),
                                 ia([s[0] for s in shapes]), pa(dB), ia([s[1] for s in shapes]), pa(out), ia([s[1] + 8 for s in shapes]), 0.25,
                                 cleared, tile, kchunk))
    torch.cuda.synchronize()
    for i, (m, nn, k) in enumerate(shapes):
        got = host(out[i])
        ref = init[i] + 0.25 * (host(dA[i][:k]).T @ host(dB[i][:k]))
        assert rel_err(got[:-1, :-8], ref) < 3e-6, i
        assert np.all(got[-1] == -7.0) and np.all(got[:, -8:] == -7.0)


@pytest.mark.parametrize("dtype,force", [(0, 0), (1, 0), (1, 10), (1, 11), (1, 12), (1, 13), (1, 14), (1, 15), (1, 16)])
def test_gemm_epilogues_and_strides(dtype, force):
    rng = np.random.default_rng(5)
    M, N, K = 264, 200, 136
    lda, ldb, ldc = K + 8, N + 16, N + 24
    A = rng.standard_normal((M, lda)).astype(np.float32)
    B = (rng.standard_normal((K, ldb)) * 0.2).astype(np.float32)
    bias = rng.standard_normal(N).astype(np.float32)
    R = rng.standard_normal((M, N)).astype(np.float32)
    dA, dB, dR = dev(A, dtype), dev(B, dtype), dev(R, dtype)
    dbias = torch.from_numpy(bias).cuda()
    tdt = torch.bfloat16 if dtype else torch.float32
    out = torch.zeros((M, ldc), dtype=tdt, device="cuda")
    Z = torch.zeros((M, N), dtype=tdt, device="cuda")
    a64, b64 = host(dA)[:, :K], host(dB)[:, :N]
    pre = a64 @ b64 + bias
    # bias + GELU (writes Z) + residual
    ok(L().ouro_op_gemm(stream(), dtype, 0, 0, M, N, K, 1.0, p(dA), lda, p(dB), ldb, p(out), ldc, 0, 0, p(dbias), p(dR), N,
                        1, p(Z), N, force))
    torch.cuda.synchronize()
    assert rel_err(host(Z), pre) < TOL[dtype]
    assert rel_err(host(out)[:, :N], O.gelu(pre) + host(dR)) < TOL[dtype]
    assert np.all(host(out)[:, N:] == 0)
    # multiply by GELU'(Z)
    out2 = torch.zeros((M, N), dtype=tdt, device="cuda")
    ok(L().ouro_op_gemm(stream(), dtype, 0, 0, M, N, K, 1.0, p(dA), lda, p(dB), ldb, p(out2), N, 0, 0, None, None, 0,
                        2, p(Z), N, force))
    torch.cuda.synchronize()
    assert rel_err(host(out2), (a64 @ b64) * O.gelu_grad(host(Z))) < TOL[dtype]
    # accumulate (split-K path for bf16): C += A^T-form product
    M2, N2, K2 = 136, 264, 4096
    A2 = rng.standard_normal((K2, M2)).astype(np.float32)
    B2 = rng.standard_normal((K2, N2)).astype(np.float32)
    dA2, dB2 = dev(A2, dtype), dev(B2, dtype)
    acc = torch.ones((M2, N2), dtype=torch.float32, device="cuda")
    ok(L().ouro_op_gemm(stream(), dtype, 1, 0, M2, N2, K2, 1.0, p(dA2), M2, p(dB2), N2, p(acc), N2, 1, 1, None, None, 0,
                        0, None, 0, force))
    torch.cuda.synchronize()
    assert rel_err(host(acc), 1.0 + host(dA2).T @ host(dB2)) < 3e-6


@pytest.mark.parametrize("force", [21, 22])
@pytest.mark.parametrize("tA", [0, 1])
@pytest.mark.parametrize("tB", [0, 1])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 31, 7), (64, 64, 32), (32, 96, 128), (65, 130, 97), (40, 84, 412), (200, 64, 516), (63, 65, 2050)])
def test_gemm_f32_matrix_core_forms(force, tA, tB, M, N, K):
    """The two fp32 forms (21: 64x64 tiles, 22: 32x32 tiles with the K-tiles dealt to the waves) at edges of tiles, of
    K-tiles and of the 16-byte alignment (4-byte loads otherwise); overwriting and accumulating.  fp32 sums of K products:
    2e-6 in the norm, as test_gemm_forms holds them to."""
    rng = np.random.default_rng(M + 7 * N + 13 * K + tA * 2 + tB)
    A = rng.standard_normal((K, M) if tA else (M, K)).astype(np.float32)
    B = rng.standard_normal((N, K) if tB else (K, N)).astype(np.float32)
    dA, dB = dev(A, 0), dev(B, 0)
    ref = (A.T if tA else A).astype(np.float64) @ (B.T if tB else B).astype(np.float64)
    for acc in (0, 1):
        out = torch.ones((M, N), dtype=torch.float32, device="cuda")
        ok(L().ouro_op_gemm(stream(), 0, tA, tB, M, N, K, 1.0, p(dA), dA.shape[1], p(dB), dB.shape[1], p(out), N, 1, acc, None, None, 0, 0, None, 0, force))
        torch.cuda.synchronize()
        assert rel_err(host(out), ref + acc) < 2e-6


@pytest.mark.parametrize("force", [0, 21, 22])
def test_gemm_f32_rows_far_apart(force):
    """Rows 2^26 floats apart: the 32-bit offset of the tile's row 16 would come round to row 0.  Such an operand takes the
    plain kernel whatever is asked for."""
    K, M, N, ld = 2, 40, 36, 1 << 26
    rng = np.random.default_rng(3)
    wide = torch.empty((K, ld), dtype=torch.float32, device="cuda")
    wide[:, :M + N] = torch.from_numpy(rng.standard_normal((K, M + N)).astype(np.float32))
    A, B = wide[:, :M], wide[:, M:M + N]
    out = torch.empty((M, N), dtype=torch.float32, device="cuda")
    ok(L().ouro_op_gemm(stream(), 0, 1, 0, M, N, K, 1.0, p(A), ld, p(B), ld, p(out), N, 1, 0, None, None, 0, 0, None, 0, force))
    torch.cuda.synchronize()
    assert rel_err(host(out), host(A).T @ host(B)) < 2e-6


@pytest.mark.parametrize("force", [21, 22])
def test_gemm_f32_matrix_core_epilogues(force):
    """Bias, GELU and its gradient, residuals, LayerNorm residual and dropout in the epilogue of both fp32 forms."""
    test_gemm_epilogues_and_strides(0, force)
    for ln in (0, 1):
        test_gemm_with_fp32_layernorm_residual(0, force, 72, 136, 96, ln)
    test_gemm_with_fused_dropout(0, force, 72, 136, 96)


# -------------------------------------------------------------------------- attention
def _attn_case(dtype, B, H, T, Mv, dh, rel, seed, force=1):
    rng = np.random.default_rng(seed)
    S = Mv + T
    d = H * dh
    q = rng.standard_normal((B * T, d)).astype(np.float32)
    kv = rng.standard_normal((B * S, 2 * d)).astype(np.float32)
    do = rng.standard_normal((B * T, d)).astype(np.float32)
    u = (rng.standard_normal((H, dh)) * 0.5).astype(np.float32)
    vb = (rng.standard_normal((H, dh)) * 0.5).astype(np.float32)
    r = rng.standard_normal((S, d)).astype(np.float32)
    dq_, dkv, ddo, du_, dvb_, dr_ = (dev(x, dtype) for x in (q, kv, do, u, vb, r))
    tdt = torch.bfloat16 if dtype else torch.float32
    o = torch.zeros((B * T, d), dtype=tdt, device="cuda")
    lse = torch.zeros((B, H, T), dtype=torch.float32, device="cuda")
    scale = 1.0 / math.sqrt(dh)
    kptr = C.c_void_p(dkv.data_ptr())
    vptr = C.c_void_p(dkv.data_ptr() + d * dkv.element_size())
    ok(L().ouro_op_attention_fwd(stream(), dtype, B, H, T, S, dh, Mv, scale, p(dq_), d, kptr, 2 * d, vptr, 2 * d, p(o), d,
                                 p(lse), rel, p(du_), p(dvb_), p(dr_), d, force))
    # oracle on the same (rounded) inputs
    q64 = host(dq_).reshape(B, T, H, dh).transpose(0, 2, 1, 3)
    k64 = host(dkv)[:, :d].reshape(B, S, H, dh).transpose(0, 2, 1, 3)
    v64 = host(dkv)[:, d:].reshape(B, S, H, dh).transpose(0, 2, 1, 3)
    r64 = host(dr_).reshape(S, H, dh).transpose(1, 0, 2)
    if rel:
        oo, cache = O.attention_core_fwd(q64, k64, v64, Mv, scale, host(du_), host(dvb_), r64)
    else:
        oo, cache = O.attention_core_fwd(q64, k64, v64, Mv, scale)
    torch.cuda.synchronize()
    tol = TOL[dtype]
    assert rel_err(host(o), oo.transpose(0, 2, 1, 3).reshape(B * T, d)) < tol
    assert np.abs(host(lse) - cache["lse"]).max() < (1e-4 if dtype == 0 else 2e-2)
    # backward
    n_scr = L().ouro_op_attention_bwd_scratch(B, H, T, S, dh)
    scr = torch.zeros(max(n_scr, 1), dtype=torch.float32, device="cuda")
    gq = torch.zeros((B * T, d), dtype=tdt, device="cuda")
    gkv = torch.zeros((B * S, 2 * d), dtype=tdt, device="cuda")
    gu = torch.zeros((H, dh), dtype=torch.float32, device="cuda")
    gvb = torch.zeros((H, dh), dtype=torch.float32, device="cuda")
    gr = torch.zeros((S, d), dtype=torch.float32, device="cuda")
    gk = C.c_void_p(gkv.data_ptr())
    gv = C.c_void_p(gkv.data_ptr() + d * gkv.element_size())
    ok(L().ouro_op_attention_bwd(stream(), dtype, B, H, T, S, dh, Mv, scale, p(dq_), d, kptr, 2 * d, vptr, 2 * d, p(o), d,
                                 p(lse), p(ddo), d, p(gq), d, gk, 2 * d, gv, 2 * d, rel, p(du_), p(dvb_), p(dr_), d,
                                 p(gu), p(gvb), p(gr), p(scr), force))
    torch.cuda.synchronize()
    do64 = host(ddo).reshape(B, T, H, dh).transpose(0, 2, 1, 3)
    rq, rk, rv, ru, rvb, rr = O.attention_core_bwd(do64, cache)
    mh = lambda x, n: x.transpose(0, 2, 1, 3).reshape(B * n, d)
    btol = tol * 2
    assert rel_err(host(gq), mh(rq, T)) < btol
    assert rel_err(host(gkv)[:, :d], mh(rk, S)) < btol
    assert rel_err(host(gkv)[:, d:], mh(rv, S)) < btol
    if rel:
        assert rel_err(host(gu), ru) < btol
        assert rel_err(host(gvb), rvb) < btol
        assert rel_err(host(gr), rr.transpose(1, 0, 2).reshape(S, d)) < btol


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("B,H,T,Mv,dh,rel", [(2, 2, 32, 0, 32, 0), (1, 3, 70, 0, 41, 0), (2, 2, 24, 17, 16, 1),
                                               (1, 2, 67, 130, 41, 1), (1, 1, 1, 0, 8, 0), (2, 1, 5, 0, 8, 1)])
def test_attention_general_kernel(dtype, B, H, T, Mv, dh, rel):
    _attn_case(dtype, B, H, T, Mv, dh, rel, seed=B + H + T + Mv + dh)


@pytest.mark.parametrize("B,H,T,Mv", [(2, 2, 128, 0), (1, 3, 200, 0), (2, 1, 96, 40), (1, 2, 512, 0), (1, 1, 33, 0),
                                      (1, 2, 300, 77), (1, 2, 100, 300), (4, 16, 512, 0), (8, 16, 300, 0), (32, 16, 256, 0), (16, 16, 384, 0),
                                      (16, 16, 300, 90)])
def test_attention_mfma_kernel(B, H, T, Mv):
    """Fused matrix-core kernels (bf16, head size 64): several query/key blocks, ragged
    tails, and a key prefix (Mv) that every query sees.  Up to 512 workgroups the backward pass is one launch (unequal block
    counts; the largest one), beyond it two.  The last three cases have enough
    (batch, head) pairs for the backward kernels to take two blocks per workgroup (an even
    count, an odd one whose middle block goes alone, and unequal query / key block counts)."""
    _attn_case(1, B, H, T, Mv, 64, 0, seed=100 + T + Mv, force=0)


@pytest.mark.parametrize("B,H,T,Mv", [(2, 2, 128, 0), (1, 3, 200, 0), (2, 1, 96, 40), (1, 2, 384, 384), (1, 1, 33, 0),
                                      (1, 2, 300, 77), (2, 2, 150, 150), (3, 2, 20, 5), (2, 3, 64, 200),
                                      (4, 2, 150, 150), (33, 8, 100, 60)])
def test_attention_xl_mfma_kernel(B, H, T, Mv):
    """Fused matrix-core kernels with the relative-position term (bf16, head size 64): with and
    without memory, several query/key blocks, ragged tails, fewer keys than a contraction tile
    (dK, dV and dr are contractions of what the dQ kernel leaves), memory longer than the segment."""
    _attn_case(1, B, H, T, Mv, 64, 1, seed=200 + T + Mv, force=0)


def _xl_fwd(q, kv, r, u, vb, B, H, T, Mv, parts):
    """Output and log-sum-exp of the relative-position forward kernel on bf16 device tensors, and the number of parts of the keys."""
    S, d = Mv + T, H * 64
    n = L().ouro_op_attention_fwd_parts_floats(B, H, T, S)
    o = torch.full((B * T, d), 3.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, H, T), 3.0, device="cuda")
    kp, vp = C.c_void_p(kv.data_ptr()), C.c_void_p(kv.data_ptr() + 2 * d)
    if parts:
        ws = torch.full((max(n, 4),), float("nan"), device="cuda")
        ok(L().ouro_op_attention_fwd_parts(stream(), B, H, T, S, Mv, 0.125, p(q), d, kp, 2 * d, vp, 2 * d, p(o), d, p(lse), p(u), p(vb), p(r), d, p(ws)))
    else:
        ok(L().ouro_op_attention_fwd(stream(), 1, B, H, T, S, 64, Mv, 0.125, p(q), d, kp, 2 * d, vp, 2 * d, p(o), d, p(lse), 1, p(u), p(vb), p(r), d, 0))
    torch.cuda.synchronize()
    return host(o), host(lse), n // (B * H * T * 66) if n else 1


def _xl_inputs(B, H, T, Mv, seed):
    rng = np.random.default_rng(seed)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    S, d = Mv + T, H * 64
    return [dev(x, 1) for x in (f(B * T, d), f(B * S, 2 * d), f(S, d), 0.5 * f(H, 64), 0.5 * f(H, 64))]


PARTS = [(1, 2, 150, 700, 2), (2, 3, 33, 900, 2), (1, 1, 200, 1000, 3), (1, 2, 70, 1500, 4), (1, 2, 1537, 0, 4), (1, 1, 1030, 1000, 4)]


@pytest.mark.parametrize("B,H,T,Mv,n", PARTS)
def test_attention_xl_forward_in_parts(B, H, T, Mv, n):
    """The keys of a query block dealt to two, three and four workgroups, ragged query and key blocks, and (no memory) early query
    blocks with fewer key blocks than parts: output and log-sum-exp against the oracle, bounds of _attn_case."""
    ins = _xl_inputs(B, H, T, Mv, T + Mv)
    o, lse, parts = _xl_fwd(*ins, B, H, T, Mv, True)
    assert parts == n
    S, d = Mv + T, H * 64
    heads = lambda x, rows: x.reshape(B, rows, H, 64).transpose(0, 2, 1, 3)
    q, kv, r, u, vb = (host(x) for x in ins)
    ref, cache = O.attention_core_fwd(heads(q, T), heads(kv[:, :d], S), heads(kv[:, d:], S), Mv, 0.125, u, vb, r.reshape(S, H, 64).transpose(1, 0, 2))
    assert rel_err(o, ref.transpose(0, 2, 1, 3).reshape(B * T, d)) < TOL[1]
    assert np.abs(lse - cache["lse"]).max() < 2e-2


@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("what", ["q", "k", "v", "keys of a part", "all keys"])
@pytest.mark.parametrize("B,H,T,Mv,n", PARTS[:5])
def test_attention_xl_parts_keep_what_is_not_finite(B, H, T, Mv, n, what, value):
    """A NaN or infinity in a query, a key, a value, in all keys that one workgroup takes or in all there are reaches the same
    outputs and log-sum-exps as in the kernel that keeps a query block's keys together; the finite ones are alike (bf16 outputs of
    two orders of summation)."""
    ins = _xl_inputs(B, H, T, Mv, T + Mv)
    S, d = Mv + T, H * 64
    if what == "q": ins[0][T // 2, 5] = value
    elif what == "k": ins[1][S // 3, 7] = value
    elif what == "v": ins[1][S // 3, d + 7] = value
    elif what == "all keys": ins[1][:S, 9] = value
    else: ins[1][:(S + 63) // 64 // n * 64, 9] = value          # the first part of the last query block
    (o, lse, parts), (o1, lse1, _) = (_xl_fwd(*ins, B, H, T, Mv, x) for x in (True, False))
    assert parts == n
    assert not np.isfinite(o1).all()
    for x, y, tol in ((o, o1, TOL[1]), (lse, lse1, 1e-5)):
        fin = np.isfinite(y)
        assert np.array_equal(np.isfinite(x), fin)
        assert not fin.any() or rel_err(x[fin], y[fin]) < tol


@pytest.mark.parametrize("B,H,T,Mv,dh", [(1, 1, 1, 0, 64), (2, 1, 10, 200, 32), (2, 2, 33, 0, 32), (1, 3, 70, 5, 41), (2, 2, 128, 0, 64), (1, 2, 150, 40, 48),
                                         (2, 1, 257, 0, 7), (1, 2, 31, 97, 36)])
def test_attention_f32_kernel(B, H, T, Mv, dh):
    """fp32 attention on the matrix cores: one query, ragged tiles on both axes, memory before the segment, head sizes that
    take the narrow and the wide instance, aligned (16-byte loads) and not; fp32 bound of _attn_case."""
    _attn_case(0, B, H, T, Mv, dh, 0, seed=300 + T + Mv + dh, force=0)


def _attn_f32(q, kv, do, B, H, T, Mv, dh, force):
    """o, lse, dq, and dk | dv of the fp32 kernels."""
    S, d = Mv + T, H * dh
    q, kv, do = (torch.from_numpy(x).cuda() for x in (q, kv, do))
    o, gq, gkv = torch.zeros_like(q), torch.zeros_like(q), torch.zeros_like(kv)
    lse = torch.zeros((B, H, T), device="cuda")
    scr = torch.zeros(max(L().ouro_op_attention_bwd_scratch(B, H, T, S, dh), 1), device="cuda")
    half = lambda t: C.c_void_p(t.data_ptr() + 4 * d)
    sc = 1.0 / math.sqrt(dh)
    ok(L().ouro_op_attention_fwd(stream(), 0, B, H, T, S, dh, Mv, sc, p(q), d, p(kv), 2 * d, half(kv), 2 * d, p(o), d, p(lse), 0, None, None, None, 0, force))
    ok(L().ouro_op_attention_bwd(stream(), 0, B, H, T, S, dh, Mv, sc, p(q), d, p(kv), 2 * d, half(kv), 2 * d, p(o), d, p(lse), p(do), d, p(gq), d,
                                 p(gkv), 2 * d, half(gkv), 2 * d, 0, None, None, None, 0, None, None, None, p(scr), force))
    torch.cuda.synchronize()
    return host(o), host(lse), host(gq), host(gkv)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("what", ["k", "v", "q", "d"])
@pytest.mark.parametrize("B,H,T,Mv,dh,pos", [(1, 2, 96, 0, 64, 40), (2, 1, 70, 5, 41, 69), (1, 1, 33, 20, 32, 0), (1, 2, 20, 0, 7, 13), (2, 1, 64, 0, 64, 31)])
def test_attention_f32_non_finite_rows(B, H, T, Mv, dh, pos, what, value):
    """An infinity or NaN at one position reaches what depends on it and nothing else (keys and values the queries that
    see them, queries and output gradients the keys they see): the matrix-core kernels against the per-row ones, which
    never touch what is not visible.  Finite values to the fp32 bound of _attn_case."""
    rng = np.random.default_rng(T + pos)
    S, d = Mv + T, H * dh
    q, kv, do = (rng.standard_normal((B, n, m)).astype(np.float32) for n, m in ((T, d), (S, 2 * d), (T, d)))
    at = {"k": kv[B - 1, :, :d], "v": kv[B - 1, :, d:], "q": q[B - 1], "d": do[B - 1]}[what]
    at[Mv + pos if what in "kv" else pos] = value
    got, ref = (_attn_f32(q, kv, do, B, H, T, Mv, dh, force) for force in (0, 1))
    assert any(not np.isfinite(r).all() for r in ref)
    for name, x, y in zip(("o", "lse", "dq", "dkv"), got, ref):
        fin = np.isfinite(y)
        assert np.array_equal(np.isfinite(x), fin), name
        assert not fin.any() or rel_err(x[fin], y[fin]) < 2 * TOL[0], name


@pytest.mark.parametrize("dtype,force", [(0, 0), (1, 1), (1, 0), (1, 10), (1, 11), (1, 12), (1, 13), (1, 14), (1, 15), (1, 16)])
@pytest.mark.parametrize("M,N,K,ln", [(200, 136, 328, 1), (384, 520, 192, 1), (130, 88, 128, 0), (260, 256, 64, 1)])
def test_gemm_with_fp32_layernorm_residual(dtype, force, M, N, K, ln):
    """C = A B + bias + R with R the LayerNorm of an fp32 matrix recomputed in the epilogue (ln = 1) or
    that fp32 matrix itself (ln = 0); fp32 result; every contraction kernel, ragged tiles."""
    rng = np.random.default_rng(M + N + K + force + ln)
    A = rng.standard_normal((M, K)).astype(np.float32); B = rng.standard_normal((K, N)).astype(np.float32) / math.sqrt(K)
    bias = rng.standard_normal(N).astype(np.float32)
    S_ = (rng.standard_normal((M, N)) * 2 + 0.3).astype(np.float32)
    g = (1 + 0.3 * rng.standard_normal(N)).astype(np.float32); b = (0.2 * rng.standard_normal(N)).astype(np.float32)
    dA, dB = dev(A, dtype), dev(B, dtype)
    dS, dbias, dg, db = (torch.from_numpy(x).cuda() for x in (S_, bias, g, b))
    R, cache = O.layernorm_fwd(S_.astype(np.float64), g.astype(np.float64), b.astype(np.float64))
    mean = torch.from_numpy(S_.astype(np.float64).mean(axis=1).astype(np.float32)).cuda()      # row statistics are inputs here
    rstd = torch.from_numpy(cache[1][:, 0].astype(np.float32)).cuda()
    Cc = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    ok(L().ouro_op_gemm_ln_residual(stream(), dtype, 0, 0, M, N, K, p(dA), K, p(dB), N, p(Cc), N, 1, p(dbias), p(dS), N,
                                    p(mean) if ln else None, p(rstd) if ln else None, p(dg) if ln else None,
                                    p(db) if ln else None, force))
    torch.cuda.synchronize()
    ref = host(dA) @ host(dB) + bias + (R if ln else S_.astype(np.float64))
    assert rel_err(host(Cc), ref) < TOL[dtype]
    assert np.abs(host(Cc) - ref).max() < (1e-4 if dtype == 0 else 0.1) * np.abs(ref).max()


@pytest.mark.parametrize("force", [11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("M,N", [(32, 40), (130, 88), (200, 100), (264, 200), (300, 530), (520, 392)])
@pytest.mark.parametrize("kind", ["bias", "fp32", "gelu", "gelu_grad", "residual", "fp32_residual", "layernorm", "residual_dropout", "layernorm_dropout"])
def test_gemm_fused_epilogues(kind, M, N, force):
    """Two row-form operands with each epilogue a layer uses: whole tiles, tiles over the edge, columns that do and do not
    end at a multiple of 8, results with a row pitch; nothing outside the result is written."""
    rng = np.random.default_rng(M + N + force)
    K, pitch = 128, (N + 7) // 8 * 8 + 8
    A = dev(rng.standard_normal((M, K)), 1); B = dev(rng.standard_normal((N, K)) / math.sqrt(K), 1)
    fp32 = kind == "fp32" or "residual" in kind or "layernorm" in kind
    full = torch.full((M + 2, pitch), 7.0, dtype=torch.float32 if fp32 else torch.bfloat16, device="cuda")
    side = dev(rng.standard_normal((M, pitch)), 0 if kind == "fp32_residual" or "layernorm" in kind else 1)      # what the epilogue reads, or Z
    bias, g, b = (dev(rng.standard_normal(N), 0) for _ in range(3))
    mean, rstd = dev(rng.standard_normal(M), 0), dev(rng.random(M) + 0.5, 0)
    C_, ref, R = full[1:], host(A) @ host(B).T, host(side)[:, :N]
    if kind in ("fp32_residual", "layernorm"):
        ln = kind == "layernorm"
        ok(L().ouro_op_gemm_ln_residual(stream(), 1, 0, 1, M, N, K, p(A), K, p(B), K, p(C_), pitch, 1, p(bias) if ln else None, p(side), pitch,
                                        p(mean) if ln else None, p(rstd) if ln else None, p(g) if ln else None, p(b) if ln else None, force))
        ref = ref + (host(bias) + (R - host(mean)[:, None]) * host(rstd)[:, None] * host(g) + host(b) if ln else R)
    elif "dropout" in kind:
        ln, pr, seed, sid, dld = kind == "layernorm_dropout", 0.375, 99 + M, 3, N + 5
        mask = O.dropout_mask(O.Config(n_layer=1, d_model=2, n_head=1, d_head=2, d_ff=1, vocab=2, seq_len=1, batch=1, dropout=pr), seed, sid, (M, dld))[:, :N]
        ok(L().ouro_op_gemm_dropout_residual(stream(), 0, 1, M, N, K, p(A), K, p(B), K, p(C_), pitch, p(bias) if ln else None, None if ln else p(side), pitch,
                                             p(side) if ln else None, pitch, p(mean) if ln else None, p(rstd) if ln else None, p(g) if ln else None,
                                             p(b) if ln else None, pr, seed, sid, dld, force))
        ref = (ref + host(bias)) * mask + (R - host(mean)[:, None]) * host(rstd)[:, None] * host(g) + host(b) if ln else ref * mask + R
    else:
        epi = {"gelu": 1, "gelu_grad": 2}.get(kind, 0)
        use_bias = kind in ("bias", "gelu")
        ok(L().ouro_op_gemm(stream(), 1, 0, 1, M, N, K, 1.0, p(A), K, p(B), K, p(C_), pitch, int(fp32), 0, p(bias) if use_bias else None,
                            p(side) if kind == "residual" else None, pitch, epi, p(side) if epi else None, pitch, force))
        if use_bias: ref = ref + host(bias)
        if kind == "residual": ref = ref + R
        if kind == "gelu_grad": ref = ref * O.gelu_grad(R)
        if kind == "gelu":
            torch.cuda.synchronize()
            assert rel_err(host(side)[:, :N], ref) < TOL[1]
            ref = O.gelu(ref)
    torch.cuda.synchronize()
    out = host(full)
    # fp32 results: sums of 128 exact products, a few operations behind them (2^-24 each); bf16: one rounding
    got, tol = out[1:M + 1, :N], 1e-5 if fp32 else TOL[1]
    assert rel_err(got, ref) < tol
    assert np.abs(got - ref).max() < tol * np.abs(ref).max()
    assert np.all(out[0] == 7) and np.all(out[M + 1] == 7) and np.all(out[1:, N:] == 7)


# ------------------------------------------------------------------ row-wise kernels
@pytest.mark.parametrize("dtype", [0, 1, 2])
@pytest.mark.parametrize("rows,d", [(37, 64), (130, 512), (9, 410), (5, 1024), (3, 4100), (517, 1024), (66, 2048)])
def test_layernorm(dtype, rows, d):
    """dtype 2: fp32 rows read, bf16 rows written (the bf16 model's form)."""
    rng = np.random.default_rng(rows + d)
    x = (rng.standard_normal((rows, d)) * 2 + 0.5).astype(np.float32)
    dy = rng.standard_normal((rows, d)).astype(np.float32)
    g = (1 + 0.3 * rng.standard_normal(d)).astype(np.float32)
    b = (0.2 * rng.standard_normal(d)).astype(np.float32)
    dx_, ddy = dev(x, 1 if dtype == 1 else 0), dev(dy, 1 if dtype == 1 else 0)
    dg_, db_ = torch.from_numpy(g).cuda(), torch.from_numpy(b).cuda()
    tdt = torch.bfloat16 if dtype else torch.float32
    y = torch.zeros((rows, d), dtype=tdt, device="cuda")
    mean = torch.zeros(rows, device="cuda"); rstd = torch.zeros(rows, device="cuda")
    ok(L().ouro_op_layernorm_fwd(stream(), dtype, p(dx_), p(dg_), p(db_), p(y), p(mean), p(rstd), rows, d, 0))
    yr, cache = O.layernorm_fwd(host(dx_), g.astype(np.float64), b.astype(np.float64))
    torch.cuda.synchronize()
    assert rel_err(host(y), yr) < TOL[min(dtype, 1)]
    assert rel_err(host(rstd), cache[1][:, 0]) < 1e-5
    gx = torch.zeros((rows, d), dtype=tdt, device="cuda")
    gg = torch.full((d,), 7.0, device="cuda"); gb = torch.full((d,), 7.0, device="cuda")
    ok(L().ouro_op_layernorm_bwd(stream(), dtype, p(ddy), p(dx_), p(dg_), p(mean), p(rstd), p(gx), p(gg), p(gb), rows, d, 0))
    torch.cuda.synchronize()
    rx, rg, rb = O.layernorm_bwd(host(ddy), g.astype(np.float64), cache)
    assert rel_err(host(gx), rx) < TOL[min(dtype, 1)]
    assert rel_err(host(gg), rg) < 1e-4
    assert rel_err(host(gb), rb) < 1e-4


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("rows,dn,d", [(37, 410, 448), (9, 41, 64), (130, 100, 101)])
def test_layernorm_zero_padded_rows(dtype, rows, dn, d):
    """Rows of d columns whose last d-dn are zero padding: statistics over dn columns only, the
    padding stays zero in y and dx, and the first dn columns equal LayerNorm of the unpadded rows."""
    rng = np.random.default_rng(rows + d)
    x = np.zeros((rows, d), np.float32); dy = np.zeros((rows, d), np.float32)
    g = np.zeros(d, np.float32); b = np.zeros(d, np.float32)
    x[:, :dn] = rng.standard_normal((rows, dn)) * 2 + 0.5
    dy[:, :dn] = rng.standard_normal((rows, dn))
    g[:dn] = 1 + 0.3 * rng.standard_normal(dn); b[:dn] = 0.2 * rng.standard_normal(dn)
    dx_, ddy = dev(x, dtype), dev(dy, dtype)
    dg_, db_ = torch.from_numpy(g).cuda(), torch.from_numpy(b).cuda()
    tdt = torch.bfloat16 if dtype else torch.float32
    y = torch.full((rows, d), 3.0, dtype=tdt, device="cuda")
    mean = torch.zeros(rows, device="cuda"); rstd = torch.zeros(rows, device="cuda")
    ok(L().ouro_op_layernorm_fwd(stream(), dtype, p(dx_), p(dg_), p(db_), p(y), p(mean), p(rstd), rows, d, dn))
    yr, cache = O.layernorm_fwd(host(dx_)[:, :dn], g[:dn].astype(np.float64), b[:dn].astype(np.float64))
    torch.cuda.synchronize()
    assert rel_err(host(y)[:, :dn], yr) < TOL[dtype]
    assert not host(y)[:, dn:].any()
    assert rel_err(host(rstd), cache[1][:, 0]) < 1e-5
    gx = torch.full((rows, d), 3.0, dtype=tdt, device="cuda")
    gg = torch.full((d,), 7.0, device="cuda"); gb = torch.full((d,), 7.0, device="cuda")
    ok(L().ouro_op_layernorm_bwd(stream(), dtype, p(ddy), p(dx_), p(dg_), p(mean), p(rstd), p(gx), p(gg), p(gb), rows, d, dn))
    torch.cuda.synchronize()
    rx, rg, rb = O.layernorm_bwd(host(ddy)[:, :dn], g[:dn].astype(np.float64), cache)
    assert rel_err(host(gx)[:, :dn], rx) < TOL[dtype]
    assert not host(gx)[:, dn:].any()
    assert rel_err(host(gg)[:dn], rg) < 1e-4 and not host(gg)[dn:].any()
    assert rel_err(host(gb)[:dn], rb) < 1e-4 and not host(gb)[dn:].any()


# ---------------------------------------------------------------------------- dropout
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("rows,cols,ld,drop_ld", [(37, 64, 64, 64), (130, 410, 448, 410), (3, 5, 9, 7)])
def test_dropout_mask_bit_exact(dtype, rows, cols, ld, drop_ld):
    """The kernel's generator against the oracle's: every element kept or dropped alike (integer
    work: bit-exact), kept elements scaled by 1/(1-p); element index = row * drop_ld + column."""
    pr, seed, sid = 0.3125, 0xDEADBEEF12345678, 11   # rates are dyadic: the same number in fp32 (boundary) and fp64 (oracle)
    cfg = O.Config(n_layer=1, d_model=2, n_head=1, d_head=2, d_ff=1, vocab=2, seq_len=1, batch=1, dropout=pr)
    src = np.zeros((rows, ld), np.float32)
    src[:, :cols] = 1.0 + np.arange(rows * cols, dtype=np.float32).reshape(rows, cols) % 7
    d_src = dev(src, dtype)
    dst = torch.zeros_like(d_src)
    ok(L().ouro_op_dropout(stream(), dtype, p(d_src), p(dst), rows, cols, ld, pr, seed, sid, drop_ld))
    torch.cuda.synchronize()
    mask = O.dropout_mask(cfg, seed, sid, (rows, drop_ld))[:, :cols]
    got = host(dst)[:, :cols]
    assert np.array_equal(got != 0, mask != 0)
    assert rel_err(got, host(d_src)[:, :cols] * mask) < TOL[dtype]
    assert 0.58 < (mask != 0).mean() < 0.8 or mask.size < 100


@pytest.mark.parametrize("dtype,force", [(0, 0), (1, 1), (1, 0), (1, 10), (1, 11), (1, 12), (1, 13), (1, 14), (1, 15), (1, 16)])
@pytest.mark.parametrize("M,N,K", [(200, 136, 328), (384, 520, 192), (130, 82, 128)])
def test_gemm_with_fused_dropout(dtype, force, M, N, K):
    """C = dropout(A B + bias) + residual in every contraction kernel's epilogue (16-byte and
    scalar store paths, ragged tiles): the mask is the oracle's at element m*N + n."""
    rng = np.random.default_rng(M + N + K + force)
    A = rng.standard_normal((M, K)).astype(np.float32); B = rng.standard_normal((K, N)).astype(np.float32) / math.sqrt(K)
    bias = rng.standard_normal(N).astype(np.float32); R = rng.standard_normal((M, N)).astype(np.float32)
    pr, seed, sid = 0.25, 424242, 5
    cfg = O.Config(n_layer=1, d_model=2, n_head=1, d_head=2, d_ff=1, vocab=2, seq_len=1, batch=1, dropout=pr)
    dA, dB, dR = dev(A, dtype), dev(B, dtype), dev(R, dtype)
    dbias = torch.from_numpy(bias).cuda()
    Cc = torch.zeros((M, N), dtype=dA.dtype, device="cuda")
    ok(L().ouro_op_gemm_dropout(stream(), dtype, 0, 0, M, N, K, p(dA), K, p(dB), N, p(Cc), N, p(dbias), p(dR), N,
                                pr, seed, sid, N, force))
    torch.cuda.synchronize()
    mask = O.dropout_mask(cfg, seed, sid, (M, N))
    ref = (host(dA) @ host(dB) + bias) * mask + host(dR)
    assert rel_err(host(Cc), ref) < TOL[dtype]


UPDATE_GROUPS = {
    # matrices (rows, cols) and runs of vectors (n,) of each group
    "small tiles of several groups": [[(64, 128), (100,), (70, 36), (3,)], [(130, 260)], [(1,)], [(33, 50), (7,), (50, 33), (129, 2)]],
    "more groups than a launch takes": [[(40 + i, 8 * i + 4), (5,)] for i in range(20)],
    "whole tiles, one launch of more than 512": [[(16384, 512)], [(512, 2048), (4100,), (2048, 512), (1000, 130)], [(9000,)]],
    "more than 512 tiles off every alignment": [[(17, 31), (8500, 510)], [(9001,), (515, 1026)]],
}


@pytest.mark.parametrize("adam", [0, 1])
@pytest.mark.parametrize("name", list(UPDATE_GROUPS))
def test_update_of_groups_in_one_launch(name, adam):
    """Every group's weights, moments and bf16 copies bit for bit those of the update of one group and of a transposition: groups of
    one launch and of several, tiles dealt to four blocks and to one, edges, pieces between the matrices, groups with two gradients, one and
    none; the cells between the transposed rows stay as they were."""
    rng = np.random.default_rng(adam)
    groups, f = UPDATE_GROUPS[name], lambda n, s=1.0: torch.from_numpy((rng.standard_normal(n) * s).astype(np.float32)).cuda()
    data, tabs = [], []
    for i, g in enumerate(groups):
        entries, off, tile, reach = [], 0, 0, 0
        last = max((j for j, e in enumerate(g) if len(e) == 2), default=-1)
        for j, e in enumerate(g):                              # the last matrix with padded transposed rows (V in a model)
            rows, cols, ld = (1, e[0], 0) if len(e) == 1 else (e[0], e[1], (e[0] + 63) // 64 * 64 if j == last else e[0])
            entries.append((off, rows, cols, ld, tile))
            tile += L().ouro_op_update_tiles(rows, cols, ld)
            reach = max(reach, off + cols * ld)
            off += rows * cols
        t = np.array(entries, dtype=[("off", "u8"), ("rows", "i4"), ("cols", "i4"), ("ld", "i4"), ("tile0", "i4")])
        tabs.append((entries, torch.from_numpy(t.view(np.uint8)).cuda(), tile, off))
        data.append(dict(w=f(off), m=f(off, 0.1), v=f(off, 0.1).abs(), g0=f(off) if i % 3 < 2 else None, g1=f(off) if i % 3 == 0 else None,
                         sh=torch.full((off,), 5.0, dtype=torch.bfloat16, device="cuda"),
                         st=torch.full((max(reach, 1),), 5.0, dtype=torch.bfloat16, device="cuda")))
    ref = [dict(d, w=d["w"].clone(), m=d["m"].clone(), v=d["v"].clone(), sh=d["sh"].clone()) for d in data]
    for d in ref:
        ok(L().ouro_op_update(stream(), p(d["w"]), p(d["m"]), p(d["v"]), p(d["sh"]), p(d["g0"]), 0.5, p(d["g1"]), 0.25, d["w"].numel(), adam, 0.01, 0.9, 0.999, 1e-8, 7))
    n = len(groups)
    ptrs = lambda key: (C.c_void_p * n)(*[None if d[key] is None else d[key].data_ptr() for d in data])
    ints = lambda xs: (C.c_int * n)(*xs)
    ok(L().ouro_op_update_groups(stream(), n, ptrs("w"), ptrs("m"), ptrs("v"), ptrs("sh"), ptrs("st"),
                                 ptrs("g0"), (C.c_float * n)(*[0.5] * n), ptrs("g1"), (C.c_float * n)(*[0.25] * n), (C.c_size_t * n)(*[t[3] for t in tabs]),
                                 (C.c_void_p * n)(*[t[1].data_ptr() for t in tabs]), ints([len(t[0]) for t in tabs]), ints([t[2] for t in tabs]), adam, 0.01, 0.9, 0.999, 1e-8, 7))
    torch.cuda.synchronize()
    for d, r, (entries, _, _, _) in zip(data, ref, tabs):
        for key in ("w", "m", "v", "sh"):
            assert torch.equal(d[key], r[key]), key
        want = torch.full_like(d["st"], 5.0)
        for off, rows, cols, ld, _ in entries:
            if ld:
                torch.as_strided(want, (cols, rows), (ld, 1), off).copy_(r["sh"][off:off + rows * cols].view(rows, cols).t())
        assert torch.equal(d["st"], want)


@pytest.mark.parametrize("dtype", [0, 1])
def test_colsum(dtype):
    rng = np.random.default_rng(3)
    x = rng.standard_normal((333, 200)).astype(np.float32)
    dx_ = dev(x, dtype)
    out = torch.full((150,), 3.0, device="cuda")
    ok(L().ouro_op_colsum(stream(), dtype, p(dx_), 200, p(out), 333, 150))
    torch.cuda.synchronize()
    assert rel_err(host(out), host(dx_)[:, :150].sum(0)) < 1e-5


@pytest.mark.parametrize("dtype", [0, 1])
def test_embedding_gather_scatter(dtype):
    rng = np.random.default_rng(4)
    vocab, d, T, B = 50, 24, 7, 5
    N = B * T
    V = rng.standard_normal((vocab, d)).astype(np.float32)
    tok = rng.integers(0, vocab, N).astype(np.int32)
    tok[:6] = 3                                           # a hot row
    dV = dev(V, dtype)
    dtok = torch.from_numpy(tok).cuda()
    pe = rng.standard_normal((T, d)).astype(np.float32)
    dpe = torch.from_numpy(pe).cuda()
    tdt = torch.bfloat16 if dtype else torch.float32
    h = torch.zeros((N, d), dtype=tdt, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ok(L().ouro_op_embed_fwd(stream(), dtype, p(dtok), p(dV), None, p(h), N, T, d, vocab, 1.0, p(flag)))
    torch.cuda.synchronize()
    assert torch.equal(h, dV[torch.from_numpy(tok.astype(np.int64)).cuda()])      # row selection is bit-exact
    ok(L().ouro_op_embed_fwd(stream(), dtype, p(dtok), p(dV), p(dpe), p(h), N, T, d, vocab, 1.5, p(flag)))
    torch.cuda.synchronize()
    ref = 1.5 * host(dV)[tok] + np.tile(pe, (B, 1))
    assert rel_err(host(h), ref) < (1e-6 if dtype == 0 else 4e-3)
    assert flag.item() == 0
    dh = rng.standard_normal((N, d)).astype(np.float32)
    ddh = dev(dh, dtype)
    dVi = torch.full((vocab, d), 9.0, device="cuda")
    ok(L().ouro_op_embed_bwd(stream(), dtype, p(dtok), p(ddh), p(dVi), N, d, vocab, 1.5))
    torch.cuda.synchronize()
    refg = np.zeros((vocab, d))
    np.add.at(refg, tok, 1.5 * host(ddh))
    assert rel_err(host(dVi), refg) < 1e-6
    assert np.all(host(dVi)[np.setdiff1d(np.arange(vocab), tok)] == 0)
    # out-of-range id: flagged, row skipped, nothing dereferenced
    tok2 = tok.copy(); tok2[2] = vocab; tok2[3] = -1
    dtok2 = torch.from_numpy(tok2).cuda()
    ok(L().ouro_op_embed_fwd(stream(), dtype, p(dtok2), p(dV), None, p(h), N, T, d, vocab, 1.0, p(flag)))
    torch.cuda.synchronize()
    assert flag.item() == 1 and np.all(host(h)[2:4] == 0)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("N,vocab", [(12, 256), (7, 1000), (5, 50257), (4, 32768), (3, 65536), (3, 65537), (6, 2056)])
def test_softmax_cross_entropy(dtype, N, vocab):
    rng = np.random.default_rng(N + vocab)
    logits = (rng.standard_normal((N, vocab)) * 3).astype(np.float32)
    tgt = rng.integers(0, vocab, N).astype(np.int32)
    ld = (vocab + 7) // 8 * 8                                  # padded rows, as the model lays them out
    tdt = torch.bfloat16 if dtype else torch.float32
    dl = torch.zeros((N, ld), dtype=tdt, device="cuda")
    dl[:, :vocab] = dev(logits, dtype)
    l64 = host(dl)[:, :vocab]                                  # the (rounded) logits both sides see
    dt = torch.from_numpy(tgt).cuda()
    G = torch.zeros((N, ld), dtype=tdt, device="cuda")
    lse = torch.zeros(N, device="cuda"); rl = torch.zeros(N, device="cuda"); loss = torch.zeros(1, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ok(L().ouro_op_softmax_ce(stream(), dtype, p(dl), ld, p(dt), p(G), ld, p(lse), p(rl), p(loss), N, vocab, p(flag)))
    torch.cuda.synchronize()
    rloss, rlse = O.cross_entropy_fwd(l64, tgt)
    rG = O.cross_entropy_bwd(l64, rlse, tgt)
    assert abs(loss.item() - rloss) / rloss < 1e-5
    assert np.abs(host(lse) - rlse).max() < 1e-4
    assert rel_err(host(G)[:, :vocab], rG) < (1e-5 if dtype == 0 else 5e-3)
    assert flag.item() == 0
    # in place: G written over the logits
    dl2 = dl.clone()
    ok(L().ouro_op_softmax_ce(stream(), dtype, p(dl2), ld, p(dt), p(dl2), ld, p(lse), p(rl), p(loss), N, vocab, p(flag)))
    torch.cuda.synchronize()
    assert torch.equal(dl2[:, :vocab], G[:, :vocab])
    # zero logits: loss = ln(vocab) (uniform softmax)
    dl.zero_()
    ok(L().ouro_op_softmax_ce(stream(), dtype, p(dl), ld, p(dt), p(G), ld, p(lse), p(rl), p(loss), N, vocab, p(flag)))
    torch.cuda.synchronize()
    assert abs(loss.item() - math.log(vocab)) < 1e-5


@pytest.mark.parametrize("adam", [0, 1])
@pytest.mark.parametrize("n", [1, 7, 4096, 100003])
def test_update_kernel(adam, n):
    rng = np.random.default_rng(n + adam)
    w = rng.standard_normal(n).astype(np.float32)
    g0 = rng.standard_normal(n).astype(np.float32); g1 = rng.standard_normal(n).astype(np.float32)
    m = (rng.standard_normal(n) * 0.1).astype(np.float32); v = (rng.random(n) * 0.1).astype(np.float32)
    dw, dg0, dg1, dm, dv = (torch.from_numpy(x.copy()).cuda() for x in (w, g0, g1, m, v))
    sh = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
    t = 5
    ok(L().ouro_op_update(stream(), p(dw), p(dm), p(dv), p(sh), p(dg0), 0.5, p(dg1), 0.5, n, adam, 0.01, 0.9, 0.999, 1e-8, t))
    torch.cuda.synchronize()
    cfg = O.Config(n_layer=1, d_model=8, n_head=2, d_head=4, d_ff=8, vocab=8, seq_len=2, batch=1, optimizer=adam)
    orc = O.Oracle.__new__(O.Oracle); orc.cfg = cfg; orc.t = t
    w64, m64, v64 = w.astype(np.float64), m.astype(np.float64), v.astype(np.float64)
    orc._apply(w64, 0.5 * g0.astype(np.float64) + 0.5 * g1.astype(np.float64), m64, v64, 0.01)
    assert rel_err(host(dw), w64) < 1e-6
    if adam:
        assert rel_err(host(dm), m64) < 1e-6 and rel_err(host(dv), v64) < 1e-6
    assert torch.equal(sh, dw.to(torch.bfloat16))            # bf16 copy = round-to-nearest-even of the master
    # zero gradient (null pointers) with zero moments leaves the weights bit-identical
    dw2 = torch.from_numpy(w.copy()).cuda(); z1 = torch.zeros(n, device="cuda"); z2 = torch.zeros(n, device="cuda")
    ok(L().ouro_op_update(stream(), p(dw2), p(z1), p(z2), None, None, 1.0, None, 0.0, n, adam, 0.01, 0.9, 0.999, 1e-8, 0))
    torch.cuda.synchronize()
    assert np.array_equal(dw2.cpu().numpy(), w) and not z1.any() and not z2.any()
