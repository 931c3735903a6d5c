"""Kernel-level parity: each HIP kernel through the C ABI vs the fp64 oracle.

Inputs are seeded, rounded to the working precision before both sides see
them.  Sizes span several tiles and end in ragged tails.  Tolerances
(normwise max-norm relative error, see gpu_util.rel_err):
  * bf16 outputs: one rounding to bf16 (2^-9 relative) on top of an fp32
    accumulation -> 8e-3;
  * fp32 outputs from bf16 inputs: products are exact in fp32, the sums round
    at 2^-24 per add -> 1e-4 for K up to a few thousand;
  * fp32 mode: 1e-5.
"""
import numpy as np
import pytest

from oracle import gpt
from paper_2403_10504_amd import atom as A
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

TOL_OUT = {"bf16": 8e-3, "f32": 1e-5}


def stream():
    return U.torch().cuda.current_stream().cuda_stream


# ---------------------------------------------------------------------- GEMM
def gemm_case(dtype, akc, bkc, M, N, K, epi, seed):
    r = U.rng(seed)
    a_shape = (M, K) if akc else (K, M)
    b_shape = (N, K) if bkc else (K, N)
    Am = U.rep(r.standard_normal(a_shape), dtype)
    Bm = U.rep(r.standard_normal(b_shape), dtype)
    Aop = Am if akc else Am.T
    Bop = Bm.T if bkc else Bm  # [K][N]
    acc = Aop.astype(np.float64) @ Bop.astype(np.float64)
    bias = U.rep(r.standard_normal(N), dtype)
    resid = r.standard_normal((M, N)).astype(np.float32)
    aux = U.rep(r.standard_normal((M, N)), dtype)
    cinit = r.standard_normal((M, N)).astype(np.float32)
    dA, dB = U.dev(Am, dtype), U.dev(Bm, dtype)
    out_f32 = epi in (A.ATOM_EPI_STORE_F32, A.ATOM_EPI_ACC_F32, A.ATOM_EPI_BIAS_RESID)
    dC = U.dev_f32(cinit) if epi == A.ATOM_EPI_ACC_F32 else U.empty((M, N), "f32" if out_f32 else dtype)
    dbias, dres, daux = U.dev(bias, dtype), U.dev_f32(resid), U.dev(aux, dtype)
    if epi == A.ATOM_EPI_BIAS_GELU:
        daux = U.empty((M, N), dtype)
    A.atom_k_gemm(U.dt_code(dtype), akc, bkc, epi, M, N, K, U.ptr(dA), a_shape[1], U.ptr(dB), b_shape[1], U.ptr(dC), N,
                  U.ptr(dbias), U.ptr(dres), U.ptr(daux), N, stream())
    U.sync()
    got = U.host(dC)
    if epi == A.ATOM_EPI_STORE or epi == A.ATOM_EPI_STORE_F32:
        ref = acc
    elif epi == A.ATOM_EPI_ACC_F32:
        ref = cinit + acc
    elif epi == A.ATOM_EPI_BIAS:
        ref = acc + bias
    elif epi == A.ATOM_EPI_BIAS_RESID:
        ref = resid + acc + bias
    elif epi == A.ATOM_EPI_BIAS_GELU:
        u = acc + bias
        assert U.rel_err(U.host(daux), u) < TOL_OUT[dtype]
        ref = gpt.gelu(U.rep(u, dtype).astype(np.float64))
    elif epi == A.ATOM_EPI_GELU_BWD:
        ref = acc * gpt.gelu_grad(aux.astype(np.float64))
    tol = 1e-4 if (out_f32 and dtype == "bf16") else TOL_OUT[dtype]
    return U.rel_err(got, ref), tol


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("M,N,K", [(200, 136, 72), (256, 384, 512), (130, 66, 520), (2, 2, 8)])
def test_gemm_layouts(dtype, akc, bkc, M, N, K):
    err, tol = gemm_case(dtype, akc, bkc, M, N, K, A.ATOM_EPI_STORE, seed=M * 7 + N + K)
    assert err < tol, err


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("epi", [A.ATOM_EPI_STORE_F32, A.ATOM_EPI_ACC_F32, A.ATOM_EPI_BIAS, A.ATOM_EPI_BIAS_GELU,
                                 A.ATOM_EPI_BIAS_RESID, A.ATOM_EPI_GELU_BWD])
def test_gemm_epilogues(dtype, epi):
    for akc, bkc in ((1, 1), (1, 0), (0, 0)):
        err, tol = gemm_case(dtype, akc, bkc, 260, 196, 136, epi, seed=epi * 3 + akc + 2 * bkc)
        assert err < tol, (akc, bkc, err)


def sampled_gemm_check(dtype, akc, bkc, M, N, K, ws_bytes=0, seed=0, rows=48):
    """Large GEMM: compare a random sample of full output rows with fp64 dot products."""
    r = U.rng(seed)
    a_shape = (M, K) if akc else (K, M)
    b_shape = (N, K) if bkc else (K, N)
    Am = U.rep(r.standard_normal(a_shape), dtype)
    Bm = U.rep(r.standard_normal(b_shape), dtype)
    dA, dB = U.dev(Am, dtype), U.dev(Bm, dtype)
    dC = U.empty((M, N), "f32")
    ws = U.empty(max(1, ws_bytes // 4), "f32")
    A.atom_k_gemm(U.dt_code(dtype), akc, bkc, A.ATOM_EPI_STORE_F32, M, N, K, U.ptr(dA), a_shape[1], U.ptr(dB),
                  b_shape[1], U.ptr(dC), N, stream=stream(), ws=U.ptr(ws) if ws_bytes else None, ws_bytes=ws_bytes)
    U.sync()
    got = U.host(dC)
    pick = np.sort(r.choice(M, size=min(rows, M), replace=False))
    pick[-1] = M - 1  # always include the ragged last row
    Aop = (Am if akc else Am.T)[pick].astype(np.float64)
    Bop = (Bm.T if bkc else Bm).astype(np.float64)
    return U.rel_err(got[pick], Aop @ Bop), got


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0)])
def test_gemm_large_tile_path(akc, bkc):
    # many output tiles with ragged edges (with both operands not k-contiguous,
    # 4100 rows are no whole 16-byte chunks: the register-staged kernel)
    err, _ = sampled_gemm_check("bf16", akc, bkc, 4100, 4104, 264, seed=akc + 2 * bkc)
    assert err < 1e-4, err


ALL_EPI = [A.ATOM_EPI_STORE, A.ATOM_EPI_STORE_F32, A.ATOM_EPI_ACC_F32, A.ATOM_EPI_BIAS, A.ATOM_EPI_BIAS_GELU,
           A.ATOM_EPI_BIAS_RESID, A.ATOM_EPI_GELU_BWD]


@pytest.mark.parametrize("K", [352, 384, 128])
@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("epi", ALL_EPI)
def test_gemm_pipelined_path(akc, bkc, epi, K):
    """bf16 problems of many tiles and short k: k a multiple of 128 (384: three loop
    trips; 128: the prologue's tiles only) and not (352: three tiles of 32 after
    two trips).  M and N end in partial tiles (ragged by 8 and 24 rows) whose
    loads are clamped to the last valid rows and whose epilogue takes the
    bounds-tested copy."""
    check_pipelined(akc, bkc, epi, 4104, 4120, K, seed=akc + 2 * bkc + 4 * epi + K)


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0)])
@pytest.mark.parametrize("epi", [A.ATOM_EPI_STORE, A.ATOM_EPI_BIAS_GELU, A.ATOM_EPI_BIAS_RESID, A.ATOM_EPI_GELU_BWD])
def test_gemm_pipelined_rotated_k(akc, bkc, epi):
    """256x256 tiles (a whole number per XCD: 256 tiles): each XCD starts its k loop
    at its own eighth of k (k = 1152: 36 tiles of 32, offsets 0, 4, ..., 28), and
    every tile takes the branch-free epilogue."""
    assert U.gemm_choice("bf16", akc, bkc, epi, 4096, 4096, 1152)[:4] == (0, 256, 256, 1)
    check_pipelined(akc, bkc, epi, 4096, 4096, 1152, seed=100 + akc + 2 * bkc + 4 * epi)


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0)])
@pytest.mark.parametrize("M,N,K,epi", [
    (3072, 4096, 1024, A.ATOM_EPI_BIAS_GELU),  # 192 tiles of 256x256: no split
    (3072, 4096, 1024, A.ATOM_EPI_GELU_BWD),
    (2048, 2048, 4096, A.ATOM_EPI_STORE),  # 64 tiles
    (1544, 1032, 2048, A.ATOM_EPI_ACC_F32),  # 35 ragged tiles
    (1544, 1032, 2048, A.ATOM_EPI_STORE_F32),
    (3072, 768, 16384, A.ATOM_EPI_STORE),  # 36 tiles; 64 MB hold seven splits at most
])
def test_gemm_four_wave_few_tiles(akc, bkc, M, N, K, epi):
    """Fewer 256x256 tiles than CUs, with a workspace: smaller tiles, or ranges of k
    whose fp32 partial sums splitk_reduce adds in order (store epilogues, as
    many as the workspace holds)."""
    seed = 200 + akc + 2 * bkc + 4 * epi + M
    check_pipelined(akc, bkc, epi, M, N, K, seed=seed, ws_bytes=64 << 20)
    if epi == A.ATOM_EPI_STORE_F32:
        # the split sum is deterministic and differs from the unsplit order
        c1 = check_pipelined(akc, bkc, epi, M, N, K, seed=seed, ws_bytes=64 << 20)
        c2 = check_pipelined(akc, bkc, epi, M, N, K, seed=seed, ws_bytes=64 << 20)
        c0 = check_pipelined(akc, bkc, epi, M, N, K, seed=seed, ws_bytes=0)
        assert np.array_equal(c1, c2)
        assert not np.array_equal(c0, c1)


def check_pipelined(akc, bkc, epi, M, N, K, seed, ws_bytes=0):
    r = U.rng(seed)
    a_shape = (M, K) if akc else (K, M)
    b_shape = (N, K) if bkc else (K, N)
    Am = U.rep(r.standard_normal(a_shape), "bf16")
    Bm = U.rep(r.standard_normal(b_shape), "bf16")
    bias = U.rep(r.standard_normal(N), "bf16")
    resid = r.standard_normal((M, N)).astype(np.float32)
    aux = U.rep(r.standard_normal((M, N)), "bf16")
    cinit = r.standard_normal((M, N)).astype(np.float32)
    dA, dB, dbias, dres = U.dev(Am, "bf16"), U.dev(Bm, "bf16"), U.dev(bias, "bf16"), U.dev_f32(resid)
    out_f32 = epi in (A.ATOM_EPI_STORE_F32, A.ATOM_EPI_ACC_F32, A.ATOM_EPI_BIAS_RESID)
    dC = U.dev_f32(cinit) if epi == A.ATOM_EPI_ACC_F32 else U.empty((M, N), "f32" if out_f32 else "bf16")
    daux = U.dev(aux, "bf16") if epi == A.ATOM_EPI_GELU_BWD else U.empty((M, N), "bf16")
    dws = U.empty((ws_bytes // 4,), "f32") if ws_bytes else None
    A.atom_k_gemm(A.ATOM_BF16, akc, bkc, epi, M, N, K, U.ptr(dA), a_shape[1], U.ptr(dB), b_shape[1], U.ptr(dC), N,
                  U.ptr(dbias), U.ptr(dres), U.ptr(daux), N, stream(), ws=U.ptr(dws) if ws_bytes else None,
                  ws_bytes=ws_bytes)
    U.sync()
    pick = np.sort(np.unique(np.concatenate([U.rng(7).choice(M, min(40, M), replace=False), [M - 9, M - 1]])))
    acc = (Am if akc else Am.T)[pick].astype(np.float64) @ (Bm.T if bkc else Bm).astype(np.float64)
    got = U.host(dC)[pick]
    if epi == A.ATOM_EPI_BIAS_GELU:
        u = acc + bias
        assert U.rel_err(U.host(daux)[pick], u) < 8e-3
        ref = gpt.gelu(U.rep(u, "bf16").astype(np.float64))
    elif epi == A.ATOM_EPI_BIAS_RESID:
        ref = resid[pick] + acc + bias
    elif epi == A.ATOM_EPI_ACC_F32:
        ref = cinit[pick] + acc
    elif epi == A.ATOM_EPI_BIAS:
        ref = acc + bias
    elif epi == A.ATOM_EPI_GELU_BWD:
        ref = acc * gpt.gelu_grad(aux[pick].astype(np.float64))
    else:
        ref = acc
    tol = 1e-4 if out_f32 else 8e-3
    assert U.rel_err(got, ref) < tol
    # the last columns (a partial tile) too
    assert U.rel_err(got[:, -24:], ref[:, -24:]) < tol
    return got


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (65, 68, 40), (31, 36, 136), (129, 260, 264), (520, 392, 520)])
def test_gemm_direct_load_edges(dtype, M, N, K):
    """The direct-load kernel at the edges of its smallest tiles (64 rows in bf16, 32
    in fp32), with k ending inside a tile of 32 and inside a group of 128 (the
    chunks past k read zeros), and row counts that only a k-contiguous operand
    may have.  Tolerances as for test_gemm_layouts."""
    for akc, bkc in ((1, 1), (1, 0), (0, 0), (0, 1)):
        Mr, Nr = (M if akc else (M + 7) // 8 * 8), (N if bkc else (N + 7) // 8 * 8)
        err, tol = gemm_case(dtype, akc, bkc, Mr, Nr, K, A.ATOM_EPI_STORE, seed=M + N + K + akc + 2 * bkc)
        assert err < tol, (akc, bkc, err)


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0)])
@pytest.mark.parametrize("M,N,K,ws", [
    (4008, 3064, 520, 0),  # 256x192 tiles, ragged rows, k ends inside a group of 128
    (1000, 8192, 2056, 0),  # 256x128 tiles, likewise
    (136, 392, 8200, 64 << 20),  # splits of k, the last one short (store epilogues)
])
@pytest.mark.parametrize("epi", ALL_EPI)
def test_gemm_direct_load_tiles(akc, bkc, M, N, K, ws, epi):
    """Tile shapes and splits that the other sizes here do not reach; tolerances as
    for the pipelined path (one bf16 rounding, or fp32 sums of exact products)."""
    check_pipelined(akc, bkc, epi, M, N, K, seed=300 + akc + 2 * bkc + 4 * epi + K, ws_bytes=ws)


# The training step's layouts and epilogues (forward, data and weight gradient).
STEP_COMBOS = [(1, 1, A.ATOM_EPI_STORE), (1, 1, A.ATOM_EPI_STORE_F32), (1, 1, A.ATOM_EPI_BIAS),
               (1, 1, A.ATOM_EPI_BIAS_GELU), (1, 1, A.ATOM_EPI_BIAS_RESID), (1, 0, A.ATOM_EPI_STORE),
               (1, 0, A.ATOM_EPI_STORE_F32), (1, 0, A.ATOM_EPI_GELU_BWD), (0, 0, A.ATOM_EPI_STORE),
               (0, 0, A.ATOM_EPI_STORE_F32), (0, 0, A.ATOM_EPI_ACC_F32)]
STORE_COMBOS = [c for c in STEP_COMBOS if c[2] <= A.ATOM_EPI_ACC_F32]


@pytest.mark.parametrize("akc,bkc,epi", STEP_COMBOS)
@pytest.mark.parametrize("tile,M,N,K", [
    # rows and columns ragged and k ending inside a group of 128, then whole tiles and whole groups
    ((256, 256), 3920, 3144, 856), ((256, 256), 3840, 3328, 896),
    ((256, 192), 2232, 3736, 1224), ((256, 192), 3840, 3264, 640),
    ((256, 128), 3472, 1176, 1072), ((256, 128), 3328, 1280, 1152),
    ((128, 128), 2808, 1224, 136), ((128, 128), 1920, 1664, 256),
    ((64, 64), 24, 32, 712), ((64, 64), 64, 128, 384)])
def test_gemm_every_tile(akc, bkc, epi, tile, M, N, K):
    """Each bf16 tile of the direct-load kernel under every epilogue of the training
    step, by the bounds-tested and the branch-free copy of the epilogue, with
    and without a k tail."""
    assert U.gemm_choice("bf16", akc, bkc, epi, M, N, K)[:4] == (0, *tile, 1)
    check_pipelined(akc, bkc, epi, M, N, K, seed=400 + akc + 2 * bkc + 4 * epi + K)


@pytest.mark.parametrize("akc,bkc,epi", STORE_COMBOS)
@pytest.mark.parametrize("tile,M,N,K", [
    ((256, 256), 1456, 2728, 3736), ((256, 256), 2304, 2048, 3456),
    ((256, 192), 648, 2184, 7800), ((256, 192), 1024, 2112, 5120),
    ((256, 128), 936, 1328, 4968), ((256, 128), 512, 2816, 5760),
    ((128, 128), 2704, 96, 4968), ((128, 128), 2816, 128, 5248),
    ((64, 64), 16, 120, 1840), ((64, 64), 64, 64, 6144)])
def test_gemm_every_tile_split(akc, bkc, epi, tile, M, N, K):
    """The same tiles over several ranges of k (the last one short in the first of
    each pair), their partials summed by splitk_reduce."""
    ws = 64 << 20
    staged, bm, bn, splits, _ = U.gemm_choice("bf16", akc, bkc, epi, M, N, K, ws)
    assert (staged, bm, bn) == (0, *tile) and splits > 1
    check_pipelined(akc, bkc, epi, M, N, K, seed=500 + akc + 2 * bkc + 4 * epi + K, ws_bytes=ws)


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("K", [8, 32, 40, 64, 96, 104, 160, 200, 224])
def test_gemm_k_tail(akc, bkc, K):
    """One to four k tiles of 32, and one to three after a whole group of four, the
    last one whole or not: only the tiles that hold k are loaded and multiplied."""
    for dtype, M, N in (("bf16", 264, 200), ("bf16", 2808, 1224), ("f32", 68, 100)):
        err, tol = gemm_case(dtype, akc, bkc, M, N, K, A.ATOM_EPI_STORE, seed=M + K + akc + 2 * bkc)
        assert err < tol, (dtype, M, err)


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("epi", ALL_EPI)
@pytest.mark.parametrize("M,N,K", [(2244, 332, 280), (2220, 324, 384)])
def test_gemm_f32_large_tile(akc, bkc, epi, M, N, K):
    """The fp32 64x64 tile: every layout and epilogue, ragged, with and without a k tail."""
    assert U.gemm_choice("f32", akc, bkc, epi, M, N, K)[:4] == (0, 64, 64, 1)
    err, tol = gemm_case("f32", akc, bkc, M, N, K, epi, seed=M + K + akc + 2 * bkc + 4 * epi)
    assert err < tol, err


def test_gemm_choice_of_short_k():
    """Where starts, epilogues and stores dominate, big tiles stay ahead of 128x128 ones."""
    for akc, bkc, epi, M, N, K in ((1, 0, A.ATOM_EPI_STORE, 14824, 12136, 384), (1, 1, A.ATOM_EPI_BIAS, 7080, 16144, 384)):
        assert U.gemm_choice("bf16", akc, bkc, epi, M, N, K)[1] == 256, (M, N, K)


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0), (0, 1)])
def test_gemm_f32_short_k(akc, bkc):
    """fp32 problems of many tiles and at most 256 k take the register-staged kernel."""
    M, N, K = 1548, 4588, 72
    assert U.gemm_choice("f32", akc, bkc, A.ATOM_EPI_STORE, M, N, K)[:4] == (1, 128, 128, 1)
    err, tol = gemm_case("f32", akc, bkc, M, N, K, A.ATOM_EPI_STORE, seed=K + akc + 2 * bkc)
    assert err < tol, err


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0)])
@pytest.mark.parametrize("epi", ALL_EPI)
def test_gemm_unaligned_large(akc, bkc, epi):
    """bf16 rows that are no whole 16-byte chunks (k-contiguous operands: no whole
    output 4-vectors), in numbers for which the register-staged kernel takes 256x256
    tiles: ragged in rows, columns and k."""
    M, N, K = 3428, 8094, 456
    assert U.gemm_choice("bf16", akc, bkc, epi, M, N, K) == (1, 256, 256, 1, 0)
    check_pipelined(akc, bkc, epi, M, N, K, seed=600 + akc + 2 * bkc + 4 * epi)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0), (0, 1)])
def test_gemm_unaligned_split_k(dtype, akc, bkc):
    """The register-staged kernel's split over k, whose sum takes columns one by one
    where N is no multiple of four."""
    M, N, K, ws = 136, 390 if dtype == "bf16" else 391, 8192, 64 << 20
    staged, _, _, splits, _ = U.gemm_choice(dtype, akc, bkc, A.ATOM_EPI_STORE_F32, M, N, K, ws)
    assert staged and splits > 1
    err, _ = sampled_gemm_check(dtype, akc, bkc, M, N, K, ws_bytes=ws, seed=akc + 2 * bkc, rows=M)
    assert err < (1e-4 if dtype == "bf16" else 1e-5), err


@pytest.mark.parametrize("N", [5496, 5504])
def test_gemm_large_result_rows(N):
    """fp32 results of more than 256 MB: stored past the caches where their rows are
    whole 128-byte lines (5504 columns), through them otherwise (5496)."""
    M, K = 12400, 72
    assert U.gemm_choice("bf16", 1, 1, A.ATOM_EPI_STORE_F32, M, N, K)[4] == (N % 32 == 0)
    err, _ = sampled_gemm_check("bf16", 1, 1, M, N, K, seed=N)
    assert err < 1e-4, err


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("epi", ALL_EPI)
@pytest.mark.parametrize("N", [392, 390])  # the direct-load and the register-staged kernel
def test_gemm_workspace_is_for_store_epilogues(dtype, epi, N):
    """The workspace contract: the three store epilogues split a long k over it, the
    others leave it as it is (a caller may share it with another stream then)."""
    M, K = 136, 8192
    a, b = U.dev(np.ones((M, K)), dtype), U.dev(np.ones((N, K)), dtype)
    c, aux, res = U.empty((M, N), "f32"), U.dev(np.zeros((M, N)), dtype), U.dev_f32(np.zeros((M, N), np.float32))
    bias = U.dev(np.zeros(N), dtype)
    c.zero_()
    ws = U.dev_f32(np.full(16 * M * N, 7.0, np.float32))
    A.atom_k_gemm(U.dt_code(dtype), 1, 1, epi, M, N, K, U.ptr(a), K, U.ptr(b), K, U.ptr(c), N, U.ptr(bias), U.ptr(res),
                  U.ptr(aux), N, stream(), ws=U.ptr(ws), ws_bytes=16 * M * N * 4)
    U.sync()
    store = epi in (A.ATOM_EPI_STORE, A.ATOM_EPI_STORE_F32, A.ATOM_EPI_ACC_F32)
    assert bool((ws == 7.0).all()) == (not store)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_gemm_split_k_is_exact_and_deterministic(dtype):
    M, N, K = 256, 392, 8192  # few output tiles, long k: splits over k
    ws = 16 * M * N * 4
    err, c1 = sampled_gemm_check(dtype, 0, 0, M, N, K, ws_bytes=ws, seed=5, rows=M)
    assert err < 1e-4, err
    _, c2 = sampled_gemm_check(dtype, 0, 0, M, N, K, ws_bytes=ws, seed=5, rows=8)
    assert np.array_equal(c1, c2)
    err0, c0 = sampled_gemm_check(dtype, 0, 0, M, N, K, ws_bytes=0, seed=5, rows=M)
    assert err0 < 1e-4
    assert not np.array_equal(c0, c1)  # the split path really ran (different summation order)


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0), (0, 1)])
@pytest.mark.parametrize("M,N,K", [(512, 1024, 8192), (1000, 2048, 4104), (96, 160, 16384), (64, 64, 512)])
def test_gemm_f32_rounding(akc, bkc, M, N, K):
    """fp32 sums take 256 products in a row (64 MFMAs of four in each of the two
    sets) before they join the totals, K / 512 of those: with each addition
    rounded by a uniform error of at most 2^-24 of the running sum, whose square
    grows evenly, the relative error is at most 2^-24 sqrt((256 + K / 512) / 6)."""
    r = U.rng(M + K)
    Am = r.standard_normal((M, K) if akc else (K, M)).astype(np.float32)
    Bm = r.standard_normal((N, K) if bkc else (K, N)).astype(np.float32)
    dA, dB, dC = U.dev_f32(Am), U.dev_f32(Bm), U.empty((M, N), "f32")
    A.atom_k_gemm(A.ATOM_F32, akc, bkc, A.ATOM_EPI_STORE, M, N, K, U.ptr(dA), Am.shape[1], U.ptr(dB), Bm.shape[1],
                  U.ptr(dC), N, stream=stream())
    U.sync()
    pick = np.sort(r.choice(M, min(M, 64), replace=False))
    ref = (Am if akc else Am.T)[pick].astype(np.float64) @ (Bm.T if bkc else Bm).astype(np.float64)
    err = np.linalg.norm(U.host(dC)[pick] - ref) / np.linalg.norm(ref)
    assert err <= 2.0**-24 * np.sqrt((256 + K / 512) / 6), err


@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0)])
@pytest.mark.parametrize("M,N,K,ranges", [(2024, 960, 5120, 8), (352, 3272, 7168, 8), (3152, 1008, 3968, 3),
                                          (536, 5488, 2944, 2), (96, 264, 16384, 16)])
def test_gemm_f32_result_rounding(akc, bkc, M, N, K, ranges):
    """fp32 results of few tiles of bf16 operands, given a workspace: no less exact than
    256-row tiles split until 192 workgroups run (or 128-row tiles in ranges of
    1024 k), which is rebuilt here: a product without workspace per range, summed
    in order in fp32.  Both errors are norms of M N independent ones, whose ratio
    has a standard deviation of about 1 / sqrt(M N): 2 % is more than three."""
    r = U.rng(M + N + K)
    Am = U.rep(r.standard_normal((M, K) if akc else (K, M)), "bf16")
    Bm = U.rep(r.standard_normal((N, K) if bkc else (K, N)), "bf16")
    dA, dB, dC, ws = U.dev(Am, "bf16"), U.dev(Bm, "bf16"), U.empty((M, N), "f32"), U.empty(16 << 20, "f32")
    A.atom_k_gemm(A.ATOM_BF16, akc, bkc, A.ATOM_EPI_STORE_F32, M, N, K, U.ptr(dA), Am.shape[1], U.ptr(dB),
                  Bm.shape[1], U.ptr(dC), N, stream=stream(), ws=U.ptr(ws), ws_bytes=64 << 20)
    step = (K // 32 + ranges - 1) // ranges * 32
    total = None
    for k0 in range(0, K, step):
        k1 = min(K, k0 + step)
        a = (dA[:, k0:k1] if akc else dA[k0:k1]).contiguous()
        b = (dB[:, k0:k1] if bkc else dB[k0:k1]).contiguous()
        part = U.empty((M, N), "f32")
        A.atom_k_gemm(A.ATOM_BF16, akc, bkc, A.ATOM_EPI_STORE_F32, M, N, k1 - k0, U.ptr(a), a.shape[1], U.ptr(b),
                      b.shape[1], U.ptr(part), N, stream=stream())
        U.sync()
        total = part if total is None else total + part
    ref = (dA if akc else dA.T).double() @ (dB.T if bkc else dB).double().contiguous()
    err, split = float((dC - ref).norm()), float((total - ref).norm())
    assert err <= 1.02 * split, (err, split)


def test_gemm_rejects_unsupported_shapes():
    t = U.empty((64, 64), "bf16")
    with pytest.raises(A.AtomError):  # K not a multiple of 8
        A.atom_k_gemm(A.ATOM_BF16, 1, 1, 0, 64, 64, 60, U.ptr(t), 64, U.ptr(t), 64, U.ptr(t), 64)
    with pytest.raises(A.AtomError):  # odd rows for a non-k-contiguous bf16 operand
        A.atom_k_gemm(A.ATOM_BF16, 0, 1, 0, 63, 64, 64, U.ptr(t), 64, U.ptr(t), 64, U.ptr(t), 64)


# ----------------------------------------------------------------- LayerNorm
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,d", [(37, 256), (130, 768), (17, 320), (5, 4096), (3, 5120), (4100, 256),
                                    (300, 2048), (1031, 5120), (77, 1088), (16, 8192), (41, 1024),
                                    # 512 blocks of rows, the last one partial: 256 threads up to 4096 columns
                                    (4091, 2112), (4091, 3072), (4091, 4096)])
def test_layernorm_fwd_bwd(dtype, rows, d):
    r = U.rng(rows + d)
    x = (r.standard_normal((rows, d)) * 2 + 0.5).astype(np.float32)
    g = U.rep(1 + 0.2 * r.standard_normal(d), dtype)
    b = U.rep(0.1 * r.standard_normal(d), dtype)
    dy = U.rep(r.standard_normal((rows, d)), dtype)
    dres0 = r.standard_normal((rows, d)).astype(np.float32)
    y_ref, (xhat, rstd) = gpt.layer_norm(x.astype(np.float64), g, b)
    dx_ref, dg_ref, db_ref = gpt.layer_norm_backward(dy.astype(np.float64), xhat, rstd, g)
    dx, dg_, db_ = U.dev_f32(x), U.dev(g, dtype), U.dev(b, dtype)
    y = U.empty((rows, d), dtype)
    mean, rs = U.empty(rows, "f32"), U.empty(rows, "f32")
    A.atom_k_layernorm_fwd(U.dt_code(dtype), U.ptr(dx), U.ptr(dg_), U.ptr(db_), U.ptr(y), U.ptr(mean), U.ptr(rs),
                           rows, d, stream())
    U.sync()
    assert U.rel_err(U.host(y), y_ref) < TOL_OUT[dtype]
    assert U.rel_err(U.host(rs), rstd[:, 0]) < 1e-5
    assert U.rel_err(U.host(mean), x.astype(np.float64).mean(axis=1)) < 1e-5
    for acc in (0, 1):
        ddy = U.dev(dy, dtype)
        dres = U.dev_f32(dres0)
        lp = U.empty((rows, d), dtype)
        dgam, dbet = U.empty(d, "f32"), U.empty(d, "f32")
        part = U.empty(A.atom_k_layernorm_bwd_part_floats(rows, d), "f32")
        A.atom_k_layernorm_bwd(U.dt_code(dtype), U.ptr(ddy), U.ptr(dx), U.ptr(mean), U.ptr(rs), U.ptr(dg_),
                               U.ptr(dres), U.ptr(lp), acc, U.ptr(dgam), U.ptr(dbet), U.ptr(part), rows, d, stream())
        U.sync()
        ref = dx_ref + (dres0 if acc else 0)
        assert U.rel_err(U.host(dres), ref) < 1e-4
        assert U.rel_err(U.host(lp), ref) < TOL_OUT[dtype]
        assert U.rel_err(U.host(dgam), dg_ref) < 1e-4
        assert U.rel_err(U.host(dbet), db_ref) < 1e-4


# ----------------------------------------------------------------- attention
# ragged T, T = 1, several heads and batches, and long loops (many key and
# query tiles through the two-stage pipelines) at both head sizes; B*H a
# multiple of 8 takes the per-XCD split of the heads in the work-item order
ATTN_CASES = [(2, 100, 2, 64), (1, 128, 3, 128), (1, 1, 1, 64), (2, 200, 1, 128), (1, 64, 2, 64), (1, 257, 1, 64),
              (1, 1000, 2, 128), (2, 600, 1, 64), (2, 300, 4, 64), (1, 520, 16, 128), (4, 130, 6, 64)] + [
    # above every rule for small problems: the 128-row kernels in forward and backward
    (36, 130, 12, 64), (18, 333, 12, 64), (18, 130, 10, 128), (11, 333, 8, 128)]


def attn_inputs(B, T, H, dh, dtype, seed):
    r = U.rng(seed)
    d = H * dh
    qkv = U.rep(r.standard_normal((B * T, 3 * d)), dtype)
    do = U.rep(r.standard_normal((B * T, d)), dtype)
    return qkv, do


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,T,H,dh", ATTN_CASES)
def test_attention_fwd_bwd(dtype, B, T, H, dh):
    d = H * dh
    qkv, do = attn_inputs(B, T, H, dh, dtype, seed=B * 1000 + T + H + dh)
    o_ref, lse_ref = gpt.causal_attention(qkv.reshape(B, T, 3 * d).astype(np.float64), H)
    dqkv_ref = gpt.causal_attention_backward(do.reshape(B, T, d).astype(np.float64),
                                             qkv.reshape(B, T, 3 * d).astype(np.float64), H)
    dq = U.dev(qkv, dtype)
    o = U.empty((B * T, d), dtype)
    lse = U.empty((B, H, T), "f32")
    A.atom_k_attn_fwd(U.dt_code(dtype), U.ptr(dq), U.ptr(o), U.ptr(lse), B, T, H, dh, stream())
    U.sync()
    # bf16: P is rounded to bf16 before the P V product, then o is stored in bf16
    tol = 1.5e-2 if dtype == "bf16" else 1e-5
    assert U.rel_err(U.host(o), o_ref.reshape(B * T, d)) < tol
    assert np.max(np.abs(U.host(lse) - lse_ref)) < 1e-4 * max(1.0, np.max(np.abs(lse_ref)))
    ddo = U.dev(do, dtype)
    delta = U.empty((B, H, T), "f32")
    dqkv = U.empty((B * T, 3 * d), dtype)
    A.atom_k_attn_bwd(U.dt_code(dtype), U.ptr(dq), U.ptr(o), U.ptr(ddo), U.ptr(lse), U.ptr(delta), U.ptr(dqkv), B, T,
                      H, dh, stream())
    U.sync()
    got = U.host(dqkv).reshape(B, T, 3 * d)
    tol = 2e-2 if dtype == "bf16" else 1e-4
    for part in range(3):
        sl = slice(part * d, (part + 1) * d)
        assert U.rel_err(got[:, :, sl], dqkv_ref[:, :, sl]) < tol, part


def test_attention_cases_take_every_variant():
    """The cases above reach the split and unsplit small kernels and the large ones at both head sizes."""
    for dh in (64, 128):
        seen = {U.attn_choice(*c) for c in ATTN_CASES if c[3] == dh}
        for f in (0, 2):  # forward, backward
            assert {v[f:f + 2] for v in seen} == {(False, False), (True, False), (True, True)}, (dh, f)


@pytest.mark.parametrize("T,BH,small", [(64, 1280, True), (64, 1281, False), (128, 384, True), (128, 385, False),
                                        (256, 192, True), (256, 193, False), (512, 96, True), (512, 97, False),
                                        (576, 142, True), (576, 143, False)])
def test_attention_forward_variant(T, BH, small):
    """Where the forward of d_h 64 takes 64-row workgroups: up to five per CU, three at 65 to 512 rows."""
    assert U.attn_choice(BH, T, 1, 64)[0] == small


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("T", [1, 63, 64, 65, 128, 129, 333, 2048, 2049])
def test_attention_small_and_large_problems_agree(T, dh):
    """Few heads take workgroups of 64 rows and one backward launch, many take 128
    rows and two launches (as does the backward beyond 2048 rows); a head's
    arithmetic is the same in both, so its results are the same bits.  Very few
    heads of more than 256 rows also split the tiles between two groups of
    waves: fp32 sums in another order and another reference maximum, so P and
    dS round differently to bf16 (2^-9 each, before the outputs' own 2^-9)."""
    H = 4
    n64 = H * ((T + 63) // 64)
    middle = (256 if dh == 128 else 512) // n64 + 1  # past the split rules
    copies = 1280 // n64 + 1                         # past every small rule
    d = H * dh
    qkv, do = attn_inputs(1, T, H, dh, "bf16", seed=T + dh)
    outs = []
    for B in (1, middle, copies):
        dq, ddo = U.dev(qkv, "bf16").repeat(B, 1), U.dev(do, "bf16").repeat(B, 1)
        o, lse, delta = U.empty((B * T, d), "bf16"), U.empty((B, H, T), "f32"), U.empty((B, H, T), "f32")
        dqkv = U.empty((B * T, 3 * d), "bf16")
        A.atom_k_attn_fwd(U.dt_code("bf16"), U.ptr(dq), U.ptr(o), U.ptr(lse), B, T, H, dh, stream())
        A.atom_k_attn_bwd(U.dt_code("bf16"), U.ptr(dq), U.ptr(o), U.ptr(ddo), U.ptr(lse), U.ptr(delta), U.ptr(dqkv),
                          B, T, H, dh, stream())
        U.sync()
        outs.append([x.reshape(B, -1) for x in (o, lse, delta, dqkv)])
    for few, some, many in zip(*outs):
        assert (some == some[:1]).all() and (many == some[:1]).all()
        if T <= 256:
            assert (few == many[:1]).all()
        else:
            assert U.rel_err(U.host(few[0]), U.host(many[0])) < 2.0**-8


# ------------------------------------------------------- cross-entropy etc.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,V,ld", [(33, 1000, 1024), (5, 50257, 50304), (1, 7, 128), (3, 4097, 4100), (4, 1003, 1003),
                                      (2, 65000, 65536)])
def test_cross_entropy_rows(dtype, rows, V, ld):
    r = U.rng(rows + V)
    z = np.zeros((rows, ld), np.float32)
    z[:, :V] = (r.standard_normal((rows, V)) * 3).astype(np.float32)
    y = r.integers(0, V, rows).astype(np.int32)
    scale = 1.0 / (rows * 4)
    loss_ref, dz_ref = gpt.cross_entropy_rows(z[:, :V].astype(np.float64), y, scale)
    dzt = U.dev_f32(z)
    dy = U.dev_i32(y)
    dz = U.dev(np.full((rows, ld), 7.0, np.float32), dtype)
    loss = U.empty(rows, "f32")
    A.atom_k_xent(U.dt_code(dtype), U.ptr(dzt), ld, U.ptr(dy), U.ptr(dz), ld, U.ptr(loss), rows, V, scale, stream())
    U.sync()
    assert U.rel_err(U.host(loss), loss_ref) < 1e-5
    g = U.host(dz)
    assert U.rel_err(g[:, :V], dz_ref) < TOL_OUT[dtype] + 1e-5
    assert np.all(g[:, V:] == 0)


def test_logits_larger_than_the_cache():
    """fp32 logits of more than 256 MB (1400 x 50304 here) are stored, and read and
    their gradient stored, past the caches: product and cross-entropy against the
    oracle on sampled rows, and the gradient's padding columns."""
    t = U.torch()
    rows, V, ld, K = 1400, 50257, 50304, 72
    g = t.Generator(device="cuda").manual_seed(9)
    a = t.randn(rows, K, device="cuda", generator=g).to(t.bfloat16)
    w = t.randn(ld, K, device="cuda", generator=g).to(t.bfloat16)
    z = t.empty(rows, ld, device="cuda")
    dz = t.full((rows, ld), 7.0, device="cuda", dtype=t.bfloat16)
    y = t.randint(0, V, (rows,), device="cuda", generator=g, dtype=t.int32)
    loss = t.empty(rows, device="cuda")
    A.atom_k_gemm(A.ATOM_BF16, 1, 1, A.ATOM_EPI_STORE_F32, rows, ld, K, U.ptr(a), K, U.ptr(w), K, U.ptr(z), ld,
                  stream=stream())
    A.atom_k_xent(A.ATOM_BF16, U.ptr(z), ld, U.ptr(y), U.ptr(dz), ld, U.ptr(loss), rows, V, 0.5, stream())
    U.sync()
    pick = np.array([0, 1, 700, 1398, 1399])
    zp = U.host(z[pick])
    assert U.rel_err(zp, U.host(a[pick]) @ U.host(w).T) < 1e-4
    loss_ref, dz_ref = gpt.cross_entropy_rows(zp[:, :V], y.cpu().numpy()[pick], 0.5)
    assert U.rel_err(U.host(loss[pick]), loss_ref) < 1e-5
    got = U.host(dz[pick])
    assert U.rel_err(got[:, :V], dz_ref) < TOL_OUT["bf16"]
    assert np.all(got[:, V:] == 0)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_colsum(dtype):
    r = U.rng(3)
    for rows, cols in ((1000, 300), (64, 2304), (7, 5), (4100, 64), (130, 12292), (33, 1030)):
        x = U.rep(r.standard_normal((rows, cols)), dtype)
        dx = U.dev(x, dtype)
        out = U.empty(cols, "f32")
        part = U.empty(A.atom_k_colsum_part_floats(rows, cols), "f32")
        A.atom_k_colsum(U.dt_code(dtype), U.ptr(dx), rows, cols, U.ptr(out), U.ptr(part), stream())
        U.sync()
        assert U.rel_err(U.host(out), x.astype(np.float64).sum(axis=0)) < 1e-5


def chain_sum(rows):
    """fp32 sum of the given rows, one after the other."""
    s = np.zeros_like(rows[0])
    for r in rows:
        s = s + r
    return s


@pytest.mark.parametrize("cols", [256, 4096, 4100, 20480])
@pytest.mark.parametrize("rows", [1, 16, 64, 65, 100, 520, 1024, 1025])
def test_colsum_rounding(rows, cols):
    """Up to 1024 rows the sum is one launch; its error against 64 bits is no larger
    than that of the order beyond (partials of 16 rows, summed in 16 slices),
    computed here in fp32.  Both are norms of `cols` independent errors, whose
    ratio has a standard deviation of 1 / sqrt(cols): three of them."""
    x = U.rng(rows + cols).standard_normal((rows, cols)).astype(np.float32)
    ref = x.astype(np.float64).sum(axis=0)
    parts = [chain_sum(x[i:i + 16]) for i in range(0, rows, 16)]
    two = chain_sum([chain_sum(parts[i::16]) for i in range(min(16, len(parts)))])
    dx, out = U.dev_f32(x), U.empty(cols, "f32")
    part = U.empty(A.atom_k_colsum_part_floats(rows, cols), "f32")
    A.atom_k_colsum(A.ATOM_F32, U.ptr(dx), rows, cols, U.ptr(out), U.ptr(part), stream())
    U.sync()
    err = np.linalg.norm(U.host(out) - ref)
    assert err <= (1 + 3 / np.sqrt(cols)) * np.linalg.norm(two.astype(np.float64) - ref)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_embedding_forward(dtype):
    r = U.rng(4)
    V, T, d, B = 300, 50, 128, 3
    wte = U.rep(r.standard_normal((V, d)), dtype)
    wpe = U.rep(r.standard_normal((T, d)), dtype)
    tok = r.integers(0, V, (B, T)).astype(np.int32)
    ref = gpt.embed_forward(tok, {"wte": wte, "wpe": wpe}).reshape(B * T, d)
    # every device buffer stays referenced until the kernel has finished
    dtok, dwte, dwpe = U.dev_i32(tok), U.dev(wte, dtype), U.dev(wpe, dtype)
    x = U.empty((B * T, d), "f32")
    A.atom_k_embed_fwd(U.dt_code(dtype), U.ptr(dtok), U.ptr(dwte), U.ptr(dwpe), U.ptr(x), B * T, T, V, d, stream())
    U.sync()
    assert U.rel_err(U.host(x), ref) < 1e-7
    # an id outside [0, V) yields a NaN row, never an out-of-range read
    bad = tok.copy()
    bad[1, 3] = V
    bad[2, 0] = -5
    dbad = U.dev_i32(bad)
    A.atom_k_embed_fwd(U.dt_code(dtype), U.ptr(dbad), U.ptr(dwte), U.ptr(dwpe), U.ptr(x), B * T, T, V, d, stream())
    U.sync()
    got = U.host(x).reshape(B, T, d)
    assert np.all(np.isnan(got[1, 3])) and np.all(np.isnan(got[2, 0]))
    assert np.array_equal(np.isnan(got).any(axis=2), (bad < 0) | (bad >= V))
