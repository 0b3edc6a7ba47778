"""GPU parity of the FP32 matrix-core product and the float64 product postcondition."""
import numpy as np
import pytest

import oracle
import workloads as W
from oracle import matrix as OM
from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(sg):
    return sg.Context(0)


def gemm(sg, ctx, A, B):
    t = to_dev({"A": A, "B": B})
    a, b = ctx.wrap(t["A"]), ctx.wrap(t["B"])
    c = a.matmul(b)
    ctx.execute(c)
    return c.to_host().reshape(A.shape[0], B.shape[1])


@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (128, 16, 128), (200, 300, 130), (257, 129, 513), (512, 1024, 256),
                                   (1200, 64, 300), (2176, 48, 1040), (1536, 32, 256)])
def test_gemm_small_within_rounding_bound(sg, ctx, M, K, N):
    say("gemm", M, K, N)
    A = W.normal_f32(M * K, 31, 1.0 / np.sqrt(K)).reshape(M, K)
    B = W.normal_f32(K * N, 32, 1.0 / np.sqrt(K)).reshape(K, N)
    C = gemm(sg, ctx, A, B)
    C64 = OM.matmul64(A, B)
    bound = OM.gamma(K) * OM.matmul_bound(A, B)
    assert np.all(np.abs(C.astype(np.float64) - C64) <= bound)


@pytest.mark.parametrize("M,K,N", [(1, 4096, 1), (64, 4096, 64), (65, 1000, 3), (63, 31, 64), (64, 32, 65), (3, 33, 129),
                                   (127, 255, 1), (130, 257, 2), (1000, 1531, 777), (513, 640, 511), (2049, 33, 2049),
                                   (2050, 17, 2047), (2048, 16, 2048), (4096, 1, 1024)])
def test_gemm_tiles_parts_and_tails(sg, ctx, M, K, N):
    """64- and 128-wide tiles, products cut along K, slices and rows that end anywhere, and a
    row of NaN and a column of infinities that must not reach other entries."""
    say("gemm tiles", M, K, N)
    A = W.normal_f32(M * K, 31, 1.0 / np.sqrt(K)).reshape(M, K)
    B = W.normal_f32(K * N, 32, 1.0 / np.sqrt(K)).reshape(K, N)
    C64 = OM.matmul64(A, B)
    bound = OM.gamma(K) * OM.matmul_bound(A, B)
    assert np.all(np.abs(gemm(sg, ctx, A, B).astype(np.float64) - C64) <= bound)
    A[-1] = np.nan
    B[:, -1] = np.inf
    C = gemm(sg, ctx, A, B)
    assert np.all(np.isnan(C[-1])) and not np.any(np.isfinite(C[:, -1]))
    assert np.all(np.abs(C[:-1, :-1].astype(np.float64) - C64[:-1, :-1]) <= bound[:-1, :-1])


@pytest.mark.parametrize("M,K,N", [(64, k, n) for n in (1, 2, 3) for k in (33, 34, 35, 66)] +
                         [(40_000, k, 1) for k in (17, 18, 19)])
def test_gemm_few_columns_behind_a_whole_slice(sg, ctx, M, K, N):
    """One to three rows of B behind the last whole slice of K, and rows shorter than 16 bytes: the
    slice's last loads end at B's end.  Whole numbers, so the product is exact."""
    say("gemm few columns", M, K, N)
    g = np.random.default_rng(M + K + N)
    A = g.integers(-8, 9, size=(M, K)).astype(np.float32)
    B = g.integers(-8, 9, size=(K, N)).astype(np.float32)
    assert np.array_equal(gemm(sg, ctx, A, B), (A.astype(np.int64) @ B.astype(np.int64)).astype(np.float32))


@pytest.mark.parametrize("M,K,N", [(2048, 512, 1700), (1921, 513, 1793), (2050, 1000, 2047), (3713, 520, 3800)])
def test_gemm_parts_of_values(sg, ctx, M, K, N):
    """The product on bfloat16 parts (tiles of 128 and 256, slices and rows that end anywhere):
    the float32 bound, exact products of values by powers of two, and magnitudes at the limits
    of the parts' range."""
    say("gemm parts", M, K, N)
    A = W.normal_f32(M * K, 31, 1.0 / np.sqrt(K)).reshape(M, K)
    B = W.normal_f32(K * N, 32, 1.0 / np.sqrt(K)).reshape(K, N)
    A[:, ::3] *= np.float32(2.0 ** 40)
    B[::3] *= np.float32(2.0 ** -25)
    B[1::3] *= np.float32(2.0 ** 50)
    A[np.abs(A) < 2.0 ** -40] = 0
    B[np.abs(B) < 2.0 ** -40] = 0
    C64, bound = OM.matmul64(A, B), OM.gamma(K) * OM.matmul_bound(A, B)
    assert np.all(np.abs(gemm(sg, ctx, A, B).astype(np.float64) - C64) <= bound)
    S = np.zeros((K, N), np.float32)
    S[np.arange(N) % K, np.arange(N)] = np.float32(2.0) ** (np.arange(N) % 61 - 30)
    assert np.array_equal(gemm(sg, ctx, A, S), A[:, np.arange(N) % K] * S[np.arange(N) % K, np.arange(N)])


@pytest.mark.parametrize("value", [np.nan, np.inf, 3e38, 2.0 ** 60, 2.0 ** -41, 1e-42])
@pytest.mark.parametrize("side", ["A", "B"])
def test_gemm_value_without_parts(sg, ctx, value, side):
    """One entry outside the parts' range: the product is that of the FP32 kernel."""
    M, K, N = 1920, 512, 1920
    say("gemm without parts", value, side)
    A = W.normal_f32(M * K, 31, 1.0 / np.sqrt(K)).reshape(M, K)
    B = W.normal_f32(K * N, 32, 1.0 / np.sqrt(K)).reshape(K, N)
    (A if side == "A" else B)[300, 77] = value
    C = gemm(sg, ctx, A, B).astype(np.float64)
    with np.errstate(invalid="ignore", over="ignore"):
        C64, bound = OM.matmul64(A, B), OM.gamma(K) * OM.matmul_bound(A, B)
    ok = np.isfinite(C64) & (np.abs(C64) < 3e38)
    assert np.array_equal(np.isnan(C[~ok]), np.isnan(C64[~ok]))
    assert np.all(np.abs(C[ok] - C64[ok]) <= bound[ok])


@pytest.mark.parametrize("M,K,N", [(200, 300, 130), (1000, 1531, 777), (2048, 512, 1700), (3713, 520, 3800)])
@pytest.mark.parametrize("side", ["A", "B"])
def test_gemm_single_products_are_rounded_once(sg, ctx, M, K, N, side):
    """One nonzero entry per row of A (or column of B), of any value: each entry of the product is
    one float32 product, rounded to nearest, at every size (no operand is shortened)."""
    say("gemm single products", M, K, N, side)
    A = W.normal_f32(M * K, 31).reshape(M, K)
    B = W.normal_f32(K * N, 32).reshape(K, N)
    if side == "A":
        k, keep = np.arange(M) * 7 % K, np.zeros((M, K), bool)
        keep[np.arange(M), k] = True
        A[~keep] = 0
        want = A[np.arange(M), k][:, None] * B[k]
    else:
        k, keep = np.arange(N) * 7 % K, np.zeros((K, N), bool)
        keep[k, np.arange(N)] = True
        B[~keep] = 0
        want = A[:, k] * B[k, np.arange(N)][None]
    assert np.array_equal(gemm(sg, ctx, A, B), want)


def test_gemm_empty_inner_dimension(sg, ctx):
    import torch
    c = ctx.wrap(torch.zeros((5, 0), device="cuda")).matmul(ctx.wrap(torch.zeros((0, 7), device="cuda")))
    ctx.execute(c)
    assert np.array_equal(c.to_host(), np.zeros(35, np.float32))


def exact_up_to_zero_sign(got, want):
    """Bit-exact, except that a -0 entry may come out +0: the sum -0 + (+0) is +0 in IEEE
    arithmetic, in the float64 oracle as on the matrix cores."""
    nz = want != 0
    return np.array_equal(got, want) and np.array_equal(got[nz].view(np.uint32), want[nz].view(np.uint32))


def test_gemm_identity_and_permutation_bit_exact(sg, ctx):
    n = 4096
    inp = W.cfg3_inputs(n, case="identity")
    say("gemm identity 4096")
    C = gemm(sg, ctx, inp["A"], inp["B"])
    assert exact_up_to_zero_sign(C, inp["A"])
    assert np.array_equal(C, oracle.matmul64(inp["A"], inp["B"]).astype(np.float32))
    P, perm = W.permutation_matrix_f32(n, 34)
    say("gemm permutation 4096")
    C = gemm(sg, ctx, inp["A"], P)
    assert exact_up_to_zero_sign(C, np.ascontiguousarray(inp["A"][:, perm]))


def test_gemm_integer_matrices_exact(sg, ctx):
    g = np.random.default_rng(5)
    A = g.integers(-8, 9, size=(384, 4096)).astype(np.float32)
    B = g.integers(-8, 9, size=(4096, 256)).astype(np.float32)
    C = gemm(sg, ctx, A, B)
    assert np.array_equal(C, (A.astype(np.int64) @ B.astype(np.int64)).astype(np.float32))


def test_cfg3_full_size_product_and_contract(sg, ctx):
    """4096^3 product with the product postcondition; sampled rows against float64."""
    n = 4096
    spec = W.cfg3_spec(n)
    inp = W.cfg3_inputs(n)
    say("cfg3 full")
    t = to_dev(inp)
    built = sg.build_spec(ctx, spec, t)
    status, verdicts = built.program.execute()
    assert status == "ok" and verdicts[0].holds == 1 and verdicts[0].first_index == -1
    C = built["C"].to_host().reshape(n, n)
    rows = np.random.default_rng(0).choice(n, 48, replace=False)
    C64 = inp["A"][rows].astype(np.float64) @ inp["B"].astype(np.float64)
    bound = OM.gamma(n) * (np.abs(inp["A"][rows]).astype(np.float64) @ np.abs(inp["B"]).astype(np.float64))
    err = np.abs(C[rows].astype(np.float64) - C64)
    assert np.all(err <= bound)
    rel = np.linalg.norm(err) / np.linalg.norm(C64)
    say("relative Frobenius error on sampled rows", rel)
    # random-sign float32 accumulation: error grows like u * sqrt(K) (u = 2^-24, K = 4096)
    assert rel < 4 * 2.0 ** -24 * np.sqrt(n)
    # the check's measure is a ratio well inside the tolerance
    assert 0 < verdicts[0].measure < OM.gamma(n)


def _product_spec(M, K, N, nvec):
    return {"inputs": [{"name": "A", "dtype": "f32", "rows": M, "cols": K},
                       {"name": "B", "dtype": "f32", "rows": K, "cols": N},
                       {"name": "C", "dtype": "f32", "rows": M, "cols": N},
                       {"name": "R", "dtype": "f32", "rows": nvec, "cols": N}],
            "nodes": [],
            "contracts": [{"kind": "ensure", "check": "product", "node": "C", "a": "A", "b": "B", "r": "R"}],
            "outputs": []}


@pytest.mark.parametrize("nvec", [1, 2, 4])
def test_product_check_parity_with_oracle(sg, ctx, nvec):
    g = np.random.default_rng(8 + nvec)
    M, K, N = 300, 517, 259
    A = g.integers(-8, 9, size=(M, K)).astype(np.float32)
    B = g.integers(-8, 9, size=(K, N)).astype(np.float32)
    R = g.integers(-8, 9, size=(nvec, N)).astype(np.float32)
    C = (A.astype(np.int64) @ B.astype(np.int64)).astype(np.float32)
    spec = _product_spec(M, K, N, nvec)
    for case in ("exact", "perturbed", "nan"):
        Cc = C.copy()
        if case == "perturbed":
            Cc[211, 17] += 1000.0
            Cc[57, 3] += 1000.0
        if case == "nan":
            Cc[99, 9] = np.nan
        inp = {"A": A, "B": B, "C": Cc, "R": R}
        say("product", nvec, case)
        built = sg.build_spec(ctx, spec, to_dev(inp))
        status, verdicts = built.program.execute()
        ref = oracle.evaluate(spec, inp)
        assert status == ref.status, (status, ref.status)
        v, r = verdicts[0], ref.verdicts[0]
        assert (v.holds, v.first_index) == (r.holds, r.first_index), (v, r)
        if case == "exact":
            assert v.measure == 0.0


def test_gemm_then_stream_pass(sg, ctx):
    """A matrix product feeding a fused element-wise chain (sum of ReLU-like filter)."""
    M = K = N = 256
    A = W.normal_f32(M * K, 1).reshape(M, K)
    B = W.normal_f32(K * N, 2).reshape(K, N)
    t = to_dev({"A": A, "B": B})
    a, b = ctx.wrap(t["A"]), ctx.wrap(t["B"])
    c = a.matmul(b)
    pos = c.filter(sg.Pred.cmp("gt", 0.0))
    s = pos.reduce("count")
    prog = sg.Program(ctx)
    prog.add_root(s)
    prog.add_root(c)
    status, _ = prog.execute()
    Cg = c.to_host()
    assert s.scalar()[1] == int(np.count_nonzero(Cg > 0))


@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (15, 513, 17), (17, 511, 1023), (1000, 1531, 777),  # made where staged
                                   (1023, 1025, 1024), (2047, 1024, 1025), (3, 1 << 18, 16), (1 << 18, 3, 16)])
def test_product_check_shapes(sg, ctx, M, K, N):
    """Row and column remainders of the check's passes, on both sides of the size from which the
    right-hand sides are written first.  Entries are whole numbers, so every sum is exact: the true
    product has measure 0, and with positive probes a wrong row is reported at its index."""
    g = np.random.default_rng(M + K + N)
    A = g.integers(-2, 3, size=(M, K)).astype(np.float32)
    B = g.integers(-2, 3, size=(K, N)).astype(np.float32)
    R = g.integers(1, 4, size=(3, N)).astype(np.float32)
    C = (A.astype(np.float64) @ B.astype(np.float64)).astype(np.float32)
    for row in (None, 0, M // 2, M - 1):
        Cc = C.copy()
        if row is not None:
            Cc[row, N - 1] += 1e6
            Cc[M - 1, 0] = np.nan
        say("product check", M, K, N, row)
        built = sg.build_spec(ctx, _product_spec(M, K, N, 3), to_dev({"A": A, "B": B, "C": Cc, "R": R}))
        v = built.program.execute()[1][0]
        if row is None:
            assert v.holds and v.measure == 0.0
        else:
            assert not v.holds and v.first_index == row
