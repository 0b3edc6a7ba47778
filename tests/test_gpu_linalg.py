"""GPU parity of the matrix/vector API of Sections 2.1 and 3.4 (transpose, right/left
matrix-vector products, Listing 1's fused transpose-product) and of compwise_divide with its
built-in clauses (Listing 2), on both the interpreter and kernels compiled for the program."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import compare, run_spec, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[False, True], ids=["interp", "spec"])
def ctx(sg, request):
    c = sg.Context(0)
    c.set_specialize(request.param)
    return c


@pytest.mark.parametrize("r,c", [(1, 1), (1, 100), (100, 1), (63, 65), (64, 64), (1000, 777), (1000, 1000), (100, 4096),
                                 (4096, 4096)])
def test_transpose_bit_exact_in_a_chain(sg, ctx, r, c):
    say("transpose", r, c)
    M = W.normal_f32(r * c, 3).reshape(r, c)
    spec = {"inputs": [{"name": "M", "dtype": "f32", "rows": r, "cols": c}],
            "nodes": [{"name": "T", "op": "transpose", "src": "M"},
                      {"name": "k", "op": "filter", "src": "T", "pred": ["cmp", "gt", 0.5]},
                      {"name": "s", "op": "reduce", "src": "k", "red": "sum"}],
            "contracts": [{"kind": "ensure", "check": "for_all", "node": "T", "pred": ["isfinite"]},
                          {"kind": "ensure", "check": "exists", "node": "T", "pred": ["cmp", "gt", 3.0]}],
            "outputs": ["T", "k", "s"]}
    built, status, verdicts, _ = run_spec(sg, ctx, spec, {"M": M})
    compare(spec, built, status, verdicts, oracle.evaluate(spec, {"M": M}))


@pytest.mark.parametrize("r,c", [(1, 1), (7, 300), (300, 7), (1000, 1000), (4096, 4096), (10000, 10), (5, 100000)])
@pytest.mark.parametrize("side", ["right", "left"])
def test_matvec(sg, ctx, r, c, side):
    say("matvec", side, r, c)
    M = W.normal_f32(r * c, 4).reshape(r, c)
    v = W.normal_f32(c if side == "right" else r, 5)
    spec = {"inputs": [{"name": "M", "dtype": "f32", "rows": r, "cols": c},
                       {"name": "v", "dtype": "f32", "n": v.size}],
            "nodes": [{"name": "y", "op": "matvec", "m": "M", "v": "v", "side": side}],
            "contracts": [], "outputs": ["y"]}
    built, status, verdicts, _ = run_spec(sg, ctx, spec, {"M": M, "v": v})
    compare(spec, built, status, verdicts, oracle.evaluate(spec, {"M": M, "v": v}))


def test_listing1_transpose_right_multiply(sg, ctx):
    """matrix.transpose.right_multiply(vector): planned as a left product of the matrix (the
    transpose is not materialized); rows = matrix.columns, columns = 1; the vector's count must
    equal the matrix's rows."""
    r, c = 3000, 1700
    M = W.normal_f32(r * c, 6).reshape(r, c)
    v = W.normal_f32(r, 7)
    spec = {"inputs": [{"name": "M", "dtype": "f32", "rows": r, "cols": c},
                       {"name": "v", "dtype": "f32", "n": r}],
            "nodes": [{"name": "T", "op": "transpose", "src": "M"},
                      {"name": "y", "op": "matvec", "m": "T", "v": "v", "side": "right"}],
            "contracts": [], "outputs": ["y"]}
    ctx.set_timing(True)
    ctx.timing_reset()
    try:
        built, status, verdicts, _ = run_spec(sg, ctx, spec, {"M": M, "v": v})
        assert ctx.timing("transpose")[1] == 0  # fused away
    finally:
        ctx.set_timing(False)
    compare(spec, built, status, verdicts, oracle.evaluate(spec, {"M": M, "v": v}))
    assert built["y"].to_host().size == c
    t = to_dev({"M": M, "w": W.normal_f32(c, 8)})
    with pytest.raises(sg.SafeGPUError) as e:
        ctx.wrap(t["M"]).transpose().right_multiply(ctx.wrap(t["w"]))  # require matrix.rows = vector.count
    assert e.value.status_name == "shape"


def div_spec(n):
    return {"inputs": [{"name": "a", "dtype": "f32", "n": n}, {"name": "b", "dtype": "f32", "n": n}],
            "nodes": [{"name": "q", "op": "zip", "a": "a", "b": "b", "binop": "div"},
                      {"name": "e", "op": "map", "src": "q", "fn": ["affine", 0.3, 0.7]},
                      {"name": "k", "op": "filter", "src": "e", "pred": ["cmp", "gt", 0.0]},
                      {"name": "s", "op": "reduce", "src": "k", "red": "sum"}],
            "contracts": [{"kind": "ensure", "check": "for_all", "node": "q", "pred": ["isfinite"]}],
            "outputs": ["q", "k", "s"]}


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("case", ["ok", "zero", "nan", "tiny", "bigratio"])
def test_compwise_divide_with_builtin_clauses(sg, ctx, fused, case):
    n = 200_003
    a = W.normal_f32(n, 9)
    b = W.normal_f32(n, 10)
    if case == "zero":
        b[[1234, 99999]] = [0.0, -0.0]
    elif case == "nan":
        b[500] = np.nan
    elif case == "tiny":
        a[::97] = 1e-30
        b[::97] = 1e15  # quotients in the subnormal range
    elif case == "bigratio":
        a[::101] = 3e38
        b[::101] = 1e-3  # overflow: the product cannot give a back
    say("divide", case, fused)
    ctx.set_fusion(fused)
    try:
        spec = div_spec(n)
        built, status, verdicts, _ = run_spec(sg, ctx, spec, {"a": a, "b": b})
    finally:
        ctx.set_fusion(True)
    ref = oracle.evaluate(spec, {"a": a, "b": b})
    assert len(verdicts) == 3  # require b /= 0, ensure quotient, then the user's clause
    compare(spec, built, status, verdicts, ref)
    if case == "zero":
        assert status == "pre_violated" and verdicts[0].first_index == 1234
    with pytest.raises(sg.SafeGPUError) as e:
        ctx.wrap(to_dev({"i": np.ones(4, np.int32)})["i"]).zip(ctx.wrap(to_dev({"j": np.ones(4, np.int32)})["j"]), "div")
    assert e.value.status_name == "dtype"


@pytest.mark.parametrize("rows,cols", [(1, 1), (3, 1023), (3, 1024), (3, 1025), (4095, 5), (4096, 5), (4097, 1030), (31, 257),
                                       (33, 2049), (100, 255), (65, 4099), (2, 5003), (300, 3)])
@pytest.mark.parametrize("offset", [0, 1])
def test_matvec_row_and_column_edges(sg, ctx, rows, cols, offset):
    """Rows shared by one or four waves, stretches and chunks that end anywhere, unaligned rows:
    the float64 sum of exact products, rounded once."""
    import torch
    say("matvec edges", rows, cols, offset)
    M = W.normal_f32(rows * cols, 71).reshape(rows, cols)
    v, u = W.normal_f32(cols, 72), W.normal_f32(rows, 73)
    dev = torch.from_numpy(np.concatenate([np.zeros(offset, np.float32), M.ravel()])).cuda()[offset:].view(rows, cols)
    m = ctx.wrap(dev)
    tv, tu = to_dev({"v": v, "u": u}).values()
    y, z = m.right_multiply(ctx.wrap(tv)), m.left_multiply(ctx.wrap(tu))
    ctx.execute(y, z)
    for got, a, b in ((y.to_host(), M, v), (z.to_host(), M.T, u)):
        ex = a.astype(np.float64) @ b.astype(np.float64)
        ab = np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64)
        # half an ulp of the result, and the float64 additions of both sides
        assert np.all(np.abs(got.astype(np.float64).ravel() - ex) <= 2.0 ** -24 * np.abs(ex) + 2.0 ** -40 * ab)


@pytest.mark.parametrize("rows", [4095, 4096, 4111])
@pytest.mark.parametrize("cols", [1, 3, 4, 5, 63, 64, 65, 511, 512, 513, 1027])
def test_matvec_short_rows(sg, ctx, rows, cols):
    """Rows of 16 lanes each, at the limits of that form and a last block cut short."""
    test_matvec_row_and_column_edges(sg, ctx, rows, cols, 0)


@pytest.mark.parametrize("rows,cols", [(64, 64), (128, 192), (130, 67), (257, 1028), (3, 5)])
def test_checks_of_a_transposed_matrix(sg, ctx, rows, cols):
    """Class and range tests of a transpose, evaluated while it is made: the first failing index
    in the transpose's order, on the same program as elements start and stop failing."""
    import torch
    say("transpose checks", rows, cols)
    M = W.normal_f32(rows * cols, 81).reshape(rows, cols)
    t = torch.from_numpy(M.copy()).cuda()
    T = ctx.wrap(t).transpose()
    p = sg.Program(ctx)
    p.add_root(T)
    p.ensure_for_all(T, sg.Pred.isfinite())
    p.ensure_for_all(T, sg.Pred.in_range(-50.0, 50.0))
    for bad in ([], [(0, 0, np.nan)], [], [(rows - 1, cols - 1, -np.inf)], [(rows // 2, cols // 3, 51.0)], [],
                [(rows - 1, 0, -51.0), (1, cols // 2, np.inf)]):
        A = M.copy()
        for r, c, x in bad:
            A[r, c] = x
        t.copy_(torch.from_numpy(A))
        status, v = p.execute()
        flat = A.T.ravel()
        for got, ok in zip(v, (np.isfinite(flat), (flat >= -50) & (flat <= 50))):
            first = int(np.argmin(ok)) if not ok.all() else -1
            assert (got.holds, got.first_index) == (int(ok.all()), first)
        assert status == ("ok" if not bad else "post_violated")
        assert np.array_equal(T.to_host().view(np.uint32), flat.view(np.uint32))


def test_checks_of_a_transposed_int_matrix(sg, ctx):
    import torch
    A = W.uniform_i32(100 * 68, 82, -9, 9).reshape(100, 68)
    A[77, 3] = 10
    T = ctx.wrap(torch.from_numpy(A).cuda()).transpose()
    p = sg.Program(ctx)
    p.add_root(T)
    p.ensure_for_all(T, sg.Pred.in_range(-9, 9))
    status, v = p.execute()
    assert status == "post_violated" and v[0].first_index == 3 * 100 + 77
