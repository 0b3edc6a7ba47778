"""GPU parity of the lean streaming kernel (programs with one running value, at most two inputs
and no compaction) at the edges of its sub-tiles and tiles, against the CPU oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import compare, say, to_dev

pytestmark = pytest.mark.gpu

SUB = 256 * 8  # elements of a sub-tile at the default launch (256 threads, unroll 2)


@pytest.fixture(scope="module")
def ctx(sg):
    return sg.Context(0)


def f32_spec(n):
    """Every float operation and check of the kernel: maps, zips, predicates, filters (no output
    compacted), checks that hold and that fail, all reductions, and a dense output."""
    return {"inputs": [{"name": "x", "dtype": "f32", "n": n}, {"name": "y", "dtype": "f32", "n": n}],
            "nodes": [{"name": "a", "op": "map", "src": "x", "fn": ["affine", 1.5, -0.25]},
                      {"name": "b", "op": "zip", "a": "a", "b": "y", "binop": "mul"},
                      {"name": "c", "op": "zip", "a": "b", "b": "y", "binop": "sub"},
                      {"name": "d", "op": "map", "src": "c", "fn": ["sqrt_abs"]},
                      {"name": "k", "op": "filter", "src": "d", "pred": ["cmp", "gt", 0.4]},
                      {"name": "k2", "op": "filter", "src": "k",
                       "pred": ["or", ["cmp", "le", 1.0], ["not", ["in_range", 0.5, 1.5]]]},
                      {"name": "t", "op": "reduce", "src": "k2", "red": "sum"},
                      {"name": "m", "op": "reduce", "src": "k2", "red": "max"},
                      {"name": "l", "op": "reduce", "src": "k2", "red": "min"},
                      {"name": "q", "op": "reduce", "src": "k", "red": "count"}],
            "contracts": [{"kind": "require", "check": "for_all", "node": "x", "pred": ["isfinite"]},
                          {"kind": "require", "check": "for_all", "node": "y", "pred": ["in_range", -9.0, 9.0]},
                          {"kind": "ensure", "check": "for_all", "node": "d", "pred": ["in_range", 0.0, 2.0]},
                          {"kind": "ensure", "check": "exists", "node": "d", "pred": ["cmp", "gt", 3.0]},
                          {"kind": "ensure", "check": "close", "node": "t", "abs_tol": 0.0, "rel_tol": 1e-5}],
            "outputs": ["d", "t", "m", "l", "q"]}


def i32_spec(n):
    return {"inputs": [{"name": "x", "dtype": "i32", "n": n}, {"name": "y", "dtype": "i32", "n": n}],
            "nodes": [{"name": "a", "op": "map", "src": "x", "fn": ["affine", 3, -7]},
                      {"name": "b", "op": "zip", "a": "a", "b": "y", "binop": "sub"},
                      {"name": "c", "op": "map", "src": "b", "fn": ["abs"]},
                      {"name": "k", "op": "filter", "src": "c", "pred": ["cmp", "ne", 11]},
                      {"name": "s", "op": "reduce", "src": "k", "red": "sum"},
                      {"name": "m", "op": "reduce", "src": "k", "red": "max"},
                      {"name": "l", "op": "reduce", "src": "c", "red": "min"}],
            "contracts": [{"kind": "require", "check": "for_all", "node": "y", "pred": ["in_range", -1000, 1000]},
                          {"kind": "ensure", "check": "for_all", "node": "c", "pred": ["in_range", 0, 3990]}],
            "outputs": ["c", "s", "m", "l"]}


EDGES = [0, 1, 63, 257, SUB - 1, SUB, SUB + 1, 2 * SUB + 255]
LARGE = [512 * SUB, 512 * SUB + 1, 1024 * SUB - 3, 2048 * SUB + 77]
CASES = [(n, 0, (256, 2)) for n in EDGES + LARGE] + \
        [(n, o, l) for o, l in ((1, (256, 4)), (0, (64, 1)), (3, (192, 2))) for n in EDGES]


@pytest.mark.parametrize("n,offset,launch", CASES)
def test_lean_chains(sg, ctx, n, offset, launch):
    """Edges of sub-tiles, tiles and grids, unaligned inputs, other launch shapes."""
    say("lean", n, offset, launch)
    for spec, inp in ((f32_spec(n), {"x": W.normal_f32(n, 5), "y": W.uniform_f32(n, 6)}),
                      (i32_spec(n), {"x": W.uniform_i32(n, 7, -999, 999), "y": W.uniform_i32(n, 8, -999, 999)})):
        dev = to_dev({k: np.concatenate([np.zeros(offset, v.dtype), v]) for k, v in inp.items()})
        dev = {k: v[offset:] for k, v in dev.items()}
        ctx.set_launch(*launch)
        try:
            built = sg.build_spec(ctx, spec, dev)
            status, verdicts = built.program.execute()
        finally:
            ctx.set_launch(256, 2)
        compare(spec, built, status, verdicts, oracle.evaluate(spec, inp))


@pytest.mark.parametrize("dtype", ["f32", "i32"])
@pytest.mark.parametrize("n", [2, SUB, SUB + 1, 3 * SUB + 130])
def test_lean_sorted_pairs_across_lanes_chunks_and_subtiles(sg, ctx, n, dtype):
    """One pair out of order at each kind of boundary, and at the vector's end."""
    base = np.arange(n).astype(np.float32 if dtype == "f32" else np.int32)
    for i in sorted({0, 2, 3, 254, 255, 256, 511, 512, 2046, 2047, 2048, 4095, n - 2} & set(range(n - 1))):
        x = base.copy()
        x[i] += 2  # pair (i, i + 1) is out of order
        say("lean sorted", dtype, n, i)
        spec = {"inputs": [{"name": "x", "dtype": dtype, "n": n}], "nodes": [],
                "contracts": [{"kind": "ensure", "check": "sorted", "node": "x"}], "outputs": []}
        built = sg.build_spec(ctx, spec, to_dev({"x": x}))
        status, verdicts = built.program.execute()
        assert status == "post_violated" and (verdicts[0].holds, verdicts[0].first_index) == (0, i)


@pytest.mark.parametrize("bad,pred", [(np.nan, ["in_range", -2.0, 2.0]), (np.inf, ["isfinite"]), (-np.inf, ["isfinite"]),
                                      (np.nan, ["isfinite"]), (2.5, ["in_range", -2.0, 2.0]), (-2.5, ["in_range", -2.0, 2.0])])
@pytest.mark.parametrize("at", [0, 777, 2 * SUB + 3, 5 * SUB + 8])
def test_lean_check_finds_the_first_failing_element(sg, ctx, bad, pred, at):
    n = 5 * SUB + 9
    x = W.uniform_f32(n, 4)
    x[at] = bad
    x[-1] = bad
    say("lean check", bad, pred, at)
    spec = {"inputs": [{"name": "x", "dtype": "f32", "n": n}], "nodes": [],
            "contracts": [{"kind": "ensure", "check": "for_all", "node": "x", "pred": pred}], "outputs": []}
    built = sg.build_spec(ctx, spec, to_dev({"x": x}))
    status, verdicts = built.program.execute()
    assert status == "post_violated" and verdicts[0].first_index == at


@pytest.mark.parametrize("specialize", [False, True])
@pytest.mark.parametrize("n", [100, 1 << 20, 4096 * SUB])
def test_a_finalizer_that_gives_up_is_reported(sg, n, specialize):
    """Results without a product check come to the host from the kernel itself, the error word with
    them: a wait that gives up is an error of that execution, and the next one is clean."""
    c = sg.Context(0)
    c.set_specialize(specialize)
    spec, inp = W.cfg1_spec(n), W.cfg1_inputs(n)
    built = sg.build_spec(c, spec, to_dev(inp))
    want = oracle.evaluate(spec, inp)
    for rep in range(3):
        c.set_wait_limit(0)
        try:
            say("lean forced wait failure", n, specialize, rep)
            with pytest.raises(sg.SafeGPUError) as e:
                built.program.execute()
            assert e.value.status_name == "device"
        finally:
            c.set_wait_limit(-1)
        status, verdicts = built.program.execute()
        compare(spec, built, status, verdicts, want)


@pytest.mark.parametrize("n", [1, 777, 37 * 8192, 37 * 8192 + 5001])
@pytest.mark.parametrize("plan", [(256, 2, 4), (64, 1, 8), (128, 4, 2)])
@pytest.mark.parametrize("batched", [False, True])
def test_lean_and_general_interpreter_give_the_same_bits(sg, n, plan, batched):
    """A chain with one running value runs on the lean kernel; with a maximum over exp(x) beside it
    the same chain runs on the general one.  At one launch shape every float64 sum, element and
    extremum has the same bits."""
    import torch
    c = sg.Context(0)
    x, y = (torch.from_numpy(W.normal_f32(n, s)).cuda() for s in (21, 22))
    say("lean and general", n, plan, batched)
    got = []
    for general in (False, True):
        a, b = c.wrap(x), c.wrap(y)
        z = a.map(sg.Fn.affine(1.5, -0.25)).zip(b, "mul")
        k = z.filter(sg.Pred.cmp("gt", -0.5))
        roots = [z.reduce("sum"), k.reduce("sum"), k.reduce("max"), z.reduce("min")]
        p = sg.Program(c)
        for r in roots:
            p.add_root(r)
        if not batched:
            p.add_root(z)
        if general:
            p.add_root(a.map(sg.Fn.unary("exp")).reduce("max"))
        if batched:
            c.set_launch(*plan[:2])
            c.set_batch_substeps(plan[2])
            sg.Batch(c, [p], use_graph=False).run()
        else:
            p.set_plan(plan + (-1,))
            assert p.features(plan + (-1,))[21] == 1
            p.execute()
            assert c.last_launch()[:4] == (min(c.last_launch()[0], -(-n // (plan[0] * 4 * plan[1] * plan[2]))),) + plan
        bits = [np.array([r.shadow(), r.scalar()[0]]).view(np.uint64).tolist() for r in roots]
        got.append((bits, z.to_host().view(np.uint32).tolist() if not batched else None, c.last_launch()[0]))
    assert got[0] == got[1]
