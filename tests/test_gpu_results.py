"""Result arrays on their way out: host and device destinations, dense and padded rows, results larger than the pinned staging
memory, and destinations at odd addresses, against the oracle."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2205_03251_amd import gpeval as g
    c = g.Context(0)
    yield c
    c.close()


def same(a, b):
    a, b = np.asarray(a), np.asarray(b)
    return bool(((a.view(np.uint32) == b.view(np.uint32)) | (np.isnan(a) & np.isnan(b))).all())


# T = 512 and 1024: dense rows; 4099 x 300 rows exceed the 4 MiB of staging; 1, 49: a few words a row
@pytest.mark.parametrize("n_trees,T", [(1, 1), (100, 49), (7, 512), (1100, 1024), (300, 4099)])
def test_float_results_to_host_and_device(ctx, n_trees, T):
    import torch

    from paper_2205_03251_amd import gpeval as g
    pop = gen.sized_population(5 + T, n_trees, 3, 31)
    cases = gen.float_cases(6, T)
    with np.errstate(all="ignore"):
        want_r, want_f = oracle.eval_population_f32(pop, cases.x, cases.y)
    ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
    ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets)
    big = torch.full((n_trees * T + 8,), 7.0, dtype=torch.float32, device="cuda")
    for shift in (None, 1, 4):          # host; one float past a 16-byte boundary; aligned
        if shift is None:
            r, f, _ = ctx.evaluate_full(ph, ch, g.GP_F32, n_trees, T)
        else:
            buf = big[shift:shift + n_trees * T]
            r, f, _ = ctx.evaluate_full(ph, ch, g.GP_F32, n_trees, T, device=True, root_buf=buf)
            assert float(big[shift - 1]) == 7.0 and float(big[shift + n_trees * T]) == 7.0
            r, f = r.cpu().numpy().reshape(n_trees, T), f.cpu().numpy()
            big.fill_(7.0)
            torch.cuda.synchronize()
        assert same(r, want_r)
        assert ((f == want_f) | (np.isnan(f) & np.isnan(want_f))).all()
    r, f = ctx.population_results(ph, ch, g.GP_F32, T)
    assert same(r, want_r)
    with np.errstate(all="ignore"):
        f = ctx.fitness(ch, g.GP_F32, want_r)
    assert ((f == want_f) | (np.isnan(f) & np.isnan(want_f))).all()
    ctx.free(ph)
    ctx.free(ch)


@pytest.mark.parametrize("n_trees,k", [(1000, 6), (40, 9), (160, 18)])      # 1, 8 and 4096 words a row
def test_boolean_results_to_host_and_device(ctx, n_trees, k):
    from paper_2205_03251_amd import gpeval as g
    pop = gen.sized_population(60 + k, n_trees, 3, 31, n_terms=k, vtype=gen.VT_BOOL)
    cases = gen.bool_cases(k)
    want_r, want_f = oracle.eval_population_bool(pop, cases.inputs, cases.target, cases.T)
    ch = ctx.set_cases(g.GP_BOOL, cases.inputs, cases.target, n_cases=cases.T)
    ph = ctx.load_population(g.GP_BOOL, pop.ops, pop.offsets, n_inputs=k)
    r, f, _ = ctx.evaluate_full(ph, ch, g.GP_BOOL, n_trees, cases.T)
    assert np.array_equal(r, want_r) and np.array_equal(f, want_f)
    r, f, _ = ctx.evaluate_full(ph, ch, g.GP_BOOL, n_trees, cases.T, device=True)
    assert np.array_equal(r.cpu().numpy().view(np.uint64), want_r) and np.array_equal(f.cpu().numpy(), want_f)
    assert np.array_equal(ctx.fitness(ch, g.GP_BOOL, want_r), want_f)
    ctx.free(ph)
    ctx.free(ch)


# one tree of many chunks: more counters to set back than a block per row covers; 300 trees: a block per tree
@pytest.mark.parametrize("vt", ["f32", "bool"])
@pytest.mark.parametrize("n_trees,n_nodes", [(1, 200001), (300, 301)])
def test_every_run_sets_its_counters_back(ctx, vt, n_trees, n_nodes):
    from paper_2205_03251_amd import gpeval as g
    if vt == "f32":
        t, cases = g.GP_F32, gen.float_cases(22, 97)
        pop = gen.sized_population(21, n_trees, n_nodes, n_nodes)
        with np.errstate(all="ignore"):
            want_r, want_f = oracle.eval_population_f32(pop, cases.x, cases.y)
        ch, T = ctx.set_cases(t, cases.x, cases.y), 97
        ph = ctx.load_population(t, pop.ops, pop.offsets, chunk_nodes=64)
    else:
        t, cases = g.GP_BOOL, gen.bool_cases(8)
        pop = gen.sized_population(21, n_trees, n_nodes, n_nodes, n_terms=8, vtype=gen.VT_BOOL)
        want_r, want_f = oracle.eval_population_bool(pop, cases.inputs, cases.target, cases.T)
        ch, T = ctx.set_cases(t, cases.inputs, cases.target, n_cases=cases.T), cases.T
        ph = ctx.load_population(t, pop.ops, pop.offsets, n_inputs=8, chunk_nodes=64)
    for kw in ({}, {}, {"per_tree": True}, {"graph": False}, {"per_tree": True}, {"per_tree": True, "graph": False},
               {"device": True}, {}):
        r, f, _ = ctx.evaluate_full(ph, ch, t, n_trees, T, **kw)
        if kw.get("device"):
            r, f = r.cpu().numpy().view(want_r.dtype), f.cpu().numpy()
        if vt == "f32":
            assert same(r, want_r), kw
            assert ((f == want_f) | (np.isnan(f) & np.isnan(want_f))).all(), kw
        else:
            assert np.array_equal(r, want_r) and np.array_equal(f, want_f), kw
    ctx.free(ph)
    ctx.free(ch)
