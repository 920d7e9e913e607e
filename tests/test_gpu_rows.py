"""Float interpreters that hold several input rows in registers, and those of one and two cases per lane: input counts at and
around the rows they hold, case counts at the edges of a slice, and co-evaluation's appended rows, against the oracle."""
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


def cases_of(seed, n_inputs, T):
    rng = np.random.default_rng(seed)
    x = rng.uniform(-2, 2, (n_inputs, T)).astype(np.float32)
    x[:, 0] = 0.0
    x[-1, -1] = np.inf if T > 1 else 1.0
    return x, rng.uniform(-1, 1, T).astype(np.float32)


# rows held past the first: 15 (K = 1, 2), 7 (K = 4), 3 (K = 8)
@pytest.mark.parametrize("n_inputs", [2, 4, 5, 8, 9, 16, 17, 64])
def test_input_rows(ctx, n_inputs):
    from paper_2205_03251_amd import gpeval as g
    names = g.variant_names()
    pop = gen.sized_population(n_inputs, 24, 3, 1501, n_terms=n_inputs)
    for T, want in ((1, "f32r_k1"), (64, "f32r_k1"), (65, "f32r_k2"), (128, "f32r_k2"), (129, "f32r_k4"), (513, "f32r_k4")):
        x, y = cases_of(T, n_inputs, T)
        with np.errstate(all="ignore"):
            want_r, want_f = oracle.eval_population_f32(pop, x, y)
        ch = ctx.set_cases(g.GP_F32, x, y)
        ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets, n_inputs=n_inputs, chunk_nodes=64)
        for v in [-1] + [i for i, nm in enumerate(names) if nm.startswith(("f32r_", "f32d_k1", "f32d_k2"))]:
            ctx.set_variant(v)
            r, f, st = ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T)
            if v < 0:
                assert names[st["variant"]].startswith(want)
            same = (r.view(np.uint32) == want_r.view(np.uint32)) | (np.isnan(r) & np.isnan(want_r))
            assert same.all(), (names[st["variant"]], T)
            assert ((f == want_f) | (np.isnan(f) & np.isnan(want_f))).all()
        ctx.set_variant(-1)
        ctx.free(ph)
        ctx.free(ch)


@pytest.mark.parametrize("n_inputs,T", [(3, 50), (3, 700), (12, 100)])
def test_coevaluation_with_several_inputs(ctx, n_inputs, T):
    """The mother's chunk values a sibling contains arrive as rows past the case set's own."""
    from paper_2205_03251_amd import gpeval as g
    pop = gen.sized_population(70 + n_inputs, 12, 301, 6001, n_terms=n_inputs)
    kids = gen.crossover_children(71, pop, 24, donor_hi=60, n_terms=n_inputs)
    x, y = cases_of(T, n_inputs, T)
    ch = ctx.set_cases(g.GP_F32, x, y)
    ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets, n_inputs=n_inputs, chunk_nodes=64)
    ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T)
    r, f, info = ctx.evaluate_incremental(ph, ch, g.GP_F32, T, kids.parent, kids.point, kids.donors.ops,
                                          kids.donors.offsets, coeval=True)
    for i in range(24):
        with np.errstate(all="ignore"):
            w_r, w_l, _, w_f = oracle.incremental_f32(pop.tree(int(kids.parent[i])), int(kids.point[i]),
                                                      kids.donors.tree(i), x, y)
        assert info["stop_level"][i] == w_l
        assert ((r[i].view(np.uint32) == w_r.view(np.uint32)) | (np.isnan(r[i]) & np.isnan(w_r))).all()
        assert f[i] == w_f or (np.isnan(f[i]) and np.isnan(w_f))
    ctx.free(ph)
    ctx.free(ch)
