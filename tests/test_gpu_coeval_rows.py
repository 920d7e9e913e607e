"""Co-evaluation on a case set that provides more inputs than the population reads: the mother's chunk values come after the
case set's rows, not after the population's."""
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


@pytest.mark.parametrize("n_inputs,provided,T", [(1, 2, 50), (1, 9, 300), (2, 20, 700), (3, 3, 100)])
def test_case_set_with_more_inputs(ctx, n_inputs, provided, T):
    from paper_2205_03251_amd import gpeval as g
    pop = gen.sized_population(170 + n_inputs, 12, 301, 6001, n_terms=n_inputs)
    kids = gen.crossover_children(171, pop, 24, donor_hi=60, n_terms=n_inputs)
    rng = np.random.default_rng(T)
    x = rng.uniform(-1, 1, (provided, T)).astype(np.float32)
    y = rng.uniform(-1, 1, T).astype(np.float32)
    ch = ctx.set_cases(g.GP_F32, x, y)
    ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets, n_inputs=n_inputs, chunk_nodes=64)
    ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T)
    r, f, info = ctx.evaluate_incremental(ph, ch, g.GP_F32, T, kids.parent, kids.point, kids.donors.ops,
                                          kids.donors.offsets, coeval=True)
    for i in range(24):
        with np.errstate(all="ignore"):
            w_r, w_l, _, w_f = oracle.incremental_f32(pop.tree(int(kids.parent[i])), int(kids.point[i]),
                                                      kids.donors.tree(i), x, y)
        assert info["stop_level"][i] == w_l, i
        assert ((r[i].view(np.uint32) == w_r.view(np.uint32)) | (np.isnan(r[i]) & np.isnan(w_r))).all(), i
        assert f[i] == w_f or (np.isnan(f[i]) and np.isnan(w_f)), i
    ctx.free(ph)
    ctx.free(ch)
