"""One launch per tree: each tree has its own item counters, one below and sixteen or four above a number of items, and a
population of many small trees does not hold a set of cache lines for each."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


def test_counters_of_small_and_large_trees():
    from paper_2205_03251_amd import gpeval as g
    # with 64 cases to a slice: 1, 4 and 256 items from one chunk, several times 256 from more chunks
    trees = [np.array([0], np.uint8), np.array([0x80, 0, 0], np.uint8)]
    trees += [gen.sized_tree(np.random.default_rng(n), n) for n in (31, 301, 2001, 6001)]
    pop = gen.pack(trees * 3)
    names = g.variant_names()
    with g.Context(0) as ctx:
        ctx.set_variant(names.index("f32d_k1_s10"))
        for T in (50, 256, 16384 - 64, 16384):
            cases = gen.float_cases(T, T)
            ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
            ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets, chunk_nodes=128)
            with np.errstate(all="ignore"):
                want, fit = oracle.eval_population_f32(pop, cases.x, cases.y)
            for graph in (True, False, True):          # captured, direct, replayed
                r, f, _ = ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T, per_tree=True, graph=graph)
                assert ((r.view(np.uint32) == want.view(np.uint32)) | (np.isnan(r) & np.isnan(want))).all(), (T, graph)
                assert ((f == fit) | (np.isnan(f) & np.isnan(fit))).all(), (T, graph)
            ctx.free(ph)
            ctx.free(ch)


def test_memory_of_many_small_trees():
    from paper_2205_03251_amd import gpeval as g
    pop, cases = gen.pack([np.array([0x80, 0, 0], np.uint8)] * 3000), gen.float_cases(1, 64)
    with g.Context(0) as ctx:
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        used = []
        for per_tree in (False, True):
            ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets)
            ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, 64, per_tree=per_tree)
            used.append(ctx.population_info(ph)["device_bytes"])
            ctx.free(ph)
        assert used[1] < used[0] + 16 * 3000           # 2048 bytes a tree before
