"""Calls that run short of device memory: what fits without side chunks (a vector of all cases per chunk, 4.4 times as many
chunks at 1024 nodes) is not refused, and a chunk size that does not fit does not end the tuning."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
T, CHUNK = 4096, 1024


@pytest.fixture(scope="module")
def made():
    """Trees, cases and, from a context without a limit, results and sizes."""
    from paper_2205_03251_amd import gpeval as g
    pop, cases = gen.sized_population(5, 24, 20001, 40001), gen.float_cases(6, T)
    kids = gen.crossover_children(7, pop, 30, donor_hi=200)
    ro = np.zeros(pop.n_trees + 1, np.int64)
    pts = [sorted({int(c) for p, c in zip(kids.parent, kids.point) if p == t}) for t in range(pop.n_trees)]
    ro[1:] = np.cumsum([len(p) for p in pts])
    rp = np.array([c for p in pts for c in p], np.int64)
    with g.Context(0) as ctx:
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets, chunk_nodes=CHUNK)
        r, f, _ = ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T)
        info = ctx.population_info(ph)
        co = ctx.evaluate_incremental(ph, ch, g.GP_F32, T, kids.parent, kids.point, kids.donors.ops, kids.donors.offsets,
                                      coeval=True)
        new, _, rec = ctx.evolve(ph, ch, 2, 3, seed=9)
        ev = (ctx.population_results(new, ch, g.GP_F32, T), rec)
    with np.errstate(all="ignore"):
        for t in (0, pop.n_trees - 1):
            assert same(r[t], oracle.eval_f32(pop.tree(t), cases.x))
    assert info["n_chunks"] > 2500                     # 670 without side chunks
    return dict(pop=pop, cases=cases, kids=kids, rp=rp, ro=ro, r=r, f=f, co=co, ev=ev)


def same(a, b):
    u = {4: np.uint32, 8: np.uint64}[a.dtype.itemsize]
    return ((a.view(u) == b.view(u)) | (np.isnan(a) & np.isnan(b))).all()


def context(megabytes):
    from paper_2205_03251_amd import gpeval as g
    return g.Context(0, budget_bytes=int(megabytes * 1e6))


# Budgets 2 to 3 % above what each of these needs when no population has side chunks (with them: 44 MB for the evaluation,
# 188 and 89 for the children, 88 for two populations, 113 for the evolution, 305 for the tuning of every size).
@pytest.mark.parametrize("how,megabytes", [("host", 11.6), ("device_compile", 25), ("postfix", 11.6)])
def test_fixed_chunk_size_under_a_tight_budget(made, how, megabytes):
    from paper_2205_03251_amd import gpeval as g
    pop, cases = made["pop"], made["cases"]
    kw = dict(chunk_nodes=CHUNK)
    ops = pop.ops
    if how == "device_compile":
        kw["device_compile"] = True
    if how == "postfix":
        kw["layout"] = g.GP_POSTFIX
        ops = np.concatenate([to_postfix(pop.tree(t)) for t in range(pop.n_trees)])
    with context(megabytes) as ctx:
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        ph = ctx.load_population(g.GP_F32, ops, pop.offsets, **kw)
        for _ in range(2):
            r, f, _ = ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T)
            assert same(r, made["r"]) and same(f, made["f"])
        assert ctx.population_info(ph)["chunk_nodes"] == CHUNK
        assert ctx.memory_used <= megabytes * 1e6
        ctx.free(ph)


def to_postfix(tree):
    out, pending = [], []
    for b in tree:
        if b & 0x80:
            pending.append([int(b), 2])
            continue
        out.append(int(b))
        while pending:
            pending[-1][1] -= 1
            if pending[-1][1]:
                break
            out.append(pending.pop()[0])
    return np.array(out, np.uint8)


@pytest.mark.parametrize("coeval,megabytes", [(False, 160), (True, 76)])
def test_children_under_a_tight_budget(made, coeval, megabytes):
    from paper_2205_03251_amd import gpeval as g
    pop, cases, kids = made["pop"], made["cases"], made["kids"]
    kw = {} if coeval else dict(record_points=made["rp"], record_offsets=made["ro"])
    with context(megabytes) as ctx:
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets, chunk_nodes=CHUNK, **kw)
        ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T)
        for _ in range(2):
            r, f, info = ctx.evaluate_incremental(ph, ch, g.GP_F32, T, kids.parent, kids.point, kids.donors.ops,
                                                  kids.donors.offsets, coeval=coeval)
            assert same(r, made["co"][0]) and same(f, made["co"][1])
            assert (info["stop_level"] == made["co"][2]["stop_level"]).all()
        r, f = ctx.population_results(ph, ch, g.GP_F32, T)
        assert same(r, made["r"]) and same(f, made["f"])


def test_a_second_population_makes_the_first_give_way(made):
    from paper_2205_03251_amd import gpeval as g
    pop, cases = made["pop"], made["cases"]
    with context(23.1) as ctx:
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        ps = []
        for _ in range(2):
            ps.append(ctx.load_population(g.GP_F32, pop.ops, pop.offsets, chunk_nodes=CHUNK))
            r, f, _ = ctx.evaluate_full(ps[-1], ch, g.GP_F32, pop.n_trees, T)
            assert same(r, made["r"]) and same(f, made["f"])
        for ph in ps:                                  # both are still evaluated
            r, f = ctx.population_results(ph, ch, g.GP_F32, T)
            assert same(r, made["r"]) and same(f, made["f"])


def test_evolution_under_a_tight_budget(made):
    from paper_2205_03251_amd import gpeval as g
    pop, cases = made["pop"], made["cases"]
    with context(58.6) as ctx:
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets, chunk_nodes=CHUNK)
        ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T)
        new, _, rec = ctx.evolve(ph, ch, 2, 3, seed=9)
        got = ctx.population_results(new, ch, g.GP_F32, T)
        assert same(got[0], made["ev"][0][0]) and same(got[1], made["ev"][0][1])
        for k in ("mother", "father", "point", "donor_node", "nodes", "stop_level", "drawn"):
            assert (rec[k] == made["ev"][1][k]).all(), k
        r, f = ctx.population_results(ph, ch, g.GP_F32, T)     # the caller's population keeps its results
        assert same(r, made["r"]) and same(f, made["f"])


def test_tuning_passes_over_sizes_that_do_not_fit(made):
    from paper_2205_03251_amd import gpeval as g
    pop, cases = made["pop"], made["cases"]
    with context(58.6) as ctx:                         # 128 nodes a chunk do not fit, 1024 and 4096 do
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets)
        ctx.autotune(ph, ch)
        assert ctx.population_info(ph)["chunk_nodes"] > 128
        r, f, _ = ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T)
        assert same(r, made["r"]) and same(f, made["f"])


def test_what_cannot_fit_is_refused_and_changes_nothing(made):
    from paper_2205_03251_amd import gpeval as g
    pop, cases = made["pop"], made["cases"]
    with context(58.6) as ctx:
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets, chunk_nodes=CHUNK)
        ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, T)
        before = ctx.population_info(ph)["n_chunks"]
        many = gen.pack([np.array([0x80, 0, 0], np.uint8)] * 30000)            # 30000 rows of 16 KiB
        p2 = ctx.load_population(g.GP_F32, many.ops, many.offsets)
        with pytest.raises(g.GPError) as e:
            ctx.evaluate_full(p2, ch, g.GP_F32, many.n_trees, T)
        assert e.value.code == g.GP_EBUDGET
        assert ctx.population_info(ph)["n_chunks"] == before
        r, f = ctx.population_results(ph, ch, g.GP_F32, T)
        assert same(r, made["r"]) and same(f, made["f"])
