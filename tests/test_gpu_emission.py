"""Device compilation of populations large enough for emission by a thread per node: the compiled form must be the host
compiler's byte for byte, at the size where that form takes over, with recorded points, several inputs, Boolean trees,
chunk targets from many tiny chunks to one chunk a tree, and combs (long chains of operands on one side)."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2205_03251_amd import gpeval as g
    c = g.Context(0)
    yield c
    c.close()


def comb(depth, left):
    t = [0x80 | (i & 3) for i in range(depth)]
    return np.array(t + [0] * (depth + 1) if left else [b for f in t for b in (f, 0)] + [0], np.uint8)


def sized(rng, total, n_terms):
    """Trees of 1001 nodes and a last one, `total` nodes in all."""
    trees = [gen.sized_tree(rng, 1001, n_terms) for _ in range(total // 1001 - 1)]
    left = total - 1001 * len(trees)
    return trees + ([gen.sized_tree(rng, left, n_terms)] if left % 2 else [gen.sized_tree(rng, left - 1, n_terms),
                                                                          np.zeros(1, np.uint8)])


def populations():
    rng = np.random.default_rng(3)
    for total in (65535, 65536, 4096 * 17, 4096 * 17 + 1):
        yield f"{total} nodes", gen.pack(sized(rng, total, 1)), 64
    big = [gen.sized_tree(rng, 60001, 3), gen.sized_tree(rng, 1, 3), gen.sized_tree(rng, 30001, 3)]
    for C in (2, 40, 1024, 8192, 100000):
        yield f"three inputs, chunk {C}", gen.pack(big, n_inputs=3), C
        yield f"Boolean, chunk {C}", gen.pack(big, vtype=gen.VT_BOOL, n_inputs=3), C
    yield "combs", gen.pack([comb(20000, True), comb(20000, False), comb(700, True)]), 256


@pytest.mark.parametrize("records", [False, True])
def test_emission_by_nodes_matches_the_host_compiler(ctx, records):
    for name, pop, C in populations():
        kw = {}
        if records:
            rng = np.random.default_rng(9)
            pts = [np.unique(rng.integers(n, size=3)) for n in pop.sizes()]
            kw = dict(record_points=np.concatenate(pts), record_offsets=np.cumsum([0] + [len(p) for p in pts]))
        dumps = []
        for dev in (False, True):
            h = ctx.load_population(pop.vtype, pop.ops, pop.offsets, n_inputs=pop.n_inputs, chunk_nodes=C,
                                    device_compile=dev, **kw)
            dumps.append(ctx.population_dump(h))
            ctx.free(h)
        assert dumps[0] == dumps[1], name
