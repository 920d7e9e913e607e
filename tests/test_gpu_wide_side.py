"""Side chunks of float populations on both sides of 10^9 nodes: from there on few enough that a launch bound by work is
not held up by their hand-offs, unless a few trees hold most of the nodes."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


# nodes per chunk: 4800 and 2400 without side chunks at 4096 and 2048 to a chunk, about 2860 and 1900 with side chunks
# wide apart, 2150 with close ones at 8192 (chosen for few large trees), 1080 at 4096 (below 10^9 nodes)
@pytest.mark.parametrize("n,tree_nodes,chunk_nodes,lo,hi", [
    (2000, 500_001, 0, 2600, 3100), (2000, 500_001, 2048, 1750, 2100),
    (1990, 500_001, 0, 1000, 1150), (60, 16_800_001, 0, 2000, 2250)])
def test_nodes_per_chunk(n, tree_nodes, chunk_nodes, lo, hi):
    from paper_2205_03251_amd import gpeval as g
    tree = gen.sized_tree(np.random.default_rng(3), tree_nodes)
    ops, offsets = np.tile(tree, n), np.arange(n + 1, dtype=np.int64) * tree_nodes
    x = np.random.default_rng(4).uniform(-1, 1, (1, 300)).astype(np.float32)
    with g.Context(0) as ctx:
        ch = ctx.set_cases(g.GP_F32, x, x[0].copy())
        _, want, _ = ctx.evaluate_full(ctx.load_population(g.GP_F32, tree, offsets[:2]), ch, g.GP_F32, 1, 300)
        chunks = []
        for device in (True, False):
            ph = ctx.load_population(g.GP_F32, ops, offsets, device_compile=device, chunk_nodes=chunk_nodes)
            chunks.append(ctx.population_info(ph)["n_chunks"])
            _, fit, _ = ctx.evaluate_full(ph, ch, g.GP_F32, n, 300, roots=False)
            ctx.free(ph)
            assert (fit.view(np.int64) == want.view(np.int64)[0]).all()
    assert chunks[0] == chunks[1]
    assert lo <= n * tree_nodes / chunks[0] <= hi, chunks
