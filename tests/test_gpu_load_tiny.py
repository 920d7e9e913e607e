"""Device compilation of populations of many tiny trees, on both sides of the nodes per chunk from which a thread per node
emits: the compiled form is the host compiler's."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi,count", [(1, 1, 70000), (1, 7, 40000), (7, 7, 12000), (9, 9, 12000), (3, 31, 12000)])
@pytest.mark.parametrize("boolean", [False, True])
def test_tiny_trees(lo, hi, count, boolean):
    from paper_2205_03251_amd import gpeval as g
    base = gen.sized_population(lo + hi, 300, lo, hi, n_terms=3)
    pop = gen.pack([base.tree(t % 300) for t in range(count)], vtype=gen.VT_BOOL if boolean else gen.VT_F32, n_inputs=3)
    vt = g.GP_BOOL if boolean else g.GP_F32
    assert len(pop.ops) >= 65536
    with g.Context(0) as ctx:
        dumps = [ctx.population_dump(ctx.load_population(vt, pop.ops, pop.offsets, n_inputs=3, device_compile=d))
                 for d in (False, True)]
    assert dumps[0] == dumps[1]
