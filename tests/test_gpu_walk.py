"""Walks of incremental evaluation taken in groups of levels: path lengths and stop levels at the edges of a group, for each
number of values a thread holds, cached and co-evaluated, against the oracle."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
LENGTHS = (1, 2, 7, 8, 9, 15, 16, 17, 33)


@pytest.fixture(scope="module")
def ctx():
    from paper_2205_03251_amd import gpeval as g
    c = g.Context(0)
    yield c
    c.close()


def path_tree(levels, stop, boolean):
    """A path of `levels` functions above node `levels` (a small subtree); at level `stop` (1-based from that node; 0: none)
    the function ignores its path operand: / (x - x), or AND false."""
    head, sibs = [], []
    for k in range(levels, 0, -1):
        head.append((0x80 if boolean else 0x83) if k == stop else (0x82 if boolean else 0x80 + k % 2))
    for k in range(1, levels + 1):
        if k == stop:
            sibs += [0x83, 0, 0x82, 0, 0] if boolean else [0x81, 0, 0]
        else:
            sibs += [1 + k % 2] if boolean else [0]
    return np.array(head + [0x80, 0, 0] + sibs, np.uint8)


# R = 1, 2, 4, 8 and 16 values a thread (float); 1 and 2 words (Boolean)
@pytest.mark.parametrize("boolean,T", [(False, 100), (False, 512), (False, 1000), (False, 2048), (False, 4096),
                                       (True, 256), (True, 1 << 15)])
@pytest.mark.parametrize("coeval", [False, True])
def test_group_edges(ctx, boolean, T, coeval):
    from paper_2205_03251_amd import gpeval as g
    vt = g.GP_BOOL if boolean else g.GP_F32
    trees, points = [], []
    for n in LENGTHS:
        for stop in sorted({0, 1, n // 2, n - 1, n}):
            if stop <= n:
                trees.append(path_tree(n, stop, boolean))
                points.append(n)
    k = max(3, (T - 1).bit_length()) if boolean else 1
    pop = gen.pack(trees, vtype=gen.VT_BOOL if boolean else gen.VT_F32, n_inputs=k)
    donors = [np.array([0x82, 1, 2] if boolean else [0x82, 0, 0], np.uint8)] * len(trees)
    doff = np.arange(0, 3 * len(trees) + 1, 3)
    if boolean:
        c = gen.bool_cases(k)
        ch = ctx.set_cases(vt, c.inputs, c.target, n_cases=c.T)
    else:
        c = gen.float_cases(T, T)
        ch = ctx.set_cases(vt, c.x, c.y)
    ph = ctx.load_population(vt, pop.ops, pop.offsets, n_inputs=k, record_points=np.array(points),
                             record_offsets=np.arange(len(trees) + 1))
    ctx.evaluate_full(ph, ch, vt, pop.n_trees, c.T)
    r, f, info = ctx.evaluate_incremental(ph, ch, vt, c.T, np.arange(len(trees)), np.array(points), np.concatenate(donors),
                                          doff, coeval=coeval)
    for i, t in enumerate(trees):
        if boolean:
            w_r, w_l, _, w_f = oracle.incremental_bool(t, points[i], donors[i], c.inputs, c.target, c.T)
            same = np.array_equal(r[i], w_r)
        else:
            with np.errstate(all="ignore"):
                w_r, w_l, _, w_f = oracle.incremental_f32(t, points[i], donors[i], c.x, c.y)
            same = ((r[i].view(np.uint32) == w_r.view(np.uint32)) | (np.isnan(r[i]) & np.isnan(w_r))).all()
        assert info["stop_level"][i] == w_l, (points[i], i)
        assert same and f[i] == w_f
    ctx.free(ph)
    ctx.free(ch)
