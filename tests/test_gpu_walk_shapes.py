"""Walks of incremental evaluation on many test cases: values held in blocks, case counts just above a power of two (threads
past the last case), the kernels for few and for many children, cached and co-evaluated, against the oracle."""
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


def path_tree(rng, levels, stop, boolean, n_inputs):
    """Functions on a path down to a small subtree, the path operand left or right; at level `stop` (1-based from the bottom;
    0: none) it is ignored.  Returns the tree and the node at the bottom."""
    bottom = [0x80, 0, 0] if not boolean else [0x80, 0, 1]
    tree, point = list(bottom), 0
    for k in range(1, levels + 1):
        if k == stop:
            f, sib, right = (0x80, [0x83, 0, 0x82, 0, 0], False) if boolean else (0x83, [0x81, 0, 0], False)
        else:
            f, sib, right = 0x80 + int(rng.integers(4 if boolean else 3)), [int(rng.integers(n_inputs))], rng.random() < 0.5
        tree = [f] + sib + tree if right else [f] + tree + sib
        point += 1 + (len(sib) if right else 0)
    return np.array(tree, np.uint8), point


# 17, 32, 33 and 64 values a thread (float); 3, 4, 5, 9 and 16 words (Boolean), whole and with a part of the last one
@pytest.mark.parametrize("boolean,T", [(False, 4097), (False, 8192), (False, 8193), (False, 16384), (True, (1 << 15) + 1),
                                       (True, 1 << 16), (True, (1 << 16) + 70), (True, (1 << 17) + 63), (True, 1 << 18)])
def test_few_and_many_children(ctx, boolean, T):
    from paper_2205_03251_amd import gpeval as g
    rng = np.random.default_rng(T)
    vt, n_inputs = (g.GP_BOOL, 5) if boolean else (g.GP_F32, 2)
    trees, points = zip(*[path_tree(rng, n, s, boolean, n_inputs)
                          for n in (1, 3, 4, 5, 8, 9, 18) for s in sorted({0, 1, n // 2, n})])
    pop = gen.pack(trees, vtype=gen.VT_BOOL if boolean else gen.VT_F32, n_inputs=n_inputs)
    donor = np.array([0x82, 1, 2] if boolean else [0x81, 0, 1], np.uint8)
    if boolean:                                        # bits past the last case are arbitrary
        x = rng.integers(0, 1 << 64, (n_inputs, (T + 63) // 64), dtype=np.uint64)
        y = rng.integers(0, 1 << 64, (T + 63) // 64, dtype=np.uint64)
    else:
        x, y = rng.uniform(-1, 1, (n_inputs, T)).astype(np.float32), rng.uniform(-1, 1, T).astype(np.float32)
    ch = ctx.set_cases(vt, x, y, n_cases=T)
    ph = ctx.load_population(vt, pop.ops, pop.offsets, n_inputs=n_inputs, record_points=np.array(points),
                             record_offsets=np.arange(len(trees) + 1))
    ctx.evaluate_full(ph, ch, vt, pop.n_trees, T)
    want = []
    for t in range(pop.n_trees):
        with np.errstate(all="ignore"):
            want.append(oracle.incremental_bool(pop.tree(t), points[t], donor, x, y, T) if boolean else
                        oracle.incremental_f32(pop.tree(t), points[t], donor, x, y))
    w_root = np.stack([w[0] for w in want])
    w_stop, w_fit = np.array([w[1] for w in want]), np.array([w[3] for w in want])
    assert len(set(w_stop.tolist())) >= 4              # the root, and several levels
    last = np.uint64((1 << (T % 64)) - 1) if T % 64 else np.uint64(2**64 - 1)
    for n in (pop.n_trees, 513, 1025):
        which = np.arange(n) % pop.n_trees
        for coeval in (False, True):
            r, f, info = ctx.evaluate_incremental(ph, ch, vt, T, which, np.array(points)[which], np.tile(donor, n),
                                                  3 * np.arange(n + 1), coeval=coeval)
            assert (info["stop_level"] == w_stop[which]).all(), (n, coeval)
            if boolean:
                r, w = r.copy(), w_root.copy()
                r[:, -1] &= last
                w[:, -1] &= last
                assert (r == w[which]).all() and (f == w_fit[which]).all(), (n, coeval)
            else:
                w = w_root[which]
                assert ((r.view(np.uint32) == w.view(np.uint32)) | (np.isnan(r) & np.isnan(w))).all(), (n, coeval)
                assert ((f == w_fit[which]) | (np.isnan(f) & np.isnan(w_fit[which]))).all(), (n, coeval)
    ctx.free(ph)
    ctx.free(ch)
