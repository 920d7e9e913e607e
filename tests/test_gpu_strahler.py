"""Strahler numbers and parents of subtrees that leave their block of 4096 positions, against the oracle: ends at and beside
block edges, numbers that rise only across blocks, spines over many blocks, and invalid neighbours."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
F = 0x80


@pytest.fixture(scope="module")
def ctx():
    from paper_2205_03251_amd import gpeval as g
    c = g.Context(0)
    yield c
    c.close()


def complete(depth):
    t = [0]
    for _ in range(depth):
        t = [F] + t + t
    return t


def comb(parts, left):
    """parts joined by a spine that runs through the left or the right children."""
    if left:
        return [F] * (len(parts) - 1) + sum(parts, [])
    return sum(([F] + p for p in parts[:-1]), []) + parts[-1]


def shapes(seed):
    rng = np.random.default_rng(90 + seed)
    yield [complete(13)] * 3                                             # 16383 nodes each: ends at every offset of a block
    yield [complete(d) for d in (11, 0, 11, 12, 0, 0, 12, 14)]
    yield [comb([complete(int(d)) for d in rng.integers(0, 11, 60)], bool(i & 1)) for i in range(6)]
    yield [comb([comb([[0]] * 3000, bool(i & 1)), complete(9), comb([[0]] * 2500, bool(i & 2))], bool(i & 4)) for i in range(8)]
    for n in (4095, 4097, 8191, 8193, 12287, 65537, 300001):
        yield [gen.sized_tree(rng, n, n_terms=1).tolist(), [0]] * 2


@pytest.mark.parametrize("shift", [0, 1, 15, 16, 4095])
@pytest.mark.parametrize("seed", [0, 1])
def test_numbers_across_blocks(ctx, seed, shift):
    import torch
    for trees in shapes(seed):
        trees = [[0]] * shift + [np.array(t, np.uint8) for t in trees] + [[F, 0], [0, 0, F]]      # the last two are invalid
        trees = [np.asarray(t, np.uint8) for t in trees]
        offs = np.zeros(len(trees) + 1, np.int64)
        offs[1:] = np.cumsum([len(t) for t in trees])
        ops = torch.from_numpy(np.concatenate(trees)).to("cuda:0")
        valid, end, parent, sn, _ = ctx.index_trees(ops, torch.from_numpy(offs).to("cuda:0"), 1, strahler=True)
        sn, valid, parent = sn.cpu().numpy(), valid.cpu().numpy(), parent.cpu().numpy()
        assert valid[:-2].all() and not valid[-2:].any()
        want = np.concatenate([oracle.strahler(t) for t in trees[:-2]] + [np.zeros(5, np.uint8)])
        assert np.array_equal(sn, want), (seed, shift, len(ops))
        assert np.array_equal(parent, np.concatenate([oracle.parents(t) for t in trees[:-2]] + [np.full(5, -1)]))
