"""Kept device blocks: a reused block counts with its whole size against the budget, and an emptied context holds few."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def cases_of(ctx, T):
    from paper_2205_03251_amd import gpeval as g
    return ctx.set_cases(g.GP_F32, np.zeros((1, T), np.float32), np.zeros(T, np.float32))


def test_reused_blocks_count_whole():
    from paper_2205_03251_amd import gpeval as g
    budget = 4 << 20
    with g.Context(0, budget_bytes=budget) as ctx:
        small = [cases_of(ctx, 64)]
        before = free_bytes()
        for _ in range(400):                 # two blocks of 64 KiB freed, then two of 2 KiB wanted
            ctx.free(cases_of(ctx, 16384))
            small.append(cases_of(ctx, 64))
        held = before - free_bytes()
        assert held <= budget + (4 << 20)    # 51 MB when the whole blocks are not counted; the allocator rounds up to 2 MiB
        assert ctx.memory_used <= budget
        ch = small[-1]
        ph = ctx.load_population(g.GP_F32, np.array([0x80, 0, 0], np.uint8), np.array([0, 3]))
        r, _, _ = ctx.evaluate_full(ph, ch, g.GP_F32, 1, 64)
        assert (r == 0).all()


def test_an_emptied_context_gives_its_blocks_back():
    from paper_2205_03251_amd import gpeval as g
    pop, cases = gen.sized_population(3, 160, 3001, 9001), gen.float_cases(4, 16384)
    with g.Context(0, budget_bytes=64 << 30) as ctx:
        before = free_bytes()
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        ph = ctx.load_population(g.GP_F32, pop.ops, pop.offsets, chunk_nodes=64)
        ctx.evaluate_full(ph, ch, g.GP_F32, pop.n_trees, cases.T)
        held = ctx.memory_used
        assert held > 700 << 20
        ctx.free(ph)
        assert before - free_bytes() > held // 2                 # kept for the next population
        ctx.free(ch)
        assert before - free_bytes() < 272 << 20


def test_the_latest_blocks_are_kept():
    from paper_2205_03251_amd import gpeval as g
    with g.Context(0, budget_bytes=32 << 20) as ctx:             # keeps up to 2 MiB
        cases_of(ctx, 64)
        sizes = [64, 4096, 16384, 1024]
        for k in range(200):                                     # more than it keeps, in changing sizes
            hs = [cases_of(ctx, sizes[(k + i) % 4]) for i in range(1 + k % 20)]
            for h in hs:
                ctx.free(h)
        assert ctx.memory_used <= 8192
