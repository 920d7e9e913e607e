"""Admission by budget: a large job is admitted under a budget that holds its vectors without side chunks."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


def test_a_large_job_near_the_budget():
    from paper_2205_03251_amd import gpeval as g
    T = 4096
    tree, cases = gen.sized_tree(np.random.default_rng(1), 1000001), gen.float_cases(2, T)
    with g.Context(0) as ctx:
        ch = ctx.set_cases(g.GP_F32, cases.x, cases.y)
        # 832 chunks of 16 KiB and 2 MB of program in 1024-node chunks without side chunks: 15.8 MB
        ctx.server_start(n_streams=1, max_batch_jobs=1, prep_threads=1, budget_bytes=16_500_000)
        r = None
        ticket = ctx.server_submit(g.GP_JOB_FULL, ch, tree)
        while r is None:
            r = ctx.server_poll(ticket, g.GP_F32, T)
        ctx.server_stop()
    assert r["status"] == g.GP_OK
    with np.errstate(all="ignore"):
        want = oracle.eval_f32(tree, np.ascontiguousarray(cases.x[:, ::32]))
    got = r["root"][::32]
    assert ((got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))).all()
