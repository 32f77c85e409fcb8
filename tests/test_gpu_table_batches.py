"""Retier, Promote, acquire, release and Finish over tables at the edges of the batches
that their single-workgroup kernels keep in registers (4,096 entries for releases,
8,192 for plans): tables, tags, free lists and reference counts equal the oracle's."""
import dataclasses

import numpy as np
import pytest

import mkv_workloads as wl
from _harness import Twin

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_req,max_pages", [(1, 1), (65, 1), (4, 1024), (3, 1366), (8, 1024), (5, 1639), (16, 1000)])
def test_table_batches(n_req, max_pages):
    import paper_2608_23834_amd as mk
    rng = np.random.default_rng(n_req * 10_000 + max_pages)
    full = 16 * max_pages
    lens = [full] + [max(1, int(full * f)) for f in rng.uniform(0.01, 0.2, n_req - 1)]
    lens[-1] = full  # the last row's last entry is in use
    w = dataclasses.replace(wl.scaled(wl.workload(1), tuple(lens), n_layers=1, name=f"table-{n_req}-{max_pages}"),
                            n_q_heads=1, n_kv_heads=1)
    tw = Twin(w, lens=lens, recent=16)
    mask = lambda p: (rng.random((n_req, max_pages)) < p).astype(np.uint8)

    def check():
        tw.check_tables()
        tw.check_refcounts()
        assert mk.kv_pool_check_errors(tw.gpu) == 0

    tw.fill_to([max(1, n - 17) for n in lens])
    tw.migrate(mask(0.1))
    check()
    tw.promote(mask(0.3))
    check()
    # every mapped page of the first and the last row once more, some pages twice in the list
    rows = sorted({0, n_req - 1})
    ids = np.concatenate([tw.obt[r][tw.obt[r] >= 0] for r in rows])
    tags = np.concatenate([tw.otags[r][tw.obt[r] >= 0] for r in rows])
    tw.acquire(ids, tags)
    tw.acquire(ids[::3], tags[::3])
    check()
    tw.migrate(mask(0.0))  # shared pages stay
    check()
    order = rng.permutation(len(ids) + len(ids[::3]))
    tw.release(np.concatenate([ids, ids[::3]])[order], np.concatenate([tags, tags[::3]])[order])
    check()
    tw.finish(rows)
    check()
    tw.fill_to([min(n, 40) for n in lens])  # the freed pages come back in the oracle's order
    check()
    # a list with one entry more than a page's references changes nothing
    live = tw.obt[0][:1]
    mk.kv_pages_release(tw.gpu, *(__import__("torch").from_numpy(x).cuda() for x in (
        np.repeat(live, 2).astype(np.int32), np.repeat(tw.otags[0][:1], 2))))
    assert mk.kv_pool_check_errors(tw.gpu, clear=True) != 0
    check()


@pytest.mark.parametrize("n_req,max_pages", [(4, 1024), (5, 1024)])
def test_finish_of_a_bad_row(n_req, max_pages):
    """Finish over rows of which one names a page outside the pool, or a free one (one batch
    of entries, and two): the reference error alone, nothing changed, and the same rows
    finish once they are sound."""
    import paper_2608_23834_amd as mk
    import torch
    lens = [16 * max_pages] + [500] * (n_req - 1)
    w = dataclasses.replace(wl.scaled(wl.workload(1), tuple(lens), n_layers=1, name=f"finish-{n_req}"),
                            n_q_heads=1, n_kv_heads=1)
    tw = Twin(w, lens=lens, recent=16)
    tw.fill_to([n - 17 for n in lens])
    tw.migrate(np.zeros((n_req, max_pages), np.uint8))
    free = int(tw.orc.fp8_stack[0])
    rows = torch.arange(n_req, dtype=torch.int32, device="cuda")
    state = lambda: [x.clone() for x in (tw.bt, tw.tags, tw.gpu.ctrl[3:])]  # (but for the error word)
    for at, bad in (((n_req - 1, 3), tw.n_tq3), ((0, max_pages - 1), free), ((0, 0), 1 << 30)):
        keep, tag = int(tw.bt[at]), int(tw.tags[at])
        tw.bt[at] = bad
        if bad == free:
            tw.tags[at] = 0
        before = state()
        for _ in range(10):
            mk.kv_request_finish(tw.gpu, rows, tw.bt, tw.tags)
            assert mk.kv_pool_check_errors(tw.gpu, clear=True) == mk.DEVERR["REFCOUNT"]
        assert all(torch.equal(a, b) for a, b in zip(state(), before))
        tw.bt[at], tw.tags[at] = keep, tag
    tw.finish(list(range(n_req)))
    tw.check_tables()
    tw.check_refcounts()
