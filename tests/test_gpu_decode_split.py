"""Decode workspaces, pages outside the pool, and the decode merge at the edges of its shapes: as many chunk slots as one round of one
wave, of two, four and eight waves takes, one more, a second round of eight waves;
every slot filled, and most of them past the request's end.  Against the oracle with
the tolerance of the other decode tests."""
import dataclasses

import numpy as np
import pytest

import mkv_workloads as wl
from _harness import Twin, max_abs

pytestmark = pytest.mark.gpu

TOL = 1e-3
RECENT = 16


def _pages(slots):
    """The widest table that one request and one KV head cut into `slots` chunks: 2
    cost units per page outside the window, 3 for the window's one, 32 per chunk."""
    return (32 * slots - 3) // 2 + 1


@pytest.mark.parametrize("d", [128, 256])
@pytest.mark.parametrize("slots", [4, 5, 16, 17, 32, 33, 129])
def test_merge_slots(d, slots):
    import paper_2608_23834_amd as mk
    n = _pages(slots) * 16 - 3
    w = dataclasses.replace(wl.scaled(wl.workload(1 if d == 128 else 5), (n,), n_layers=1, name=f"merge-{slots}"),
                            n_q_heads=3, n_kv_heads=1)
    tw = Twin(w, lens=[n], recent=RECENT)
    for cur in (min(700, n // 2), n - 1):
        tw.fill_to([cur])
        tw.migrate()
        r = tw.decode()
        err = max(max_abs(r["out"], r["ref_out"]), max_abs(r["lse"], r["ref_lse"]))
        print(f"d {d} slots {slots} length {cur}: {err:.2e}", flush=True)
        assert np.all(np.isfinite(r["out"])) and err <= TOL
    r = tw.decode_append()
    err = max(max_abs(r["out"], r["ref_out"]), max_abs(r["lse"], r["ref_lse"]))
    assert np.all(np.isfinite(r["out"])) and err <= TOL
    assert mk.kv_pool_check_errors(tw.gpu) == 0


@pytest.mark.parametrize("d,hq", [(128, 6), (256, 16), (256, 24)])
def test_pages_outside_the_pool_are_left_out(d, hq):
    """Ids outside the pool set the error word and are left out; page 0, here without valid
    contents, does not stand in for them.  The bad pages are the last ones, so the shorter
    request is the reference."""
    import paper_2608_23834_amd as mk
    import torch
    n, keep = 700, 39  # pages 39 .. 42 go bad: TQ3 pages, then the last ones in FP8
    w = dataclasses.replace(wl.scaled(wl.workload(1 if d == 128 else 5), (n,), n_layers=1, name=f"bad-{hq}"),
                            n_q_heads=hq, n_kv_heads=2)
    tw = Twin(w, lens=[n], recent=32)
    tw.fill_to([n])
    tw.migrate(np.zeros((1, tw.max_pages), np.uint8))
    bt, tags = tw.obt.copy(), tw.otags
    assert tags[0, keep] == 2 and tags[0, -1] == 0
    good = tw.decode(seq_lens=[16 * keep])
    live8, live3 = bt[0, :keep][tags[0, :keep] < 2], bt[0, :keep][tags[0, :keep] == 2]
    free = lambda count, live: torch.from_numpy(np.setdiff1d(np.arange(count), live)).cuda()
    tw.gpu.fp8_scales_view()[:, free(tw.n_fp8, live8)] = float("nan")
    tw.gpu.tq3_view()[:, free(tw.n_tq3, live3), :, 12 * d:] = 0xFF
    tw.orc = None
    for bad in (-1, 1 << 30):
        tw.bt[0, keep:] = bad
        r = tw.decode()
        assert mk.kv_pool_check_errors(tw.gpu, clear=True) == mk.DEVERR["RANGE"]
        err = max(max_abs(r["out"], good["ref_out"]), max_abs(r["lse"], good["ref_lse"]))
        print(f"d {d} heads {hq} id {bad}: {err:.2e}", flush=True)
        assert np.all(np.isfinite(r["out"])) and err <= TOL


@pytest.mark.parametrize("d,hq", [(128, 6), (256, 16), (256, 24)])
@pytest.mark.parametrize("n", [5, 700])
def test_fused_append_to_a_page_outside_the_pool(d, hq, n):
    """The page that the new token lands in has no valid id: the fused step fails as a whole
    (range error, zero rows, nothing changed), whether or not the chunk holds other pages."""
    import paper_2608_23834_amd as mk
    import torch
    w = dataclasses.replace(wl.scaled(wl.workload(1 if d == 128 else 5), (n, 90), n_layers=1, name=f"app-{hq}-{n}"),
                            n_q_heads=hq, n_kv_heads=2)
    tw = Twin(w, lens=[n, 90], recent=32, headroom=16)
    tw.fill_to([n, 90])
    tw.migrate(np.zeros((2, tw.max_pages), np.uint8))
    tw.orc = None
    tw.bt[0, n // 16] = tw.n_fp8
    state = lambda: [x.clone() for x in (tw.bt, tw.tags, tw.gpu.ctrl[3:], tw.gpu.fp8, tw.gpu.fp8_scales, tw.gpu.tq3)]
    before = state()
    r = tw.decode_append()
    assert mk.kv_pool_check_errors(tw.gpu, clear=True) == mk.DEVERR["RANGE"]
    assert (r["out"] == 0).all() and np.isneginf(r["lse"]).all()
    assert all(torch.equal(a, b) for a, b in zip(state(), before))


def test_pool_without_tq3_pages():
    """A Stale tag in a pool that holds no TQ3 page: left out, whatever follows it."""
    import paper_2608_23834_amd as mk
    w = dataclasses.replace(wl.scaled(wl.workload(1), (300,), n_layers=1, name="no-tq3"), n_q_heads=4, n_kv_heads=1)
    tw = Twin(w, lens=[300], recent=1 << 20, n_tq3=0)
    tw.fill_to([300])
    good = tw.decode(seq_lens=[16 * 16])
    tw.orc = None
    tw.tags[0, 16:] = 2
    r = tw.decode()
    assert mk.kv_pool_check_errors(tw.gpu, clear=True) == mk.DEVERR["RANGE"]
    assert max_abs(r["out"], good["ref_out"]) <= TOL and max_abs(r["lse"], good["ref_lse"]) <= TOL


@pytest.mark.parametrize("d", [128, 256])
@pytest.mark.parametrize("pages,waves", [(70, 2), (200, 4), (500, 8)])
def test_merge_of_huge_values_without_weight(d, pages, waves):
    """The tokens of the first wave's slots have values near the largest fp32 number and
    scores so low that their weight is zero: the wave's sums are infinite, and must not
    reach the output (all ones)."""
    import paper_2608_23834_amd as mk
    n = 16 * pages
    w = dataclasses.replace(wl.scaled(wl.workload(1 if d == 128 else 5), (n,), n_layers=1, name=f"huge-{pages}"),
                            n_q_heads=3, n_kv_heads=1)
    tw = Twin(w, lens=[n], recent=1 << 20)
    slots = -(-3 * pages // 32)  # 3 cost units per page, 32 per chunk
    first = -(-32 * (-(-slots // waves)) // 3)  # pages of the first wave's slots
    low = (np.arange(n) < 16 * first)[:, None, None]
    k = np.broadcast_to(np.where(low, -8.0, 8.0), (n, 1, d)).astype(np.float32)
    v = np.broadcast_to(np.where(low, 3.3e38, 1.0), (n, 1, d)).astype(np.float32)
    tw.append([n], layer_kv=(wl.bf16_round(k)[None], wl.bf16_round(v)[None]))
    r = tw.decode(q=wl.bf16_round(np.full((1, 3, d), 1.0, np.float32)))
    print(f"d {d}, {pages} pages: {r['out'].min()} to {r['out'].max()}", flush=True)
    assert max_abs(r["out"], 1.0) <= TOL and max_abs(r["out"], r["ref_out"]) <= TOL
    assert mk.kv_pool_check_errors(tw.gpu) == 0


def _pool(d, hq, hkv, recent):
    import paper_2608_23834_amd as mk
    return mk.Pool(1, hq, hkv, d, 1, 1, recent, np.ones(d, np.int8))


@pytest.mark.parametrize("d,hq,hkv", [(256, 24, 4), (128, 32, 8), (128, 8, 1), (128, 16, 1), (256, 16, 2)])
def test_workspace_sizes(d, hq, hkv):
    """A workspace sized for more requests or pages is never the smaller one."""
    import paper_2608_23834_amd as mk
    for recent in (16, 1024, 1 << 20):
        p = _pool(d, hq, hkv, recent)
        size = np.array([[mk.paged_attn_workspace_bytes(p, r, m) for m in (1, 2, 15, 48, 161, 231, 1986, 4096, 65536)]
                         for r in (1, 2, 7, 8, 12, 13, 27, 31, 32, 33, 36, 40, 63, 64, 65, 127, 128, 300, 5000)])
        assert (np.diff(size, axis=0) >= 0).all() and (np.diff(size, axis=1) >= 0).all()


@pytest.mark.parametrize("d,hq,hkv,more,n,max_pages", [(128, 32, 8, 13, 12, 161), (128, 32, 8, 64, 63, 60),
                                                       (256, 24, 4, 8, 7, 1986), (128, 8, 1, 300, 299, 40)])
def test_workspace_serves_fewer_requests(d, hq, hkv, more, n, max_pages):
    """A decode of n requests on the workspace of `more` (the smaller call needs more
    slots), with the tables as wide as the workspace was sized for."""
    import paper_2608_23834_amd as mk
    import torch
    lens = [16 * max_pages - 5] + [37 + 11 * (r % 9) for r in range(n - 1)]
    w = dataclasses.replace(wl.scaled(wl.workload(1 if d == 128 else 5), tuple(lens), n_layers=1, name=f"ws-{n}-{max_pages}"),
                            n_q_heads=hq, n_kv_heads=hkv)
    tw = Twin(w, lens=lens, recent=1024)
    assert tw.max_pages == max_pages
    tw.fill_to(lens)
    tw.migrate()
    ws = mk.workspace(tw.gpu, more, max_pages)
    guard = torch.full((ws.numel() + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    tw._ws = lambda ws_fill: guard[:ws.numel()]
    r = tw.decode()
    err = max(max_abs(r["out"], r["ref_out"]), max_abs(r["lse"], r["ref_lse"]))
    print(f"d {d}: {n} requests on the workspace of {more}: {err:.2e}", flush=True)
    assert np.all(np.isfinite(r["out"])) and err <= TOL
    assert bool((guard[ws.numel():] == 0xA5).all())
    assert mk.kv_pool_check_errors(tw.gpu) == 0
