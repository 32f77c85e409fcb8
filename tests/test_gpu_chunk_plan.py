"""Chunk attention where its plan and its page ring can go wrong: blocks cut into
parts along the pages, page-list blocks that end short, odd page counts, pages
that only later rows see, more requests than the plan keeps in LDS.  Against the
oracle; the tolerance is that of the other chunk tests (three-term E4M3 queries)."""
import dataclasses

import numpy as np
import pytest

import mkv_workloads as wl
from _harness import Twin

pytestmark = pytest.mark.gpu

TOL = 1e-3


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def _bound(w, t, res):
    """What the score product allows, for every row, head and channel.  Three E4M3 terms leave
    2^-14 of an entry of the rotated query (each term half a unit of its four significant
    bits), or 2^-10, half E4M3's smallest step, where that is more, with the largest entry
    scaled to 128 or above: in 2-norm at most (2^-14 + 2^-17 sqrt(d)) |q|.  A score moves by
    that times the request's largest |k| / sqrt(d), a weight by the same share, and a channel
    by that share of the spread of its values, at most 2 max |v| (and 1e-5 of them for the
    rest: fp32 sums, and weights of 22 bits)."""
    f = lambda x: wl.bf16_to_f32(x).astype(np.float64)
    group = w.n_q_heads // w.n_kv_heads
    most = np.empty(res["out"].shape)
    for r, n in enumerate(t.cur):
        k, v = (f(x) for x in wl.kv_layer(w, 0, n, token_offset=r * 1_000_000))
        kn = np.repeat(np.sqrt((k ** 2).sum(-1)).max(0), group)             # [head]
        vc = np.repeat(np.abs(v).max(0), group, axis=0)                     # [head][channel]
        rows = slice(res["cu"][r], res["cu"][r + 1])
        qn = np.sqrt((f(res["q"][rows]) ** 2).sum(-1))                      # [row][head]
        share = (2.0 ** -14 + 2.0 ** -17 * np.sqrt(w.head_dim)) * qn * kn / np.sqrt(w.head_dim) + 1e-5
        most[rows] = share[..., None] * 2 * vc
    return most


def _twin(d, hq, hkv, lens, recent):
    w = dataclasses.replace(wl.workload(2), n_q_heads=hq, n_kv_heads=hkv, head_dim=d, ctx=tuple(lens),
                            n_req=len(lens), n_layers=1, recent=recent)
    return w, Twin(w, lens=lens, recent=recent)


def _run(d, hq, hkv, ctx, nq, recent, stride=1, migrate_after=False, tol=lambda *a: TOL):
    import paper_2608_23834_amd as mk
    w, t = _twin(d, hq, hkv, [c + q for c, q in zip(ctx, nq)], recent)
    t.fill_to(ctx)
    t.migrate(np.zeros((t.n_req, t.max_pages), np.uint8))
    t.append(nq)
    if migrate_after:
        t.migrate(np.zeros((t.n_req, t.max_pages), np.uint8))
    res = t.chunk(nq, sample_stride=stride)
    assert mk.kv_pool_check_errors(t.gpu) == 0
    ref, out = res["ref_out"], res["out"]
    assert np.isfinite(out).all()
    ok = np.isfinite(ref)
    err, most = np.abs(out[ok] - ref[ok]), np.broadcast_to(tol(w, t, res), out.shape)[ok]
    print(f"chunk d{d} {hq}/{hkv} ctx {ctx[:4]} nq {nq[:4]}: max abs error {err.max():.2e}, of the bound "
          f"{(err / most).max():.2f}", flush=True)
    assert (err <= most).all()


@pytest.mark.parametrize("d", [128, 256])
@pytest.mark.parametrize("ctx,nq,recent", [
    ([7000], [1], 64),                    # one query: many parts, nearly all TQ3
    ([4097], [5], 1 << 20),               # all FP8, an odd count
    ([2080 + 48], [3], 48),               # 65 TQ3 pairs: a list block of one pair, then FP8
    ([4128 + 64, 33, 700], [17, 40, 2], 64),  # 129 pairs beside short requests
    ([0, 16], [250, 31], 32),             # no context: rows end at different pages
])
def test_chunk_cut_and_lists(torch_cuda, d, ctx, nq, recent):
    _run(d, 8, 2, ctx, nq, recent)


@pytest.mark.parametrize("d", [128, 256])
def test_chunk_tq3_past_early_rows(torch_cuda, d):
    """The chunk's own pages are already TQ3: early rows skip TQ3 pairs."""
    _run(d, 12, 2, [96, 500], [220, 130], 16, migrate_after=True)


@pytest.mark.parametrize("d", [128, 256])
def test_chunk_fp8_value_scales(torch_cuda, d):
    """FP8 pages only, values of every size.  Values times a power of two (scales of 2^-15 to
    2^7 here) give the rows times it, up to what the products make of the same operands: a
    weight keeps 22 bits and the values' conversion is exact, whatever the scale.  2^-20 of
    the rows' 2-norm is two units of a weight's last bit."""
    import paper_2608_23834_amd as mk
    ctx, nq = [700, 33], [150, 40]
    rows = {}
    for power in (0, -8, -5, 4, 11):
        w, t = _twin(d, 8, 2, [c + q for c, q in zip(ctx, nq)], 1 << 20)
        for counts in (ctx, nq):
            k, v = zip(*(wl.kv_layer(w, 0, n, token_offset=r * 1_000_000 + t.cur[r]) for r, n in enumerate(counts)))
            v = wl.bf16_round(wl.bf16_to_f32(np.concatenate(v)) * np.float32(2.0 ** power))
            t.append(counts, layer_kv=(np.concatenate(k)[None], v[None]))
        assert (t.otags != 2).all()
        scales = t.gpu.fp8_scales_view()[0, :, :, 1]
        scales = scales[scales > 0]
        assert float(scales.min()) >= 2.0 ** -15 and float(scales.max()) < 2.0 ** 8
        res = t.chunk(nq)
        rows[power] = res["out"] * np.float32(2.0 ** -power)
        ref = res["ref_out"] * 2.0 ** -power
        err, moved = (float(np.linalg.norm(rows[power] - x) / np.linalg.norm(ref)) for x in (ref, rows[0]))
        print(f"chunk d{d}, values times 2^{power}: relative error {err:.2e}, off the unscaled rows by "
              f"{moved:.2e}", flush=True)
        assert float(np.max(np.abs(rows[power] - ref))) <= TOL
        assert moved <= 2.0 ** -20
        assert mk.kv_pool_check_errors(t.gpu) == 0


def test_chunk_many_requests(torch_cuda):
    # 4,000 rows over at most 42 tokens, many of them nearly one token's value: held
    # to the bound of the score product instead of the long contexts' tolerance
    n = 1030
    _run(128, 2, 1, [(7 * r) % 40 for r in range(n)], [1 + r % 3 for r in range(n)], 16, tol=_bound)


@pytest.mark.parametrize("n_q", [70_000, 540_000])
def test_chunk_overlapping_ranges_of_many_requests(torch_cuda, n_q):
    """Every second request claims all queries: 2^28 row blocks, and more than 2^31 where the
    call may have 133,035.  The range error, and nothing is written."""
    import paper_2608_23834_amd as mk
    n_req, hq = 65535, 16
    pool = mk.Pool(1, hq, 1, 128, 1, 1, 16, np.ones(128, np.int8))
    cu = torch_cuda.zeros(n_req + 1, dtype=torch_cuda.int32, device="cuda")
    cu[1::2] = n_q
    q = torch_cuda.empty((n_q, hq, 128), dtype=torch_cuda.int16, device="cuda")
    out = torch_cuda.full((n_q, hq, 128), 7.0, device="cuda")
    bt = torch_cuda.zeros((n_req, 1), dtype=torch_cuda.int32, device="cuda")
    tags = torch_cuda.zeros((n_req, 1), dtype=torch_cuda.uint8, device="cuda")
    sl = torch_cuda.ones(n_req, dtype=torch_cuda.int32, device="cuda")
    ws = mk.workspace(pool, n_req, 1, n_q)
    mk.paged_attn_chunk(pool, 0, q, cu, bt, tags, sl, out, ws)
    assert mk.kv_pool_check_errors(pool, clear=True) == mk.DEVERR["RANGE"]
    assert bool((out == 7.0).all())
    print(f"{n_q} queries claimed by {n_req // 2 + 1} requests: refused", flush=True)


def _chunk_and_decode(torch, t, w, q):
    """The last query of every request by the chunk call and by the decode, with the error
    word of each."""
    import paper_2608_23834_amd as mk
    n, rows = t.n_req, torch.from_numpy(q.view(np.int16)).cuda()
    cu = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    sl = torch.tensor(t.cur, dtype=torch.int32, device="cuda")
    out = torch.full((n, w.n_q_heads, w.head_dim), float("nan"), device="cuda")
    ref = out.clone()
    mk.paged_attn_chunk(t.gpu, 0, rows, cu, t.bt, t.tags, sl, out, mk.workspace(t.gpu, n, t.max_pages, n))
    e0 = mk.kv_pool_check_errors(t.gpu, clear=True)
    mk.paged_attn_decode(t.gpu, 0, rows, t.bt, t.tags, sl, ref, None, mk.workspace(t.gpu, n, t.max_pages))
    return out.cpu().numpy(), ref.cpu().numpy(), e0, mk.kv_pool_check_errors(t.gpu, clear=True)


@pytest.mark.parametrize("d", [128, 256])
def test_chunk_leaves_out_pages_outside_the_pool(torch_cuda, d):
    """Ids outside the pool set the error word and are left out, as in the decode; page 0,
    here without valid contents, does not stand in for them."""
    import paper_2608_23834_amd as mk
    w, t = _twin(d, 8, 2, [700, 333], 128)
    t.orc = None
    t.fill_to([700, 333])
    t.migrate(np.zeros((2, t.max_pages), np.uint8))
    bt, tags = t.bt.cpu().numpy(), t.tags.cpu().numpy()
    for bad8, bad3 in ((t.n_fp8, t.n_tq3), (-5, -1), (1 << 30, 1 << 30)):
        t.bt.copy_(torch_cuda.from_numpy(bt))
        for r in range(2):
            t.bt[r, int(np.argmax(tags[r] == 2))] = bad3       # the first of its format: page a of a pair
            t.bt[r, int(np.argmax(tags[r] == 2)) + 5] = bad3
            t.bt[r, int(np.argmax(tags[r] == 0))] = bad8
            t.bt[r, int(np.argmax(tags[r] == 0)) + 1] = bad8
        live = t.bt.cpu().numpy()
        # contents that are no numbers where no live page lies
        f8, f3 = ((np.setdiff1d(np.arange(n), live[m]), n) for n, m in ((t.n_fp8, tags < 2), (t.n_tq3, tags == 2)))
        t.gpu.fp8_scales_view()[:, torch_cuda.from_numpy(f8[0]).cuda()] = float("nan")
        t.gpu.tq3_view()[:, torch_cuda.from_numpy(f3[0]).cuda(), :, 12 * d:] = 0xFF
        out, ref, e0, e1 = _chunk_and_decode(torch_cuda, t, w, wl.q_decode(w, 0)[:2])
        assert e0 == e1 == mk.DEVERR["RANGE"]
        assert np.isfinite(ref).all() and np.isfinite(out).all()
        assert float(np.max(np.abs(out - ref))) <= TOL


def test_chunk_pool_without_tq3_pages(torch_cuda):
    """A Stale tag in a pool that holds no TQ3 page."""
    import paper_2608_23834_amd as mk
    w = dataclasses.replace(wl.workload(2), n_q_heads=8, n_kv_heads=2, head_dim=128, ctx=(300, 90), n_req=2,
                            n_layers=1, recent=1 << 20)
    t = Twin(w, lens=[300, 90], recent=1 << 20, n_tq3=0, with_oracle=False)
    t.fill_to([300, 90])
    t.tags[0, 3:5] = 2
    t.tags[1, 0] = 2
    out, ref, e0, e1 = _chunk_and_decode(torch_cuda, t, w, wl.q_decode(w, 0)[:2])
    assert e0 == e1 == mk.DEVERR["RANGE"]
    assert np.isfinite(out).all() and float(np.max(np.abs(out - ref))) <= TOL


@pytest.mark.parametrize("d", [128, 256])
def test_chunk_rows_without_the_other_requests(torch_cuda, d):
    """On a deterministic pool the rows of a request are the same, bit for bit, alone and
    beside the others of a call; otherwise its blocks are cut in other places, and both are
    within the other tests' tolerance of the exact rows."""
    import paper_2608_23834_amd as mk
    lens, nq = [8200, 900, 5000, 64, 3000], [64, 33, 40, 64, 10]
    w, t = _twin(d, 12, 2, lens, 256)
    t.orc = None
    t.fill_to(lens)
    t.migrate(np.zeros((t.n_req, t.max_pages), np.uint8))
    for fixed in (False, True):
        mk.paged_attn_set_deterministic(t.gpu, fixed)
        both = t.chunk(nq)
        q = torch_cuda.from_numpy(both["q"].view(np.int16)).cuda()
        for r in range(t.n_req):
            a, b = both["cu"][r], both["cu"][r + 1]
            out = torch_cuda.full((nq[r], 12, d), float("nan"), device="cuda")
            mk.paged_attn_chunk(t.gpu, 0, q[a:b].contiguous(), torch_cuda.tensor([0, nq[r]], dtype=torch_cuda.int32, device="cuda"),
                                t.bt[r:r + 1].contiguous(), t.tags[r:r + 1].contiguous(),
                                torch_cuda.tensor(lens[r:r + 1], dtype=torch_cuda.int32, device="cuda"), out,
                                mk.workspace(t.gpu, 1, t.max_pages, nq[r]))
            alone = out.cpu().numpy()
            off = float(np.max(np.abs(alone - both["out"][a:b])))
            print(f"d{d} deterministic {fixed}: request {r} alone and beside the others: {off:.2e}", flush=True)
            assert off == 0 if fixed else off <= 2 * TOL
    mk.paged_attn_set_deterministic(t.gpu, False)
    assert mk.kv_pool_check_errors(t.gpu) == 0


def test_chunk_workspace_sizes(torch_cuda):
    """A workspace sized for more queries, requests or pages is never the smaller one."""
    import paper_2608_23834_amd as mk
    for d, hq, hkv in ((256, 24, 4), (128, 32, 8), (128, 16, 1)):
        _, t = _twin(d, hq, hkv, [16], 16)
        size = lambda r, p, q: mk.paged_attn_workspace_bytes(t.gpu, r, p, q)
        qs = [1, 2, 7, 64, 127, 128, 500, 2047, 2048, 2049, 2730, 2731, 4096, 8192, 65536, 1 << 20]
        for r in (1, 3, 64, 1030):
            for p in (1, 2, 40, 63, 4096):
                now = [size(r, p, q) for q in qs]
                assert all(a <= b for a, b in zip(now, now[1:]))
                assert all(size(r, p, q) <= min(size(r + 1, p, q), size(r, p + 1, q)) for q in qs[::3])


@pytest.mark.parametrize("nq", [[2100, 40], [900, 7, 1300, 1]])
def test_chunk_workspace_serves_smaller_calls(torch_cuda, nq):
    """One workspace, sized for the first chunk of a prompt (too many blocks to be cut), for
    the chunks after it as well."""
    import paper_2608_23834_amd as mk
    _, t = _twin(128, 32, 8, [sum(nq)], 256)
    ws = mk.workspace(t.gpu, 1, t.max_pages, max(nq))
    for n in nq:
        t.append([n])
        t.migrate(np.zeros((1, t.max_pages), np.uint8))
        res = t.chunk([n], sample_stride=max(1, n // 40), ws=ws)
        ok = np.isfinite(res["ref_out"])
        err = float(np.max(np.abs(res["out"][ok] - res["ref_out"][ok])))
        print(f"chunk of {n}: max abs error {err:.2e}", flush=True)
        assert np.isfinite(res["out"]).all() and err <= TOL
    assert mk.kv_pool_check_errors(t.gpu) == 0


def test_chunk_least_workspace(torch_cuda):
    """The smallest workspace that is taken (it does not depend on the queries): blocks
    left whole, and more of them than it holds work items for."""
    import paper_2608_23834_amd as mk
    ctx, nq = [300, 0, 40], [4200, 70, 5]
    _, t = _twin(128, 16, 1, [c + q for c, q in zip(ctx, nq)], 64)
    t.fill_to([c + q for c, q in zip(ctx, nq)])
    t.migrate(np.zeros((t.n_req, t.max_pages), np.uint8))
    full = t.chunk(nq, sample_stride=301)
    lo, hi = 0, mk.paged_attn_workspace_bytes(t.gpu, t.n_req, t.max_pages, 1)
    one = torch_cuda.zeros((3, 16, 128), dtype=torch_cuda.int16, device="cuda")
    out = torch_cuda.zeros((3, 16, 128), device="cuda")
    cu = torch_cuda.tensor([0, 1, 2, 3], dtype=torch_cuda.int32, device="cuda")
    sl = torch_cuda.tensor(t.cur, dtype=torch_cuda.int32, device="cuda")
    big = torch_cuda.zeros(hi, dtype=torch_cuda.uint8, device="cuda")
    while hi - lo > 1:  # (a size that is too small is refused on the host)
        mid = (lo + hi) // 2
        try:
            mk.paged_attn_chunk(t.gpu, 0, one, cu, t.bt, t.tags, sl, out, big[:mid])
            hi = mid
        except mk.MkvError as e:
            assert e.code == 3
            lo = mid
    assert hi < 3 * 8 * 3 * (t.max_pages + 2) + 3 * 1280 + 3 * 256 + 512 * 48 + 256
    small = t.chunk(nq, sample_stride=301, ws=big[:hi])
    err = float(np.max(np.abs(full["out"] - small["out"])))
    print(f"least workspace {hi} bytes, max abs difference {err:.2e}", flush=True)
    assert np.isfinite(small["out"]).all()
    assert err == 0  # (with room for parts so many blocks are left whole as well)
    ok = np.isfinite(small["ref_out"])
    assert float(np.max(np.abs(small["out"][ok] - small["ref_out"][ok]))) <= TOL
    assert mk.kv_pool_check_errors(t.gpu) == 0
