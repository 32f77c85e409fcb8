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
    """What the score product allows: the rotated query is held to 2^-15 of each
    entry (three E4M3 terms of four significant bits), so a score moves by up to
    2^-15 |q| |k| / sqrt(d), a weight by that share, and an output by that share of
    the spread of the values, at most 2 max |v|."""
    norm = lambda x: float(np.sqrt((wl.bf16_to_f32(x).astype(np.float64) ** 2).sum(-1)).max())
    kv = [wl.kv_layer(w, 0, n, token_offset=r * 1_000_000) for r, n in enumerate(t.cur)]
    k = max(norm(k) for k, _ in kv)
    v = max(float(np.abs(wl.bf16_to_f32(v)).max()) for _, v in kv)
    return 2.0 ** -15 * norm(res["q"]) * k / np.sqrt(w.head_dim) * 2 * v


def _run(d, hq, hkv, ctx, nq, recent, stride=1, migrate_after=False, tol=lambda *a: TOL):
    import paper_2608_23834_amd as mk
    lens = [c + q for c, q in zip(ctx, nq)]
    w = dataclasses.replace(wl.workload(2), n_q_heads=hq, n_kv_heads=hkv, head_dim=d, ctx=tuple(lens),
                            n_req=len(lens), n_layers=1, recent=recent)
    t = Twin(w, lens=lens, recent=recent)
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
    err = float(np.max(np.abs(out[ok] - ref[ok])))
    print(f"chunk d{d} {hq}/{hkv} ctx {ctx[:4]} nq {nq[:4]}: max abs error {err:.2e}", flush=True)
    assert err <= tol(w, t, res)


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


def test_chunk_many_requests(torch_cuda):
    # 4,000 rows over at most 42 tokens, many of them nearly one token's value: held
    # to the bound of the score product instead of the long contexts' tolerance
    n = 1030
    _run(128, 2, 1, [(7 * r) % 40 for r in range(n)], [1 + r % 3 for r in range(n)], 16, tol=_bound)
