"""Prompt-sized appends and the TQ3 encode at the edges of their kernels, bit for
bit against the oracle."""
import dataclasses

import numpy as np
import pytest

import mkv_workloads as wl
from _harness import Twin

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def _twin(d, hkv, lens, n_layers=1, recent=1 << 20, **kw):
    w = dataclasses.replace(wl.workload(2), n_q_heads=hkv, n_kv_heads=hkv, head_dim=d, ctx=tuple(lens),
                            n_req=len(lens), n_layers=n_layers, recent=recent)
    return Twin(w, n_layers=n_layers, **kw)


def _rows(rng, n, h, d, scale=1.0):
    return rng.standard_normal((n, h, d)).astype(np.float32) * np.float32(scale)


@pytest.mark.parametrize("d", [128, 256])
def test_append_page_edges(torch_cuda, d):
    """Partial, whole and continued pages (old codes kept or re-rounded), zero
    rows, negative zeros and scales at both ends of the fp32 range, through the
    plan + quantize path (more tokens than a decode-step append takes)."""
    rng = np.random.default_rng(7 + d)
    h = 2
    first = [1, 15, 16, 17, 3, 400, 20, 33, 0, 31]
    second = [15, 2, 16, 30, 13, 90, 45, 1, 70, 64]
    mags = [1.0, 1e-30, 1e30, 1.0, 3e-38, 1.0, 0.0, 1.0, 1.0, 1e-20]
    grow = [8.0, 1.0, 0.5, 100.0, 1.0, 1e-3, 1.0, 1e6, 1.0, 1.0]
    t = _twin(d, h, [a + b for a, b in zip(first, second)], headroom=16)
    for counts, scales in ((first, mags), (second, [m * g for m, g in zip(mags, grow)])):
        kv = []
        for _ in range(2):
            x = np.concatenate([_rows(rng, n, h, d, s) for n, s in zip(counts, scales)])
            x[::5, :, 3] = -0.0
            x[2::7, :, :] *= np.float32(2.0 ** -30)
            kv.append(wl.bf16_round(x)[None])
        assert sum(counts) > 256
        t.append(counts, layer_kv=tuple(kv))
        t.check_tables()
        t.check_pages()


@pytest.mark.parametrize("n_req,n", [(1, 70000), (3, 22000), (1100, 17), (1030, 1)])
def test_append_plan_sizes(torch_cuda, n_req, n):
    """Calls of more than one batch of table entries and of more than one run of
    requests (the ids, tables and free lists of every page)."""
    lens = [n + (r % 3) for r in range(n_req)]
    t = _twin(128, 1, lens)
    rng = np.random.default_rng(n_req)
    k = wl.bf16_round(_rows(rng, sum(lens), 1, 128))[None]
    t.append(lens, layer_kv=(k, k[:, ::-1].copy()))
    t.check_tables()
    t.check_pages()


@pytest.mark.parametrize("n_req", [65, 130, 200, 256])
@pytest.mark.parametrize("every", [2, 3, 64])
def test_small_append_of_many_fresh_pages(torch_cuda, n_req, every):
    """One token to more than 64 requests, some of which need a fresh page and some not: the
    64th fresh page falls inside a group of 64 requests."""
    t = _twin(128, 1, [40] * n_req)
    rng = np.random.default_rng(n_req + every)

    def step(counts):
        k = wl.bf16_round(_rows(rng, sum(counts), 1, 128))[None]
        t.append(counts, layer_kv=(k, k[:, ::-1].copy()))
        t.check_tables()
        t.check_pages()
        t.check_refcounts()

    step([1 if r % every == 0 else 16 if r % 5 else 0 for r in range(n_req)])
    for _ in range(2):
        step([1] * n_req)


@pytest.mark.parametrize("n_req", [257, 1024, 1025])
def test_append_no_tokens(torch_cuda, n_req):
    """A call without new tokens, of more requests than a decode-step append takes:
    the plan lists nothing and nothing changes."""
    lens = [1 + r % 3 for r in range(n_req)]
    t = _twin(128, 1, lens)
    rng = np.random.default_rng(n_req)
    k = wl.bf16_round(_rows(rng, sum(lens), 1, 128))[None]
    t.append(lens, layer_kv=(k, k))
    state = lambda: [x.clone() for x in (t.gpu.fp8, t.gpu.fp8_scales, t.gpu.tq3, t.gpu.ctrl, t.bt, t.tags)]
    none = np.zeros((1, 0, 1, 128), np.uint16)
    t.append([0] * n_req, layer_kv=(none, none))  # (the second call meets the first one's empty list)
    before = state()
    t.append([0] * n_req, layer_kv=(none, none))
    assert all(torch_cuda.equal(a, b) for a, b in zip(state(), before))
    t.check_tables()
    t.check_pages()
    t.check_refcounts()


def _special_pages(d, h, rng):
    """Blocks of 16 tokens whose codes sit on decision boundaries."""
    blocks = []
    one = np.zeros((16, h, d), np.float32)
    for i in range(16):
        one[i, :, (i * 37) % d] = (-1.0) ** i * 2.0 ** (i % 4)
    blocks.append(one)                                        # basis vectors: exact ties, y = 0
    blocks.append(np.zeros((16, h, d), np.float32))           # zero keys
    blocks.append(np.ones((16, h, d), np.float32))            # constant values (scale 0)
    two = np.zeros((16, h, d), np.float32)
    two[:, :, 0], two[:, :, 1] = 1.0, -1.0
    blocks.append(two)
    ramp = np.tile((np.arange(16, dtype=np.float32) * 0.5)[:, None, None], (1, h, d))
    blocks.append(ramp)                                       # values on half-code boundaries
    blocks.append(ramp - 448.0)
    blocks.append(np.tile((np.arange(16) % 2 * 13.0 + 1.0).astype(np.float32)[:, None, None], (1, h, d)))
    blocks.append(_rows(rng, 16, h, d, 1e-7))                 # binary16 subnormal metadata
    blocks.append(_rows(rng, 16, h, d, 1e-30))
    blocks.append(_rows(rng, 16, h, d, 1e6))                  # saturating metadata
    blocks.append(np.sign(_rows(rng, 16, h, d)) * 448.0)      # the largest integer sums
    big = _rows(rng, 16, h, d)
    big[:, :, :4] *= 64.0
    blocks.append(big)
    off = _rows(rng, 16, h, d, 1e-2) + 100.0                  # zero >> scale: wide guard band
    blocks.append(off)
    blocks += [_rows(rng, 16, h, d, 2.0 ** s) for s in (-8, 0, 6)]
    return np.concatenate(blocks)


@pytest.mark.parametrize("d", [128, 256])
def test_encode_special_pages(torch_cuda, d):
    rng = np.random.default_rng(d)
    h = 3
    x = _special_pages(d, h, rng)
    n = x.shape[0]
    t = _twin(d, h, [n, n], recent=16, n_layers=2)
    k = wl.bf16_round(np.concatenate([x, x[::-1]]))
    v = wl.bf16_round(np.concatenate([x[::-1], x]))
    t.append([n, n], layer_kv=(np.stack([k, v]), np.stack([v, k])))
    t.check_pages()
    t.migrate(np.zeros((2, t.max_pages), np.uint8))
    t.check_tables()
    n8, n3 = t.check_pages()
    assert n3 >= 2 * (n // 16 - 1)


@pytest.mark.parametrize("d", [128, 256])
def test_encode_infinite_values(torch_cuda, d):
    """A page with an infinite value has an infinite V scale; its other values are zero
    codes, no numbers, and count for neither bound of their channel.  Their metadata stays
    finite: zero 65504 and scale -65504 (the bounds that saw nothing), codes 0; a channel
    that holds an infinity has zero -65504."""
    t = _twin(d, 1, [32], recent=16, with_oracle=False)
    rng = np.random.default_rng(d)
    x = _rows(rng, 32, 1, d)
    for ch in (5, d - 1):
        x[3, 0, ch] = np.inf
    k, v = wl.bf16_round(_rows(rng, 32, 1, d))[None], wl.bf16_round(x)[None]
    t.append([32], layer_kv=(k, v))
    t.migrate(np.zeros((1, 2), np.uint8))
    page = int(t.bt[0, 0])
    assert int(t.tags[0, 0]) == 2
    reg = t.gpu.tq3_view()[0, page, 0].cpu().numpy()
    scale, zero = (reg[a: a + 2 * d].view(np.float16) for a in (12 * d + 32, 14 * d + 32))
    inf = np.zeros(d, bool)
    inf[[5, d - 1]] = True
    assert (zero[~inf] == 65504).all() and (scale[~inf] == -65504).all()
    assert (zero[inf] == -65504).all() and np.isnan(scale[inf]).all()
    assert (reg[6 * d: 12 * d] == 0).all()


@pytest.mark.parametrize("d", [128, 256])
def test_promote_special_pages(torch_cuda, d):
    """The same pages back to FP8: zero scales, scales without a fast division, saturated
    and subnormal metadata; every byte as the oracle's."""
    rng = np.random.default_rng(d + 1)
    h = 3
    x = _special_pages(d, h, rng)
    n = x.shape[0]
    t = _twin(d, h, [n, n], recent=16, n_layers=2)
    k = wl.bf16_round(np.concatenate([x, x[::-1]]))
    v = wl.bf16_round(np.concatenate([x[::-1], x]))
    t.append([n, n], layer_kv=(np.stack([k, v]), np.stack([v, k])))
    t.migrate(np.zeros((2, t.max_pages), np.uint8))
    assert t.promote((t.otags == 2).astype(np.uint8)) >= 2 * (n // 16 - 1)
    t.check_tables()
    t.check_pages()
