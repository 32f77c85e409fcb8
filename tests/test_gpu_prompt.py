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
