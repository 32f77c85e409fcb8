"""Decode merge at the edges of its shapes: as many chunk slots as one round of one
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
