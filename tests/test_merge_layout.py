"""Merger.layout: counts and offsets read back in one wait or in several, and the
packs planned from them, against the definition; several threads at once."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

from paper_2606_04484_amd import actor


def _merger(n_tl, n_seg, dev, seed):
    """A merger of n_tl timelines of 3 tokens whose outputs are filled in by hand."""
    i32 = dict(dtype=torch.int32, device=dev)
    tl = dict(tok=torch.zeros(3 * n_tl, **i32), tl_tok_off=3 * torch.arange(n_tl + 1, device=dev),
              traj_tl_off=torch.tensor([0, n_tl], **i32))
    m = actor.Merger(tl)
    lens = np.random.default_rng(seed).integers(1, 9, n_seg).astype(np.int32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    for k, v in (("cu_seqlens", cu), ("cu_targets", cu // 2)):
        m.out[k][:n_seg + 1] = torch.from_numpy(v).to(dev)
    m.out["counts"].copy_(torch.tensor([n_seg, int(cu[-1]), int(cu[-1] // 2),
                                        int(lens.max(initial=0))]))
    return m, cu


def _check(L, cu, pack):
    n = len(cu) - 1
    assert (L.n_seg, L.n_tok, L.n_mask) == (n, cu[-1], cu[-1] // 2)
    np.testing.assert_array_equal(L.cu_host, cu)
    np.testing.assert_array_equal(L.cut_host, cu // 2)
    at = 0
    for p in L.packs:
        a, b = p["s0"], p["s1"]
        assert a == at and b > a
        assert (p["t0"], p["t1"], p["r0"], p["r1"]) == (cu[a], cu[b], cu[a] // 2, cu[b] // 2)
        assert p["max_len"] == np.diff(cu[a:b + 1]).max()
        assert cu[b] - cu[a] <= pack or b == a + 1
        assert b == n or cu[b + 1] - cu[a] > pack
        at = b
    assert at == n


@pytest.mark.parametrize("limit", [0, 1 << 20])   # offsets after the counts, and with them
@pytest.mark.parametrize("n_tl,n_seg", [(1, 0), (1, 1), (37, 20), (500, 500)])
def test_layout(monkeypatch, n_tl, n_seg, limit):
    monkeypatch.setattr(actor.Merger, "ONE_COPY_TL", limit)
    m, cu = _merger(n_tl, n_seg, "cpu", n_tl)
    for pack in (1, 8, 31, 1 << 30):
        _check(m.layout(pack), cu, pack)


@pytest.mark.gpu
def test_layout_from_threads():
    m, cu = _merger(500, 431, "cuda", 5)
    with ThreadPoolExecutor(4) as pool:
        for i, L in enumerate(pool.map(m.layout, [8 + i for i in range(64)])):
            _check(L, cu, 8 + i)
