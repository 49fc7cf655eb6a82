"""A non-finite row stays with the rows that attend to it: in the plain attention
(float32, and bfloat16 head dims other than 64 and 128) a masked key or query
adds nothing, whatever it holds.

A pack of several segments, ended inside the kernels' 16-row products and 64-row
tiles, runs through the block once clean and once with one bad row.  Rows that do
not attend to it keep the clean pass's values: of other segments, and (forward)
earlier ones of its own.  The bad row moves its 16-row products to ordered
multiply-adds, so those values may differ by their float32 rounding (bfloat16: by
a rounding of the storage type that it tips over).
"""
import dataclasses

import numpy as np
import pytest
import torch

from tests.gpu_cases import bf16_case_model
from workloads.configs import ModelConfig

pytestmark = pytest.mark.gpu

LENS = (37, 5, 90, 16, 70)
F32 = ModelConfig(d_model=64, n_q_heads=4, n_kv_heads=2, head_dim=16, d_ff=64, vocab=64, dtype="f32",
                  vocab_chunk=64)
MODELS = {f"f32-{hd}": dataclasses.replace(F32, head_dim=hd) for hd in (16, 32, 64, 128)}
MODELS["bf16-40"] = bf16_case_model(hd=40, d=64, ff=64)


def _inputs(m):
    g = torch.Generator(device="cuda").manual_seed(7)
    dt = torch.bfloat16 if m.dtype == "bf16" else torch.float32
    d, q, hq, f = m.d_model, m.qkv_dim, m.n_q_heads * m.head_dim, m.d_ff
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    w = dict(attn_norm=torch.ones(d, device="cuda"), mlp_norm=torch.ones(d, device="cuda"),
             w_qkv=rnd(q, d) / 8, w_o=rnd(d, hq) / 8, w_gate_up=rnd(2 * f, d) / 8, w_down=rnd(d, f) / 8)
    n = sum(LENS)
    return {k: v.to(dt) for k, v in w.items()}, rnd(n, d).to(dt), rnd(n, d)


def _block(m, w, x, dy):
    from paper_2606_04484_amd import capi
    n, cfg = x.shape[0], capi.block_cfg(m)
    u8 = lambda b: torch.empty(b, dtype=torch.uint8, device="cuda")
    cu = torch.tensor(np.concatenate([[0], np.cumsum(LENS)]), dtype=torch.int32, device="cuda")
    pos = torch.cat([torch.arange(v, dtype=torch.int32, device="cuda") for v in LENS])
    y, dx = torch.empty_like(x), torch.empty_like(dy)
    saved, ws = u8(capi.aj_block_saved_bytes(cfg, n)), u8(capi.aj_block_workspace_bytes(cfg, n, len(LENS)))
    g = {k: torch.zeros(v.shape, device="cuda") for k, v in w.items()}
    capi.aj_varlen_block_fwd(cfg, w, cu, pos, max(LENS), x, y, saved)
    capi.aj_varlen_block_bwd(cfg, w, cu, pos, max(LENS), x, saved, dy, dx, g, ws)
    torch.cuda.synchronize()
    return y.float(), dx


@pytest.mark.parametrize("where", ["x", "dy"])
@pytest.mark.parametrize("seg", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("name", list(MODELS))
def test_a_bad_row_reaches_only_its_own_segment(name, seg, where):
    """x: a NaN row (so its query, key and value are NaN); dy: an infinite one."""
    m = MODELS[name]
    print(f"non-finite {name} segment {seg} in {where}", flush=True)
    w, x, dy = _inputs(m)
    y0, dx0 = _block(m, w, x, dy)
    assert y0.isfinite().all() and dx0.isfinite().all()
    s0 = sum(LENS[:seg])
    bad = s0 + LENS[seg] // 2
    (x if where == "x" else dy)[bad] = float("nan") if where == "x" else float("inf")
    y, dx = _block(m, w, x, dy)
    other = torch.ones(len(x), dtype=torch.bool, device="cuda")
    other[s0:s0 + LENS[seg]] = False
    before = other.clone()
    before[s0:bad] = True
    tol = 2 ** -6 if m.dtype == "bf16" else 1e-5
    for got, ref, rows in ((y, y0, before if where == "x" else torch.ones_like(other)), (dx, dx0, other)):
        assert got[rows].isfinite().all()
        assert (got[rows] - ref[rows]).abs().max() <= tol * ref.abs().max()
    assert not (y if where == "x" else dx)[bad].isfinite().any()
