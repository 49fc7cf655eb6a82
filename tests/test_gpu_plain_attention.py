"""The float32 products and the attention of head dims other than 64 and 128, at
the edges of their tiles: whole actor updates against the float64 oracle at the
bounds of the other actor tests (float32: 1e-4 everywhere; bfloat16: log-prob
2e-2, loss and gradients 1e-2, cosine 0.999).

Head dims cover every count of 16-feature chunks with and without padding; the
widths make ragged 64-wide tiles and reductions; packs of 300 tokens make
segments end inside a wave's 16 rows and workgroups' 64.
"""
import dataclasses

import pytest

from tests.gpu_cases import Case, bf16_case_model, workload
from tests.test_gpu_actor import check, run_gpu
from workloads import make_lora_numpy
from workloads.configs import ModelConfig

pytestmark = pytest.mark.gpu


def _model(hd, dtype="f32", **kw):
    base = dict(d_model=136, n_q_heads=4, n_kv_heads=2, head_dim=hd, d_ff=200, vocab=1000,
                dtype=dtype, vocab_chunk=384)
    return ModelConfig(**{**base, **kw})


@pytest.mark.parametrize("hd,pack", [(8, 131072), (16, 300), (24, 131072), (32, 300), (40, 131072),
                                     (64, 300), (72, 131072), (128, 300)])
def test_float32(hd, pack):
    print(f"f32 hd={hd} pack={pack}", flush=True)
    case = Case(workload(_model(hd), n_traj=3, seed=hd), margin=0.01)
    check(case, run_gpu(case, True, pack_tokens=pack), True, 1e-4, 1e-4, 1e-4, 0.99999)


@pytest.mark.parametrize("widths", [dict(d_model=8, d_ff=8, vocab=9, vocab_chunk=8),
                                    dict(d_model=264, d_ff=72, vocab=65, vocab_chunk=64)])
def test_float32_small_and_odd_widths(widths):
    print(f"f32 {widths}", flush=True)
    case = Case(workload(_model(16, **widths), n_traj=2), margin=0.01)
    check(case, run_gpu(case, False), False, 1e-4, 1e-4, 1e-4, 0.99999)


def test_float32_adapters_with_ragged_rank():
    m = dataclasses.replace(_model(24), n_layers=2)
    lora = make_lora_numpy(m, 40, seed=2000, b_std=0.05)
    case = Case(workload(m, n_traj=2), margin=0.01, lora=lora, lora_scale=2.0)
    check(case, run_gpu(case, True), True, 1e-4, 1e-4, 1e-4, 0.99999)


@pytest.mark.parametrize("hd", [16, 40, 96])
def test_bfloat16(hd):
    print(f"bf16 hd={hd}", flush=True)
    case = Case(workload(bf16_case_model(hd=hd, d=256), n_traj=4), noise_std=0.3, margin=0.05)
    check(case, run_gpu(case, True), True, 2e-2, 1e-2, 1e-2, 0.999)
