"""The MFMA main loop at the edges of its tiles and k-steps, through the LM head.

The LM head's three products cover every operand layout the loop takes, with
every one of its sizes free: logits = hn W^T (K = d; W as stored or
transposed), d hn = dz W (K = vocab chunk) and dW = dz^T hn (K = targets).  The
reference is float64 on the same bfloat16 storage (hn and dz rounded once).

Tolerances: a product's float32 sums are exact to ~1e-6 here; what differs is
the storage rounding (relative 2^-9 at most per element of hn and dz, an
element of either side a neighbour apart at most).  So log-probs agree to
2^-8 of the largest logit, dW = dz^T hn to a relative L2 of 2^-8, and dh, the
norm's backward of dz W, to 2^-7.
"""
import numpy as np
import pytest
import torch

from tests import plans

pytestmark = pytest.mark.gpu

# (targets, d, vocab, chunk): reductions below one k-step, of 1 to 9 steps (so
# every remainder of the four-stage ring), ragged ends; one row to two tiles
SIZES = [(1, 8, 8, 8), (31, 24, 40, 40), (33, 40, 264, 96), (255, 64, 256, 256), (257, 104, 520, 264),
         (300, 136, 1000, 512), (64, 160, 96, 96), (129, 264, 288, 144), (700, 32, 2056, 2056),
         (96, 520, 130, 128),
         # reductions in pieces (PIECES): every tile's (few tiles), and those of the
         # tiles past a full round of 256 (65 x 5 tiles of d hidden)
         (300, 136, 4104, 4104), (2000, 264, 2600, 2600), (16500, 1032, 2056, 2056)]
# of these the plans of d hidden and of dW: (tile, whole tiles, pieces of the rest)
PIECES = {(300, 4104): ((128, 0, 15), (128, 66, 1)), (2000, 2600): ((128, 0, 5), (128, 0, 4)),
          (16500, 2056): ((256, 256, 3), (256, 0, 5))}


def _bf(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16)


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("n,d,vocab,chunk", SIZES)
def test_lm_head_products(n, d, vocab, chunk, transposed):
    from paper_2606_04484_amd import capi
    if transposed and vocab % 8:
        pytest.skip("the transposed copy needs vocab % 8 == 0")
    print(f"lm head n={n} d={d} vocab={vocab} chunk={chunk} transposed={transposed}", flush=True)
    if (n, vocab) in PIECES:
        cap = max(plans.partial_floats(chunk, d), plans.partial_floats(n, d))
        p = [plans.gemm_plan(n, d, chunk, cap), plans.gemm_plan(chunk, d, n, cap)]
        assert tuple((x.tile, x.whole, x.split) for x in p) == PIECES[n, vocab]
    rng = np.random.default_rng(n * 7 + d)
    h = _bf(rng.standard_normal((n + 1, d)))
    gain = _bf(1 + 0.1 * rng.standard_normal(d))
    w = _bf(0.1 * rng.standard_normal((vocab, d)))
    tok = rng.integers(0, vocab, n + 1).astype(np.int32)
    adv = rng.standard_normal(n + 1).astype(np.float32)
    eps, rms = 0.2, 1e-6

    h64, g64, w64 = (t.double().numpy() for t in (h, gain, w))
    r = 1 / np.sqrt((h64[:n] ** 2).mean(1) + rms)
    hn = _bf(h64[:n] * r[:, None] * g64).double().numpy()
    z = hn @ w64.T
    lse = np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)
    t = tok[1:]
    lp = z[np.arange(n), t] - lse
    old = np.zeros(n + 1, np.float32)
    old[1:] = lp + 0.05 * np.sign(rng.standard_normal(n))        # well inside the clip range
    ratio = np.exp(lp - old[1:])
    g = -adv[1:] * ratio / n
    onehot = np.zeros((n, vocab))
    onehot[np.arange(n), t] = 1
    dz = _bf(g[:, None] * (onehot - np.exp(z - lse[:, None]))).double().numpy()
    dw_ref = dz.T @ hn
    dhn = dz @ w64
    gd = g64 * dhn
    dh_ref = r[:, None] * (gd - h64[:n] * (r ** 2)[:, None] * (gd * h64[:n]).mean(1, keepdims=True))

    cfg = capi.LossCfg(d, vocab, chunk, eps, rms, capi.AJ_BF16, 0)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    u8 = lambda b: torch.empty(b, dtype=torch.uint8, device="cuda")
    hg, gg, wg = h.cuda(), gain.cuda(), w.cuda()
    wt = wg.t().contiguous() if transposed else None
    saved, ws = u8(capi.aj_loss_saved_bytes(cfg, n)), u8(capi.aj_loss_workspace_bytes(cfg, n))
    lp_g, lse_g, stats = (torch.zeros(k, device="cuda") for k in (n, n, 5))
    dh, dg, dw = torch.zeros(n + 1, d, device="cuda"), torch.zeros(d, device="cuda"), torch.zeros(vocab, d, device="cuda")
    args = (dev(np.arange(1, n + 1, dtype=np.int32)), dev(tok), dev(old), dev(adv), 1.0 / n, hg, gg, wg, saved)
    capi.aj_logprob_pg_loss_fwd(cfg, *args, lp_g, lse_g, stats, ws, w_vocab_t=wt)
    capi.aj_logprob_pg_loss_bwd(cfg, *args, lp_g, lse_g, dh, dg, dw, ws, w_vocab_t=wt)
    torch.cuda.synchronize()
    assert np.max(np.abs(lp_g.cpu().numpy() - lp)) <= 2 ** -8 * max(1.0, np.abs(z).max())
    rel = lambda a, b: np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b)
    assert rel(dw, dw_ref) <= 2 ** -8
    assert rel(dh[:n], dh_ref) <= 2 ** -7
    assert not dh[n].any()


@pytest.mark.parametrize("rank", [8, 40, 136, 256])
def test_second_segment_steps(rank):
    """The adapters' second reduction segment from one k-step to eight (more
    than the loop's stages): with A and B zero in all but the first 8 of `rank`
    rows, the update is that of rank 8, up to one bfloat16 rounding of each
    layer's outputs, whose sums may run in another order."""
    import dataclasses
    from tests.gpu_cases import Case, bf16_case_model, rel_l2, workload
    from tests.test_gpu_actor import run_gpu
    from workloads import make_lora_numpy
    print(f"second segment rank={rank}", flush=True)
    m = dataclasses.replace(bf16_case_model(hd=64, d=256, hq=4, hkv=2, ff=512), n_layers=1)
    base = make_lora_numpy(m, 8, seed=2001, b_std=0.05)
    wide = {}
    for k, v in base.items():
        pad = np.zeros((rank, v.shape[1]) if k.startswith("lora_a") else (v.shape[0], rank), np.float32)
        pad[tuple(slice(0, s) for s in v.shape)] = v
        wide[k] = pad
    case = Case(workload(m, n_traj=2), noise_std=0.3, margin=0.05, lora=base, lora_scale=0.5)
    a = run_gpu(case, True)
    case.lora = wide
    b = run_gpu(case, True)
    np.testing.assert_allclose(a["lp"], b["lp"], atol=2e-2, rtol=0)
    for k, v in base.items():
        assert rel_l2(b["grads"][k][tuple(slice(0, s) for s in v.shape)], a["grads"][k]) <= 1e-2, k


def test_second_segment_in_pieces():
    """A down projection of 4104 features over few tokens runs in pieces, its
    adapters' segment with the first of them: against the float64 oracle at the
    bounds of the other bfloat16 actor tests (log-prob 2e-2, loss and gradients
    1e-2, cosine 0.999)."""
    import dataclasses
    from tests.gpu_cases import Case, bf16_case_model, workload
    from tests.test_gpu_actor import check, run_gpu
    from workloads import make_lora_numpy
    print("second segment in pieces", flush=True)
    m = dataclasses.replace(bf16_case_model(hd=64, d=256, hq=4, hkv=2, ff=4104), n_layers=1)
    case = Case(workload(m, n_traj=2), noise_std=0.3, margin=0.05,
                lora=make_lora_numpy(m, 40, seed=2001, b_std=0.05), lora_scale=0.5)
    n = case.merged.n_tok
    assert plans.gemm_plan(n, m.d_model, m.d_ff, min(2000 * n, 256 * 65536), True).split > 1
    check(case, run_gpu(case, True), True, 2e-2, 1e-2, 1e-2, 0.999)


@pytest.mark.parametrize("hq,hkv,hd,ff,parts", [(7, 1, 64, 128, 1), (7, 1, 64, 512, 4),
                                                (7, 1, 64, 1024, 7), (6, 2, 128, 1536, 3),
                                                (4, 4, 128, 512, 1)])
def test_key_gradients_in_parts(hq, hkv, hd, ff, parts):
    """The dK/dV pass with a group's query heads in one part (128 and the group
    of one head), in uneven ones (512: the scratch holds 4 parts of 7 heads) and
    one head each: against the oracle at the same bounds."""
    from tests.gpu_cases import Case, bf16_case_model, workload
    from tests.test_gpu_actor import check, run_gpu
    print(f"dK/dV parts hq={hq} hkv={hkv} hd={hd} ff={ff}", flush=True)
    m = bf16_case_model(hd=hd, d=256, hq=hq, hkv=hkv, ff=ff)
    case = Case(workload(m, n_traj=2), noise_std=0.3, margin=0.05)
    # the backward's scratch is d gate and d up: n rows of ff floats
    n, n_seg = case.merged.n_tok, case.merged.n_seg
    b = plans.AttnBwdArgs(n_tok=n, n_seg=n_seg, Hq=hq, Hkv=hkv, hd=hd, part=256, part_floats=n * ff)
    assert plans.attn_dkv_parts(b) == parts
    check(case, run_gpu(case, True), True, 2e-2, 1e-2, 1e-2, 0.999)
