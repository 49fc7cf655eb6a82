"""The whole actor update at the 1.5B-class block's FULL model shapes against
the float64 oracle, element by element: d 1536, 12 query / 2 key-value heads
of 128, SwiGLU 8960, the full 151936-word LM head streamed in 32768-column
chunks, bfloat16, one pack in the benchmark's launch configuration.

The batch is episodes 0 and 1 of the seeded block1.5b-64x8 workload (37824
unmerged -> 7147 merged tokens in two segments of ~3.6k, 2751 loss tokens),
small enough for the oracle's float64 update (a few tens of seconds on the
host) and large enough that every long-reduction GEMM layout runs the way it
does in the benchmark:
  * NN, 4 waves: d h = d z W_chunk (reduction = the 32768-wide vocab chunk)
    and the gate/up input gradient (reduction 2 d_ff = 17920);
  * NN, 4 waves, also the down projection forward (reduction d_ff = 8960),
    whose weight the step reads from its transposed [in][out] copy;
  * TN, 4 waves: every block weight gradient (reduction = 7147 tokens);
the test asserts that each of these kernel classes actually launched (the
NT layout, which the forward runs on the [out][in] weights, is compared with
the oracle at small shapes in tests/test_gpu_actor.py).

Checked (Section 4.2 step (4): the update; Section 4.4.2: on merged
timelines): every target's log-prob (absolute 2e-2), the loss (relative
1e-2 of max(|L|, mean |term|)), and every gradient tensor -- embedding,
both norm gains, W_qkv, W_o, W_gate_up, W_down, the final gain and the
vocab matrix -- at relative L2 <= 1e-2 with cosine >= 0.999.

Rollout log-probs: the oracle's own log-probs of the merged layout plus the
generator's N(0, 0.05) noise, kept 0.05 (log space) off the clip kinks so
that both sides take the same clip branch.
"""
import numpy as np
import pytest
import torch

from oracle import merge as om
from oracle import model as M
from tests.gpu_cases import cosine, loss_rel_err, nudge_old, rel_l2
from workloads import get_config, make_timelines, make_weights_torch

pytestmark = pytest.mark.gpu

EPISODES = [0, 1]


def _episodes(tl, old):
    return om.episodes_from_flat(tl.traj_tl_off, tl.tl_tok_off, tl.tok, tl.flags, old, tl.adv)


@pytest.fixture(scope="module")
def case():
    cfg = get_config(1)
    m = cfg.model
    tl = make_timelines(cfg).subset(EPISODES)
    Wd = make_weights_torch(m, seed=1000, device="cuda", gain_std=0.1)
    W = {k: v.float().cpu().numpy() for k, v in Wd.items()}
    del Wd
    torch.cuda.empty_cache()
    print(f"full shapes, episodes {EPISODES}: {tl.n_tok} unmerged tokens", flush=True)
    # the source token of every merged position: merge with old = token index
    idx, _ = om.merge_batch(_episodes(tl, np.arange(tl.n_tok, dtype=np.float64)))
    cur_m = M.current_logprob(idx, W, m)
    sel = idx.mask == 1
    cur = np.zeros(tl.n_tok)
    cur[idx.old_logprob[sel].astype(np.int64)] = np.nan_to_num(cur_m[sel])
    llm = (tl.flags & 3) == 2
    old = nudge_old(cur, tl.lp_noise, llm, m.clip_eps, 0.05)
    merged, _ = om.merge_batch(_episodes(tl, old))
    print(f"oracle merge: {merged.n_tok} tokens, segments {np.diff(merged.cu_seqlens)}",
          flush=True)
    ref = M.actor_update(merged, W, m)
    print(f"oracle update done: loss {ref['loss']:.6g}, {ref['n_mask']} loss tokens", flush=True)
    return m, tl, old, W, merged, ref


@pytest.fixture(scope="module")
def gpu_run(case):
    from paper_2606_04484_amd import actor, capi
    m, tl, old, W, merged, ref = case
    dev = actor.upload_timelines(tl, old)
    L = actor.merge(dev, merged=True, pack_tokens=m.pack_tokens)
    Wd = {k: torch.from_numpy(v).to(device="cuda", dtype=torch.bfloat16) for k, v in W.items()}
    A = actor.ActorUpdate(m, Wd)
    A.prepare(L)
    A.zero_grads()
    capi.aj_timing_enable(True)
    A.step(L)
    torch.cuda.synchronize()
    rec = capi.aj_timing_read()
    capi.aj_timing_enable(False)
    out = dict(lp=A.logprob[:L.n_mask].cpu().numpy().astype(np.float64),
               targets=L.targets[:L.n_mask].cpu().numpy(), stats=A.stats.cpu().numpy(),
               err=int(A.err.cpu()[0]), packs=len(L.packs), n_tok=L.n_tok,
               grads={k: v.cpu().numpy() for k, v in A.G.items()}, rec=rec)
    del A, Wd
    torch.cuda.empty_cache()
    print("kernel classes launched: " +
          ", ".join(f"{k} {v[1]}" for k, v in rec.items() if v[1]), flush=True)
    return out


def test_long_reduction_layouts_ran(gpu_run):
    """The step as the actor runs it: the forward projections read the
    transposed weight copies, so its long reductions run the NN or TN layout,
    those in whole 256x256 tiles or long pieces on the 4-wave kernel (the NT one
    is compared in test_gpu_gemm_plans.py)."""
    rec = gpu_run["rec"]
    for k in ("gemm4_nn", "gemm4_tn", "lm_fwd", "lm_dz", "attn_fwd", "attn_bwd"):
        assert rec[k][1] > 0, k
    assert rec["gemm4_nt"][1] == 0 and rec["gemm_nt"][1] == 0
    # one block forward and backward and one loss forward and backward per pack,
    # each bracketing the kernels it launched
    n = gpu_run["packs"]
    assert rec["stage_block"][1] == 2 * n and rec["stage_loss"][1] == 2 * n
    inner = sum(rec[k][0] for k in ("attn_fwd", "attn_bwd"))
    assert rec["stage_block"][0] > inner > 0
    assert rec["stage_loss"][0] > rec["lm_fwd"][0] + rec["lm_dz"][0] > 0


def test_targets_and_logprobs(case, gpu_run):
    m, tl, old, W, merged, ref = case
    got = gpu_run
    assert got["err"] == 0 and got["packs"] == 1 and got["n_tok"] == merged.n_tok
    tgt = ref["tgt"][merged.mask[ref["tgt"]] == 1]
    np.testing.assert_array_equal(got["targets"], tgt)
    err = np.abs(got["lp"] - ref["logprob"][tgt])
    print(f"log-prob |err|: max {err.max():.4g}, rms {np.sqrt(np.mean(err ** 2)):.4g} "
          f"over {len(tgt)} targets", flush=True)
    assert err.max() <= 2e-2


def test_loss(case, gpu_run):
    m, tl, old, W, merged, ref = case
    got = gpu_run
    assert got["stats"][3] == ref["n_mask"]
    le = loss_rel_err(float(got["stats"][0]), ref["loss"], ref["term"])
    print(f"loss {got['stats'][0]:.6g} vs oracle {ref['loss']:.6g}: rel {le:.3g}", flush=True)
    assert le <= 1e-2


def test_every_gradient(case, gpu_run):
    m, tl, old, W, merged, ref = case
    got = gpu_run["grads"]
    assert set(got) == set(ref["grads"])
    bad = []
    for k in sorted(ref["grads"]):
        r, c = rel_l2(got[k], ref["grads"][k]), cosine(got[k], ref["grads"][k])
        print(f"{k}: rel_l2 {r:.3g} cos {c:.6f}", flush=True)
        if not (r <= 1e-2 and c >= 0.999):
            bad.append((k, r, c))
    cat_g = np.concatenate([got[k].ravel() for k in sorted(got)])
    cat_r = np.concatenate([ref["grads"][k].ravel() for k in sorted(got)])
    print(f"all gradients: rel_l2 {rel_l2(cat_g, cat_r):.3g} cos {cosine(cat_g, cat_r):.6f}",
          flush=True)
    assert not bad, bad
