"""The work that a user of this framework has it do, as cases that can be timed.

A training program's step over one batch of multi-turn episodes is: merge the
timelines, then for each pack of merged segments the embedding, the decoder
block(s) and the fused LM head + clipped policy-gradient loss, forward and
backward, then AdamW.  Each kind below is one of these stages through its entry
point, and "update" is the whole step through `actor.ActorUpdate`:

  update  merge + one actor update (all weights, or LoRA adapters)
  merge   Algorithm 1 with token-level Match, counts read back, packs planned
  text    the same with text-level Match and its consistency report
  block   the decoder block over one pack, forward only or forward + backward
  loss    LM head + loss over one pack's targets, forward + backward
  embed   the embedding gather and its gradient
  adamw   the optimizer over one flat group of parameters

Shapes are those of `workloads/configs.py`; lengths are ragged as merged
episodes are.  Gradients accumulate from pass to pass, as over the packs of a
batch; "update" clears them first, as a step does.
"""
import dataclasses
import functools
import math
import random

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_2606_04484_amd import actor
from paper_2606_04484_amd import capi
from workloads import get_config, layer_key, lora_key, lora_shapes, make_timelines
from workloads.gen import weight_shapes

DEV = "cuda"
WORKLOADS = {"tiny": 0, "1.5b": 1, "7b": 2, "multi7b": 3, "32b": 4}
LORA_PROJ = ("w_qkv", "w_o", "w_gate_up", "w_down")
BLOCK = ("attn_norm", "w_qkv", "w_o", "mlp_norm", "w_gate_up", "w_down")


def listed():
    return [
        # the smallest whole step: the float32 workload, 8 short episodes, where
        # launches and the host path weigh most
        dict(name="update-tiny-f32", kind="update", shape="tiny", episodes=8, layers=1, rank=0, pack=131072),
        # adapters only, on a two-layer policy of 1.5B-class blocks: 4 episodes
        dict(name="update-lora-1.5b", kind="update", shape="1.5b", episodes=4, layers=2, rank=32, pack=131072),
        # the merge of one batch at its own size (1.2M tokens of 64 episodes)
        dict(name="merge-1.5b", kind="merge", shape="1.5b", episodes=64, copies=1),
        # the merge of a large collection (16 x 32 agent episodes, ~100M tokens)
        dict(name="merge-large", kind="merge", shape="7b", episodes=32, copies=16),
        # text-level Match where the chat template strips earlier thinking
        dict(name="merge-text-7b", kind="text", shape="7b", episodes=32, think=1.0),
        # scoring one short episode (reference or rollout log-probs): forward only
        dict(name="block-fwd-1.5b-short", kind="block", shape="1.5b", tokens=2347, segs=2, train=False),
        # one small pack of multi-agent segments, forward + backward
        dict(name="block-train-7b", kind="block", shape="7b", tokens=19437, segs=5, train=True),
        # one merged long-horizon episode (60 calls in one segment), forward + backward
        dict(name="block-train-32b-long", kind="block", shape="32b", tokens=45769, segs=1, train=True),
        # the LM head over two episodes' targets, with the KL penalty
        dict(name="loss-1.5b-kl", kind="loss", shape="1.5b", tokens=7147, targets=2751, kl=0.002, keep=False),
        # the LM head over one long-horizon episode's targets
        dict(name="loss-32b", kind="loss", shape="32b", tokens=45769, targets=18897, kl=0.0, keep=False),
        # the embedding of a nearly full pack, ids drawn as natural text's are
        dict(name="embed-7b", kind="embed", shape="7b", tokens=118943, zipf=1.1),
        # every parameter of the 1.5B-class workload (block, embedding, LM head)
        dict(name="adamw-1.5b", kind="adamw", n=513544704, copy="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("update", "merge", "text", "block", "block", "loss", "embed", "adamw"))
    if kind == "update":
        if rng.random() < 0.5:
            return dict(kind=kind, shape="tiny", episodes=_log(rng, 2, 24), layers=rng.randint(1, 3),
                        rank=rng.choice((0, 0, 8)), pack=rng.choice((700, 4096, 131072)))
        return dict(kind=kind, shape="1.5b", episodes=rng.randint(1, 6), layers=rng.randint(1, 2),
                    rank=rng.choice((0, 8, 16, 32, 64)), pack=rng.choice((16384, 131072)))
    if kind == "merge":
        shape = rng.choice(("tiny", "1.5b", "7b", "multi7b", "32b"))
        top = get_config(WORKLOADS[shape]).n_traj
        return dict(kind=kind, shape=shape, episodes=rng.randint(1, top), copies=_log(rng, 1, 8))
    if kind == "text":
        shape = rng.choice(("1.5b", "7b", "multi7b", "32b"))
        top = get_config(WORKLOADS[shape]).n_traj
        return dict(kind=kind, shape=shape, episodes=rng.randint(1, top), think=rng.choice((0.5, 1.0)))
    if kind == "block":
        shape = rng.choice(("1.5b", "7b", "32b"))
        tokens = _log(rng, 600, {"1.5b": 100000, "7b": 48000, "32b": 24000}[shape])
        return dict(kind=kind, shape=shape, tokens=tokens, segs=_log(rng, 1, max(1, tokens // 500)),
                    train=rng.random() < 0.6)
    if kind == "loss":
        shape = rng.choice(("1.5b", "7b", "32b"))
        tokens = _log(rng, 500, 40000)
        targets = max(1, int(tokens * rng.uniform(0.1, 0.45)))
        return dict(kind=kind, shape=shape, tokens=tokens, targets=targets, kl=rng.choice((0.0, 0.002)),
                    keep=rng.random() < 0.25)
    if kind == "embed":
        return dict(kind=kind, shape=rng.choice(("1.5b", "7b", "32b")), tokens=_log(rng, 700, 131072),
                    zipf=rng.choice((0.0, 1.1)))
    return dict(kind="adamw", n=_log(rng, 1000, 500000000), copy=rng.choice(("bf16", "f32", "none")))


# ---------------------------------------------------------------- inputs

def _config(case):
    cfg = get_config(WORKLOADS[case["shape"]])
    m = dataclasses.replace(cfg.model, n_layers=case.get("layers", 1))
    return dataclasses.replace(cfg, model=m, n_traj=case.get("episodes", cfg.n_traj))


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(g, *shape, std=1.0, dtype=torch.float32):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32).mul_(std).to(dtype)


def _storage(m):
    return torch.bfloat16 if m.dtype == "bf16" else torch.float32


def _weights(m, g, names):
    shapes = weight_shapes(m)
    out = {}
    for k in names:
        if k.split(".")[0].endswith("norm"):
            out[k] = (1.0 + _randn(g, *shapes[k], std=0.1)).to(_storage(m))
        else:
            out[k] = _randn(g, *shapes[k], std=m.init_std, dtype=_storage(m))
    return out


def _seg_lens(tokens, segs):
    """Ragged segment lengths that add up to `tokens` (a case has the same ones for every seed)."""
    r = random.Random(tokens * 1009 + segs)
    w = [r.uniform(0.5, 2.0) for _ in range(segs)]
    lens = [max(1, int(tokens * v / sum(w))) for v in w]
    while sum(lens) > tokens:
        lens[lens.index(max(lens))] -= 1
    lens[-1] += tokens - sum(lens)
    return lens


def _scored(tokens, want):
    """`want` of the positions 1..tokens-1 in runs, as responses are: sorted int64."""
    r = random.Random(tokens * 31 + want)
    share = want / max(1, tokens - 1)
    pos, at = [], 1
    while at < tokens:
        n = r.randint(50, 400)
        at += int(n * (1 - share) / share * r.uniform(0.5, 1.5)) if share < 1 else 0
        pos.extend(range(at, min(tokens, at + n)))
        at += n
    got = np.array(pos[:want], np.int64)
    if len(got) < want:
        left = np.setdiff1d(np.arange(1, tokens), got)
        got = np.sort(np.concatenate([got, left[len(left) - (want - len(got)):]]))
    return got


@functools.lru_cache(maxsize=4)
def _recipe(shape, episodes, think):
    """The batch whose lengths and shared prefixes every seed of a case has."""
    cfg = dataclasses.replace(get_config(WORKLOADS[shape]), n_traj=episodes)
    return make_timelines(cfg, seed=0, think_p=think)


def _timelines(case, seed):
    """A batch of the case's lengths with ids, advantages and noise of its own: ids are relabelled one to one, so
    that what was a shared prefix stays one."""
    tl = _recipe(case["shape"], case["episodes"], case.get("think"))
    rng = np.random.default_rng(seed)
    vocab = get_config(WORKLOADS[case["shape"]]).model.vocab
    label = rng.permutation(vocab).astype(np.int32)
    llm = (tl.flags & 3) == 2
    adv = np.repeat(rng.standard_normal(tl.n_tl).astype(np.float32), np.diff(tl.tl_tok_off))
    noise = np.zeros(tl.n_tok, np.float32)
    noise[llm] = rng.normal(0.0, 0.05, int(llm.sum()))
    return dataclasses.replace(tl, tok=label[tl.tok], adv=np.where(llm, adv, np.float32(0)), lp_noise=noise)


@functools.lru_cache(maxsize=None)
def _counts(shape, episodes):
    """(unmerged, llm, merged and scored tokens, (query, key) pairs) of a batch."""
    tl = _recipe(shape, episodes, None)
    old = np.zeros(tl.n_tok, np.float32)
    merged, tgt, seg2 = 0, 0, 0
    for lens, m, *_ in _merge_host(tl, old):
        merged += int(sum(lens))
        tgt += int(m.sum())
        seg2 += sum(n * (n + 1) // 2 for n in lens)
    return tl.n_tok, int(((tl.flags & 3) == 2).sum()), merged, tgt, seg2


def _merge_host(tl, old):
    """Algorithm 1 with token-level Match, on the host: per surviving timeline ([length], mask, tok, old
    log-prob, advantage, source position of each llm token)."""
    out = []
    for e in range(len(tl.traj_tl_off) - 1):
        a, b = int(tl.traj_tl_off[e]), int(tl.traj_tl_off[e + 1])
        spans = [(int(tl.tl_tok_off[i]), int(tl.tl_tok_off[i + 1])) for i in range(a, b)]
        gone = [False] * len(spans)
        kept = []
        for i in range(len(spans) - 1, -1, -1):
            if gone[i]:
                continue
            s, t = spans[i]
            tok, flags = tl.tok[s:t], tl.flags[s:t]
            llm = (flags & 3) == 2
            src = np.where(llm, np.arange(s, t), -1)
            for j in range(i - 1, -1, -1):
                sj, tj = spans[j]
                n = tj - sj
                if gone[j] or n > t - s or (n < t - s and not flags[n] & 4):
                    continue
                fj = tl.flags[sj:tj]
                if not np.array_equal(tl.tok[sj:tj], tok[:n]) or np.any((fj ^ flags[:n]) & 4):
                    continue
                gone[j] = True
                take = ((fj & 3) == 2) & ~llm[:n]
                src[:n][take] = np.arange(sj, tj)[take]
                llm[:n] |= take
            at = np.maximum(src, 0)
            kept.append(([t - s], llm, tok, np.where(llm, old[at], 0).astype(np.float32),
                         np.where(llm, tl.adv[at], 0).astype(np.float32), src))
        out.extend(reversed(kept))
    return out


def _ids(g, n, vocab, zipf):
    if not zipf:
        return torch.randint(0, vocab, (n,), generator=g, device=DEV, dtype=torch.int32)
    cdf = torch.arange(1, vocab + 1, device=DEV, dtype=torch.float64).pow_(-zipf).cumsum_(0)
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * cdf[-1]
    return torch.searchsorted(cdf, u).clamp_(max=vocab - 1).to(torch.int32)


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return globals()["_run_" + state["kind"]](state)


# ---------------------------------------------------------------- update

def _update_inputs(case, seed):
    cfg = _config(case)
    m = cfg.model
    g = _gen(seed)
    tl = _timelines(case, seed)
    W = _weights(m, g, weight_shapes(m))
    lora = None
    if case["rank"]:
        lora = {}
        for k, shape in lora_shapes(m, case["rank"]).items():
            std = 1.0 / math.sqrt(shape[1]) if k.startswith("lora_a") else 0.01
            lora[k] = _randn(g, *shape, std=std, dtype=_storage(m))
    segs = _merge_host(tl, np.zeros(tl.n_tok, np.float32))
    # the rollout policy is the current one up to the engines' numerical noise
    with torch.no_grad():
        lp, pos = _policy(W, lora, m, segs, torch.float32)
    src = np.concatenate([s[5] for s in segs])[pos.cpu().numpy()]
    old = np.zeros(tl.n_tok, np.float32)
    old[src] = lp.float().cpu().numpy() + tl.lp_noise[src]
    return cfg, tl, W, lora, old


def _prepare_update(case, seed):
    cfg, tl, W, lora, old = _update_inputs(case, seed)
    m = cfg.model
    dev = actor.upload_timelines(tl, old, DEV)
    merger = actor.Merger(dev)
    A = actor.ActorUpdate(m, W, DEV, lora=lora, lora_rank=case["rank"], lora_scale=2.0)
    merger.launch(True)
    A.prepare(merger.layout(case["pack"]))
    return dict(kind="update", merger=merger, A=A, pack=case["pack"])


def _run_update(s):
    A = s["A"]
    s["merger"].launch(True)
    L = s["merger"].layout(s["pack"])
    A.zero_grads()
    A.step(L)
    return dict(logprob=A.logprob[:L.n_mask], stats=A.stats, grads=A.G)


# ---------------------------------------------------------------- merge, text

def _prepare_merge(case, seed):
    cfg = _config(case)
    tl = _timelines(case, seed)
    old = np.where((tl.flags & 3) == 2, tl.lp_noise - 11.0, 0).astype(np.float32)
    d = actor.upload_timelines(tl, old, DEV)
    R = case["copies"]
    if R > 1:   # other episodes of the same recipe: other ids, same lengths
        k = torch.arange(R, device=DEV)
        n, t = tl.n_tok, tl.n_tl
        ids = (d["tok"].long() + 7919 * k.view(-1, 1)) % cfg.model.vocab
        d = dict(traj_tl_off=torch.cat([(d["traj_tl_off"][:-1] + t * k.view(-1, 1)).flatten(),
                                        torch.tensor([R * t], device=DEV)]).to(torch.int32),
                 tl_tok_off=torch.cat([(d["tl_tok_off"][:-1] + n * k.view(-1, 1)).flatten(),
                                       torch.tensor([R * n], device=DEV)]),
                 tok=ids.flatten().to(torch.int32), flags=d["flags"].repeat(R),
                 old_logprob=d["old_logprob"].repeat(R), adv=d["adv"].repeat(R))
    return dict(kind="merge", merger=actor.Merger(d))


def _run_merge(s):
    s["merger"].launch(True)
    L = s["merger"].layout(131072)
    o, n, k = s["merger"].out, L.n_tok, L.n_seg
    return dict(absorber=o["absorber"], cu_seqlens=o["cu_seqlens"][:k + 1], seg_src=o["seg_src"][:k],
                cu_targets=o["cu_targets"][:k + 1], counts=o["counts"], tok=o["tok"][:n], pos=o["pos"][:n],
                mask=o["mask"][:n], old_logprob=o["old_logprob"][:n], adv=o["adv"][:n],
                targets=o["targets"][:L.n_mask], packs=len(L.packs))


def _prepare_text(case, seed):
    tl = _timelines(case, seed)
    old = np.where((tl.flags & 3) == 2, tl.lp_noise - 11.0, 0).astype(np.float32)
    return dict(kind="text", merger=actor.Merger(actor.upload_timelines(tl, old, DEV), text=True))


def _run_text(s):
    return dict(_run_merge(s), ti=s["merger"].ti)


# ---------------------------------------------------------------- block

def _block_inputs(case, seed):
    m = _config(case).model
    g = _gen(seed)
    n = case["tokens"]
    w = _weights(m, g, BLOCK)
    x = _randn(g, n, m.d_model, dtype=_storage(m))
    dy = None
    if case["train"]:
        # the loss reaches the rows that feed a scored token, about a third
        dy = torch.zeros(n, m.d_model, device=DEV)
        rows = torch.from_numpy(_scored(n + 1, max(1, int(0.35 * n))) - 1).to(DEV)
        dy[rows] = _randn(g, len(rows), m.d_model, std=1e-4)
    return m, w, x, dy


def _prepare_block(case, seed):
    m, w, x, dy = _block_inputs(case, seed)
    n = case["tokens"]
    for k in LORA_PROJ:   # the actor keeps these beside the weights
        if m.dtype == "bf16":
            w[k + "_t"] = w[k].t().contiguous()
    lens = _seg_lens(n, case["segs"])
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device=DEV)
    pos = torch.cat([torch.arange(v, dtype=torch.int32, device=DEV) for v in lens])
    cfg = capi.block_cfg(m)
    u8 = lambda b: torch.empty(max(1, b), dtype=torch.uint8, device=DEV)
    s = dict(kind="block", cfg=cfg, w=w, cu=cu, pos=pos, longest=max(lens), x=x, dy=dy, y=torch.empty_like(x),
             saved=u8(capi.aj_block_saved_bytes(cfg, n)))
    if dy is not None:
        s.update(ws=u8(capi.aj_block_workspace_bytes(cfg, n, case["segs"])), dx=torch.empty_like(dy),
                 g={k: torch.zeros(w[k].shape, dtype=torch.float32, device=DEV) for k in BLOCK})
    return s


def _run_block(s):
    capi.aj_varlen_block_fwd(s["cfg"], s["w"], s["cu"], s["pos"], s["longest"], s["x"], s["y"], s["saved"])
    if s["dy"] is None:
        return dict(y=s["y"])
    capi.aj_varlen_block_bwd(s["cfg"], s["w"], s["cu"], s["pos"], s["longest"], s["x"], s["saved"], s["dy"],
                             s["dx"], s["g"], s["ws"])
    return dict(y=s["y"], dx=s["dx"], grads=s["g"])


# ---------------------------------------------------------------- loss

def _loss_inputs(case, seed):
    m = _config(case).model
    g = _gen(seed)
    n, k = case["tokens"], case["targets"]
    w = _weights(m, g, ("final_norm", "w_vocab"))
    h = _randn(g, n, m.d_model, std=2.0, dtype=_storage(m))
    tg = torch.from_numpy(_scored(n, k)).to(DEV)
    tok = _ids(g, n, m.vocab, 0.0)
    with torch.no_grad():
        lp = _head(h, w["final_norm"], w["w_vocab"], tg, tok, m, _storage(m)).float()
    old, adv = (torch.zeros(n, device=DEV) for _ in range(2))
    old[tg] = lp + _randn(g, k, std=0.05)
    adv[tg] = _randn(g, 64).repeat_interleave(-(-k // 64))[:k]
    ref = lp + _randn(g, k, std=0.1) if case["kl"] else None
    return m, w, h, tg, tok, old, adv, ref


def _prepare_loss(case, seed):
    m, w, h, tg, tok, old, adv, ref = _loss_inputs(case, seed)
    k = case["targets"]
    cfg = capi.loss_cfg(m, keep_logits=case["keep"])
    u8 = lambda b: torch.empty(max(1, b), dtype=torch.uint8, device=DEV)
    wt = w["w_vocab"].t().contiguous() if m.dtype == "bf16" else None   # the actor keeps it beside the weight
    f32 = lambda *shape: torch.zeros(*shape, device=DEV)
    return dict(kind="loss", cfg=cfg, w=w, wt=wt, h=h, tg=tg.to(torch.int32), tok=tok, old=old, adv=adv, ref=ref,
                kl=case["kl"], inv=1.0 / k, saved=u8(capi.aj_loss_saved_bytes(cfg, k)),
                ws=u8(capi.aj_loss_workspace_bytes(cfg, k)), logprob=f32(k), lse=f32(k), stats=f32(5),
                dh=f32(*h.shape), dg=f32(m.d_model), dw=f32(m.vocab, m.d_model),
                err=torch.zeros(1, dtype=torch.int32, device=DEV))


def _run_loss(s):
    w = s["w"]
    capi.aj_logprob_pg_loss_fwd(s["cfg"], s["tg"], s["tok"], s["old"], s["adv"], s["inv"], s["h"], w["final_norm"],
                                w["w_vocab"], s["saved"], s["logprob"], s["lse"], s["stats"], s["ws"], s["err"],
                                ref_logprob=s["ref"], kl_coef=s["kl"], w_vocab_t=s["wt"])
    capi.aj_logprob_pg_loss_bwd(s["cfg"], s["tg"], s["tok"], s["old"], s["adv"], s["inv"], s["h"], w["final_norm"],
                                w["w_vocab"], s["saved"], s["logprob"], s["lse"], s["dh"], s["dg"], s["dw"],
                                s["ws"], ref_logprob=s["ref"], kl_coef=s["kl"], w_vocab_t=s["wt"])
    return dict(logprob=s["logprob"], lse=s["lse"], stats=s["stats"], dh=s["dh"], dg=s["dg"], dw=s["dw"])


# ---------------------------------------------------------------- embed

def _embed_inputs(case, seed):
    m = _config(case).model
    g = _gen(seed)
    tok = _ids(g, case["tokens"], m.vocab, case["zipf"])
    return m, tok, _weights(m, g, ("emb",))["emb"], _randn(g, case["tokens"], m.d_model, std=1e-4)


def _prepare_embed(case, seed):
    m, tok, emb, dx = _embed_inputs(case, seed)
    n, d = dx.shape
    return dict(kind="embed", tok=tok, emb=emb, dx=dx, x=torch.empty(n, d, dtype=emb.dtype, device=DEV),
                err=torch.zeros(1, dtype=torch.int32, device=DEV), demb=torch.zeros(emb.shape, device=DEV),
                ws=torch.empty(capi.aj_embed_bwd_workspace_bytes(n, d), dtype=torch.uint8, device=DEV))


def _run_embed(s):
    capi.aj_embed_fwd(s["tok"], s["emb"], s["x"], s["err"])
    capi.aj_embed_bwd(s["tok"], s["dx"], s["demb"], s["ws"])
    return dict(x=s["x"], demb=s["demb"], err=s["err"])


# ---------------------------------------------------------------- adamw

ADAM = dict(lr=1e-6, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, step=10)


def _adamw_inputs(case, seed):
    g = _gen(seed)
    n = case["n"]
    return (_randn(g, n, std=0.02), _randn(g, n, std=1e-4), _randn(g, n, std=1e-5),
            _randn(g, n, std=1e-4).square_())


def _prepare_adamw(case, seed):
    p, g, m, v = _adamw_inputs(case, seed)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32, "none": None}[case["copy"]]
    return dict(kind="adamw", p=p, g=g, m=m, v=v, copy=None if dt is None else torch.empty_like(p, dtype=dt))


def _run_adamw(s):
    capi.aj_adamw_step(s["p"], s["g"], s["m"], s["v"], grad_scale=1.0, param_copy=s["copy"], **ADAM)
    out = dict(p=s["p"], m=s["m"], v=s["v"])
    if s["copy"] is not None:
        out["copy"] = s["copy"]
    return out


# ---------------------------------------------------------------- work

def _block_flops(m, tokens, pairs, train):
    """Products of one block over `tokens` with `pairs` (query, key) pairs; the backward twice the
    forward's projections and 2.5 times its attention."""
    return (6 if train else 2) * m.block_params() * tokens + \
        (3.5 if train else 1) * 4 * m.head_dim * m.n_q_heads * pairs


def work(case):
    kind = case["kind"]
    if kind == "adamw":
        return dict(bytes=case["n"] * {"bf16": 30, "f32": 32, "none": 28}[case["copy"]], flops=12 * case["n"])
    m = _config(case).model
    es = 2 if m.dtype == "bf16" else 4
    d, V = m.d_model, m.vocab
    if kind in ("merge", "text"):
        un, llm, merged, tgt, _ = _counts(case["shape"], case["episodes"])
        R = case.get("copies", 1)
        return dict(bytes=R * (5 * un + 8 * llm + 17 * merged + 4 * tgt), flops=0)
    if kind == "update":
        un, llm, merged, tgt, pairs = _counts(case["shape"], case["episodes"])
        full = case["rank"] == 0
        # frozen weights get no weight gradient: one of the backward's two products less
        fl = m.n_layers * _block_flops(m, merged, pairs, True) + 6 * d * V * tgt
        if not full:
            fl -= m.n_layers * 2 * m.block_params() * merged + 2 * d * V * tgt
            rank_params = sum(int(np.prod(s)) for s in lora_shapes(m, case["rank"]).values())
            fl += 6 * rank_params * merged
        blk = m.n_layers * m.block_params()
        grads = 4 * (blk + 2 * V * d) if full else 4 * rank_params
        return dict(bytes=5 * un + es * (blk + 2 * V * d) + grads, flops=fl)
    if kind == "block":
        n, train = case["tokens"], case["train"]
        pairs = sum(v * (v + 1) // 2 for v in _seg_lens(n, case["segs"]))
        by = es * (m.block_params() + 2 * n * d)
        if train:
            by += 4 * (2 * n * d + 2 * m.block_params())
        return dict(bytes=by, flops=_block_flops(m, n, pairs, train))
    if kind == "loss":
        n, k = case["tokens"], case["targets"]
        return dict(bytes=es * (k * d + V * d) + 4 * (n * d + 2 * V * d), flops=6 * d * V * k)
    n = case["tokens"]   # embed: rows read and written; the gradient's rows read, the touched ones updated
    touched = min(n, V) if not case["zipf"] else min(n, V) * 0.3
    return dict(bytes=int(n * (8 + 2 * es * d + 4 * d) + 8 * d * touched), flops=n * d)


def tolerance(case):
    """About four times the largest error against exact() over the ranges (in brackets), where that is more than
    rounding to the output's type alone makes."""
    kind = case["kind"]
    if kind in ("merge", "text"):
        return "exact"
    if kind == "adamw":     # a bfloat16 copy rounds the other way once in ~1e5 values
        return dict(rel=2e-5, max=1e-2) if case["copy"] == "bf16" else dict(rel=2e-7, max=1e-6)
    if kind == "embed":     # (3.1e-7, max 8.2e-5)
        return dict(rel=1.2e-6, max=3.5e-4)
    if kind == "loss":      # (3.4e-3, max 0.16)
        return dict(rel=0.014, max=0.6)
    if kind == "block":     # (8.5e-3, max 0.093)
        return dict(rel=0.03, max=0.4)
    if case["shape"] == "tiny":   # (1.2e-6)
        return dict(rel=5e-6, max=1e-3)
    return dict(rel=0.03, max=0.45)   # (1.24e-2, max 0.11)


# ---------------------------------------------------------------- 64-bit results

def _norm(x, g, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g


def _rope(x, pos, theta):
    half = x.shape[-1] // 2
    inv = theta ** (-torch.arange(half, device=DEV, dtype=torch.float64) / half)
    a = pos.double()[:, None] * inv[None, :]
    c, s = a.cos()[:, None, :].to(x.dtype), a.sin()[:, None, :].to(x.dtype)
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


def _head_attn(q, k, v):
    """One query head over one segment; queries in strips, so that the scores stay small."""
    out, n = [], q.shape[0]
    for a in range(0, n, 4096):
        b = min(n, a + 4096)
        s = q[a:b] @ k[:b].t() * (1.0 / math.sqrt(q.shape[1]))
        s = s.masked_fill(torch.arange(a, b, device=DEV)[:, None] < torch.arange(b, device=DEV)[None, :], -math.inf)
        out.append(s.softmax(-1) @ v[:b])
    return torch.cat(out)


def _block_ref(w, x, lens, m):
    n, hd, hq, hk = x.shape[0], m.head_dim, m.n_q_heads, m.n_kv_heads
    pos = torch.cat([torch.arange(v, device=DEV) for v in lens])
    qkv = (_norm(x, w["attn_norm"], m.rms_eps) @ w["w_qkv"].t()).view(n, hq + 2 * hk, hd)
    qk = _rope(qkv[:, :hq + hk], pos, m.rope_theta)
    rows, at = [], 0
    for v in lens:
        heads = [checkpoint(_head_attn, qk[at:at + v, h], qk[at:at + v, hq + h * hk // hq],
                            qkv[at:at + v, hq + hk + h * hk // hq], use_reentrant=False) for h in range(hq)]
        rows.append(torch.cat(heads, 1))
        at += v
    x1 = x + torch.cat(rows) @ w["w_o"].t()
    gate, up = (_norm(x1, w["mlp_norm"], m.rms_eps) @ w["w_gate_up"].t()).split(m.d_ff, 1)
    return x1 + (torch.nn.functional.silu(gate) * up) @ w["w_down"].t()


def _head(h, gain, w_vocab, tg, tok, m, dt, lse_out=None):
    """log-probs of the targets `tg` (positions), rows in strips."""
    out = []
    gain, w_vocab = gain.to(dt), w_vocab.to(dt)

    def strip(rows, ids, gn, wv):
        z = (_norm(rows.to(dt), gn, m.rms_eps) @ wv.t()).to(torch.float64 if dt == torch.float64 else torch.float32)
        l = torch.logsumexp(z, 1)
        return z.gather(1, ids[:, None])[:, 0] - l, l

    for a in range(0, len(tg), 2048):
        t = tg[a:a + 2048]
        lp, l = checkpoint(strip, h[t - 1], tok[t].long(), gain, w_vocab, use_reentrant=False)
        out.append(lp)
        if lse_out is not None:
            lse_out.append(l.detach())
    return torch.cat(out)


def _policy(W, lora, m, segs, dt):
    """log-probs of every scored token of the merged segments, and their positions; W, lora: leaves or plain."""
    lens = [s[0][0] for s in segs]
    tok = torch.from_numpy(np.concatenate([s[2] for s in segs])).to(DEV)
    mask = np.concatenate([s[1] for s in segs])
    start = np.zeros(len(mask), bool)
    start[np.concatenate([[0], np.cumsum(lens)[:-1]])] = True
    tg = torch.from_numpy(np.flatnonzero(mask & ~start)).to(DEV)
    x = W["emb"].to(dt)[tok.long()]
    for layer in range(m.n_layers):
        w = {k: W[layer_key(k, layer)].to(dt) for k in BLOCK}
        if lora:
            for k in LORA_PROJ:
                w[k] = w[k] + 2.0 * lora[lora_key("b", k, layer)].to(dt) @ lora[lora_key("a", k, layer)].to(dt)
        x = _block_ref(w, x, lens, m)
    return _head(x, W["final_norm"], W["w_vocab"], tg, tok, m, dt), tg


def _objective(lp, old, adv, inv, m, ref, kl_coef):
    """The loss and the five statistics of the clipped objective."""
    r = (lp - old).exp()
    rc = r.clamp(1 - m.clip_eps, 1 + m.clip_eps)
    loss = -torch.minimum(r * adv, rc * adv).sum() * inv
    clipped = (((adv > 0) & (r > 1 + m.clip_eps)) | ((adv < 0) & (r < 1 - m.clip_eps))).sum()
    kl = lp.new_zeros(())
    if ref is not None:
        delta = ref - lp
        kl = (delta.exp() - delta - 1).clamp(-10, 10).sum()
        loss = loss + kl_coef * kl * inv
    stats = [loss, clipped, r.sum(), torch.tensor(len(lp)), kl]
    return loss, torch.stack([v.detach().double().to(DEV) for v in stats])


def _leaf(t):
    return t.double().requires_grad_(True)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("merge", "text"):
        return None
    if kind == "adamw":
        p, g, m, v = (t.double() for t in _adamw_inputs(case, seed))
        f = {k: float(np.float32(x)) for k, x in ADAM.items()}   # the entry point takes 32-bit numbers
        m = f["beta1"] * m + (1 - f["beta1"]) * g
        v = f["beta2"] * v + (1 - f["beta2"]) * g * g
        mh, vh = m / (1 - f["beta1"] ** ADAM["step"]), v / (1 - f["beta2"] ** ADAM["step"])
        p = p - f["lr"] * f["weight_decay"] * p - f["lr"] * mh / (vh.sqrt() + f["eps"])
        out = dict(p=p, m=m, v=v)
        return out if case["copy"] == "none" else dict(out, copy=p)
    if kind == "embed":
        _, tok, emb, dx = _embed_inputs(case, seed)
        demb = torch.zeros(emb.shape, dtype=torch.float64, device=DEV).index_add_(0, tok.long(), dx.double())
        return dict(x=emb[tok.long()].double(), demb=demb, err=None)
    if kind == "loss":
        m, w, h, tg, tok, old, adv, ref = _loss_inputs(case, seed)
        hd, gain, wv = _leaf(h), _leaf(w["final_norm"]), _leaf(w["w_vocab"])
        lse = []
        lp = _head(hd, gain, wv, tg, tok, m, torch.float64, lse)
        loss, stats = _objective(lp, old[tg].double(), adv[tg].double(), 1.0 / len(tg), m,
                                 None if ref is None else ref.double(), case["kl"])
        loss.backward()
        return dict(logprob=lp.detach(), lse=torch.cat(lse), stats=stats, dh=hd.grad, dg=gain.grad, dw=wv.grad)
    if work(case)["flops"] > 1.2e14:   # too long in 64 bits
        return None
    if kind == "block":
        m, w, x, dy = _block_inputs(case, seed)
        lens = _seg_lens(case["tokens"], case["segs"])
        if dy is None:
            with torch.no_grad():
                return dict(y=_block_ref({k: v.double() for k, v in w.items()}, x.double(), lens, m))
        w, x = {k: _leaf(v) for k, v in w.items()}, _leaf(x)
        y = _block_ref(w, x, lens, m)
        y.backward(dy.double())
        return dict(y=y.detach(), dx=x.grad, grads={k: w[k].grad for k in BLOCK})
    cfg, tl, W, lora, old = _update_inputs(case, seed)
    segs = _merge_host(tl, old)
    if lora:
        W, lora = {k: v.double() for k, v in W.items()}, {k: _leaf(v) for k, v in lora.items()}
    else:
        W = {k: _leaf(v) for k, v in W.items()}
    lp, tg = _policy(W, lora, cfg.model, segs, torch.float64)
    at = tg.cpu().numpy()
    pick = lambda i: torch.from_numpy(np.concatenate([s[i] for s in segs])[at]).to(DEV).double()
    loss, stats = _objective(lp, pick(3), pick(4), 1.0 / len(at), cfg.model, None, 0.0)
    loss.backward()
    return dict(logprob=lp.detach(), stats=stats, grads={k: v.grad for k, v in (lora or W).items()})
