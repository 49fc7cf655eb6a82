"""The bfloat16 attention kernels at either side of their dispatch rules, with the
rule's choice asserted: waves per workgroup of the forward and dQ passes (4 or 8)
and parts of a group's query heads in the dK/dV pass, at head_dim 64 and 128, with
segments that begin and end inside one workgroup's rows and tiles.

The reference is the definition in float64 on the same bfloat16 operands, a head and
a segment at a time (2-D products).  The kernels round the weights P (and in the
backward also dS = P (dP - delta)) to bfloat16 before a product, relative 2^-9 at
most per term, and each result once more; the backward's delta comes from the
forward's rounded O.  Each of these is at most 2^-9 of the norm it acts on (measured:
a tensor differs by 0.0018 to 0.0026), so a relative L2 of 2^-7 holds for every
tensor.
"""
import math

import pytest
import torch

from tests import plans

pytestmark = pytest.mark.gpu

# (segment lengths, query heads, KV heads, head_dim, part scratch in heads' sums): (waves, parts)
LONG = (5000, 37, 150, 4000)           # 9187 tokens, mean above 2048: 8 waves past 256 workgroups
CASES = [
    (LONG, 8, 2, 128, 0, (8, 1)),
    (LONG, 8, 2, 64, 0, (8, 1)),
    (LONG, 8, 1, 64, 7, (8, 4)),
    (LONG, 7, 1, 128, 7, (4, 7)),          # 252 workgroups of 8 waves
    (LONG, 7, 1, 64, 3, (4, 3)),
    ((2100, 1, 300, 1999, 255, 257, 30), 12, 2, 128, 4, (4, 3)),
    ((2100, 1, 300, 1999, 255, 257, 30), 12, 2, 64, 0, (4, 1)),
    ((33,), 6, 2, 128, 3, (4, 3)),
]


def _reference(qkv, dout, lens, hq, hkv, hd):
    """o, lse (log2 units), dq|dk|dv in float64."""
    x = qkv.double().view(-1, hq + 2 * hkv, hd)
    do = dout.double().view(-1, hq, hd)
    o, d = torch.zeros_like(do), torch.zeros_like(x)
    lse = torch.zeros(hq, len(x), dtype=torch.float64, device=x.device)
    scale, t0 = 1 / math.sqrt(hd), 0
    for n in lens:
        s = slice(t0, t0 + n)
        t0 += n
        above = torch.ones(n, n, dtype=torch.bool, device=x.device).triu(1)
        for h in range(hq):
            g = h * hkv // hq
            q, k, v = x[s, h], x[s, hq + g], x[s, hq + hkv + g]
            z = (q @ k.t() * scale).masked_fill_(above, -math.inf)
            lse[h, s] = torch.logsumexp(z, 1) / math.log(2)
            p = torch.softmax(z, 1)
            o[s, h] = p @ v
            d[s, hq + hkv + g] += p.t() @ do[s, h]
            ds = p * (do[s, h] @ v.t() - (do[s, h] * o[s, h]).sum(1, keepdim=True)) * scale
            d[s, h] = ds @ k
            d[s, hq + g] += ds.t() @ q
    return o, lse, d


@pytest.mark.parametrize("lens,hq,hkv,hd,scratch,want", CASES)
def test_attention(lens, hq, hkv, hd, scratch, want):
    n, dev = sum(lens), "cuda"
    print(f"attention {lens} heads {hq}/{hkv} of {hd}", flush=True)
    gen = torch.Generator(device=dev).manual_seed(n + hd)
    rnd = lambda w: torch.randn(n, w, generator=gen, device=dev).to(torch.bfloat16)
    qkv, dout = rnd((hq + 2 * hkv) * hd), rnd(hq * hd)
    o, dqkv = torch.zeros_like(dout), torch.zeros_like(qkv)
    lse, delta = torch.zeros(hq, n, device=dev), torch.zeros(hq, n, device=dev)
    cu = torch.tensor([0, *torch.tensor(lens).cumsum(0).tolist()], dtype=torch.int32, device=dev)
    floats = scratch * n * 2 * hkv * hd
    part = torch.empty(max(floats, 1), device=dev)
    st = torch.cuda.current_stream().cuda_stream
    scale = 1 / math.sqrt(hd)
    f = plans.AttnArgs(n, len(lens), hq, hkv, hd, 0, cu.data_ptr(), qkv.data_ptr(), o.data_ptr(),
                       lse.data_ptr(), scale)
    b = plans.AttnBwdArgs(n, len(lens), hq, hkv, hd, 0, cu.data_ptr(), qkv.data_ptr(), o.data_ptr(),
                          dout.data_ptr(), lse.data_ptr(), delta.data_ptr(), dqkv.data_ptr(), scale,
                          part.data_ptr() if floats else None, floats)
    assert (plans.attn_row_waves(n, len(lens), hq), plans.attn_dkv_parts(b)) == want
    plans.attn_fwd_bf16(f, st)
    plans.attn_bwd_bf16(b, st)
    torch.cuda.synchronize()
    ro, rl, rd = _reference(qkv, dout, lens, hq, hkv, hd)
    rel = lambda a, r: ((a.double() - r).norm() / r.norm()).item()
    d = dqkv.view(n, -1, hd)
    errs = dict(o=rel(o.view(n, hq, hd), ro), lse=rel(lse, rl), dq=rel(d[:, :hq], rd[:, :hq]),
                dk=rel(d[:, hq:hq + hkv], rd[:, hq:hq + hkv]), dv=rel(d[:, hq + hkv:], rd[:, hq + hkv:]))
    print(" ".join(f"{k} {v:.2e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= 2 ** -7
