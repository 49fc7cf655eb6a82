"""The bfloat16 products on every kernel that gemm_plan sends them to, bit-exact:
operands are integers in [-2, 2], so every float32 sum is exact in any order
(|sum| <= 4 K < 2^24) and a bfloat16 result is that sum rounded once.

Sizes end in partial tiles and ragged k-steps.  The plan (tile, 4-wave, whole
tiles, pieces) is asserted, so that a change of its cost model cannot empty the
test, and so is the class that the launch record counts the product in.
"""
import pytest
import torch

from tests import plans

pytestmark = pytest.mark.gpu

# (layout, M, N, K): (tile, 4-wave, whole tiles, pieces each of the rest)
CASES = [
    # 256x256 tiles, 4 waves: whole; whole and pieces; pieces
    ("NT", 3901, 3899, 4104, (256, True, 256, 1)),
    ("TN", 3896, 3904, 4104, (256, True, 256, 1)),
    ("NN", 16501, 1032, 4104, (256, True, 256, 3)),
    ("NT", 519, 1033, 66008, (256, True, 0, 16)),
    ("NN", 519, 1032, 66008, (256, True, 0, 16)),
    ("TN", 520, 1032, 66007, (256, True, 0, 16)),
    # 8 waves
    ("NT", 5001, 8999, 264, (256, False, 720, 1)),
    ("NN", 6001, 3304, 1544, (256, False, 256, 3)),
    ("TN", 2600, 2600, 4104, (256, False, 0, 2)),
    # 128x128 tiles
    ("NT", 131, 265, 520, (128, False, 6, 1)),
    ("NN", 2347, 1536, 1536, (128, False, 228, 1)),
    ("NN", 301, 520, 66040, (128, False, 0, 16)),
    ("TN", 72, 1032, 3001, (128, False, 0, 11)),
]


@pytest.mark.parametrize("layout,M,N,K,plan", CASES, ids=[f"{c[0]}-{c[1]}x{c[2]}x{c[3]}" for c in CASES])
def test_product(layout, M, N, K, plan):
    from paper_2606_04484_amd import capi
    print(f"{layout} {M}x{N} K={K}", flush=True)
    cap = plans.partial_floats(M, N)
    p = plans.gemm_plan(M, N, K, cap)
    assert (p.tile, p.long_k, p.whole, p.split) == plan
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    ints = lambda *s, m=2: torch.randint(-m, m + 1, s, generator=gen, device="cuda").to(torch.bfloat16)
    a_k, b_k = layout != "TN", layout == "NT"
    A = ints(M, K) if a_k else ints(K, M)
    B = ints(N, K) if b_k else ints(K, N)
    ref = (A if a_k else A.t()).double() @ (B.t() if b_k else B).double()
    part = torch.empty(cap, device="cuda")
    ldc = N + 4
    R = ints(M, ldc, m=100)
    C0 = ints(M, ldc, m=100).float()
    capi.aj_timing_enable(True)
    for accum in (True, False):
        out = C0.clone() if accum else R.clone()
        g = plans.Gemm(M=M, N=N, K=K, A=A.data_ptr(), lda=A.shape[1], a_kmajor=a_k, B=B.data_ptr(),
                       ldb=B.shape[1], b_kmajor=b_k, C=out.data_ptr(), ldc=ldc, out=int(accum),
                       R=None if accum else R.data_ptr(), partial=part.data_ptr(), partial_cap=cap)
        plans.gemm_bf16(g, torch.cuda.current_stream().cuda_stream)
        if accum:
            assert torch.equal(out[:, :N], C0[:, :N] + ref.float())
            assert torch.equal(out[:, N:], C0[:, N:])
        else:
            assert torch.equal(out[:, :N], (R[:, :N].double() + ref).float().to(torch.bfloat16))
            assert torch.equal(out[:, N:], R[:, N:])
    rec = capi.aj_timing_read()
    capi.aj_timing_enable(False)
    cls = ("gemm4_" if p.long_k else "gemm_") + layout.lower()
    assert {k: v[1] for k, v in rec.items() if v[1]} == {cls: 2}
