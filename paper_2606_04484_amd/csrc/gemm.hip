// GEMMs of the block and the LM head.
//
// bfloat16: v_mfma_f32_16x16x32_bf16 tiles, float32 accumulation, 256x256
// workgroup tiles on 8 waves (128x64 per wave) or 4 (128x128).
// Operands are copied into LDS in their memory order: a K-major one as
// [row][k], an M/N-major one (the weight-gradient GEMMs read activations
// [tokens, features]) as [k][row], whose MFMA fragments come out of LDS
// already transposed through ds_read_tr16_b64.  Workgroup ids are
// remapped so that each XCD (ids are dealt round-robin over the 8 XCDs) walks
// a contiguous, row-grouped run of tiles and its L2 sees the reuse.
//
// float32, and bfloat16 operands that the copies above cannot take:
// v_mfma_f32_16x16x4_f32 on 64x64 tiles.
#include "ops.h"
#include "gemm_core.h"

namespace aj {
namespace {

struct EpArgs {
  int M, N;
  void *C; int64_t ldc;
  int c_f32, accum;
  const void *R;
  int vec;   // 4-column vector stores are aligned (C, R, partial rows)
  const bf16_t *gu;   // SwiGLU backward: [gate | up] rows (stride ldc), else null
};

// d gate, d up of one SwiGLU element from d s (float32) and bf16 gate / up
AJ_DEV void swiglu_grad(float ds, float g, float u, float &dg, float &du) {
  const float sg = 1.f / (1.f + __expf(-g));
  dg = ds * u * sg * (1.f + g * (1.f - sg));
  du = ds * g * sg;
}

using gemm_core::f32x4_t;
using gemm_core::Seg;

// Output modes of the epilogue's fast path (interior tiles, aligned rows).
enum { kEpPartial, kEpAccum, kEpF32, kEpF32R, kEpBf16, kEpBf16R, kEpSwiglu };

// One pass of the fast epilogue: the staged rows (32 of each wave row), 4
// columns per thread and instruction; every LDS read of the pass is issued
// before the first store.
template <int MODE, typename Cfg>
AJ_DEV void store_pass(const float *stage, int i, int m0, int n0, int64_t ldo, float *P,
                       const EpArgs &ep) {
  constexpr int LDW = Cfg::BN + 4, C4 = Cfg::BN / 4;
  constexpr int Q = 32 * Cfg::WM * C4 / Cfg::NT;
  float4 v[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int c = threadIdx.x + Cfg::NT * q;
    v[q] = *reinterpret_cast<const float4 *>(stage + (c / C4) * LDW + (c % C4) * 4);
  }
  auto offset = [&](int q) {
    const int c = threadIdx.x + Cfg::NT * q;
    const int row = c / C4;
    return (int64_t)(m0 + (row >> 5) * Cfg::WTM + 32 * i + (row & 31)) * ldo + n0 + (c % C4) * 4;
  };
  if constexpr (MODE == kEpAccum || MODE == kEpF32R) {
    const float *src = MODE == kEpAccum ? (const float *)ep.C : (const float *)ep.R;
    float4 u[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) u[q] = *reinterpret_cast<const float4 *>(src + offset(q));
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float4 w = make_float4(v[q].x + u[q].x, v[q].y + u[q].y, v[q].z + u[q].z,
                                   v[q].w + u[q].w);
      *reinterpret_cast<float4 *>((float *)ep.C + offset(q)) = w;
    }
  } else if constexpr (MODE == kEpSwiglu) {
    uint2 g4[Q], u4[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      g4[q] = *reinterpret_cast<const uint2 *>(ep.gu + offset(q));
      u4[q] = *reinterpret_cast<const uint2 *>(ep.gu + offset(q) + ep.N);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float dsv[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
      const float gv[4] = {__uint_as_float(g4[q].x << 16), __uint_as_float(g4[q].x & 0xffff0000u),
                           __uint_as_float(g4[q].y << 16), __uint_as_float(g4[q].y & 0xffff0000u)};
      const float uv[4] = {__uint_as_float(u4[q].x << 16), __uint_as_float(u4[q].x & 0xffff0000u),
                           __uint_as_float(u4[q].y << 16), __uint_as_float(u4[q].y & 0xffff0000u)};
      float dg[4], du[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) swiglu_grad(dsv[e], gv[e], uv[e], dg[e], du[e]);
      bf16_t *cp = (bf16_t *)ep.C + offset(q);
      *reinterpret_cast<uint2 *>(cp) = make_uint2(f2bf2(dg[0], dg[1]), f2bf2(dg[2], dg[3]));
      *reinterpret_cast<uint2 *>(cp + ep.N) = make_uint2(f2bf2(du[0], du[1]), f2bf2(du[2], du[3]));
    }
  } else if constexpr (MODE == kEpBf16R) {
    uint2 u[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) u[q] = *reinterpret_cast<const uint2 *>((const bf16_t *)ep.R + offset(q));
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      uint2 out;
      out.x = f2bf2(v[q].x + __uint_as_float(u[q].x << 16),
                    v[q].y + __uint_as_float(u[q].x & 0xffff0000u));
      out.y = f2bf2(v[q].z + __uint_as_float(u[q].y << 16),
                    v[q].w + __uint_as_float(u[q].y & 0xffff0000u));
      *reinterpret_cast<uint2 *>((bf16_t *)ep.C + offset(q)) = out;
    }
  } else {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if constexpr (MODE == kEpPartial) {
        *reinterpret_cast<float4 *>(P + offset(q)) = v[q];
      } else if constexpr (MODE == kEpF32) {
        *reinterpret_cast<float4 *>((float *)ep.C + offset(q)) = v[q];
      } else {
        uint2 out;
        out.x = f2bf2(v[q].x, v[q].y);
        out.y = f2bf2(v[q].z, v[q].w);
        *reinterpret_cast<uint2 *>((bf16_t *)ep.C + offset(q)) = out;
      }
    }
  }
}

// LDS writes of the staged rows (or their reads) complete, then a barrier:
// unlike __syncthreads, the tile's global stores stay in flight.
AJ_DEV void epi_barrier() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  gemm_core::bar_nofence();
}

// The epilogue of four consecutive columns (m, n) .. (m, n + 3) of the output, m
// and n inside it, columns past N left out.
AJ_DEV void store4(const EpArgs &ep, int m, int n, const float4 &v) {
  const int64_t o = (int64_t)m * ep.ldc + n;
  const float vv[4] = {v.x, v.y, v.z, v.w};
  if (ep.gu) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (n + e >= ep.N) break;
      float dg, du;
      swiglu_grad(vv[e], bf2f(ep.gu[o + e]), bf2f(ep.gu[o + e + ep.N]), dg, du);
      ((bf16_t *)ep.C)[o + e] = f2bf(dg);
      ((bf16_t *)ep.C)[o + e + ep.N] = f2bf(du);
    }
  } else if (ep.vec && n + 4 <= ep.N) {
    if (ep.c_f32) {
      float4 *cp = reinterpret_cast<float4 *>((float *)ep.C + o);
      float4 w = v;
      if (ep.accum || ep.R) {
        const float4 u = ep.accum ? *cp : *reinterpret_cast<const float4 *>((const float *)ep.R + o);
        w.x += u.x; w.y += u.y; w.z += u.z; w.w += u.w;
      }
      *cp = w;
    } else {
      float w0 = v.x, w1 = v.y, w2 = v.z, w3 = v.w;
      if (ep.R) {
        const uint2 u = *reinterpret_cast<const uint2 *>((const bf16_t *)ep.R + o);
        w0 += __uint_as_float(u.x << 16); w1 += __uint_as_float(u.x & 0xffff0000u);
        w2 += __uint_as_float(u.y << 16); w3 += __uint_as_float(u.y & 0xffff0000u);
      }
      *reinterpret_cast<uint2 *>((bf16_t *)ep.C + o) = make_uint2(f2bf2(w0, w1), f2bf2(w2, w3));
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (n + e >= ep.N) break;
      if (ep.accum) ((float *)ep.C)[o + e] += vv[e];
      else if (ep.c_f32) ((float *)ep.C)[o + e] = vv[e] + (ep.R ? ((const float *)ep.R)[o + e] : 0.f);
      else ((bf16_t *)ep.C)[o + e] = f2bf(vv[e] + (ep.R ? bf2f(((const bf16_t *)ep.R)[o + e]) : 0.f));
    }
  }
}

// Which output tiles a launch runs whole and which in pieces: tiles [0, whole)
// of the walk take one workgroup each; each of the rest takes `split`, on
// ranges of k_piece, whose float32 sums go to `partial` (a BM x BN block per
// piece, pieces of one range side by side) for gemm_pieces_kernel to add up.
struct Pieces {
  int whole, rest, split, k_piece;
  float *partial;
};

// Shared body of the GEMM kernels: main loop of configuration Cfg (and the
// second segment's, SEG2), then the epilogue through LDS.
template <bool A_K, bool B_K, typename Cfg, bool SEG2 = false>
AJ_DEV void gemm_tile(int M, int N, int K, const bf16_t *A, int64_t lda, const bf16_t *B,
                      int64_t ldb, const EpArgs &ep, const Pieces &pc,
                      gemm_core::Smem<Cfg, A_K, B_K> &sm, const Seg &s2 = Seg{}) {
  const int tiles_m = (M + Cfg::BM - 1) / Cfg::BM, tiles_n = (N + Cfg::BN - 1) / Cfg::BN;
  int t, kbeg = 0, kend = K;
  float *P = nullptr;
  if ((int)blockIdx.x < pc.whole) {
    t = gemm_core::xcd_item(blockIdx.x, pc.whole);
  } else {
    // an XCD's pieces are of neighbouring tiles over one range of k
    const int p = gemm_core::xcd_item(blockIdx.x - pc.whole, pc.rest * pc.split);
    t = pc.whole + p % pc.rest;
    kbeg = (p / pc.rest) * pc.k_piece;
    kend = min(K, kbeg + pc.k_piece);
    P = pc.partial + (int64_t)p * (Cfg::BM * Cfg::BN);
  }
  const gemm_core::TileIdx ti = gemm_core::tile_at(t, tiles_m, tiles_n);
  const int m0 = ti.tm * Cfg::BM, n0 = ti.tn * Cfg::BN;
  const int lane = threadIdx.x & 63, wave = gemm_core::wave_id();
  const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
  f32x4_t acc[Cfg::TM][Cfg::TN];
  if constexpr (SEG2) {
    // the second segment goes with the first piece
    const Seg t2{s2.A, s2.lda, s2.B, s2.ldb, s2.kbeg, kbeg == 0 ? s2.kend : s2.kbeg};
    gemm_core::mainloop<Cfg, A_K, B_K, true>(acc, Seg{A, lda, B, ldb, kbeg, kend}, M, N, m0, n0,
                                             sm, t2);
  } else {
    gemm_core::mainloop<Cfg, A_K, B_K>(acc, Seg{A, lda, B, ldb, kbeg, kend}, M, N, m0, n0, sm);
  }
  epi_barrier();

  // Epilogue through LDS, 32 rows of each wave row (two accumulator rows of
  // tiles) at a time: a lane's four consecutive columns of a row go out as one
  // 16-byte write, then rows are stored 4 columns per lane.  The padding of 4
  // floats per row puts the 16 rows of a write on different banks.
  // Pieces, and interior tiles with aligned rows, take a pass specialised to
  // the output mode (no per-element branches, the pass's LDS reads issued
  // together); edge tiles go four columns at a time.
  float *stage = reinterpret_cast<float *>(&sm);
  constexpr int LDW = Cfg::BN + 4, C4 = Cfg::BN / 4;
  // the SwiGLU pass is for tiles of 128 accumulators and fewer: with 256 it
  // pushes the epilogue past full unrolling and the accumulators into scratch
  constexpr bool kSwiglu = Cfg::TM * Cfg::TN <= 32;
  const bool fast = P || (ep.vec && m0 + Cfg::BM <= M && n0 + Cfg::BN <= N && (kSwiglu || !ep.gu));
  const int mode = P ? kEpPartial
                   : ep.gu ? kEpSwiglu
                   : ep.accum ? kEpAccum
                   : ep.c_f32 ? (ep.R ? kEpF32R : kEpF32)
                              : (ep.R ? kEpBf16R : kEpBf16);
#pragma unroll
  for (int i = 0; i < Cfg::TM / 2; ++i) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < Cfg::TN; ++j)
        *reinterpret_cast<f32x4_t *>(stage + (wm * 32 + 16 * h + (lane & 15)) * LDW +
                                     gemm_core::acc_col<Cfg>(wn, j, lane)) = acc[2 * i + h][j];
    epi_barrier();
    if (fast) {
      const int64_t ldo = ep.ldc;
      switch (mode) {
        case kEpPartial: store_pass<kEpPartial, Cfg>(stage, i, 0, 0, Cfg::BN, P, ep); break;
        case kEpAccum: store_pass<kEpAccum, Cfg>(stage, i, m0, n0, ldo, P, ep); break;
        case kEpF32: store_pass<kEpF32, Cfg>(stage, i, m0, n0, ldo, P, ep); break;
        case kEpF32R: store_pass<kEpF32R, Cfg>(stage, i, m0, n0, ldo, P, ep); break;
        case kEpBf16: store_pass<kEpBf16, Cfg>(stage, i, m0, n0, ldo, P, ep); break;
        case kEpSwiglu:
          if constexpr (kSwiglu) store_pass<kEpSwiglu, Cfg>(stage, i, m0, n0, ldo, P, ep);
          break;
        default: store_pass<kEpBf16R, Cfg>(stage, i, m0, n0, ldo, P, ep); break;
      }
    } else {
#pragma unroll 4
      for (int q = 0; q < 32 * Cfg::WM * C4 / Cfg::NT; ++q) {
        const int c = threadIdx.x + Cfg::NT * q;
        const int row = c / C4, c4 = (c % C4) * 4;
        const int m = m0 + (row >> 5) * Cfg::WTM + 32 * i + (row & 31), n = n0 + c4;
        if (m < M && n < N)
          store4(ep, m, n, *reinterpret_cast<const float4 *>(stage + row * LDW + c4));
      }
    }
    epi_barrier();
  }
}

// Cfg8 is the default, Cfg4 takes reductions of kLongK and more, CfgS (two
// workgroups to a CU) products of few tiles.
template <typename Cfg, bool A_K, bool B_K>
__global__ __launch_bounds__(Cfg::NT, Cfg::BM == 128 ? 2 : 1) void gemm_mfma_kernel(
    int M, int N, int K, const bf16_t *A, int64_t lda, const bf16_t *B, int64_t ldb, EpArgs ep,
    Pieces pc) {
  __shared__ __attribute__((aligned(16))) gemm_core::Smem<Cfg, A_K, B_K> sm;
  gemm_tile<A_K, B_K, Cfg>(M, N, K, A, lda, B, ldb, ep, pc, sm);
}

// The same with a second reduction segment with the operand layouts of the
// first, C = A B + A2 B2 (Cfg8 with either reduction length, or CfgS).
template <typename Cfg, bool A_K, bool B_K>
__global__ __launch_bounds__(Cfg::NT, Cfg::BM == 128 ? 2 : 1) void gemm_mfma_seg2_kernel(
    int M, int N, int K, const bf16_t *A, int64_t lda, const bf16_t *B, int64_t ldb, Seg s2,
    EpArgs ep, Pieces pc) {
  __shared__ __attribute__((aligned(16))) gemm_core::Smem<Cfg, A_K, B_K> sm;
  gemm_tile<A_K, B_K, Cfg, true>(M, N, K, A, lda, B, ldb, ep, pc, sm, s2);
}

// The pieces of each split tile added up in the order of their k ranges, then
// the epilogue.  One workgroup per 1024 outputs of a tile, 4 columns per thread;
// four pieces' loads are in flight at a time (one at a time, and 4096 outputs
// per workgroup, took 18.5 us for 16 pieces of 32 64 x 64 tiles).  The partials
// were written just before and mostly sit in the last-level cache.
template <int BM, int BN>
__global__ __launch_bounds__(256) void gemm_pieces_kernel(EpArgs ep, Pieces pc) {
  constexpr int PER = BM * BN / 1024;
  const int r = blockIdx.x / PER, e = (blockIdx.x % PER) * 1024 + (int)threadIdx.x * 4;
  const int tiles_m = (ep.M + BM - 1) / BM, tiles_n = (ep.N + BN - 1) / BN;
  const gemm_core::TileIdx ti = gemm_core::tile_at(pc.whole + r, tiles_m, tiles_n);
  const int m = ti.tm * BM + e / BN, n = ti.tn * BN + e % BN;
  if (m >= ep.M || n >= ep.N) return;
  const float *P = pc.partial + (int64_t)r * (BM * BN) + e;
  const int64_t step = (int64_t)pc.rest * (BM * BN);
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int z = 0; z < pc.split; z += 4) {
    float4 u[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (z + q < pc.split) u[q] = *reinterpret_cast<const float4 *>(P + (z + q) * step);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (z + q < pc.split) { v.x += u[q].x; v.y += u[q].y; v.z += u[q].z; v.w += u[q].w; }
  }
  store4(ep, m, n, v);
}

constexpr int kLongK = 4096;

// ---------------------------------------------------------------- float32
// 64 x 64 outputs by four waves of 32 x 32 on v_mfma_f32_16x16x4_f32 (float32
// products and sums throughout), 32-wide k-steps in two LDS buffers, the next
// step's operands loaded into registers beside the current one's products.  Any
// size, stride and alignment: operands go through registers, four elements of
// the contiguous dimension at a time where they are aligned.  The float32
// workload's products are small (3443 tokens, widths 128 .. 1024), so what
// matters is that every CU has a tile: hence the small tile, and reductions over
// the tokens in pieces.  Its 15 products (a 64x64 tile of plain FMAs before):
// 2880 -> 300 us.
constexpr int kFTile = 64, kFBK = 32, kFLd = kFBK + 4;

struct FOperand {
  const void *p;
  int64_t ld;
  bool kmajor, vec;     // vec: 4-element loads are aligned
};

template <typename T>
AJ_DEV float4 load_elems(const T *p, int n, bool vec) {
  if (vec && n >= 4) {
    if constexpr (sizeof(T) == 4) {
      return *reinterpret_cast<const float4 *>(p);
    } else {
      const uint2 u = *reinterpret_cast<const uint2 *>(p);
      return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                         __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
    }
  }
  return make_float4(n > 0 ? ldf(p) : 0.f, n > 1 ? ldf(p + 1) : 0.f, n > 2 ? ldf(p + 2) : 0.f,
                     n > 3 ? ldf(p + 3) : 0.f);
}

// this thread's q-th four elements (q = 0, 1) of the 64 x 32 operand tile at (r0, k0)
template <typename T>
AJ_DEV float4 f32_fetch(const T *p, int64_t ld, bool kmajor, bool vec, int q, int r0, int rows,
                        int k0, int kend) {
  const int idx = threadIdx.x + 256 * q;
  const int r = r0 + (kmajor ? idx / 8 : idx % 16 * 4), k = k0 + (kmajor ? idx % 8 * 4 : idx / 16);
  if (r >= rows || k >= kend) return make_float4(0.f, 0.f, 0.f, 0.f);
  return load_elems(p + (kmajor ? r * ld + k : k * ld + r), kmajor ? kend - k : rows - r, vec);
}
AJ_DEV void f32_stage(float *lds, bool kmajor, int q, const float4 &v) {
  const int idx = threadIdx.x + 256 * q;
  if (kmajor) {
    *reinterpret_cast<float4 *>(lds + idx / 8 * kFLd + idx % 8 * 4) = v;
  } else {
    float *p = lds + idx % 16 * 4 * kFLd + idx / 16;
    p[0] = v.x; p[kFLd] = v.y; p[2 * kFLd] = v.z; p[3 * kFLd] = v.w;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void gemm_f32_kernel(int M, int N, int K, FOperand A, FOperand B,
                                                       int K2, FOperand A2, FOperand B2, EpArgs ep,
                                                       Pieces pc) {
  __shared__ __attribute__((aligned(16))) float As[2][kFTile * kFLd], Bs[2][kFTile * kFLd];
  const int tiles_m = (M + kFTile - 1) / kFTile, tiles_n = (N + kFTile - 1) / kFTile;
  int t = blockIdx.x, kbeg = 0, kend = K;
  float *P = nullptr;
  if (t >= pc.whole) {
    const int p = t - pc.whole;
    t = pc.whole + p % pc.rest;
    kbeg = (p / pc.rest) * pc.k_piece;
    kend = min(K, kbeg + pc.k_piece);
    P = pc.partial + (int64_t)p * (kFTile * kFTile);
  }
  const gemm_core::TileIdx ti = gemm_core::tile_at(t, tiles_m, tiles_n);
  const int m0 = ti.tm * kFTile, n0 = ti.tn * kFTile;
  const int lane = threadIdx.x & 63, wave = gemm_core::wave_id(), wm = wave >> 1, wn = wave & 1;
  // steps of the first segment, then of the second
  const int n1 = kend > kbeg ? (kend - kbeg + kFBK - 1) / kFBK : 0;
  const int nk = n1 + (K2 + kFBK - 1) / kFBK;
  float4 va[2], vb[2];
  auto fetch = [&](int s) {
    const bool two = s >= n1;
    const int k0 = two ? (s - n1) * kFBK : kbeg + s * kFBK;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      va[q] = f32_fetch((const T *)(two ? A2.p : A.p), two ? A2.ld : A.ld, A.kmajor,
                        two ? A2.vec : A.vec, q, m0, M, k0, two ? K2 : kend);
      vb[q] = f32_fetch((const T *)(two ? B2.p : B.p), two ? B2.ld : B.ld, B.kmajor,
                        two ? B2.vec : B.vec, q, n0, N, k0, two ? K2 : kend);
    }
  };
  f32x4_t acc[2][2] = {};
  if (nk > 0) fetch(0);
  for (int s = 0; s < nk; ++s) {
    float *as = As[s & 1], *bs = Bs[s & 1];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      f32_stage(as, A.kmajor, q, va[q]);
      f32_stage(bs, B.kmajor, q, vb[q]);
    }
    __syncthreads();   // (the other buffer's readers are all past the barrier before this one)
    if (s + 1 < nk) fetch(s + 1);
    // lane l: row l%16, k = 4 (l/16) + j at the j-th product of each 16 k
#pragma unroll
    for (int c = 0; c < kFBK / 16; ++c) {
      f32x4_t fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[i] = *reinterpret_cast<const f32x4_t *>(as + (wm * 32 + i * 16 + (lane & 15)) * kFLd + 16 * c + 4 * (lane >> 4));
        fb[i] = *reinterpret_cast<const f32x4_t *>(bs + (wn * 32 + i * 16 + (lane & 15)) * kFLd + 16 * c + 4 * (lane >> 4));
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int jn = 0; jn < 2; ++jn)
            acc[i][jn] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[jn][j], fa[i][j], acc[i][jn], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int jn = 0; jn < 2; ++jn) {
      const int r = wm * 32 + i * 16 + (lane & 15), c = wn * 32 + jn * 16 + 4 * (lane >> 4);
      const float4 v = make_float4(acc[i][jn][0], acc[i][jn][1], acc[i][jn][2], acc[i][jn][3]);
      if (P) *reinterpret_cast<float4 *>(P + r * kFTile + c) = v;
      else if (m0 + r < M && n0 + c < N) store4(ep, m0 + r, n0 + c, v);
    }
}

template <bool A_K, bool B_K>
void launch_mfma(const Gemm &g, const EpArgs &ep, const GemmPlan &pl, hipStream_t s) {
  const Pieces pc{pl.whole, pl.tiles - pl.whole, pl.split, pl.k_piece, g.partial};
  const int grid = pc.whole + pc.rest * pc.split;
  const bf16_t *A = (const bf16_t *)g.A, *B = (const bf16_t *)g.B;
  if (g.K2 > 0) {
    const Seg s2{(const bf16_t *)g.A2, g.lda2, (const bf16_t *)g.B2, g.ldb2, 0, g.K2};
    if (pl.tile == 128)
      gemm_mfma_seg2_kernel<gemm_core::CfgS, A_K, B_K><<<grid, gemm_core::CfgS::NT, 0, s>>>(
          g.M, g.N, g.K, A, g.lda, B, g.ldb, s2, ep, pc);
    else
      gemm_mfma_seg2_kernel<gemm_core::Cfg8, A_K, B_K><<<grid, gemm_core::Cfg8::NT, 0, s>>>(
          g.M, g.N, g.K, A, g.lda, B, g.ldb, s2, ep, pc);
  } else if (pl.tile == 128) {
    gemm_mfma_kernel<gemm_core::CfgS, A_K, B_K><<<grid, gemm_core::CfgS::NT, 0, s>>>(
        g.M, g.N, g.K, A, g.lda, B, g.ldb, ep, pc);
  } else if (pl.long_k) {
    gemm_mfma_kernel<gemm_core::Cfg4, A_K, B_K><<<grid, gemm_core::Cfg4::NT, 0, s>>>(
        g.M, g.N, g.K, A, g.lda, B, g.ldb, ep, pc);
  } else {
    gemm_mfma_kernel<gemm_core::Cfg8, A_K, B_K><<<grid, gemm_core::Cfg8::NT, 0, s>>>(
        g.M, g.N, g.K, A, g.lda, B, g.ldb, ep, pc);
  }
  if (pc.rest == 0 || pc.split <= 1) return;
  if (pl.tile == 128) gemm_pieces_kernel<128, 128><<<pc.rest * 16, 256, 0, s>>>(ep, pc);
  else gemm_pieces_kernel<256, 256><<<pc.rest * 64, 256, 0, s>>>(ep, pc);
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

// Predicted times, in us, of one round of workgroups over a reduction of k.
// 256 x 256 tiles, one workgroup per CU: 7.5 us of prologue and epilogue, then
// 15.4 ns per k while few CUs work, 22.8 ns with all 256 (copy rate and power
// shared).  128 x 128 tiles, two per CU: 8.6 ns per k with one on a CU, 16.5
// with two.  Adding up pieces: a launch and its bytes.  Fitted to NN and TN
// products of M 700 .. 19437, N 1536 .. 37888, K 1536 .. 32768, which it gives
// to 10 %.
static double round_256(int tiles, double k) {
  const double busy = tiles <= 64 ? 0.0 : (tiles - 64) / 192.0;
  return 7.5 + k * (0.0154 + 0.0074 * busy);
}
static double round_128(int tiles, double k) {
  return tiles <= 256 ? 4.5 + 0.0086 * k : 6.0 + 0.0165 * k;
}
static double rounds(int tile, int tiles, double k) {
  const int per = tile == 256 ? 256 : 512, full = tiles / per, rem = tiles % per;
  auto one = [&](int t) { return tile == 256 ? round_256(t, k) : round_128(t, k); };
  return (full ? full * one(per) : 0.0) + (rem ? one(rem) : 0.0);
}

// The fastest of: every 256 x 256 tile whole; the tiles past the last full
// round of 256 in pieces (all of them, when there are fewer than 256 tiles);
// 128 x 128 tiles, whole or in pieces.  Measured either side of the lines (NN):
//   2347 x 1536, K 1536: 256 whole 31.2, 128 whole 17.8 us
//   2347 x 1536, K 8960: 256 whole 138.7, 256 in 4 pieces 70.4, 128 whole 80.2 us
//   700 x 1536, K 8960: 256 in 8 pieces 40.0, 128 in 3 pieces 36.3 us
//   14500 x 1536, K 8960 (342 tiles): whole 376.8, last 86 in 2 pieces 312.2 us
//   19437 x 3584, K 18944 (1064 tiles): whole 2140, last 40 in 6 pieces 1879 us
//   700 x 17920, K 1536 (210 tiles): 256 whole 42.2, 128 whole 48.1 us
GemmPlan gemm_plan(int M, int N, int K, size_t partial_cap, bool eight_wave) {
  auto tiles_of = [&](int t) { return ((M + t - 1) / t) * ((N + t - 1) / t); };
  GemmPlan best{256, K >= kLongK && !eight_wave, tiles_of(256), tiles_of(256), 1, K};
  if (K <= 0) return best;
  double t_best = rounds(256, best.tiles, K);
  for (int tile = 256; tile >= 128; tile /= 2) {
    const int tiles = tiles_of(tile);
    if (tile == 128) {
      const double t = rounds(128, tiles, K);
      if (t < t_best) t_best = t, best = {128, false, tiles, tiles, 1, K};
    }
    // pieces: of the last, partial round of 256 x 256 tiles, or of every tile
    const int whole = tile == 256 ? tiles / 256 * 256 : 0, rest = tiles - whole;
    if (rest == 0 || (tile == 128 && rest > 512)) continue;
    for (int S = 2; S <= kMaxSplit && K / S >= 256; ++S) {
      const int64_t pieces = (int64_t)rest * S;
      if ((size_t)pieces * tile * tile > partial_cap || pieces > 1024) break;
      const int k_piece = ((K + S - 1) / S + 31) / 32 * 32;
      const double t = rounds(tile, whole, K) + rounds(tile, (int)pieces, k_piece) + 6.0 +
                       0.03 * pieces * tile * tile / 65536.0;
      if (t < t_best) {
        t_best = t;
        best = {tile, tile == 256 && !eight_wave && (whole ? K : k_piece) >= kLongK, tiles, whole, S,
                k_piece};
      }
    }
  }
  return best;
}

int gemm_f32_pieces(int M, int N, int K, size_t partial_cap) {
  const int tiles = ((M + kFTile - 1) / kFTile) * ((N + kFTile - 1) / kFTile);
  int S = 1;
  while (S < kMaxSplit && S < K / (2 * kFBK) && tiles * S < 512 &&
         (size_t)tiles * (S + 1) * (kFTile * kFTile) <= partial_cap)
    ++S;
  return S;
}

template <typename T>
int gemm(const Gemm &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return AJ_OK;
  if (g.K2 > 0 && (!g.A2 || !g.B2))
    return fail(AJ_ERR_UNSUPPORTED, "gemm: a second segment needs its operands");
  EpArgs ep{g.M, g.N, g.C, g.ldc, g.c_f32 ? 1 : 0, g.out == OUT_ACCUM_F32 ? 1 : 0, g.R, 0,
            (const bf16_t *)g.swiglu_gu};
  if (g.swiglu_gu && (sizeof(T) != 2 || ep.accum || ep.c_f32 || g.R || g.ldc < 2 * (int64_t)g.N))
    return fail(AJ_ERR_UNSUPPORTED, "gemm: SwiGLU epilogue needs bf16 C [n, 2N], no "
                "accumulation or residual");
  if (ep.accum || sizeof(T) == 4) ep.c_f32 = 1;
  {
    const uintptr_t al = ep.c_f32 ? 15 : 7;
    ep.vec = g.ldc % 4 == 0 && ((uintptr_t)g.C & al) == 0 && ((uintptr_t)g.R & al) == 0 &&
             (!g.swiglu_gu || (g.N % 4 == 0 && ((uintptr_t)g.swiglu_gu & 7) == 0));
  }
  bool mfma = false;
  if constexpr (sizeof(T) == 2) {
    // vector loads need the contiguous dimension in whole 8-element groups
    const int a_contig = g.a_kmajor ? g.K : g.M, b_contig = g.b_kmajor ? g.K : g.N;
    mfma = a_contig % 8 == 0 && b_contig % 8 == 0 && g.lda % 8 == 0 && g.ldb % 8 == 0 &&
           aligned16(g.A) && aligned16(g.B);
    if (g.K2 > 0) {
      const int a2 = g.a_kmajor ? g.K2 : g.M, b2 = g.b_kmajor ? g.K2 : g.N;
      mfma = mfma && a2 % 8 == 0 && b2 % 8 == 0 && g.lda2 % 8 == 0 && g.ldb2 % 8 == 0 &&
             aligned16(g.A2) && aligned16(g.B2);
    }
  }
  const size_t cap = g.partial && aligned16(g.partial) ? g.partial_cap : 0;
  if (mfma) {
    const GemmPlan pl = gemm_plan(g.M, g.N, g.K, cap, g.K2 > 0 || g.swiglu_gu);
    int kc = g.a_kmajor ? (g.b_kmajor ? AJ_KC_GEMM_NT : AJ_KC_GEMM_NN) : AJ_KC_GEMM_TN;
    if (pl.long_k) kc += AJ_KC_GEMM4_NT - AJ_KC_GEMM_NT;   // the kernel that runs
    const int tk =
        timing_begin(s, kc, g.recompute ? 0.0 : 2.0 * g.M * g.N * ((double)g.K + g.K2));
    if (g.a_kmajor && g.b_kmajor) launch_mfma<true, true>(g, ep, pl, s);
    else if (g.a_kmajor) launch_mfma<true, false>(g, ep, pl, s);
    else if (g.b_kmajor) launch_mfma<false, true>(g, ep, pl, s);
    else launch_mfma<false, false>(g, ep, pl, s);
    timing_end(s, tk);
    return check_launch("gemm");
  }
  const int tiles = ((g.M + kFTile - 1) / kFTile) * ((g.N + kFTile - 1) / kFTile);
  const int S = g.K2 == 0 ? gemm_f32_pieces(g.M, g.N, g.K, cap) : 1;
  const int k_piece = ((g.K > 0 ? g.K : 0) + S - 1) / S;
  const Pieces pc{S > 1 ? 0 : tiles, S > 1 ? tiles : 0, S, (k_piece + kFBK - 1) / kFBK * kFBK,
                  g.partial};
  auto operand = [](const void *p, int64_t ld, bool kmajor) {
    return FOperand{p, ld, kmajor, ld % 4 == 0 && ((uintptr_t)p & (4 * sizeof(T) - 1)) == 0};
  };
  gemm_f32_kernel<T><<<pc.whole + pc.rest * S, 256, 0, s>>>(
      g.M, g.N, g.K > 0 ? g.K : 0, operand(g.A, g.lda, g.a_kmajor),
      operand(g.B, g.ldb, g.b_kmajor), g.K2, operand(g.A2, g.lda2, g.a_kmajor),
      operand(g.B2, g.ldb2, g.b_kmajor), ep, pc);
  if (S > 1) gemm_pieces_kernel<kFTile, kFTile><<<pc.rest * 4, 256, 0, s>>>(ep, pc);
  return check_launch("gemm");
}

template int gemm<float>(const Gemm &, hipStream_t);
template int gemm<bf16_t>(const Gemm &, hipStream_t);

}  // namespace aj
