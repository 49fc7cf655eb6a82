// Causal GQA attention over packed variable-length segments.
//
// Tiles are runs of consecutive packed rows; a row attends to the keys of its
// own segment up to itself, [seg_start(row), row], with seg_start found from
// cu_seqlens.  Query head h reads key/value head floor(h * Hkv / Hq).
//
// These kernels serve the float32 workload and head dims other than 64 and 128:
// v_mfma_f32_16x16x4_f32 (float32 products and sums), a wave per 16 rows of one
// head, four waves sharing the rows staged in LDS.  bfloat16 with head_dim 64 or
// 128 goes to the kernels in attention_mfma.hip.
//
// All products keep the wave's 16 rows on the lanes' columns: with S^T = K Q^T a
// lane holds scores of one query (its column l%16) for keys 4 (l/16) + 0..3, and
// that is the layout the next product takes as its operand (the j-th product of
// a 16-wide reduction covers elements 4 (l/16) + j), so probabilities never
// leave their registers.  Segments here are a few hundred rows: the time is one
// pass of dependent steps over a segment, which a wave per 16 rows (4 times the
// rows in flight of a thread quad per row, and 16 of a step's keys at once)
// shortens from 391 / 356 / 457 us (forward, dQ, dK and dV of 3443 tokens in 4
// heads of 32) to 29 / 31 / 39.  Loading a step's rows beside the step before and
// splitting the score products' chain in two: 22 / 25 / 32.
//
// A masked pair has weight 0 in those products, and 0 times an infinity or a NaN
// is a NaN.  So a workgroup whose sums are not all finite takes its rows again,
// with the masked pairs left out one by one: a bad row stays with the rows that
// attend to it, and finite rows pay one check at the end (a check of every step's
// rows cost 3 to 8 %).
#include <type_traits>
#include "ops.h"

namespace aj {
namespace {

constexpr int kRows = 64;     // query (or key) rows per workgroup: 16 per wave
constexpr int kMaxHd = 128;
typedef float f32x4_t __attribute__((ext_vector_type(4)));

AJ_DEV int seg_of(const int32_t *cu, int n_seg, int base, int row) {
  int lo = 0, hi = n_seg - 1;   // largest s with cu[s] - base <= row
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (cu[mid] - base <= row) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// First row of row's segment, clamped into [0, row] whatever cu_seqlens holds.
template <typename A>
AJ_DEV int seg_start(const A &a, int row) {
  const int v = a.cu_seqlens[seg_of(a.cu_seqlens, a.n_seg, a.base, row)] - a.base;
  return v < 0 ? 0 : (v > row ? row : v);
}

// One past the last row of row's segment, clamped into [row + 1, n_tok].
template <typename A>
AJ_DEV int seg_end(const A &a, int row) {
  const int v = a.cu_seqlens[seg_of(a.cu_seqlens, a.n_seg, a.base, row) + 1] - a.base;
  return v <= row ? row + 1 : (v > a.n_tok ? a.n_tok : v);
}

AJ_DEV f32x4_t mfma4(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Rows of NC 16-feature chunks in LDS: 16 NC + 4 floats apart, so that the 16
// rows of a fragment read, and the 4 row groups of a transposed one, fall on
// different banks.
template <int NC> constexpr int kLd = 16 * NC + 4;
// Rows staged per step: 64, less where two such arrays would pass 64 KB.
template <int NC> constexpr int kStep = NC <= 4 ? 64 : 32;

// The thread's share of rows [r0, r0 + kStep) of a [rows, ld] matrix's hd columns,
// in fours (zeros past `last` and past hd; hd is a multiple of 8, so four columns
// are in or out as one): loaded into registers, then put into LDS, so that a
// step's loads run beside the step before.
template <int NC> constexpr int kFours = kStep<NC> * NC * 4 / 256;
template <typename T, int NC>
AJ_DEV void fetch_rows(float4 (&v)[kFours<NC>], const T *p, int64_t ld, int hd, bool vec, int r0,
                       int last) {
#pragma unroll
  for (int q = 0; q < kFours<NC>; ++q) {
    const int e = threadIdx.x + 256 * q, r = e / (NC * 4), c = e % (NC * 4) * 4;
    v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r0 + r <= last && c < hd) {
      const T *src = p + (int64_t)(r0 + r) * ld + c;
      if (vec && sizeof(T) == 4) {
        v[q] = *reinterpret_cast<const float4 *>(src);
      } else if (vec) {
        const uint2 u = *reinterpret_cast<const uint2 *>(src);
        v[q] = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                           __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
      } else {
        v[q] = make_float4(ldf(src), ldf(src + 1), ldf(src + 2), ldf(src + 3));
      }
    }
  }
}
template <int NC>
AJ_DEV void put_rows(float *lds, const float4 (&v)[kFours<NC>]) {
#pragma unroll
  for (int q = 0; q < kFours<NC>; ++q) {
    const int e = threadIdx.x + 256 * q, r = e / (NC * 4), c = e % (NC * 4) * 4;
    *reinterpret_cast<float4 *>(lds + r * kLd<NC> + c) = v[q];
  }
}

// a lane's operand of its own row: features 16 c + 4 (l/16) + j
template <typename T, int NC>
AJ_DEV void own_row(f32x4_t (&f)[NC], const T *p, int hd, bool valid) {
  const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int k = 16 * c + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) f[c][j] = valid && k < hd ? ldf(p + k + j) : 0.f;
  }
}
template <typename T, int NC>
AJ_DEV void store_row(T *p, const f32x4_t (&f)[NC], int hd, float scale) {
  const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int k = 16 * c + 4 * g;
    if (k < hd)
#pragma unroll
      for (int j = 0; j < 4; ++j) stf(p + k + j, f[c][j] * scale);
  }
}

// (rows of LDS x the lane's row)^T: 16 rows from `rows` on against `own`; the
// lane gets rows 4 (l/16) + 0..3
template <int NC>
AJ_DEV f32x4_t rows_dot(const float *rows, const f32x4_t (&own)[NC]) {
  const int lane = threadIdx.x & 63;
  // in two chains, which issue side by side
  f32x4_t s[2] = {};
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const f32x4_t a = *reinterpret_cast<const f32x4_t *>(rows + (lane & 15) * kLd<NC> + 16 * c + 4 * (lane >> 4));
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j & 1] = mfma4(a[j], own[c][j], s[j & 1]);
  }
  return s[0] + s[1];
}
// acc[features, lane's row] += sum over 16 rows of LDS, w[row] (the lane's rows
// 4 (l/16) + j) times the row's features; w is 0 for rows without their bit in
// `in`, which EXACT leaves out whatever they hold.
template <bool EXACT, int NC>
AJ_DEV void rows_add(f32x4_t (&acc)[NC], const float *rows, const f32x4_t &w, int in) {
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  if constexpr (EXACT) {
    in <<= 4 * g;   // of the lane's column: all 16 rows
    in |= __shfl_xor(in, 16, 64);
    in |= __shfl_xor(in, 32, 64);
#pragma unroll 1
    for (int r = 0; r < 16; ++r) {
      const float wj = r & 2 ? (r & 1 ? w[3] : w[2]) : (r & 1 ? w[1] : w[0]);
      const float wr = __shfl(wj, (r >> 2) * 16 + col, 64);
      if ((in >> r) & 1)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[c][e] = fmaf(rows[r * kLd<NC> + 16 * c + 4 * g + e], wr, acc[c][e]);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        acc[c] = mfma4(rows[(4 * g + j) * kLd<NC> + 16 * c + col], w[j], acc[c]);
  }
}
// Whether any thread's sums are not finite (in every thread of the workgroup).
template <int NC>
AJ_DEV bool any_nonfinite(const f32x4_t (&f)[NC], bool valid) {
  f32x4_t z = {};
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) z[e] = fmaf(f[c][e], 0.f, z[e]);
  return __syncthreads_or(valid && !(z[0] + z[1] + z[2] + z[3] == 0.f));
}

AJ_DEV bool vec4(const void *p, int64_t ld, int es) {
  return ld % 4 == 0 && ((uintptr_t)p & (4 * es - 1)) == 0;
}

template <typename T, int NC>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) float Ks[kStep<NC> * kLd<NC>], Vs[kStep<NC> * kLd<NC>];
  const int hd = a.hd, ld = (a.Hq + 2 * a.Hkv) * hd;
  const int h = blockIdx.y, g = (h * a.Hkv) / a.Hq;
  const int row0 = blockIdx.x * kRows, last = min(row0 + kRows, a.n_tok) - 1;
  const int lane = threadIdx.x & 63, w0 = row0 + 16 * (threadIdx.x >> 6);
  const int row = w0 + (lane & 15);
  const bool valid = row < a.n_tok;
  const T *qkv = (const T *)a.qkv, *kp = qkv + (a.Hq + g) * hd, *vp = kp + a.Hkv * hd;
  const bool vec = vec4(a.qkv, ld, sizeof(T));
  const int start = valid ? seg_start(a, row) : row;
  f32x4_t q[NC], o[NC];
  own_row<T, NC>(q, qkv + (int64_t)row * ld + h * hd, hd, valid);
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int j = 0; j < 4; ++j) q[c][j] *= a.scale;
  float m, l;
  const int k_lo = seg_start(a, row0);
  float4 kr[kFours<NC>], vr[kFours<NC>];
  auto walk = [&](auto exact) __attribute__((always_inline)) {
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    fetch_rows<T, NC>(kr, kp, ld, hd, vec, k_lo, last);
    fetch_rows<T, NC>(vr, vp, ld, hd, vec, k_lo, last);
    for (int k0 = k_lo; k0 <= last; k0 += kStep<NC>) {
      __syncthreads();
      put_rows<NC>(Ks, kr);
      put_rows<NC>(Vs, vr);
      __syncthreads();
      if (k0 + kStep<NC> <= last) {
        fetch_rows<T, NC>(kr, kp, ld, hd, vec, k0 + kStep<NC>, last);
        fetch_rows<T, NC>(vr, vp, ld, hd, vec, k0 + kStep<NC>, last);
      }
      for (int t = 0; t < kStep<NC> && k0 + t <= w0 + 15; t += 16) {
        f32x4_t s = rows_dot<NC>(Ks + t * kLd<NC>, q);
        const int key = k0 + t + 4 * (lane >> 4);
        float mx = -INFINITY;
        int in = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (key + j < start || key + j > row || !valid) s[j] = -INFINITY;
          else in |= 1 << j;
          mx = fmaxf(mx, s[j]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mn = fmaxf(m, mx);
        // a query that has seen no key yet keeps zero weights (mn is -inf)
        const float sc = mn == -INFINITY ? 1.f : __expf(m - mn);
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          s[j] = s[j] == -INFINITY ? 0.f : __expf(s[j] - mn);
          sum += s[j];
        }
        l = l * sc + sum;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int j = 0; j < 4; ++j) o[c][j] *= sc;
        rows_add<decltype(exact)::value>(o, Vs + t * kLd<NC>, s, in);
        m = mn;
      }
    }
  };
  walk(std::false_type{});
  if (any_nonfinite<NC>(o, valid)) walk(std::true_type{});
  // each lane has summed its own keys' weights
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (!valid) return;
  store_row<T, NC>((T *)a.o + (int64_t)row * a.Hq * hd + h * hd, o, hd, 1.f / l);
  if (lane < 16) a.lse[(int64_t)h * a.n_tok + row] = m + logf(l);
}

// delta[h][row] = sum_d dO * O
template <typename T>
__global__ __launch_bounds__(256) void attn_delta_kernel(AttnBwdArgs a) {
  const int64_t idx = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (idx >= (int64_t)a.n_tok * a.Hq) return;
  const int row = (int)(idx / a.Hq), h = (int)(idx % a.Hq);
  const T *o = (const T *)a.o + (int64_t)row * a.Hq * a.hd + h * a.hd;
  const T *d = (const T *)a.dout + (int64_t)row * a.Hq * a.hd + h * a.hd;
  float s = 0.f;
  for (int c = lane; c < a.hd; c += 64) s += ldf(o + c) * ldf(d + c);
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) s += __shfl_xor(s, w, 64);
  if (lane == 0) a.delta[(int64_t)h * a.n_tok + row] = s;
}

// dQ rows: dq = scale * sum_j P_j (dO.V_j - delta) K_j
template <typename T, int NC>
__global__ __launch_bounds__(256) void attn_dq_f32_kernel(AttnBwdArgs a) {
  __shared__ __attribute__((aligned(16))) float Ks[kStep<NC> * kLd<NC>], Vs[kStep<NC> * kLd<NC>];
  const int hd = a.hd, ld = (a.Hq + 2 * a.Hkv) * hd;
  const int h = blockIdx.y, g = (h * a.Hkv) / a.Hq;
  const int row0 = blockIdx.x * kRows, last = min(row0 + kRows, a.n_tok) - 1;
  const int lane = threadIdx.x & 63, w0 = row0 + 16 * (threadIdx.x >> 6);
  const int row = w0 + (lane & 15);
  const bool valid = row < a.n_tok;
  const T *qkv = (const T *)a.qkv, *kp = qkv + (a.Hq + g) * hd, *vp = kp + a.Hkv * hd;
  const bool vec = vec4(a.qkv, ld, sizeof(T));
  const int start = valid ? seg_start(a, row) : row;
  const float lse = valid ? a.lse[(int64_t)h * a.n_tok + row] : 0.f;
  const float delta = valid ? a.delta[(int64_t)h * a.n_tok + row] : 0.f;
  f32x4_t q[NC], dob[NC], dq[NC];
  own_row<T, NC>(q, qkv + (int64_t)row * ld + h * hd, hd, valid);
  own_row<T, NC>(dob, (const T *)a.dout + (int64_t)row * a.Hq * hd + h * hd, hd, valid);
  const int k_lo = seg_start(a, row0);
  float4 kr[kFours<NC>], vr[kFours<NC>];
  auto walk = [&](auto exact) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < NC; ++c) dq[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    fetch_rows<T, NC>(kr, kp, ld, hd, vec, k_lo, last);
    fetch_rows<T, NC>(vr, vp, ld, hd, vec, k_lo, last);
    for (int k0 = k_lo; k0 <= last; k0 += kStep<NC>) {
      __syncthreads();
      put_rows<NC>(Ks, kr);
      put_rows<NC>(Vs, vr);
      __syncthreads();
      if (k0 + kStep<NC> <= last) {
        fetch_rows<T, NC>(kr, kp, ld, hd, vec, k0 + kStep<NC>, last);
        fetch_rows<T, NC>(vr, vp, ld, hd, vec, k0 + kStep<NC>, last);
      }
      for (int t = 0; t < kStep<NC> && k0 + t <= w0 + 15; t += 16) {
        const f32x4_t s = rows_dot<NC>(Ks + t * kLd<NC>, q);
        const f32x4_t dp = rows_dot<NC>(Vs + t * kLd<NC>, dob);
        const int key = k0 + t + 4 * (lane >> 4);
        f32x4_t ds;
        int in = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool inj = valid && key + j >= start && key + j <= row;
          ds[j] = inj ? __expf(s[j] * a.scale - lse) * (dp[j] - delta) * a.scale : 0.f;
          in |= inj << j;
        }
        rows_add<decltype(exact)::value>(dq, Ks + t * kLd<NC>, ds, in);
      }
    }
  };
  walk(std::false_type{});
  if (any_nonfinite<NC>(dq, valid)) walk(std::true_type{});
  if (valid) store_row<T, NC>((T *)a.dqkv + (int64_t)row * ld + h * hd, dq, hd, 1.f);
}

// dK, dV rows of kv head g: sum over the query heads of the group and the
// queries of the same segment at or after the key.
template <typename T, int NC>
__global__ __launch_bounds__(256) void attn_dkv_f32_kernel(AttnBwdArgs a) {
  __shared__ __attribute__((aligned(16))) float Qs[kStep<NC> * kLd<NC>], Ds[kStep<NC> * kLd<NC>];
  __shared__ __attribute__((aligned(16))) float Ls[kStep<NC>], Dl[kStep<NC>];
  const int hd = a.hd, ld = (a.Hq + 2 * a.Hkv) * hd;
  const int g = blockIdx.y;
  const int row0 = blockIdx.x * kRows;
  const int lane = threadIdx.x & 63, w0 = row0 + 16 * (threadIdx.x >> 6);
  const int row = w0 + (lane & 15);           // the key row
  const bool valid = row < a.n_tok;
  const T *qkv = (const T *)a.qkv;
  const bool vec = vec4(a.qkv, ld, sizeof(T)), vecd = vec4(a.dout, (int64_t)a.Hq * hd, sizeof(T));
  const int end = valid ? seg_end(a, row) : 0;
  const int q_hi = seg_end(a, min(row0 + kRows, a.n_tok) - 1) - 1;
  // the last query any of the wave's keys meets
  int w_hi = end - 1;
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) w_hi = max(w_hi, __shfl_xor(w_hi, o, 64));
  f32x4_t k[NC], v[NC], dk[NC], dv[NC];
  own_row<T, NC>(k, qkv + (int64_t)row * ld + (a.Hq + g) * hd, hd, valid);
  own_row<T, NC>(v, qkv + (int64_t)row * ld + (a.Hq + a.Hkv + g) * hd, hd, valid);
  const int group = a.Hq / a.Hkv;
  // the steps over every query head of the group, in one sequence
  const int n_q = q_hi >= row0 ? (q_hi - row0) / kStep<NC> + 1 : 0;
  float4 qr[kFours<NC>], dr[kFours<NC>];
  float lr = 0.f, er = 0.f;
  auto fetch = [&](int i) {
    const int h = g * group + i / n_q, q0 = row0 + i % n_q * kStep<NC>;
    fetch_rows<T, NC>(qr, qkv + h * hd, ld, hd, vec, q0, q_hi);
    fetch_rows<T, NC>(dr, (const T *)a.dout + h * hd, (int64_t)a.Hq * hd, hd, vecd, q0, q_hi);
    const int q = q0 + (int)threadIdx.x;
    if ((int)threadIdx.x < kStep<NC>) {
      lr = q <= q_hi ? a.lse[(int64_t)h * a.n_tok + q] : 0.f;
      er = q <= q_hi ? a.delta[(int64_t)h * a.n_tok + q] : 0.f;
    }
  };
  auto walk = [&](auto exact) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < NC; ++c) dk[c] = dv[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (n_q > 0) fetch(0);
    for (int i = 0; i < group * n_q; ++i) {
      const int q0 = row0 + i % n_q * kStep<NC>;
      __syncthreads();
      put_rows<NC>(Qs, qr);
      put_rows<NC>(Ds, dr);
      if ((int)threadIdx.x < kStep<NC>) Ls[threadIdx.x] = lr, Dl[threadIdx.x] = er;
      __syncthreads();
      if (i + 1 < group * n_q) fetch(i + 1);
      for (int t = 0; t < kStep<NC> && q0 + t <= w_hi; t += 16) {
        if (q0 + t + 15 < w0) continue;
        const f32x4_t s = rows_dot<NC>(Qs + t * kLd<NC>, k);
        const f32x4_t dp = rows_dot<NC>(Ds + t * kLd<NC>, v);
        const int ql = t + 4 * (lane >> 4);
        f32x4_t p, ds;
        int in = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool inj = valid && q0 + ql + j >= row && q0 + ql + j < end;
          p[j] = inj ? __expf(s[j] * a.scale - Ls[ql + j]) : 0.f;
          ds[j] = inj ? p[j] * (dp[j] - Dl[ql + j]) * a.scale : 0.f;
          in |= inj << j;
        }
        rows_add<decltype(exact)::value>(dv, Ds + t * kLd<NC>, p, in);
        rows_add<decltype(exact)::value>(dk, Qs + t * kLd<NC>, ds, in);
      }
    }
  };
  walk(std::false_type{});
  // not `||`: every thread takes both barriers
  if (any_nonfinite<NC>(dk, valid) | any_nonfinite<NC>(dv, valid)) walk(std::true_type{});
  if (!valid) return;
  T *base = (T *)a.dqkv + (int64_t)row * ld;
  store_row<T, NC>(base + (a.Hq + g) * hd, dk, hd, 1.f);
  store_row<T, NC>(base + (a.Hq + a.Hkv + g) * hd, dv, hd, 1.f);
}

// 16-feature chunks of a head, rounded up to an instantiated count
#define AJ_NC_DISPATCH(hd, CALL)                     \
  do {                                               \
    if ((hd) <= 16) { constexpr int NC = 1; CALL; }  \
    else if ((hd) <= 32) { constexpr int NC = 2; CALL; } \
    else if ((hd) <= 64) { constexpr int NC = 4; CALL; } \
    else { constexpr int NC = 8; CALL; }             \
  } while (0)

}  // namespace

template <typename T>
int attn_fwd(const AttnArgs &a, hipStream_t s) {
  if (a.n_tok <= 0) return AJ_OK;
  if (a.hd > kMaxHd || a.hd % 8) return fail(AJ_ERR_UNSUPPORTED, "attention: head_dim %d", a.hd);
  if (sizeof(T) == 2 && attn_mfma_supported(a.hd, a.qkv, a.o, a.o)) return attn_fwd_mfma(a, s);
  dim3 grid((a.n_tok + kRows - 1) / kRows, a.Hq);
  const int tk = timing_begin(s, AJ_KC_ATTN_FWD, 0.0);
  AJ_NC_DISPATCH(a.hd, (attn_fwd_f32_kernel<T, NC><<<grid, 256, 0, s>>>(a)));
  timing_end(s, tk);
  return check_launch("attention forward");
}

template <typename T>
int attn_bwd(const AttnBwdArgs &a, hipStream_t s) {
  if (a.n_tok <= 0) return AJ_OK;
  if (a.hd > kMaxHd || a.hd % 8) return fail(AJ_ERR_UNSUPPORTED, "attention: head_dim %d", a.hd);
  // the matrix-core forward saves its log-sum-exp in log2 units, the plain
  // kernels in natural ones: the backward must take the forward's path
  const bool fwd_mfma = sizeof(T) == 2 && attn_mfma_supported(a.hd, a.qkv, a.o, a.o);
  if (fwd_mfma) {
    if (!attn_mfma_supported(a.hd, a.qkv, a.dout, a.dqkv))
      return fail(AJ_ERR_UNSUPPORTED, "attention backward: d out / d qkv not 16-byte aligned");
    return attn_bwd_mfma(a, s);
  }
  const int64_t nd = (int64_t)a.n_tok * a.Hq;
  const int tk = timing_begin(s, AJ_KC_ATTN_BWD, 0.0);
  attn_delta_kernel<T><<<(unsigned)((nd + 3) / 4), 256, 0, s>>>(a);
  const int blocks = (a.n_tok + kRows - 1) / kRows;
  AJ_NC_DISPATCH(a.hd, (attn_dq_f32_kernel<T, NC><<<dim3(blocks, a.Hq), 256, 0, s>>>(a)));
  AJ_NC_DISPATCH(a.hd, (attn_dkv_f32_kernel<T, NC><<<dim3(blocks, a.Hkv), 256, 0, s>>>(a)));
  timing_end(s, tk);
  return check_launch("attention backward");
}

template int attn_fwd<float>(const AttnArgs &, hipStream_t);
template int attn_fwd<bf16_t>(const AttnArgs &, hipStream_t);
template int attn_bwd<float>(const AttnBwdArgs &, hipStream_t);
template int attn_bwd<bf16_t>(const AttnBwdArgs &, hipStream_t);

}  // namespace aj
