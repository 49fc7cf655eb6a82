// Embedding gather x = E[tok] and its backward, the scatter-add
// dE[v] += sum over positions p with tok[p] == v of dx[p], made
// deterministic without float atomics:
//   1. keys (token << 32 | position) are sorted by token with a stable radix
//      sort, so that the sorted order -- runs of equal token, positions
//      ascending inside a run -- does not depend on how it is scheduled;
//   2. the sorted rows are cut into tiles of 256 (64 rows below 65536, so that
//      small batches fill the chip); one wave per (tile,
//      256-column slice) walks its rows in order and sums each run of equal
//      token.  A run that begins and ends inside the tile is added to dE
//      right there (it has no other owner); the piece of a run that crosses
//      into the next tile goes to a tile slot: slot 1 the piece of a run
//      that begins in the tile, slot 0 the piece of one that began earlier
//      (the whole tile when the run spans it);
//   3. a run that crosses tile boundaries is finished by the boundary it
//      crosses first: slot 1 of its first tile, then slot 0 of each later
//      tile in order, added to dE once.
// Each dE row is therefore written by one owner, with the same sum order on
// every call.
#include "ops.h"

namespace aj {
namespace {

constexpr int kWaveCols = 256;         // columns per wave: 64 lanes x 4
constexpr int kTileWaves = 4;
constexpr uint32_t kNoTok = 0xffffffffu;

// Sorted rows per reduction tile.  A tile is one wave's chain of 8-row batches:
// at 3443 rows of 128 columns, 14 tiles of 256 rows took 60 us.
constexpr int kSmallRows = 65536;
int tile_rows(int n) { return n < kSmallRows ? 64 : 256; }
int64_t n_tiles(int n) { return (n + tile_rows(n) - 1) / tile_rows(n); }

// The wave's LDS accesses before it are done before those after it.
AJ_DEV void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

AJ_DEV uint32_t key_tok(uint64_t k) { return (uint32_t)(k >> 32); }
AJ_DEV uint32_t key_pos(uint64_t k) { return (uint32_t)k; }

// One wave per row.  VEC: 16 bytes per lane and load, all of a lane's loads
// before its first store (2-byte accesses moved 118943 rows of 3584 bfloat16
// values in 522 us).
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void embed_fwd_kernel(const int32_t *tok, int n, const T *emb,
                                                        int d, int vocab, T *x, int32_t *err) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= n) return;
  const int t = tok[row];
  const bool ok = t >= 0 && t < vocab;
  if (!ok && lane == 0 && err) atomicOr(err, AJ_DEVERR_TOKEN_RANGE);
  const T *src = emb + (int64_t)(ok ? t : 0) * d;
  T *dst = x + (int64_t)row * d;
  if constexpr (VEC) {
    constexpr int E = 16 / sizeof(T), U = 8;
    const int nv = d / E;
    const uint4 *s4 = reinterpret_cast<const uint4 *>(src);
    uint4 *d4 = reinterpret_cast<uint4 *>(dst);
    for (int c0 = lane; c0 < nv; c0 += 64 * U) {
      uint4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        v[u] = ok && c0 + 64 * u < nv ? s4[c0 + 64 * u] : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c0 + 64 * u < nv) d4[c0 + 64 * u] = v[u];
    }
  } else {
    for (int c = lane; c < d; c += 64) dst[c] = ok ? src[c] : T(0);
  }
}

// ---------------------------------------------------------------- sort
// Least significant digit first, one count and one scatter launch per digit of
// up to 9 bits (two digits for a 152064-word vocab).  At most 64 workgroups (256
// past 262144 rows) take a contiguous share of the rows each, so that a scatter
// workgroup can add up the counts before its own by itself: no scan launch, no
// workgroup waits for another.  118943 rows: 22 launches of a bitonic network
// 166 us, these 4 launches 43 us (the two scatters 33).
constexpr int kMaxBits = 9, kMaxBins = 1 << kMaxBits;
constexpr int kSub = 1024;             // rows per round of a workgroup: 256 per wave

int sort_blocks(int n) {
  const int most = n > 262144 ? 256 : 64;
  const int64_t b = ((int64_t)n + kSub - 1) / kSub;
  return (int)(b < most ? b : most);
}

struct Digit { int shift, bits, vocab; };

// Row i's key of the first pass (tok) or a later one; tokens out of range take
// the token field kNoTok and sort to the end, as value `vocab`.
AJ_DEV uint64_t sort_key(const int32_t *tok, const uint64_t *keys, int64_t i, int vocab) {
  if (!tok) return keys[i];
  const int t = tok[i];
  const uint32_t tt = t >= 0 && t < vocab ? (uint32_t)t : kNoTok;
  return ((uint64_t)tt << 32) | (uint32_t)i;
}
AJ_DEV int digit_of(uint64_t key, const Digit &dg) {
  const uint32_t t = key_tok(key), v = t == kNoTok ? (uint32_t)dg.vocab : t;
  return (int)((v >> dg.shift) & ((1u << dg.bits) - 1));
}

// counts[block][bin] of the block's rows
__global__ __launch_bounds__(256) void sort_count_kernel(const int32_t *tok, const uint64_t *keys,
                                                         int n, Digit dg, int share,
                                                         int32_t *counts) {
  __shared__ int32_t cnt[kMaxBins];
  const int bins = 1 << dg.bits;
  for (int b = threadIdx.x; b < bins; b += 256) cnt[b] = 0;
  __syncthreads();
  const int64_t lo = (int64_t)blockIdx.x * share, hi = min(lo + share, (int64_t)n);
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256)
    atomicAdd(&cnt[digit_of(sort_key(tok, keys, i, dg.vocab), dg)], 1);
  __syncthreads();
  for (int b = threadIdx.x; b < bins; b += 256) counts[blockIdx.x * bins + b] = cnt[b];
}

// Stable scatter of the block's rows.  A round takes 1024 of them, 256 per wave
// in row order: a lane's rank among the wave's equal digits comes from ballots
// and the wave's running counts, and the rank of the wave's share from the
// counts of the waves before it.
__global__ __launch_bounds__(256) void sort_scatter_kernel(const int32_t *tok, const uint64_t *keys,
                                                           int n, Digit dg, int share,
                                                           const int32_t *counts, uint64_t *out) {
  __shared__ int32_t base[kMaxBins];          // next output row of each digit
  __shared__ int32_t wcnt[4][kMaxBins];
  __shared__ int32_t part[4];
  const int bins = 1 << dg.bits, nb = gridDim.x, me = blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // this thread's digits: 2 tid and 2 tid + 1
  int before[2] = {0, 0}, all[2] = {0, 0};
  for (int b0 = 0; b0 < nb; b0 += 8) {
    int c[8][2];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int bin = 2 * (int)threadIdx.x + e;
        c[u][e] = b0 + u < nb && bin < bins ? counts[(b0 + u) * bins + bin] : 0;
      }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        all[e] += c[u][e];
        before[e] += b0 + u < me ? c[u][e] : 0;
      }
  }
  int x = all[0] + all[1];
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) part[w] = x;
  __syncthreads();
  int off = x - all[0] - all[1];
  for (int i = 0; i < w; ++i) off += part[i];
  if (2 * (int)threadIdx.x < bins) base[2 * threadIdx.x] = off + before[0];
  if (2 * (int)threadIdx.x + 1 < bins) base[2 * threadIdx.x + 1] = off + all[0] + before[1];
  const int64_t lo = (int64_t)me * share, hi = min(lo + share, (int64_t)n);
  for (int64_t r0 = lo; r0 < hi; r0 += kSub) {
    for (int b = threadIdx.x; b < 4 * kMaxBins; b += 256) (&wcnt[0][0])[b] = 0;
    __syncthreads();
    uint64_t key[4];
    int dig[4], rank[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = r0 + w * 256 + q * 64 + lane;
      key[q] = i < hi ? sort_key(tok, keys, i, dg.vocab) : 0;
      dig[q] = i < hi ? digit_of(key[q], dg) : -1;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint64_t peers = __ballot(dig[q] >= 0);
      for (int b = 0; b < dg.bits; ++b) {
        const uint64_t set = __ballot((dig[q] >> b) & 1);
        peers &= (dig[q] >> b) & 1 ? set : ~set;
      }
      const int below = __popcll(peers & ((1ull << lane) - 1));
      rank[q] = dig[q] >= 0 ? wcnt[w][dig[q]] + below : 0;
      wave_lds_sync();   // every lane has read its count before a leader adds
      if (dig[q] >= 0 && below == 0) wcnt[w][dig[q]] += __popcll(peers);
      wave_lds_sync();
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (dig[q] < 0) continue;
      int at = base[dig[q]] + rank[q];
      for (int i = 0; i < w; ++i) at += wcnt[i][dig[q]];
      out[at] = key[q];
    }
    __syncthreads();
    for (int b = threadIdx.x; b < bins; b += 256)
      base[b] += wcnt[0][b] + wcnt[1][b] + wcnt[2][b] + wcnt[3][b];
    __syncthreads();
  }
}

AJ_DEV void add4(float4 &a, const float4 &b) {
  a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
}

// Step 2: one wave per (tile, 256-column slice); lane l owns columns
// col0 .. col0+3.  piece: [n_tiles][2][d].
template <int kTile>
__global__ __launch_bounds__(256) void embed_tile_kernel(const uint64_t *keys, int n,
                                                         const float *dx, int d, float *demb,
                                                         float *piece) {
  __shared__ uint64_t sk[kTile];
  const int tile = blockIdx.x;
  const int r0 = tile * kTile, r1 = min(n, r0 + kTile);
  for (int t = threadIdx.x; t < r1 - r0; t += 256) sk[t] = keys[r0 + t];
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col0 = (blockIdx.y * kTileWaves + wave) * kWaveCols + 4 * lane;
  if (col0 >= d) return;
  const uint32_t prev_tok = r0 > 0 ? key_tok(keys[r0 - 1]) : kNoTok;
  const uint32_t next_tok = r1 < n ? key_tok(keys[r1]) : kNoTok;
  float *slot0 = piece + ((int64_t)tile * 2) * d + col0;
  float *slot1 = slot0 + d;
  // the first run may have started in an earlier tile
  bool began_before = key_tok(sk[0]) == prev_tok;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int r = r0; r < r1; r += 8) {
    // eight rows, and the dE rows of the runs that end among them, in flight at once
    float4 v[8], o[8];
    uint32_t tt[8];
    bool last[8];       // the row is the last of its run
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int rr = r + u;
      const uint64_t k = rr < r1 ? sk[rr - r0] : ~0ull;
      tt[u] = key_tok(k);
      last[u] = tt[u] != (rr + 1 < r1 ? key_tok(sk[rr + 1 - r0]) : next_tok);
      const bool in = rr < r1 && tt[u] != kNoTok;
      v[u] = in ? *(const float4 *)(dx + (int64_t)key_pos(k) * d + col0)
                : make_float4(0.f, 0.f, 0.f, 0.f);
      o[u] = in && last[u] ? *(const float4 *)(demb + (int64_t)tt[u] * d + col0)
                           : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (r + u >= r1 || tt[u] == kNoTok) break;
      add4(acc, v[u]);
      if (last[u]) {
        if (began_before) {
          *(float4 *)slot0 = acc;                // head piece
        } else {
          add4(o[u], acc);
          *(float4 *)(demb + (int64_t)tt[u] * d + col0) = o[u];
        }
      } else if (r + u + 1 == r1) {
        // the run goes on in the next tile: the whole tile, or a tail piece
        *(float4 *)(began_before ? slot0 : slot1) = acc;
      }
      if (last[u]) {
        began_before = false;
        acc = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  }
}

// Step 3: the run crossing boundary b = (blockIdx.x + 1) * kTile, if it
// crosses no earlier boundary; one thread per 4 columns.  A run may span every
// tile: eight of its pieces are loaded at a time, added in order (one at a time, a
// load behind each token check, 65535 rows of one token and 128 columns took 321
// us in all).
template <int kTile>
__global__ __launch_bounds__(256) void embed_cross_kernel(const uint64_t *keys, int n, int n_tiles,
                                                          int d, const float *piece, float *demb) {
  const int bt = blockIdx.x + 1;
  const int64_t b = (int64_t)bt * kTile;
  if (b >= n) return;
  const uint32_t t = key_tok(keys[b - 1]);
  if (t == kNoTok || key_tok(keys[b]) != t) return;
  if (bt > 1 && key_tok(keys[b - kTile - 1]) == t) return;     // crosses b - kTile too
  const int col0 = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (col0 >= d) return;
  float4 acc = *(const float4 *)(piece + ((int64_t)(bt - 1) * 2 + 1) * d + col0);
  // the run's later tiles [bt, end): those that begin with its token (sorted keys)
  int end = bt + 1, hi = n_tiles;
  while (end < hi) {
    const int mid = (end + hi) >> 1;
    if (key_tok(keys[(int64_t)mid * kTile]) == t) end = mid + 1; else hi = mid;
  }
  for (int u = bt; u < end; u += 8) {
    float4 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      v[q] = u + q < end ? *(const float4 *)(piece + ((int64_t)(u + q) * 2) * d + col0)
                         : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (u + q < end) add4(acc, v[q]);
  }
  float4 *o = (float4 *)(demb + (int64_t)t * d + col0);
  float4 v = *o;
  add4(v, acc);
  *o = v;
}

struct EmbedWs {
  uint64_t *keys[2];
  int32_t *counts;
  float *piece;
  size_t bytes;
};

EmbedWs carve_embed(void *ws, int n, int d) {
  Carver c(ws);
  EmbedWs w;
  w.keys[0] = c.take<uint64_t>(n);
  w.keys[1] = c.take<uint64_t>(n);
  w.counts = c.take<int32_t>((int64_t)sort_blocks(n) * kMaxBins);
  // never less for more rows: a buffer sized for the largest pack serves them all
  const int64_t tiles = n < kSmallRows ? n_tiles(n) : std::max<int64_t>(n_tiles(n), kSmallRows / 64);
  w.piece = c.take<float>(2 * tiles * (int64_t)d);
  w.bytes = c.bytes();
  return w;
}

template <int kTile>
void embed_reduce(const uint64_t *keys, int n, const float *dx, int d, float *d_emb, float *piece,
                  hipStream_t s) {
  const int tiles = (n + kTile - 1) / kTile;
  const int col_blocks = (d + kTileWaves * kWaveCols - 1) / (kTileWaves * kWaveCols);
  embed_tile_kernel<kTile><<<dim3(tiles, col_blocks), 256, 0, s>>>(keys, n, dx, d, d_emb, piece);
  if (tiles > 1)
    embed_cross_kernel<kTile><<<dim3(tiles - 1, (d / 4 + 255) / 256), 256, 0, s>>>(
        keys, n, tiles, d, piece, d_emb);
}

}  // namespace

template <typename T>
void embed_fwd(const int32_t *tok, int n, const T *emb, int d, int vocab, T *x, int32_t *err,
               hipStream_t s) {
  if (n <= 0) return;
  const bool vec = (d * sizeof(T)) % 16 == 0 && (((uintptr_t)emb | (uintptr_t)x) & 15) == 0;
  if (vec) embed_fwd_kernel<T, true><<<(n + 3) / 4, 256, 0, s>>>(tok, n, emb, d, vocab, x, err);
  else embed_fwd_kernel<T, false><<<(n + 3) / 4, 256, 0, s>>>(tok, n, emb, d, vocab, x, err);
}
template void embed_fwd<float>(const int32_t *, int, const float *, int, int, float *, int32_t *,
                               hipStream_t);
template void embed_fwd<bf16_t>(const int32_t *, int, const bf16_t *, int, int, bf16_t *,
                                int32_t *, hipStream_t);

}  // namespace aj

extern "C" int aj_embed_fwd(const int32_t *tok, int32_t n_tok, const void *emb, int32_t d,
                            int32_t vocab, int dtype, void *x, int32_t *err, void *stream) {
  AJ_REQUIRE(n_tok >= 0 && d > 0 && vocab > 0, AJ_ERR_SHAPE, "aj_embed_fwd: sizes");
  if (n_tok == 0) return AJ_OK;
  AJ_REQUIRE(tok && emb && x, AJ_ERR_NULL, "aj_embed_fwd: null pointer");
  hipStream_t st = (hipStream_t)stream;
  if (dtype == AJ_BF16)
    aj::embed_fwd<bf16_t>(tok, n_tok, (const bf16_t *)emb, d, vocab, (bf16_t *)x, err, st);
  else if (dtype == AJ_F32)
    aj::embed_fwd<float>(tok, n_tok, (const float *)emb, d, vocab, (float *)x, err, st);
  else
    return aj::fail(AJ_ERR_UNSUPPORTED, "aj_embed_fwd: dtype %d", dtype);
  return aj::check_launch("aj_embed_fwd");
}

extern "C" size_t aj_embed_bwd_workspace_bytes(int32_t n_tok, int32_t d) {
  if (n_tok < 0 || d <= 0) return 0;
  return aj::carve_embed(nullptr, n_tok, d).bytes;
}

extern "C" int aj_embed_bwd(const int32_t *tok, int32_t n_tok, const float *dx, int32_t d,
                            int32_t vocab, float *d_emb, void *ws, size_t ws_bytes,
                            void *stream) {
  using namespace aj;
  AJ_REQUIRE(n_tok >= 0 && d > 0 && vocab > 0, AJ_ERR_SHAPE, "aj_embed_bwd: sizes");
  AJ_REQUIRE(n_tok <= (1 << 30), AJ_ERR_UNSUPPORTED, "aj_embed_bwd: n_tok %d > 2^30", n_tok);
  AJ_REQUIRE(d % 4 == 0, AJ_ERR_UNSUPPORTED, "aj_embed_bwd: d %d not a multiple of 4", d);
  if (n_tok == 0) return AJ_OK;
  AJ_REQUIRE(tok && dx && d_emb && ws, AJ_ERR_NULL, "aj_embed_bwd: null pointer");
  AJ_REQUIRE(((uintptr_t)dx & 15) == 0 && ((uintptr_t)d_emb & 15) == 0, AJ_ERR_UNSUPPORTED,
             "aj_embed_bwd: dx and d_emb must be 16-byte aligned");
  const EmbedWs w = carve_embed(ws, n_tok, d);
  AJ_REQUIRE(ws_bytes >= w.bytes, AJ_ERR_WORKSPACE, "aj_embed_bwd: workspace %zu < %zu",
             ws_bytes, w.bytes);
  hipStream_t s = (hipStream_t)stream;
  // as few digits of the token (and of the value `vocab` past the last one) as
  // kMaxBits allows, evenly wide
  int bits = 1;
  while (bits < 31 && (vocab >> bits) != 0) ++bits;
  const int passes = (bits + kMaxBits - 1) / kMaxBits, width = (bits + passes - 1) / passes;
  const int blocks = sort_blocks(n_tok), share = (n_tok + blocks - 1) / blocks;
  for (int p = 0; p < passes; ++p) {
    const Digit dg{p * width, width, vocab};
    const int32_t *t = p == 0 ? tok : nullptr;
    sort_count_kernel<<<blocks, 256, 0, s>>>(t, w.keys[(p & 1) ^ 1], n_tok, dg, share, w.counts);
    sort_scatter_kernel<<<blocks, 256, 0, s>>>(t, w.keys[(p & 1) ^ 1], n_tok, dg, share, w.counts,
                                               w.keys[p & 1]);
  }
  const uint64_t *keys = w.keys[(passes - 1) & 1];
  if (tile_rows(n_tok) == 64) embed_reduce<64>(keys, n_tok, dx, d, d_emb, w.piece, s);
  else embed_reduce<256>(keys, n_tok, dx, d, d_emb, w.piece, s);
  return check_launch("aj_embed_bwd");
}
