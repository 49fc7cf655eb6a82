// The bfloat16 MFMA GEMM main loop, shared by the plain GEMM and the fused
// LM-head kernels (which only differ in what they do with the accumulators).
//
// Workgroup tiles of v_mfma_f32_16x16x32_bf16 products, 32-wide k-steps through
// a ring of LDS stages.  Operands are copied into LDS in their memory order: a
// K-major one as [row][k], an M/N-major one as [k][row], whose MFMA fragments
// come out of LDS already transposed through ds_read_b64_tr_b16.
//
// Why 16x16x32 and not 32x32x16: these products run at the chip's power limit
// (the clock falls below 1.8 GHz while they run, and from registers alone random
// operands reach 1880 TFLOP/s where constant ones reach 2480, csrc/ceiling.hip),
// and the smaller tile's accumulator traffic per product is half (a quarter of
// the accumulators, half the products).  That file's loop with 256 accumulators
// per lane and random operands: 2041 TFLOP/s with this instruction, 1788 with the
// larger one.  With it went the fragment reads' address arithmetic (one address
// per operand, constants for the rest) and the copies' (buffer resources in
// scalar registers): the loop holds MFMAs, LDS reads, copies and scalar
// instructions only.  32B-class LM head over 18897 targets 104.3 -> 89.9 ms, 32B
// block over one 45769-token segment 197.1 -> 183.9 ms, 7B block over 19437
// tokens 30.2 -> 27.3 ms.
#pragma once
#include <utility>
#include "common.h"

namespace aj {
namespace gemm_core {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// Tile rows per group of the tile walk: the 32 tiles an XCD runs at once then
// cover 4 rows x 8 columns of tiles (12 operand panels shared through its L2;
// measured 1-3 % faster than 8 x 4 on the long-reduction layouts, 16 x 2 and
// 2 x 16 slower).
constexpr int kGroupM = 4;
constexpr int kXcds = 8;

struct TileIdx { int tm, tn; };

// Workgroups are dealt to the XCDs round robin: the XCD of workgroup wg of nwg
// walks a contiguous run of items.
AJ_DEV int xcd_item(int wg, int nwg) {
  const int per = nwg / kXcds, rem = nwg % kXcds;
  const int xcd = wg % kXcds, idx = wg / kXcds;
  return xcd * per + (xcd < rem ? xcd : rem) + idx;
}
// Tile number t of the walk.
AJ_DEV TileIdx tile_at(int t, int tiles_m, int tiles_n) {
  // a skinny product runs whole tile rows (or columns) side by side, so that
  // each operand tile is fetched once for all the tiles that share it
  if (tiles_n <= 16) return {t / tiles_n, t % tiles_n};
  if (tiles_m <= 16) return {t % tiles_m, t / tiles_m};
  const int span = kGroupM * tiles_n;
  const int first_m = (t / span) * kGroupM;
  const int gm = min(tiles_m - first_m, kGroupM);
  const int r = t % span;
  return {first_m + r % gm, r / gm};
}
AJ_DEV TileIdx tile_of(int wg, int nwg, int tiles_m, int tiles_n) {
  return tile_at(xcd_item(wg, nwg), tiles_m, tiles_n);
}

template <int BM_, int BN_, int WM_, int WN_>
struct MfmaCfg {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int NW = WM * WN, NT = NW * 64;
  static constexpr int WTM = BM / WM, WTN = BN / WN;   // a wave's block
  static constexpr int TM = WTM / 16, TN = WTN / 16;   // its MFMA tiles
  static_assert(WTM % 32 == 0 && WTN % 16 == 0, "tile shape");
};
// 8 waves as 2 x 4, each 128 rows x 64 columns.
using Cfg8 = MfmaCfg<256, 256, 2, 4>;
// The LM-head kernels: 8 waves as 4 x 2, each 64 rows x 128 columns, so that a
// row's 256 columns sit in few lanes for the per-row epilogue reductions.
using CfgWide = MfmaCfg<256, 256, 4, 2>;
// Four waves, one per SIMD, as 2 x 2, each 128x128 (256 float32 accumulators
// per lane, in AGPRs).  Against 8 waves of 128x64 this reads a third less from
// LDS per MFMA; used for long reductions, where its heavier per-tile prologue
// and epilogue are amortised.
using Cfg4 = MfmaCfg<256, 256, 2, 2>;
// A quarter of that tile, four waves of 64x64, two workgroups to a CU: products
// with too few 256x256 tiles to fill the chip.
using CfgS = MfmaCfg<128, 128, 2, 2>;

constexpr int kBK = 32;       // k-step
constexpr int kStages = 4;    // LDS stages: the copies of a k-step run four steps ahead

__device__ __attribute__((aligned(16))) const uint32_t kZero16[4] = {0, 0, 0, 0};

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>): the places of
// a k-step's reads and copies are picked at compile time, with no loop for the
// unroller to give up on.
template <typename F, int... I>
AJ_DEV void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
AJ_DEV void static_for(F &&f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

AJ_DEV uint32_t lds_addr(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}
AJ_DEV int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// One k-step of an operand of R rows (M or N) x 32 k, bfloat16, in LDS, filled
// by asynchronous direct-to-LDS global loads: a wave instruction moves a block
// of 64 x 16 bytes, lane l's 16 bytes landing at block + 16*l, so the layout
// inside a block is chosen through each lane's global address.  Both layouts
// spread the 16 lanes l..l+15 of a fragment read over all 64 banks, with
// addresses that differ between the wave's fragments by a constant only.  The
// counters see no conflict on M/N-major operands; K-major ones still conflict,
// a third of the cycles the LDS is busy in a product with one of each:
//   K-major operand (rows r, k contiguous): [R][32], 16 rows a block, the
//     16-byte chunk c of row r at r*64 + 16*(c ^ ((r >> 2) & 3))  (ds_read_b128)
//   M/N-major operand (k rows, r contiguous): whole k rows, 512 / R of them a
//     block, blocks 32 bytes more than 1 KB apart.  A ds_read_b64_tr_b16 pass
//     covers 32 bytes of the 8 rows k0 + {0..3, 8..11}, which sit in 8
//     consecutive blocks: row k is in block (k & 3) + 4 ((k >> 3) & 1) (+ 8
//     ((k >> 2) & 1) for R = 256), as its row k >> 4 (for R = 128 its row
//     ((k >> 2) & 1) + 2 (k >> 4)).
// Rows past the operand's end read row `rows - 1` (their products land in
// output rows / columns that are never stored); k past K reads zeros.
template <bool KMAJOR, int R, int NW>
struct Tile {
  static_assert(R == 128 || R == 256, "block layout");
  static constexpr int kBlocks = R / 16;
  static constexpr int kBlock = KMAJOR ? 512 : 528;    // bf16 elements from block to block
  static constexpr int kHalfs = kBlocks * kBlock;      // and per stage
  static constexpr int kInstr = kBlocks / NW;          // copies per wave and k-step
  static constexpr int CH = R / 8;                     // 16-byte chunks per M/N-major k row

  AJ_DEV static int swz_k(int r) { return (r >> 2) & 3; }
  // k row of lane l's chunk of M/N-major block blk
  AJ_DEV static int row_n(int blk, int lane) {
    const int sub = lane / CH, low = (blk & 3) + 8 * ((blk >> 2) & 1);
    return R == 256 ? low + 4 * (blk >> 3) + 16 * sub : low + 4 * (sub & 1) + 16 * (sub >> 1);
  }

  // bounded copy of the k-step at k0
  AJ_DEV static void load(uint16_t *lds, const bf16_t *X, int64_t ld, int r0, int rows, int k0,
                          int K) {
    const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
    for (int q = 0; q < kInstr; ++q) {
      const int blk = wave * kInstr + q;               // 1 KB block of the stage
      const void *src;
      if (KMAJOR) {
        const int r = blk * 16 + (lane >> 2);
        const int k = k0 + 8 * ((lane & 3) ^ swz_k(r));
        const int rr = min(r0 + r, rows - 1);
        src = k < K ? (const void *)(X + (int64_t)rr * ld + k) : (const void *)kZero16;
      } else {
        const int k = k0 + row_n(blk, lane);
        const int rr = min(r0 + 8 * (lane % CH), rows - 8);
        src = k < K ? (const void *)(X + (int64_t)k * ld + rr) : (const void *)kZero16;
      }
      __builtin_amdgcn_global_load_lds(
          src, (__attribute__((address_space(3))) void *)(lds + blk * kBlock), 16, 0, 0);
    }
  }
};

// Copies of whole k-steps: a 32-bit loop-invariant offset per lane and copy, the
// step's address in scalar registers (a buffer resource), so that a copy costs
// no vector instruction beside itself and one register instead of two.
template <bool KMAJOR, int R, int NW>
struct Copier {
  using T = Tile<KMAJOR, R, NW>;
  uint32_t off[T::kInstr];
  int lds_off;              // of the wave's first block, bf16 elements
  int64_t step;

  AJ_DEV void init(int64_t ld, int r0, int rows) {
    const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
    for (int q = 0; q < T::kInstr; ++q) {
      const int blk = wave * T::kInstr + q;
      if (KMAJOR) {
        const int r = blk * 16 + (lane >> 2);
        const int rr = min(r0 + r, rows - 1) - r0;
        off[q] = (uint32_t)(((int64_t)rr * ld + 8 * ((lane & 3) ^ T::swz_k(r))) * 2);
      } else {
        const int rr = min(r0 + 8 * (lane % T::CH), rows - 8) - r0;
        off[q] = (uint32_t)(((int64_t)T::row_n(blk, lane) * ld + rr) * 2);
      }
    }
    lds_off = wave * T::kInstr * T::kBlock;
    step = KMAJOR ? kBK : kBK * ld;
  }
  AJ_DEV void issue_one(int q, uint16_t *lds, const bf16_t *tile) const {
    // raw buffer from `tile` on, 4 GB of range: every offset is inside the operand
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(tile), 0, -1, 0x00027000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rsrc, (__attribute__((address_space(3))) void *)(lds + lds_off + q * T::kBlock), 16,
        off[q], 0, 0, 0);
  }
};

// Fragment reads of N 16-row MFMA operands from a wave's first row on: lane l
// gets row l%16 and k = 8*(l/16) + 0..7.  One per-lane address serves them all;
// the stage and the fragment are immediates.  The
// reads are inline assembly: the compiler cannot tell them apart from the LDS
// writes of the in-flight direct-to-LDS copies and would otherwise wait for
// those copies before every read; the caller waits for the reads itself.
template <bool KMAJOR, int R, int N>
struct Frags {
  using T = Tile<KMAJOR, R, 4>;
  static constexpr int kStage = T::kHalfs * 2;         // bytes
  // from a lane's k rows k0..k0+3 to k0+4..k0+7
  static constexpr int kHigh = R == 256 ? 8 * T::kBlock * 2 : 256;
  static_assert(kStages * kStage <= 69632, "stage offsets are 16-bit immediates");
  uint32_t addr;

  AJ_DEV void init(const uint16_t *lds, int rb) {
    const int lane = threadIdx.x & 63, g = lane >> 4, s = lane & 15;
    const uint32_t base = lds_addr(lds);
    if (KMAJOR) {
      const int m = rb + s;
      addr = base + m * 64 + 16 * (g ^ T::swz_k(m));
    } else {
      // ds_read_b64_tr_b16: in each 16-lane group, lane j receives element j%4
      // of the 4-element run addressed by lane 4e + j/4 (e = 0..3).  Source
      // lane s points at k row k0 + s/4, rows mb + 4*(s%4)..+3, so lane j
      // receives row mb + j at k0..k0+3 (k0 = 8 g); a second read gives
      // k0+4..k0+7.
      const int blk = (s >> 2) + 4 * (g & 1), sub = R == 256 ? g >> 1 : 2 * (g >> 1);
      addr = base + (blk * T::kBlock + sub * R + rb + 4 * (s & 3)) * 2;
    }
  }
  template <int I, int ST>
  AJ_DEV bf16x8_t read() const {
    if constexpr (KMAJOR) {
      bf16x8_t v;
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr),
                   "n"(ST * kStage + I * 1024) : "memory");
      return v;
    } else {
      u32x2_t lo, hi;
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr),
                   "n"(ST * kStage + I * 32) : "memory");
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr),
                   "n"(ST * kStage + I * 32 + kHigh) : "memory");
      return __builtin_bit_cast(bf16x8_t, u32x4_t{lo[0], lo[1], hi[0], hi[1]});
    }
  }
};

// kStages of a k-step of both operands (256x256 tiles: 32 KB each, 128 KB).
template <typename C, bool A_K, bool B_K>
struct Smem {
  uint16_t a[kStages][Tile<A_K, C::BM, C::NW>::kHalfs];
  uint16_t b[kStages][Tile<B_K, C::BN, C::NW>::kHalfs];
};

// A workgroup barrier without the memory fence of __syncthreads: that fence
// waits for every outstanding vector-memory operation, the direct-to-LDS
// copies still meant to fly included.  Visibility of the copies and reads that
// must be complete is ensured by explicit vmcnt / lgkmcnt waits before it; the
// empty asm statements keep the compiler from moving memory operations across.
AJ_DEV void bar_nofence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Waits until at most n k-steps' copies (PER per wave each, n <= 3) are
// still in flight.
template <int PER>
AJ_DEV void wait_steps(int n) {
  static_assert(PER == 4 || PER == 8, "copies per wave and k-step");
  switch (n * PER) {
    case 24: __asm__ volatile("s_waitcnt vmcnt(24)" ::: "memory"); break;
    case 16: __asm__ volatile("s_waitcnt vmcnt(16)" ::: "memory"); break;
    case 12: __asm__ volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
    case 8: __asm__ volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
    case 4: __asm__ volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
    default: __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
  }
}

// Waits for every LDS read in flight; the fragments pass through empty
// statements after the wait so that no MFMA consuming them is scheduled
// above it.
template <int TM, int TN>
AJ_DEV void frag_wait(bf16x8_t (&a)[TM], bf16x8_t (&b)[TN]) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(a[i]));
#pragma unroll
  for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(b[j]));
}

// One k-step.  On entry the step's fragments (fa, fb) are in registers and, by
// the barrier that the caller has passed, the next step's stage holds its data
// for every wave and this step's stage has been read by every wave.  So the
// step's products run beside the copies of the step kStages ahead (into this
// step's stage) and the reads of the next step's fragments (na, nb), both at
// fixed places between the MFMAs; the reads end three quarters through and are
// waited for after the last MFMA, so no wave carries a read into the next step.
// The MFMA takes (b, a): a lane then holds four consecutive columns of one row.
template <typename C, bool A_K, bool B_K, int ST, bool kCopy, bool kRead = true>
AJ_DEV void kstep(f32x4_t (&acc)[C::TM][C::TN], const bf16x8_t (&fa)[C::TM],
                  const bf16x8_t (&fb)[C::TN], bf16x8_t (&na)[C::TM], bf16x8_t (&nb)[C::TN],
                  const Frags<A_K, C::BM, C::TM> &ra, const Frags<B_K, C::BN, C::TN> &rb,
                  const Copier<A_K, C::BM, C::NW> &ca, const Copier<B_K, C::BN, C::NW> &cb,
                  Smem<C, A_K, B_K> &sm, const bf16_t *ta, const bf16_t *tb) {
  constexpr int NM = C::TM * C::TN, NR = C::TM + C::TN;
  constexpr int kA = Tile<A_K, C::BM, C::NW>::kInstr, kB = Tile<B_K, C::BN, C::NW>::kInstr;
  constexpr int SP = NM / (2 * (kA + kB)), NX = (ST + 1) % kStages;
  static_assert(SP >= 1, "copies fit the first half of the step");
  static_for<NM>([&](auto tc) __attribute__((always_inline)) {
    constexpr int t = decltype(tc)::value, i = t / C::TN, j = t % C::TN;
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kCopy && t % SP == SP - 1 && t / SP < kA + kB) {
      constexpr int q = t / SP;
      if constexpr (q < kA) ca.issue_one(q, sm.a[ST], ta);
      else cb.issue_one(q - kA, sm.b[ST], tb);
    }
    // reads [q0, q1) of the next step's fragments: B's first
    constexpr int q0 = (t * 4 * NR + 3 * NM - 1) / (3 * NM), q1 = ((t + 1) * 4 * NR + 3 * NM - 1) / (3 * NM);
    static_for<(kRead && q0 < NR ? (q1 < NR ? q1 : NR) - q0 : 0)>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = q0 + decltype(qc)::value;
      if constexpr (q < C::TN) nb[q] = rb.template read<q, NX>();
      else na[q - C::TN] = ra.template read<q - C::TN, NX>();
    });
    __builtin_amdgcn_sched_barrier(0);
  });
  if constexpr (kRead) frag_wait(na, nb);
}

// A reduction segment: operands and the range [kbeg, kend) of k.
struct Seg {
  const bf16_t *A; int64_t lda;
  const bf16_t *B; int64_t ldb;
  int kbeg, kend;
};

// acc[i][j] (lane's share of the wave's block) = sum over k of A(m, k) B(n, k)
// for the tile at (m0, n0), over segment s1 and, with SEG2, s2.  The steps run
// in this order: zero steps that make their number a multiple of kStages, s2's,
// s1's ragged one, s1's full ones.  All but the full ones come first, in the
// prologue's copies, so that the loop copies full steps only and ends without a
// remainder (a branch per step there costs the accumulators their registers).
template <typename C, bool A_K, bool B_K, bool SEG2 = false>
AJ_DEV void mainloop(f32x4_t (&acc)[C::TM][C::TN], const Seg &s1, int M, int N, int m0, int n0,
                     Smem<C, A_K, B_K> &sm, const Seg &s2 = Seg{}) {
  // device code only: this compiler's host pass rejects some instances of kstep
#if defined(__HIP_DEVICE_COMPILE__)
  using TA = Tile<A_K, C::BM, C::NW>;
  using TB = Tile<B_K, C::BN, C::NW>;
  using CA = Copier<A_K, C::BM, C::NW>;
  using CB = Copier<B_K, C::BN, C::NW>;
  constexpr int PER = TA::kInstr + TB::kInstr;
  const int len1 = s1.kend > s1.kbeg ? s1.kend - s1.kbeg : 0;
  const int nfull = len1 / kBK, ragged = len1 % kBK ? 1 : 0;
  const int n2 = SEG2 && s2.kend > s2.kbeg ? (s2.kend - s2.kbeg + kBK - 1) / kBK : 0;
  const int nk = (nfull + ragged + n2 + kStages - 1) / kStages * kStages;
  const int front = nk - nfull;                 // steps before the first full one
  const int wave = wave_id();
  const int wm = wave / C::WN, wn = wave % C::WN;
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  if (nk == 0) return;
  CA ca;
  CB cb;
  ca.init(s1.lda, m0, M);
  cb.init(s1.ldb, n0, N);
  Frags<A_K, C::BM, C::TM> ra;
  Frags<B_K, C::BN, C::TN> rb;
  ra.init(sm.a[0], wm * C::WTM);
  rb.init(sm.b[0], wn * C::WTN);
  // the tiles of k-step `front` (the first full one), less `front` steps
  const bf16_t *ta = s1.A + (A_K ? (int64_t)m0 * s1.lda + s1.kbeg : (int64_t)s1.kbeg * s1.lda + m0) -
                     front * ca.step;
  const bf16_t *tb = s1.B + (B_K ? (int64_t)n0 * s1.ldb + s1.kbeg : (int64_t)s1.kbeg * s1.ldb + n0) -
                     front * cb.step;
  // all copies of k-step kt (< nk) into stage st
  auto copy_step = [&](int kt, int st) {
    if (kt >= front) {
#pragma unroll
      for (int q = 0; q < TA::kInstr; ++q) ca.issue_one(q, sm.a[st], ta + kt * ca.step);
#pragma unroll
      for (int q = 0; q < TB::kInstr; ++q) cb.issue_one(q, sm.b[st], tb + kt * cb.step);
      return;
    }
    // bounded: a step that starts at or past its segment's end reads zeros
    const int k2 = kt - (front - ragged - n2);
    const bool seg2 = SEG2 && k2 >= 0 && k2 < n2;
    const Seg &s = seg2 ? s2 : s1;
    const int k0 = seg2 ? s.kbeg + k2 * kBK : k2 < 0 ? s.kend : s.kbeg + nfull * kBK;
    TA::load(sm.a[st], s.A, s.lda, m0, M, k0, s.kend);
    TB::load(sm.b[st], s.B, s.ldb, n0, N, k0, s.kend);
  };
  bf16x8_t f0a[C::TM], f0b[C::TN], f1a[C::TM], f1b[C::TN];
#pragma unroll
  for (int st = 0; st < kStages; ++st) copy_step(st, st);
  wait_steps<PER>(kStages - 1);
  bar_nofence();
  static_for<C::TN>([&](auto q) { f0b[q] = rb.template read<decltype(q)::value, 0>(); });
  static_for<C::TM>([&](auto q) { f0a[q] = ra.template read<decltype(q)::value, 0>(); });
  frag_wait(f0a, f0b);
  // Four steps a turn, so that every stage is a constant.  Before a step the
  // next one's copies have landed (those of the two after it may fly).
  int kt = 0;
  if constexpr (SEG2)   // more than four front steps: the bounded copies, before the products
    for (; kt + kStages < front; kt += kStages) {
#define AJ_STEP(U, FA, FB, NA, NB)                                                            \
  wait_steps<PER>(2);                                                                         \
  bar_nofence();                                                                              \
  copy_step(kt + U + kStages, U);                                                             \
  kstep<C, A_K, B_K, U, false>(acc, FA, FB, NA, NB, ra, rb, ca, cb, sm, nullptr, nullptr);
      AJ_STEP(0, f0a, f0b, f1a, f1b)
      AJ_STEP(1, f1a, f1b, f0a, f0b)
      AJ_STEP(2, f0a, f0b, f1a, f1b)
      AJ_STEP(3, f1a, f1b, f0a, f0b)
#undef AJ_STEP
    }
  for (; kt + kStages < nk; kt += kStages) {
#define AJ_STEP(U, FA, FB, NA, NB)                                                            \
  wait_steps<PER>(2);                                                                         \
  bar_nofence();                                                                              \
  kstep<C, A_K, B_K, U, true>(acc, FA, FB, NA, NB, ra, rb, ca, cb, sm,                        \
                              ta + (kt + U + kStages) * ca.step,                              \
                              tb + (kt + U + kStages) * cb.step);
    AJ_STEP(0, f0a, f0b, f1a, f1b)
    AJ_STEP(1, f1a, f1b, f0a, f0b)
    AJ_STEP(2, f0a, f0b, f1a, f1b)
    AJ_STEP(3, f1a, f1b, f0a, f0b)
#undef AJ_STEP
  }
#define AJ_STEP(U, FA, FB, NA, NB, LEFT, READ)                                                \
  wait_steps<PER>(LEFT);                                                                      \
  bar_nofence();                                                                              \
  kstep<C, A_K, B_K, U, false, READ>(acc, FA, FB, NA, NB, ra, rb, ca, cb, sm, nullptr, nullptr);
  AJ_STEP(0, f0a, f0b, f1a, f1b, 2, true)
  AJ_STEP(1, f1a, f1b, f0a, f0b, 1, true)
  AJ_STEP(2, f0a, f0b, f1a, f1b, 0, true)
  AJ_STEP(3, f1a, f1b, f0a, f0b, 0, false)
#undef AJ_STEP
#endif
}

// Row / first column of accumulator tile (i, j) for this lane: the lane holds
// row lane%16 and columns 4*(lane/16) + 0..3 of each 16x16 tile.
template <typename C>
AJ_DEV int acc_row(int wm, int i, int lane) { return wm * C::WTM + i * 16 + (lane & 15); }
template <typename C>
AJ_DEV int acc_col(int wn, int j, int lane) { return wn * C::WTN + j * 16 + 4 * (lane >> 4); }

}  // namespace gemm_core
}  // namespace aj
