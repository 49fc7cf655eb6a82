// Host-only check of the scratch of split reductions against the plans that gemm()
// follows, through the library's own workspace carving: for the block, adapter and
// LM-head products of every workload, in both data types and at packs up to the
// workload's capacity,
//   - the sums of every piece a plan asks for fit the scratch the call passes,
//   - a plan's ranges cover its reduction,
//   - float32 scratch is no limit on its plans, and no more than their largest,
//   - every workspace grows with the pack, so that one sized for the largest pack
//     serves the smaller ones.
// Built with the library sources included (host compilation only; nothing is
// launched).  Exit status 1 on a violation.
#include <cstdio>
#include <algorithm>
#include <array>
#include "loss.hip"
// the two sources each define these helpers in their own unnamed namespace
#define check_cfg block_check_cfg
#define carve_saved block_carve_saved
#include "block.hip"
#undef check_cfg
#undef carve_saved
using namespace aj;
static int bad = 0;
static size_t seen[2];   // the most floats of scratch a plan used, by float32
static const char *at;

static void fail_at(const char *what, int64_t M, int64_t N, int64_t K, size_t need, size_t cap) {
  if (++bad < 20) printf("%s: %s %ldx%ld K=%ld needs %zu of %zu\n", at, what, (long)M, (long)N, (long)K, need, cap);
}

static void product(bool f32, int64_t M, int64_t N, int64_t K, size_t cap, bool eight, bool free_cap) {
  size_t need = 0;
  if (f32) {
    const int S = gemm_f32_pieces((int)M, (int)N, (int)K, cap);
    need = S > 1 ? (size_t)S * ((M + 63) / 64) * ((N + 63) / 64) * 4096 : 0;
    if (free_cap && S != gemm_f32_pieces((int)M, (int)N, (int)K, (size_t)1 << 40))
      fail_at("scratch limits the pieces of", M, N, K, need, cap);
  } else {
    const GemmPlan p = gemm_plan((int)M, (int)N, (int)K, cap, eight);
    need = p.whole < p.tiles ? (size_t)(p.tiles - p.whole) * p.split * p.tile * p.tile : 0;
    if (p.whole < p.tiles && (int64_t)p.split * p.k_piece < K) fail_at("ranges of", M, N, K, need, cap);
    if (p.whole == p.tiles && p.split != 1) fail_at("pieces of no tile of", M, N, K, need, cap);
  }
  if (need > cap) fail_at("sums of", M, N, K, need, cap);
  seen[f32] = std::max(seen[f32], need);
}

int main() {
  struct C { const char *name; int d, Hq, Hkv, hd, F, V, chunk, cap; } cs[] = {
    {"tiny", 128, 4, 4, 32, 512, 1024, 1024, 131072},
    {"1.5b", 1536, 12, 2, 128, 8960, 151936, 32768, 131072},
    {"7b", 3584, 28, 4, 128, 18944, 152064, 32768, 131072},
    {"7b-8192", 3584, 28, 4, 128, 18944, 152064, 8192, 131072},
    {"32b", 5120, 40, 8, 128, 27648, 152064, 8192, 131072},
    {"32b-32768", 5120, 40, 8, 128, 27648, 152064, 32768, 131072},
  };
  for (auto &c : cs)
    for (int f32 = 0; f32 < 2; ++f32) {
      aj_block_cfg b{};
      b.d_model = c.d; b.n_q_heads = c.Hq; b.n_kv_heads = c.Hkv; b.head_dim = c.hd; b.d_ff = c.F;
      b.dtype = f32 ? AJ_F32 : AJ_BF16;
      aj_loss_cfg l{};
      l.d_model = c.d; l.vocab = c.V; l.vocab_chunk = c.chunk; l.dtype = b.dtype;
      const int q = (c.Hq + 2 * c.Hkv) * c.hd, hq = c.Hq * c.hd, d = c.d, F = c.F;
      const int64_t gw = group_width(l), glast = c.V % gw ? c.V % gw : gw;
      at = c.name;
      size_t last[5] = {};
      for (int n = 1; n <= c.cap; n += n < 20000 ? 61 : 1021) {
        const BwdWs w = carve_bwd(b, n, nullptr);
        const Saved s = block_carve_saved(b, n, nullptr);
        const LossWs lw = carve_ws(l, n, nullptr);
        const size_t bytes[5] = {w.bytes, s.bytes, lw.bytes, carve_lora_bwd(b, 32, n, nullptr, nullptr),
                                 carve_lora_bwd(b, 256, n, nullptr, nullptr)};
        for (int i = 0; i < 5; ++i) {
          if (bytes[i] < last[i]) fail_at("smaller workspace", n, i, 0, bytes[i], last[i]);
          last[i] = bytes[i];
        }
        const size_t cap = w.splitk_floats;
        for (auto &p : {std::array<int, 2>{d, F}, {2 * F, d}, {d, hq}, {q, d}}) product(f32, p[0], p[1], n, cap, false, true);
        for (bool eight : {false, true}) {   // without and with adapters
          product(f32, n, F, d, cap, true, true);
          product(f32, n, d, 2 * F, cap, eight, true);
          product(f32, n, hq, d, cap, eight, true);
          product(f32, n, d, q, cap, eight, true);
          product(f32, n, q, d, s.part_floats, eight, false);
          product(f32, n, d, hq, s.part_floats, eight, false);
          product(f32, n, 2 * F, d, s.part_floats, eight, false);
          product(f32, n, d, F, s.part_floats, eight, false);
        }
        for (int r : {8, 32, 256}) {
          LoraBwd lb;
          carve_lora_bwd(b, r, n, nullptr, &lb);
          for (int p = 0; p < 4; ++p) {
            const int o = proj_out(b, p), i = proj_in(b, p);
            product(f32, o, r, n, lb.partial_floats, false, true);
            product(f32, n, r, o, lb.partial_floats, false, true);
            product(f32, r, i, n, lb.partial_floats, false, true);
            product(f32, n, r, i, s.part_floats, false, false);
          }
        }
        for (int64_t g : {gw, glast}) {
          product(f32, n, d, g, lw.splitk_floats, false, true);
          product(f32, g, d, n, lw.splitk_floats, false, true);
        }
        if (f32) {
          const size_t most = (size_t)1024 * 4096;
          if (std::max({cap, s.part_floats, lw.splitk_floats}) > most)
            fail_at("float32 scratch", n, 0, 0, most, std::max({cap, s.part_floats, lw.splitk_floats}));
        }
      }
      const BwdWs w = carve_bwd(b, c.cap, nullptr);
      printf("%-10s %s block %zu floats, forward %zu, LM head %zu; plans used up to %zu\n", c.name,
             f32 ? "f32 " : "bf16", w.splitk_floats, block_carve_saved(b, c.cap, nullptr).part_floats,
             carve_ws(l, c.cap, nullptr).splitk_floats, seen[f32]);
    }
  printf("violations: %d\n", bad);
  return bad != 0;
}
