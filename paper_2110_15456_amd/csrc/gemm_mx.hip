// gemm_mx.hip -- dispatch of the BFP GEMM (kernel in gemm_mx.h) over the
// group size and the operand formats: chunk planes read per operand (1 or 2)
// and whether the first plane holds FP4 codes.  Each group size and
// plane-count pair is instantiated in its own file
// (gemm_mx_{11,12,21,22}[_g32].hip) so that they compile in parallel.
#include "gemm_direct.h"
#include "gemm_mx.h"

namespace fastbfp {

FASTBFP_MX_DECLARE(1, 1, 0, 0, 16)
FASTBFP_MX_DECLARE(1, 1, 0, 1, 16)
FASTBFP_MX_DECLARE(1, 1, 1, 0, 16)
FASTBFP_MX_DECLARE(1, 1, 1, 1, 16)
FASTBFP_MX_DECLARE(1, 2, 0, 0, 16)
FASTBFP_MX_DECLARE(1, 2, 0, 1, 16)
FASTBFP_MX_DECLARE(1, 2, 1, 0, 16)
FASTBFP_MX_DECLARE(1, 2, 1, 1, 16)
FASTBFP_MX_DECLARE(2, 1, 0, 0, 16)
FASTBFP_MX_DECLARE(2, 1, 0, 1, 16)
FASTBFP_MX_DECLARE(2, 1, 1, 0, 16)
FASTBFP_MX_DECLARE(2, 1, 1, 1, 16)
FASTBFP_MX_DECLARE(2, 2, 0, 0, 16)
FASTBFP_MX_DECLARE(2, 2, 0, 1, 16)
FASTBFP_MX_DECLARE(2, 2, 1, 0, 16)
FASTBFP_MX_DECLARE(2, 2, 1, 1, 16)
FASTBFP_MX_DECLARE(1, 1, 0, 0, 32)
FASTBFP_MX_DECLARE(1, 1, 0, 1, 32)
FASTBFP_MX_DECLARE(1, 1, 1, 0, 32)
FASTBFP_MX_DECLARE(1, 1, 1, 1, 32)
FASTBFP_MX_DECLARE(1, 2, 0, 0, 32)
FASTBFP_MX_DECLARE(1, 2, 0, 1, 32)
FASTBFP_MX_DECLARE(1, 2, 1, 0, 32)
FASTBFP_MX_DECLARE(1, 2, 1, 1, 32)
FASTBFP_MX_DECLARE(2, 1, 0, 0, 32)
FASTBFP_MX_DECLARE(2, 1, 0, 1, 32)
FASTBFP_MX_DECLARE(2, 1, 1, 0, 32)
FASTBFP_MX_DECLARE(2, 1, 1, 1, 32)
FASTBFP_MX_DECLARE(2, 2, 0, 0, 32)
FASTBFP_MX_DECLARE(2, 2, 0, 1, 32)
FASTBFP_MX_DECLARE(2, 2, 1, 0, 32)
FASTBFP_MX_DECLARE(2, 2, 1, 1, 32)

#define FASTBFP_MX11_TILES_DECLARE(FA, FB)      \
  FASTBFP_MX11_TILE_DECLARE(256, 128, FA, FB)   \
  FASTBFP_MX11_TILE_DECLARE(256, 64, FA, FB)    \
  FASTBFP_MX11_TILE_DECLARE(128, 64, FA, FB)    \
  FASTBFP_MX11_TILE_DECLARE(128, 128, FA, FB)
FASTBFP_MX11_TILES_DECLARE(0, 0)
FASTBFP_MX11_TILES_DECLARE(0, 1)
FASTBFP_MX11_TILES_DECLARE(1, 0)
FASTBFP_MX11_TILES_DECLARE(1, 1)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_DECLARE, 1, 1, 16)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_DECLARE, 1, 2, 16)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_DECLARE, 2, 1, 16)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_DECLARE, 2, 2, 16)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_DECLARE, 1, 1, 32)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_DECLARE, 1, 2, 32)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_DECLARE, 2, 1, 32)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_DECLARE, 2, 2, 32)

// Tile of the one-chunk, groups-of-16, FP32-output GEMM (0..4: 256x256,
// 256x128, 256x64, 128x64, 128x128), from measurements on MI355X over the
// transformer, FFN-step and ResNet-18 im2col shapes (every tile forced, us):
//  * N <= 64: 128x64, a wider tile is mostly padding (802816 x 64 x 576 (2,2) 91
//    against 109-292 on the others, (4,4) 155 against 181-325; only (4,2) has
//    256x64 ahead, 144 against 148);
//  * A in FP4 codes: 256x128, whose two LDS stages take 60-76 KB, so that two
//    workgroups share a CU: 1-10% faster than 256x256 on 8192 x 4096, 12288 and
//    16384 x 4096 (457 against 506 on the last, (2,2)), 1-3% slower on 8192 x 4096
//    x 16384;
//  * A in FP6 codes: 256x256 (a 256x128 tile still takes 92-108 KB of LDS, one
//    workgroup per CU, and is 27-45% slower; 128x128, two per CU, 16-48%
//    slower), but 128x128 for N <= 128 or when 256x256 tiles are too few;
//  * too few: fewer than 192 tiles leave over a quarter of the 256 CUs idle;
//    then the next smaller tile, down to 128x64.
// With C converted to BFP in the epilogue (converted), A in FP4 codes gets
// the FP6 rule.  That line was drawn when a slab began with a barrier and the
// reads waited for (8192 x 16384 x 4096 (2,2) to m = 2: 600-630 us on 256x256, 710
// on 256x128).  With the pipeline through the slab barriers it is 510 against
// 440-475, 50176 x 256 x 2304 47 against 39, 8192 x 4096 x 16384 392 against 383,
// and 12544 x 512 x 4608, which has the 128x128 tile here, 41 against 45.
static int gemm_mx11_tile(int64_t M, int64_t N, int fa, bool converted) {
  constexpr int64_t MIN_TILES = 192;
  auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  if (N <= 64) return 3;
  if (fa && !converted) return tiles(256, 128) >= MIN_TILES ? 1 : 3;
  if (N > 128 && tiles(256, 256) >= MIN_TILES) return 0;
  return tiles(128, 128) >= MIN_TILES ? 4 : 3;
}

namespace {

// A product's operands as the kernels see them.
struct Product {
  const uint8_t *a_mant, *a_exp;
  int64_t a_ps;  // byte offset of A's plane 1 (its stored plane 0's size)
  const uint8_t *b_mant, *b_exp;
  int64_t b_ps;
  int M, N, ng;  // ng: 16-value halves per row (K / 16, the plane layout's unit)
  int na, nb;    // planes read
  int fa, fb;    // one plane read: it holds FP4 codes; two: split at 2 bits
  float scale;
};

// Where C goes: FP32 rows, BFP in the epilogue (qo), or the partial sums of a
// product whose K is taken in parts.
struct Output {
  float* C;
  int64_t ldc;
  const OutBFP* qo;
  int part_slabs;  // 0: all of K
  hipStream_t s;
};

template <int BM, int BN>
hipError_t launch_tile(const Product& p, const Output& o) {
#define FASTBFP_TILE(FA, FB)                                                                                         \
  return launch_mx_11_tile<BM, BN, FA, FB>(p.a_mant, p.a_exp, p.b_mant, p.b_exp, p.M, p.N, p.ng, p.scale, o.C, o.ldc, \
                                           o.qo, o.part_slabs, o.s)
  if (!p.fa && !p.fb) FASTBFP_TILE(0, 0);
  if (!p.fa) FASTBFP_TILE(0, 1);
  if (!p.fb) FASTBFP_TILE(1, 0);
  FASTBFP_TILE(1, 1);
#undef FASTBFP_TILE
}

template <int NA, int NB, int G>
hipError_t launch_fmt(const Product& p, const Output& o) {
#define FASTBFP_FMT(FA, FB)                                                                                      \
  return launch_mx_t<NA, NB, FA, FB, G>(p.a_mant, p.a_exp, p.a_ps, p.b_mant, p.b_exp, p.b_ps, p.M, p.N, p.ng,    \
                                        p.scale, o.C, o.ldc, o.qo, o.part_slabs, o.s)
  if (!p.fa && !p.fb) FASTBFP_FMT(0, 0);
  if (!p.fa) FASTBFP_FMT(0, 1);
  if (!p.fb) FASTBFP_FMT(1, 0);
  FASTBFP_FMT(1, 1);
#undef FASTBFP_FMT
}

// tile: 0 the operand formats' default, 1..4 the smaller ones (one plane per
// operand and groups of 16).
template <int G>
hipError_t launch_tiled(const Product& p, const Output& o, int tile) {
  if (tile == 1) return launch_tile<256, 128>(p, o);
  if (tile == 2) return launch_tile<256, 64>(p, o);
  if (tile == 3) return launch_tile<128, 64>(p, o);
  if (tile == 4) return launch_tile<128, 128>(p, o);
  if (p.na == 1 && p.nb == 1) return launch_fmt<1, 1, G>(p, o);
  if (p.na == 1 && p.nb == 2) return launch_fmt<1, 2, G>(p, o);
  if (p.na == 2 && p.nb == 1) return launch_fmt<2, 1, G>(p, o);
  return launch_fmt<2, 2, G>(p, o);
}

template <int NA, int NB, int G>
hipError_t launch_direct_fmt(const Product& p, const GemmPlan& plan, float* C, int64_t ldc, const direct::Out* out,
                             hipStream_t s) {
#define FASTBFP_DIRECT(FA, FB)                                                                                    \
  return launch_direct_t<NA, NB, FA, FB, G>(plan.rm, plan.rn, p.a_mant, p.a_exp, p.a_ps, p.b_mant, p.b_exp, p.b_ps, \
                                            p.M, p.N, p.ng, p.scale, C, ldc, out, s)
  if (!p.fa && !p.fb) FASTBFP_DIRECT(0, 0);
  if (!p.fa) FASTBFP_DIRECT(0, 1);
  if (!p.fb) FASTBFP_DIRECT(1, 0);
  FASTBFP_DIRECT(1, 1);
#undef FASTBFP_DIRECT
}

template <int G>
hipError_t launch_direct(const Product& p, const GemmPlan& plan, float* C, int64_t ldc, const direct::Out* out,
                         hipStream_t s) {
  if (p.na == 1 && p.nb == 1) return launch_direct_fmt<1, 1, G>(p, plan, C, ldc, out, s);
  if (p.na == 1 && p.nb == 2) return launch_direct_fmt<1, 2, G>(p, plan, C, ldc, out, s);
  if (p.na == 2 && p.nb == 1) return launch_direct_fmt<2, 1, G>(p, plan, C, ldc, out, s);
  return launch_direct_fmt<2, 2, G>(p, plan, C, ldc, out, s);
}

int fmt_flag(int m, int planes) { return planes == 1 ? plane0_fp4(m) : m <= 6; }

Product make_product(const uint8_t* a_mant, const uint8_t* a_exp, int a_m, int na, const uint8_t* b_mant,
                     const uint8_t* b_exp, int b_m, int nb, int64_t M, int64_t N, int64_t K, int g, int scale_log2) {
  return Product{a_mant, a_exp, M * (K / g) * plane_group_bytes(g, a_m, 0), b_mant, b_exp,
                 N * (K / g) * plane_group_bytes(g, b_m, 0), (int)M, (int)N, (int)(K / 16), na, nb, fmt_flag(a_m, na),
                 fmt_flag(b_m, nb), ldexpf(1.0f, scale_log2)};
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace

// The rule above, not the tile that gemm_plan found for K in parts: such a tile
// is priced on a share of K and on the workgroups of all parts.  Over all of K
// (4,4) 1024 x 4096 x 16384 takes 208 us on 64 workgroups of 256 x 256 and 139 on
// the rule's 256 of 128 x 128; 2304 x 256 x 50176 457 us on 18 of 256 x 128 and
// 278 on the rule's 72 of 128 x 64.
GemmPlan gemm_plan_whole(int a_m, int na, int nb, int64_t M, int64_t N, int g) {
  const bool one = na == 1 && nb == 1 && g == 16;
  return GemmPlan{one ? gemm_mx11_tile(M, N, fmt_flag(a_m, na), false) : 0, 0, 1, 0, 0};
}

namespace {

// The tile of a product of one-chunk operands (groups of 16) whose K is not split:
// the rule's, unless another is priced 3% below it.  In us what a workgroup takes:
// `fix` from its start to its first MFMA and out, `c` for a whole tile of C, `slab`
// for a slab; c and slab with one and with two workgroups on a CU (0: one fits),
// slab by the codes of A x B (FP6 x FP6, FP6 x FP4, FP4 x FP6, FP4 x FP4).  Slabs
// take up to kLoad more as the card fills (its L2s and the Infinity Cache serve
// every CU).  Fitted to every tile's times on 2820 products of 2^15 to 2^25 outputs
// (11-20% off, by K): the tile taken is 0.9% slower than the fastest on average, the
// rule's 2.9%.  With prices that knew only FP4 x FP4 and the rest and no start of a
// tile beyond 4 us, 27797 x 704 x 256 (2,4) took 256x256 (32 us, 256x128 25) and
// 32777 x 160 x 64 (15.8, 256x128 11.4).
int whole_tile(int64_t M, int64_t N, int64_t K, int fa, int fb, int rule) {
  struct Tile {
    int id, bm, bn;
    double fix, c[2], slab[2][4];
  };
  static const Tile kTiles[] = {{0, 256, 256, 6.67, {4.23, 0.0}, {{1.27, 1.21, 1.21, 1.14}, {0.0, 0.0, 0.0, 0.0}}},
                                {1, 256, 128, 2.97, {2.39, 6.99}, {{0.88, 0.86, 0.81, 0.77}, {0.0, 0.0, 1.03, 0.92}}},
                                {4, 128, 128, 1.23, {1.14, 3.51}, {{0.60, 0.56, 0.59, 0.48}, {0.77, 0.64, 0.67, 0.55}}},
                                {3, 128, 64, 0.41, {0.62, 1.81}, {{0.46, 0.41, 0.43, 0.35}, {0.57, 0.49, 0.47, 0.40}}}};
  constexpr double kLoad = 0.55, kRagged = 1.4, kOdd = 3.8;  // K no multiple of 128; C stored value by value
  const int fmt = 2 * fa + fb;
  const double slabs = (double)ceil_div(K / 16, mx::KG) * (K % 128 ? kRagged : 1.0);
  int best = rule;
  double best_us = 1e30;
  for (const Tile& t : kTiles) {
    const int occ = t.slab[1][fmt] > 0.0 ? 2 : 1;
    const int64_t wgs = ceil_div(M, t.bm) * ceil_div(N, t.bn), full = wgs / (256 * occ), rest = wgs % (256 * occ);
    const double used = (double)(M < t.bm ? M : t.bm) * (double)(N < t.bn ? N : t.bn) / (t.bm * t.bn) *
                        (N % 4 ? kOdd : 1.0);
    auto us = [&](int o, double load) {
      return slabs * t.slab[o][fmt] * (1.0 + kLoad * load) + t.fix + t.c[o] * used;
    };
    const double last = rest == 0 ? 0.0 : rest <= 256 ? us(0, rest / 256.0) : us(1, 1.0);
    const double sum = (2.9 + full * us(occ - 1, 1.0) + last) * (t.id == rule ? 0.97 : 1.0);
    if (sum < best_us) best_us = sum, best = t.id;
  }
  return best;
}

}  // namespace

// The plan of a product that has a workspace.  A product whose tiles fill the
// card runs as without one.  With fewer tiles, a tile's serial run of K slabs
// sets the time (dW of ResNet-18's conv2_x, 576 x 64 x 802816, has 5 tiles of
// 128 x 64 with 6272 slabs each: 3.9 ms), so the candidates below are priced
// and the cheapest is taken: every tile with K in as many parts as fill one or
// more workgroups per CU, and the few-output kernel.  Prices in us, from sweeps
// of every tile x parts and of the few-output kernel's tiles over weight
// gradients, few-token and small products on MI355X.  What the plan takes, and
// its time against bfp_gemm's (graph replays of ten calls):
//   576 x 64 x 802816 (2,2)     3949 -> 83  (128x64 in 102 parts)
//   2304 x 256 x 50176 (4,4)     264 -> 56  (256x128 in 14 parts)
//   1024 x 4096 x 16384 (4,4)    127 -> 87  (256x256 in 4 parts)
//   1024 x 1024 x 8192 (6,6)     134 -> 39  (256x128 in 8 parts)
//   16 x 16384 x 4096 (4,4)       24 -> 18  (few-output, 32 x 32)
//   1 x 4096 x 4096 (4,4)         18 -> 5.4 (few-output, 16 x 16)
//   256 x 256 x 256 (4,4)        5.2 -> 3.2 (few-output, 16 x 16)
//   2048 x 1024 x 4096 (4,4)      25 -> 25  (whole, 128x64; any split 30 or more)
GemmPlan gemm_plan(int a_m, int na, int b_m, int nb, int64_t M, int64_t N, int64_t K, int g) {
  const int fa = fmt_flag(a_m, na), fb = fmt_flag(b_m, nb);
  const bool one = na == 1 && nb == 1 && g == 16;
  GemmPlan best = gemm_plan_whole(a_m, na, nb, M, N, g);
  const int rule = best.tile;
  const int64_t slabs = ceil_div(K / 16, mx::KG);
  if (slabs == 0 || M * N > (int64_t(1) << 25)) return best;  // (at least 512 tiles of 256 x 256)

  // Tiles: rows, columns, and the time of one slab with 1 and with 2 workgroups
  // on a CU (0: they do not fit), for FP6 and for FP4 codes on both sides.
  // (Measured before the kernel's pipeline ran through the slab barriers.  With it,
  // on a full card, from K = 16384 and 49152: FP6 256x256 2.08, 256x128 1.25,
  // 128x128 1.01 and 1.34, 128x64 0.81 and 0.95; FP4 1.43, 1.02 and 1.50, 0.78
  // and 0.96, 0.58 and 0.73.)
  struct Tile {
    int id, bm, bn;
    double us[2][2];
  };
  static const Tile kTiles[] = {{0, 256, 256, {{1.8, 0.0}, {1.45, 0.0}}},
                                {1, 256, 128, {{1.2, 0.0}, {0.95, 1.35}}},
                                {4, 128, 128, {{0.95, 1.3}, {0.68, 0.92}}},
                                {3, 128, 64, {{0.72, 1.0}, {0.5, 0.7}}}};
  // The default tile of the other operand formats (launch_mx_t), priced by the
  // MFMAs of a wave and slab.
  const bool wide22 = na == 2 && nb == 2 && fa && fb;
  Tile def{0, (na == 1 || wide22) ? 256 : 128, nb == 1 ? 256 : 128, {}};
  const int per_pair = g == 32 ? na * nb : 2 * (na == 2 && fa ? nb : nb == 2 && fb ? na : na * nb == 4 ? 3 : na * nb);
  def.us[0][0] = def.us[1][0] = 0.6 + 0.0115 * (def.bm / 32) * (def.bn / 32) * per_pair;

  double best_us = 1e30;
  auto tile_us = [&](const Tile& t, int64_t parts, int64_t part_slabs) {
    const double* us = t.us[one && fa && fb];
    const int occ = us[1] > 0.0 ? 2 : 1;
    const int64_t wgs = ceil_div(M, t.bm) * ceil_div(N, t.bn) * parts;
    const int64_t full = wgs / (256 * occ), rest = wgs % (256 * occ);
    const double slab = full * us[occ - 1] + (rest == 0 ? 0.0 : rest <= 256 ? us[0] : us[1]);
    const double fix = 2.0 + 2.0 * (t.bm * t.bn) / 65536.0;  // a tile's start and its C
    // a second launch, and every part's sums written and read
    const double sum = parts > 1 ? 4.0 + 8e-6 / 5.0 * parts * M * N : 0.0;
    return part_slabs * slab + fix * (full + (rest > 0)) + sum;
  };
  auto consider = [&](const Tile& t) {
    const int64_t tiles = ceil_div(M, t.bm) * ceil_div(N, t.bn);
    for (int fill = 0; fill <= 2; ++fill) {  // whole, or in parts that fill 256 or 512 workgroups
      int64_t parts = fill == 0 ? 1 : 256 * fill / tiles;
      parts = parts < slabs / 4 ? parts : slabs / 4;  // at least four slabs in each
      if (fill > 0 && parts <= 1) continue;
      int64_t ps = fill == 0 ? slabs : ceil_div(ceil_div(slabs, parts), 2) * 2;  // (exponents come in slab pairs)
      parts = ceil_div(slabs, ps);
      if (fill > 0 && (parts <= 1 || parts * M * gemm_plan_ld(N) * 4 > (int64_t(1) << 28))) continue;
      const double us = tile_us(t, parts, ps);
      if (us < 0.95 * best_us) {
        best_us = us;
        best = GemmPlan{t.id, parts > 1 ? (int)ps : 0, (int)parts, 0, 0};
      }
    }
  };
  if (one) {
    for (const Tile& t : kTiles)  // the tile used without a workspace first: the others have to beat it
      if (t.id == rule) consider(t);
    for (const Tile& t : kTiles)
      if (t.id != rule) consider(t);
  } else {
    consider(def);
  }

  // The few-output kernel: its operand reads (every workgroup reads its rows of
  // both, 7 TB/s from L2 and the Infinity Cache) and the supersteps a wave waits for
  // in turn (1.36, 2.8 and 4.2 us each on its three tiles, half of it hidden
  // under the reads); or, with more workgroups than fit the CUs (LDS holds 16, 4
  // and 2 of the three tiles, and eight waves fill half a CU), the rounds of
  // them.  Without the rounds 23517 x 896 x 64 (2,4) went to 10304 workgroups of
  // 64 x 32, 78 us where the tiled kernel takes 20.  A tenth of margin: the tiled
  // kernel's prices are the firmer ones.
  const double va = (na == 1 && fa ? 0.5 : 0.75) + (na == 2 ? (fa ? 0.5 : 0.75) : 0.0) + 1.0 / g;
  const double vb = (nb == 1 && fb ? 0.5 : 0.75) + (nb == 2 ? (fb ? 0.5 : 0.75) : 0.0) + 1.0 / g;
  const int64_t nss = ceil_div(K, 256), per_wave = ceil_div(nss, direct::kMaxWaves);
  const int64_t waves = nss < direct::kMaxWaves ? nss : direct::kMaxWaves;
  // (The other formats' tiles start 3 us later than their price says: at K = 64, 7 to
  // 15 us where it says 5.)
  const double tiled_us = one || best.parts > 1 ? best_us : best_us + 3.0;
  double direct_us = 1e30;
  static const struct { int rm, rn, fit; double us, again; } kDirect[] = {
      {1, 1, 16, 1.36, 0.0}, {2, 2, 4, 2.8, 1.07}, {4, 2, 2, 4.2, 2.2}};
  for (const auto& d : kDirect) {
    if (ceil_div(M, 16 * d.rm) > direct::kMaxRowTiles) continue;  // does not fit its grid
    const double tm = (double)ceil_div(M, 16 * d.rm), tn = (double)ceil_div(N, 16 * d.rn);
    const double rows_a = M < 16 * d.rm ? M : 16 * d.rm, rows_b = N < 16 * d.rn ? N : 16 * d.rn;
    const double reads = 1.5 + tm * tn * K * (rows_a * va + rows_b * vb) / 7e6 + 0.5 * d.us * per_wave;
    const double more = tm * tn / (256.0 * (d.fit < 16 / waves ? d.fit : 16 / waves)) - 1.0;
    const double rounds = 1.8 + 0.5 * d.us * per_wave + more * (0.5 * (na + nb) * d.again * per_wave + 1.6);
    const double us = reads > rounds ? reads : rounds;
    if (us < direct_us && us < 0.9 * tiled_us) {
      direct_us = us;
      best = GemmPlan{rule, 0, 1, d.rm, d.rn};
    }
  }
  if (one && best.rm == 0 && best.parts == 1) best.tile = whole_tile(M, N, K, fa, fb, rule);
  return best;
}

int64_t gemm_plan_ld(int64_t N) { return (N + 3) / 4 * 4; }

hipError_t launch_gemm_mx(const uint8_t* a_mant, const uint8_t* a_exp, int a_m, int na, const uint8_t* b_mant,
                          const uint8_t* b_exp, int b_m, int nb, int64_t M, int64_t N, int64_t K, int g,
                          int scale_log2, float* C, int64_t ldc, int tile, hipStream_t s) {
  if (M == 0 || N == 0) return hipSuccess;
  const Product p = make_product(a_mant, a_exp, a_m, na, b_mant, b_exp, b_m, nb, M, N, K, g, scale_log2);
  const Output o{C, ldc, nullptr, 0, s};
  if (g == 32) return launch_tiled<32>(p, o, 0);
  if (tile < 0) tile = na == 1 && nb == 1 ? gemm_mx11_tile(M, N, p.fa, false) : 0;
  return launch_tiled<16>(p, o, tile);
}

hipError_t launch_gemm_mx_bfp(const uint8_t* a_mant, const uint8_t* a_exp, int a_m, int na, const uint8_t* b_mant,
                              const uint8_t* b_exp, int b_m, int nb, int64_t M, int64_t N, int64_t K, int g,
                              int scale_log2, int c_m, int mode, uint64_t seed, uint8_t* c_mant, uint8_t* c_exp,
                              uint32_t* status, hipStream_t s) {
  if (M == 0 || N == 0) return hipSuccess;
  const OutBFP qo{c_mant, c_mant + M * (N / 16) * plane_group_bytes(16, c_m, 0), c_exp, status, c_m, mode,
                  c_m <= 4 ? plane0_fp4(c_m) : c_m <= 6, (uint32_t)seed, (uint32_t)(seed >> 32)};
  const Product p = make_product(a_mant, a_exp, a_m, na, b_mant, b_exp, b_m, nb, M, N, K, g, scale_log2);
  const Output o{nullptr, N, &qo, 0, s};
  if (g == 32) return launch_tiled<32>(p, o, 0);
  return launch_tiled<16>(p, o, na == 1 && nb == 1 ? gemm_mx11_tile(M, N, p.fa, true) : 0);
}

hipError_t launch_gemm_plan(const GemmPlan& plan, const uint8_t* a_mant, const uint8_t* a_exp, int a_m, int na,
                            const uint8_t* b_mant, const uint8_t* b_exp, int b_m, int nb, int64_t M, int64_t N,
                            int64_t K, int g, int scale_log2, float* C, int64_t ldc, hipStream_t s) {
  if (M == 0 || N == 0) return hipSuccess;
  const Product p = make_product(a_mant, a_exp, a_m, na, b_mant, b_exp, b_m, nb, M, N, K, g, scale_log2);
  if (plan.rm > 0)
    return g == 32 ? launch_direct<32>(p, plan, C, ldc, nullptr, s) : launch_direct<16>(p, plan, C, ldc, nullptr, s);
  const Output o{C, ldc, nullptr, plan.parts > 1 ? plan.part_slabs : 0, s};
  return g == 32 ? launch_tiled<32>(p, o, 0) : launch_tiled<16>(p, o, plan.tile);
}

hipError_t launch_gemm_direct_bfp(const GemmPlan& plan, const uint8_t* a_mant, const uint8_t* a_exp, int a_m, int na,
                                  const uint8_t* b_mant, const uint8_t* b_exp, int b_m, int nb, int64_t M, int64_t N,
                                  int64_t K, int g, int scale_log2, int c_m, int mode, uint64_t seed, uint8_t* c_mant,
                                  uint8_t* c_exp, uint32_t* status, hipStream_t s) {
  const Product p = make_product(a_mant, a_exp, a_m, na, b_mant, b_exp, b_m, nb, M, N, K, g, scale_log2);
  const direct::Out out{c_mant, c_mant + M * (N / 16) * plane_group_bytes(16, c_m, 0), c_exp, status, c_m, mode,
                        (uint32_t)seed, (uint32_t)(seed >> 32)};
  return g == 32 ? launch_direct<32>(p, plan, nullptr, N, &out, s) : launch_direct<16>(p, plan, nullptr, N, &out, s);
}

}  // namespace fastbfp
