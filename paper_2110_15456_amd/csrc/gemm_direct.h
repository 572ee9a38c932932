// gemm_direct.h -- the BFP GEMM for products with few outputs: a few tokens
// against a layer's weights, or a small layer.  The same sums as gemm_mx.h
// (section III-B; the same block-scaled MFMA per chunk-plane pair), without
// LDS staging.
//
// What bounds these products is the latency and the number of bytes in flight,
// not the matrix cores: the tiled kernel gives a 16 x 16384 x 4096 product 256
// workgroups of 128 x 64, one per CU, each waiting for its own 6 KB slab 32
// times in a row.  Here a workgroup computes a small tile (16 RM x 16 RN) and its
// waves split K between them, so that the whole operand is requested by many
// waves at once; every wave loads its fragments straight into registers and the
// waves' sums are added through LDS in a fixed order.
//
// A K superstep is 16 units (of 16 values).  Lane (r = lane % 16, lb = lane /
// 16) takes row r's units 4 lb .. 4 lb + 3: 48 contiguous bytes of an FP6 plane
// (three 16-byte loads) or 32 of an FP4 or Lo2 plane (two), and their exponents
// in one load, which serve four MFMA K-steps (two with groups of 32): which
// group of a K-step a lane block holds does not matter as long as both
// operands agree.  Units past K meet zero exponents on both sides (a scale of
// 2^-254 adds nothing); rows past the end read zeros (the buffer resource ends
// at the last row).
#pragma once
#include "bfp_quant.h"

namespace fastbfp {

namespace direct {

typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int kMaxWaves = 8;
constexpr int kMaxRowTiles = 65535;  // row tiles are the grid's y, which holds no more

__device__ __forceinline__ rsrc_t make_rsrc(const uint8_t* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p), (short)0, (int)bytes, 0x00020000);
}

// One lane's four units of one plane: 12 dwords (FP6) or 8 (FP4, Lo2).
template <int KIND> struct Units {
  static constexpr int ND = KIND == kPlaneFP6 ? 12 : 8;
  int d[ND];
  __device__ __forceinline__ void load(rsrc_t r, uint32_t off) {
#pragma unroll
    for (int i = 0; i < ND / 4; ++i) {
      const v4i v = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r, off + 16 * i, 0, 0));
#pragma unroll
      for (int k = 0; k < 4; ++k) d[4 * i + k] = v[k];
    }
  }
  // Codes of unit u at dwords 0.. of w (FP6 codes for a Lo2 plane).
  __device__ __forceinline__ void codes(int u, int (&w)[3]) const {
    if constexpr (KIND == kPlaneFP6) {
      w[0] = d[3 * u];
      w[1] = d[3 * u + 1];
      w[2] = d[3 * u + 2];
    } else if constexpr (KIND == kPlaneFP4) {
      w[0] = d[2 * u];
      w[1] = d[2 * u + 1];
      w[2] = 0;
    } else {
      uint32_t t0, t1, t2;
      lo2_unpack((uint32_t)d[2 * u], (uint32_t)d[2 * u + 1], t0, t1, t2);
      w[0] = (int)t0;
      w[1] = (int)t1;
      w[2] = (int)t2;
    }
  }
  // Operand of one unit in half 0; DUP: repeated in half 1, else zeros there.
  template <bool DUP> __device__ __forceinline__ v8i half(int u) const {
    int w[3];
    codes(u, w);
    if constexpr (KIND == kPlaneFP4) return DUP ? v8i{w[0], w[1], w[0], w[1], 0, 0, 0, 0} : v8i{w[0], w[1], 0, 0, 0, 0, 0, 0};
    else return DUP ? v8i{w[0], w[1], w[2], w[0], w[1], w[2], 0, 0} : v8i{w[0], w[1], w[2], 0, 0, 0, 0, 0};
  }
  // Operand of units 2p and 2p + 1 (a group of 32).
  __device__ __forceinline__ v8i pair(int p) const {
    int a[3], b[3];
    codes(2 * p, a);
    codes(2 * p + 1, b);
    if constexpr (KIND == kPlaneFP4) return v8i{a[0], a[1], b[0], b[1], 0, 0, 0, 0};
    else return v8i{a[0], a[1], a[2], b[0], b[1], b[2], 0, 0};
  }
};
// Two FP6-coded units (of different planes) side by side.
template <int K0, int K1>
__device__ __forceinline__ v8i join(const Units<K0>& x, const Units<K1>& y, int u) {
  int a[3], b[3];
  x.codes(u, a);
  y.codes(u, b);
  return v8i{a[0], a[1], a[2], b[0], b[1], b[2], 0, 0};
}

// The exponents of one lane's four units: four bytes (groups of 16) or two
// (groups of 32), zero past the last unit.  dw: the rows' exponents start
// 4-byte aligned (2-byte for groups of 32).
template <int G>
__device__ __forceinline__ uint32_t load_exps(rsrc_t r, uint32_t off, int units_left, bool dw) {
  const int n = G == 16 ? units_left : (units_left + 1) / 2;  // exponents left (<= 0: none)
  constexpr int NE = G == 16 ? 4 : 2;
  uint32_t e = 0;
  if (dw) {
    e = G == 16 ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0)
                : (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
    if (n < NE) e &= n <= 0 ? 0u : (1u << (8 * n)) - 1u;
  } else {
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const uint32_t b = (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, off + k, 0, 0);
      e |= (k < n ? b : 0u) << (8 * k);
    }
  }
  return e;
}

template <int FMT> struct fmt { static constexpr int value = FMT == kPlaneFP4 ? 4 : 2; };

// acc += one K-step: A in format KA, B in KB (B first: a lane's four results
// are four consecutive columns of one row of C), block scales ea / eb (low byte).
template <int KA, int KB>
__device__ __forceinline__ void mma(v4f& acc, const v8i& a, const v8i& b, uint32_t ea, uint32_t eb) {
  acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b, a, acc, fmt<KB>::value, fmt<KA>::value, 0, (int)eb, 0,
                                                         (int)ea);
}

// BFP output (m and mode at run time: a group per thread, once per workgroup).
struct Out {
  uint8_t *mant0, *mant1, *exps;
  uint32_t* status;
  int m, mode;
  uint32_t key0, key1;
};
// Converts the 16 values at b as quantize_groups does and stores them as group
// gid; true if one was Inf or NaN.
__device__ __forceinline__ bool convert(const uint32_t (&b)[16], int64_t gid, const Out& o) {
  const uint32_t E = group_exponent<16>(b), m = (uint32_t)o.m, qmax = (1u << m) - 1u;
  uint32_t q[16], noise[4] = {0u, 0u, 0u, 0u};
  if (o.mode == kStochastic) {
    group_noise<16>((uint64_t)gid, o.key0, o.key1, noise);
#pragma unroll
    for (int t = 0; t < 16; ++t)
      q[t] = value_magnitude<kStochastic, false>(b[t], magnitude_align<kStochastic>(m, E), noise[t >> 2], t, qmax);
  } else if (o.mode == kNearest) {
#pragma unroll
    for (int t = 0; t < 16; ++t)
      q[t] = value_magnitude<kNearest, false>(b[t], magnitude_align<kNearest>(m, E), 0u, t, qmax);
  } else {
#pragma unroll
    for (int t = 0; t < 16; ++t)
      q[t] = value_magnitude<kTruncate, false>(b[t], magnitude_align<kTruncate>(m, E), 0u, t, qmax);
  }
  const uint32_t lo_bits = m <= 4 ? 0u : (uint32_t)low_chunk_bits(o.m), lo_mask = (1u << lo_bits) - 1u;
  uint32_t w0[4] = {0u, 0u, 0u, 0u}, w1[4] = {0u, 0u, 0u, 0u};
  auto put6 = [](uint32_t(&w)[4], int t, uint32_t code) {
    const int wi = 6 * t >> 5, sh = 6 * t & 31;
    w[wi] |= code << sh;
    if (sh > 26) w[wi + 1] |= code >> (32 - sh);
  };
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const uint32_t neg = b[t] >> 31, hi = q[t] >> lo_bits, lo = q[t] & lo_mask;
    if (m <= 2) w0[t >> 3] |= (hi ? (neg << 3) | hi : 0u) << (4 * (t & 7));
    else put6(w0, t, hi ? (neg << 5) | e2m3_half_code(hi) : 0u);
    if (m > 4) put6(w1, t, lo ? (neg << 5) | (m > 6 ? e2m3_half_code(lo) : lo) : 0u);
  }
  o.exps[gid] = (uint8_t)E;
  if (m <= 2) store_plane<16, true>(o.mant0, gid, w0);
  else store_plane<16, false>(o.mant0, gid, w0);
  if (m > 6) {
    store_plane<16, false>(o.mant1, gid, w1);
  } else if (m > 4) {
    const uint2 d = lo2_pack(w1[0], w1[1], w1[2]);
    const uint32_t w[2] = {d.x, d.y};
    store_plane<16, true>(o.mant1, gid, w);
  }
  return E == 255u;
}

// One row tile's fragments of one superstep.
template <int NP, int K0, int K1> struct Frag {
  Units<K0> p0;
  Units<K1> p1;
  uint32_t e;
};

}  // namespace direct

// NA / NB, FA / FB, G: as mx::Cfg (planes read; FP4 codes, or split at 2 bits).
// BOUT: C is written as BFP (N a multiple of 16).
template <int NA, int NB, int FA, int FB, int G, int RM, int RN, bool BOUT>
__global__ __launch_bounds__(64 * direct::kMaxWaves) void k_gemm_direct(
    const uint8_t* __restrict__ a_mant, const uint8_t* __restrict__ a_exp, int64_t a_ps,
    const uint8_t* __restrict__ b_mant, const uint8_t* __restrict__ b_exp, int64_t b_ps, int M, int N, int ng,
    float scale, float* __restrict__ C, int64_t ldc, direct::Out out) {
  using namespace direct;
  constexpr int KA0 = (NA == 1 && FA) ? kPlaneFP4 : kPlaneFP6, KB0 = (NB == 1 && FB) ? kPlaneFP4 : kPlaneFP6;
  constexpr int KA1 = FA ? kPlaneLo2 : kPlaneFP6, KB1 = FB ? kPlaneLo2 : kPlaneFP6;
  constexpr bool SA = NA == 2 && FA, SB = NB == 2 && FB;  // split at 2 bits
  constexpr int SROW = 16 * RN + 4;                       // LDS row stride in floats (padding spreads the banks)
  __shared__ __attribute__((aligned(16))) float part[kMaxWaves][16 * RM * SROW];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int lr = lane & 15, lb = lane >> 4;
  const int row0 = blockIdx.y * (16 * RM), col0 = blockIdx.x * (16 * RN);
  const int a_rows = min(16 * RM, M - row0), b_rows = min(16 * RN, N - col0);
  const int ng_e = ng * 16 / G;
  constexpr int UA0 = KA0 == kPlaneFP6 ? 12 : 8, UB0 = KB0 == kPlaneFP6 ? 12 : 8;  // bytes per unit
  constexpr int UA1 = KA1 == kPlaneFP6 ? 12 : 8, UB1 = KB1 == kPlaneFP6 ? 12 : 8;
  const rsrc_t ra0 = make_rsrc(a_mant + (int64_t)row0 * ng * UA0, (uint32_t)a_rows * ng * UA0);
  const rsrc_t rb0 = make_rsrc(b_mant + (int64_t)col0 * ng * UB0, (uint32_t)b_rows * ng * UB0);
  const rsrc_t ra1 = make_rsrc(a_mant + a_ps + (int64_t)row0 * ng * UA1, NA == 2 ? (uint32_t)a_rows * ng * UA1 : 0u);
  const rsrc_t rb1 = make_rsrc(b_mant + b_ps + (int64_t)col0 * ng * UB1, NB == 2 ? (uint32_t)b_rows * ng * UB1 : 0u);
  const rsrc_t rea = make_rsrc(a_exp + (int64_t)row0 * ng_e, (uint32_t)a_rows * ng_e);
  const rsrc_t reb = make_rsrc(b_exp + (int64_t)col0 * ng_e, (uint32_t)b_rows * ng_e);
  constexpr int EA = G == 16 ? 4 : 2;  // exponent bytes per lane and superstep
  const bool dw = ng_e % EA == 0 && (reinterpret_cast<uintptr_t>(a_exp) % EA) == 0 &&
                  (reinterpret_cast<uintptr_t>(b_exp) % EA) == 0;

  v4f acc[RM][RN];
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < RN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

  // this wave's contiguous run of supersteps
  const int nss = (ng + 15) / 16, per = (nss + nw - 1) / nw;
  const int ss0 = wave * per, ss1 = min(nss, ss0 + per);
  for (int ss = ss0; ss < ss1; ++ss) {
    const int u0 = ss * 16 + 4 * lb;
    Frag<NA, KA0, KA1> fa[RM];
    Frag<NB, KB0, KB1> fb[RN];
#pragma unroll
    for (int j = 0; j < RN; ++j) {
      const uint32_t r = 16 * j + lr;
      fb[j].p0.load(rb0, (r * ng + u0) * UB0);
      if constexpr (NB == 2) fb[j].p1.load(rb1, (r * ng + u0) * UB1);
      fb[j].e = load_exps<G>(reb, G == 16 ? r * ng_e + u0 : r * ng_e + u0 / 2, ng - u0, dw);
    }
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      const uint32_t r = 16 * i + lr;
      fa[i].p0.load(ra0, (r * ng + u0) * UA0);
      if constexpr (NA == 2) fa[i].p1.load(ra1, (r * ng + u0) * UA1);
      fa[i].e = load_exps<G>(rea, G == 16 ? r * ng_e + u0 : r * ng_e + u0 / 2, ng - u0, dw);
    }
#pragma unroll
    for (int u = 0; u < (G == 16 ? 4 : 2); ++u) {
#pragma unroll
      for (int i = 0; i < RM; ++i) {
        const auto& x = fa[i];
        const uint32_t ea = (x.e >> (8 * u)) & 0xFFu;
#pragma unroll
        for (int j = 0; j < RN; ++j) {
          const auto& y = fb[j];
          const uint32_t eb = (y.e >> (8 * u)) & 0xFFu;
          v4f& c = acc[i][j];
          // The chunk weights on the scale bytes and the pairing of planes
          // are those of gemm_mx.h.
          if constexpr (G == 32) {
            constexpr int wa0 = NA == 1 ? 0 : SA ? 2 : 4, wa1 = SA ? 2 : 0;
            constexpr int wb0 = NB == 1 ? 0 : SB ? 2 : 4, wb1 = SB ? 2 : 0;
            mma<KA0, KB0>(c, x.p0.pair(u), y.p0.pair(u), ea + wa0, eb + wb0);
            if constexpr (NA == 2) mma<KA1, KB0>(c, x.p1.pair(u), y.p0.pair(u), ea + wa1, eb + wb0);
            if constexpr (NB == 2) mma<KA0, KB1>(c, x.p0.pair(u), y.p1.pair(u), ea + wa0, eb + wb1);
            if constexpr (NA == 2 && NB == 2) mma<KA1, KB1>(c, x.p1.pair(u), y.p1.pair(u), ea + wa1, eb + wb1);
          } else if constexpr (SA) {
            // A's [q >> 2 | q & 3] block against each plane of B repeated
            const v8i av = join(x.p0, x.p1, u);
            constexpr int wb0 = NB == 1 ? 0 : SB ? 2 : 4, wb1 = SB ? 2 : 0;
            mma<kPlaneFP6, KB0>(c, av, y.p0.template half<true>(u), ea + 2, eb + wb0);
            if constexpr (NB == 2) mma<kPlaneFP6, KB1>(c, av, y.p1.template half<true>(u), ea + 2, eb + wb1);
          } else if constexpr (SB) {
            const v8i bv = join(y.p0, y.p1, u);
            constexpr int wa0 = NA == 1 ? 0 : 4;
            mma<KA0, kPlaneFP6>(c, x.p0.template half<true>(u), bv, ea + wa0, eb + 2);
            if constexpr (NA == 2) mma<KA1, kPlaneFP6>(c, x.p1.template half<true>(u), bv, ea, eb + 2);
          } else if constexpr (NA == 2 && NB == 2) {
            // split at 4 bits on both sides: the two cross products share one MFMA
            mma<KA0, KB0>(c, x.p0.template half<false>(u), y.p0.template half<false>(u), ea + 4, eb + 4);
            mma<KA1, KB1>(c, x.p1.template half<false>(u), y.p1.template half<false>(u), ea, eb);
            mma<kPlaneFP6, kPlaneFP6>(c, join(x.p0, x.p1, u), join(y.p1, y.p0, u), ea + 4, eb);
          } else {
            constexpr int wa0 = NA == 1 ? 0 : 4, wb0 = NB == 1 ? 0 : 4;
            mma<KA0, KB0>(c, x.p0.template half<false>(u), y.p0.template half<false>(u), ea + wa0, eb + wb0);
            if constexpr (NA == 2)
              mma<KA1, KB0>(c, x.p1.template half<false>(u), y.p0.template half<false>(u), ea, eb + wb0);
            if constexpr (NB == 2)
              mma<KA0, KB1>(c, x.p0.template half<false>(u), y.p1.template half<false>(u), ea + wa0, eb);
          }
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < RN; ++j)
      *reinterpret_cast<v4f*>(&part[wave][(16 * i + lr) * SROW + 16 * j + 4 * lb]) = acc[i][j];
  __syncthreads();
  // C: the waves' sums added in wave order, four columns (or a group of 16) per
  // thread.
  if constexpr (BOUT) {
    const int nact = min(nw, (nss + per - 1) / max(per, 1));
    bool bad = false;
    for (int q = threadIdx.x; q < 16 * RM * RN; q += blockDim.x) {
      const int r = q / RN, j = q % RN;
      uint32_t b[16];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v4f v = *reinterpret_cast<const v4f*>(&part[0][r * SROW + 16 * j + 4 * k]);
        for (int w = 1; w < nact; ++w) v += *reinterpret_cast<const v4f*>(&part[w][r * SROW + 16 * j + 4 * k]);
#pragma unroll
        for (int t = 0; t < 4; ++t) b[4 * k + t] = __float_as_uint(v[t] * scale);
      }
      if (row0 + r < M && col0 + 16 * j < N)
        bad |= convert(b, (int64_t)(row0 + r) * (N / 16) + col0 / 16 + j, out);
    }
    if (out.status && bad) atomicOr(out.status, 1u);
    return;
  }
  const bool vec = (ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0;
  const int nact = min(nw, (nss + per - 1) / max(per, 1));  // waves that had a superstep
  for (int q = threadIdx.x; q < 16 * RM * 4 * RN; q += blockDim.x) {
    const int r = q / (4 * RN), k = 4 * (q % (4 * RN));
    v4f v = *reinterpret_cast<const v4f*>(&part[0][r * SROW + k]);
    for (int w = 1; w < nact; ++w) v += *reinterpret_cast<const v4f*>(&part[w][r * SROW + k]);
    const int row = row0 + r, col = col0 + k;
    if (row >= M) continue;
    float* p = C + (int64_t)row * ldc + col;
    if (vec && col + 3 < N) {
      *reinterpret_cast<float4*>(p) = make_float4(v[0] * scale, v[1] * scale, v[2] * scale, v[3] * scale);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (col + t < N) p[t] = v[t] * scale;
    }
  }
}

template <int NA, int NB, int FA, int FB, int G>
hipError_t launch_direct_t(int rm, int rn, const uint8_t* a_mant, const uint8_t* a_exp, int64_t a_ps,
                           const uint8_t* b_mant, const uint8_t* b_exp, int64_t b_ps, int M, int N, int ng, float scale,
                           float* C, int64_t ldc, const direct::Out* out, hipStream_t s) {
  const int nss = (ng + 15) / 16;
  const int nw = nss < 1 ? 1 : nss > direct::kMaxWaves ? direct::kMaxWaves : nss;
  const dim3 grid((unsigned)((N + 16 * rn - 1) / (16 * rn)), (unsigned)((M + 16 * rm - 1) / (16 * rm)));
  if (grid.y > (unsigned)direct::kMaxRowTiles) return hipErrorInvalidValue;  // (gemm_plan does not plan it)
#define FASTBFP_DIRECT_LAUNCH(RM, RN)                                                                                 \
  if (rm == RM && rn == RN) {                                                                                         \
    if (out)                                                                                                          \
      hipLaunchKernelGGL((k_gemm_direct<NA, NB, FA, FB, G, RM, RN, true>), grid, dim3(64 * nw), 0, s, a_mant, a_exp,  \
                         a_ps, b_mant, b_exp, b_ps, M, N, ng, scale, C, ldc, *out);                                   \
    else                                                                                                              \
      hipLaunchKernelGGL((k_gemm_direct<NA, NB, FA, FB, G, RM, RN, false>), grid, dim3(64 * nw), 0, s, a_mant, a_exp, \
                         a_ps, b_mant, b_exp, b_ps, M, N, ng, scale, C, ldc, direct::Out{});                          \
    return hipGetLastError();                                                                                         \
  }
  FASTBFP_DIRECT_LAUNCH(1, 1)
  FASTBFP_DIRECT_LAUNCH(2, 2)
  FASTBFP_DIRECT_LAUNCH(4, 2)
#undef FASTBFP_DIRECT_LAUNCH
  return hipErrorInvalidValue;
}

// One operand-format combination's dispatch over the group sizes.
#define FASTBFP_DIRECT_INSTANTIATE(NA, NB, FA, FB, G)                                                            \
  template hipError_t launch_direct_t<NA, NB, FA, FB, G>(int, int, const uint8_t*, const uint8_t*, int64_t,      \
                                                         const uint8_t*, const uint8_t*, int64_t, int, int, int, \
                                                         float, float*, int64_t, const direct::Out*, hipStream_t);
#define FASTBFP_DIRECT_DECLARE(NA, NB, FA, FB, G) extern FASTBFP_DIRECT_INSTANTIATE(NA, NB, FA, FB, G)
#define FASTBFP_DIRECT_ALL(DO, NA, NB, G) DO(NA, NB, 0, 0, G) DO(NA, NB, 0, 1, G) DO(NA, NB, 1, 0, G) DO(NA, NB, 1, 1, G)

}  // namespace fastbfp
