// repack.hip -- re-encodes a stored BFP tensor into the chunk-plane layout that
// the block-scaled GEMM kernel (gemm_mx.h) reads, so that the products it does
// not take directly still run on it (bfp_gemm_ws):
//   * a precision below the stored width: each magnitude truncated to its top
//     m_use bits (the discard of low-order bits, section V-D) and stored as an
//     m_use-bit tensor, with the same exponents;
//   * groups of 4 or 8: each group becomes one 16-value unit holding its g
//     values and 16 - g zeros, with the group's exponent (the other operand
//     gets the same padding, so the zeros meet zeros and every product is the
//     group's own);
//   * groups of 64: two groups of 32 that share the group's exponent (the
//     sum of their exact products is the 64-value group's);
//   * the packed storage of section V-D: unpacked, each group at its stored
//     exponent E = base + e.
// The values stay exactly what the stored tensor stands for at m_use bits, so
// a GEMM on the repacked operands computes the same per-group terms T_G.
#include <type_traits>

#include "bfp_decode.h"

namespace fastbfp {

namespace {

typedef uint32_t u2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u3_t __attribute__((ext_vector_type(3)));

// OR a 6-bit code into position t of 16 little-endian packed FP6 codes.
__device__ __forceinline__ void put6(uint32_t (&w)[3], int t, uint32_t code) {
  const int bit = 6 * t, wi = bit >> 5, sh = bit & 31;
  w[wi] |= code << sh;
  if (sh > 26) w[wi + 1] |= code >> (32 - sh);
}

// One thread per output 16-value unit: unit u of row r, idx = r * units_out + u.
// G: the source group size.
template <int G>
__global__ __launch_bounds__(256) void k_repack(Opnd src, int64_t units_out, int64_t total, int m_out,
                                                uint8_t* __restrict__ p0, uint8_t* __restrict__ p1,
                                                uint8_t* __restrict__ exps_out) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int row = (int)(idx / units_out);
  const int64_t u = idx % units_out;
  // source unit, source group, and (G < 16) the group's first value in its unit
  const int64_t src_unit = G < 16 ? (u * G) / 16 : u;
  const int64_t grp = G < 16 ? u : (u * 16) / G;
  const int first = G < 16 ? (int)((u * G) % 16) : 0;
  int a[8], b[8], s[16];
  decode_q8(src, row, src_unit, 0, a);
  decode_q8(src, row, src_unit, 1, b);
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    s[t] = a[t];
    s[8 + t] = b[t];
  }
  int q[16];
  if constexpr (G < 16) {
#pragma unroll
    for (int t = 0; t < 16; ++t) q[t] = 0;
#pragma unroll
    for (int k = 0; k < 16; k += G)
      if (first == k) {
#pragma unroll
        for (int t = 0; t < G; ++t) q[t] = s[k + t];
      }
  } else {
#pragma unroll
    for (int t = 0; t < 16; ++t) q[t] = s[t];
  }
  // planes of the m_out-bit tensor (launch.h): FP4 for m <= 2, FP6 for m <= 4,
  // FP6 of q >> 2 and Lo2 of q & 3 for m = 5, 6, FP6 of q >> 4 and q & 15 for m = 7, 8
  const int lo_bits = m_out <= 4 ? 0 : low_chunk_bits(m_out);
  uint32_t w0[3] = {0u, 0u, 0u}, w1[3] = {0u, 0u, 0u};
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const uint32_t mag = (uint32_t)(q[t] < 0 ? -q[t] : q[t]), neg = q[t] < 0 ? 1u : 0u;
    const uint32_t hi = mag >> lo_bits, lo = mag & ((1u << lo_bits) - 1u);
    if (m_out <= 2) {
      w0[t >> 3] |= (hi ? (neg << 3) | hi : 0u) << (4 * (t & 7));
    } else {
      put6(w0, t, hi ? (neg << 5) | e2m3_half_code(hi) : 0u);
      if (m_out > 6) put6(w1, t, lo ? (neg << 5) | e2m3_half_code(lo) : 0u);
      else if (m_out > 4) put6(w1, t, lo ? (neg << 5) | lo : 0u);  // FP6 code of +-lo/8 (subnormal)
    }
  }
  if (m_out <= 2) {
    *reinterpret_cast<u2_t*>(p0 + idx * 8) = u2_t{w0[0], w0[1]};
  } else {
    *reinterpret_cast<u3_t*>(p0 + idx * 12) = u3_t{w0[0], w0[1], w0[2]};
    if (m_out > 6) {
      *reinterpret_cast<u3_t*>(p1 + idx * 12) = u3_t{w1[0], w1[1], w1[2]};
    } else if (m_out > 4) {
      const uint2 d = lo2_pack(w1[0], w1[1], w1[2]);
      *reinterpret_cast<u2_t*>(p1 + idx * 8) = u2_t{d.x, d.y};
    }
  }
  // exponents: one per output group of 16, or of 32 (source groups of 32 and 64)
  const int e = opnd_exponent(src, row, grp);
  if (G <= 16)
    exps_out[idx] = (uint8_t)e;
  else if ((u & 1) == 0)
    exps_out[idx / 2] = (uint8_t)e;
}

// The three faster forms below run at the widths whose planes are already
// there: the stored one, or the upper chunk plane alone.  They move and
// re-encode whole words of codes; only a precision between chunk boundaries goes
// value by value (k_repack).

// Fields of 3 bits to a spacing of 6: fields 0..3 of x at bits 0, 6, 12, 18.
__device__ __forceinline__ uint32_t spread6(uint32_t x) {
  x = (x | (x << 6)) & 0x0003F03Fu;
  return (x | (x << 3)) & 0x001C71C7u;
}
// The FP6 E2M3 codes (24 bits each) of values 0..3 and 4..7 whose upper and
// lower 2-bit chunks, with signs, are the eight 3-bit fields of hi and lo.  With
// c = (q3 q2 q1 q0), the code of c/2 is, by c's top bit: 1 1 q2 q1 q0; 1 0 q1 q0
// 0; 0 1 q0 0 0; 0 0 q0 0 0 -- bit logic on all eight values at once.
__device__ __forceinline__ void fp6_of_chunks(uint32_t hi, uint32_t lo, uint32_t& c0, uint32_t& c1) {
  constexpr uint32_t B = 0x249249u;  // bit 0 of each field
  const uint32_t q3 = (hi >> 1) & B, q2 = hi & B, q1 = (lo >> 1) & B, q0 = lo & B;
  const uint32_t b4 = q3 | q2, b3 = q3 | (q1 & ~q2);
  const uint32_t b2 = (q3 & q2) | (~q3 & ((q2 & q1) | (~q2 & q0)));
  const uint32_t b1 = (q3 & q1) | (~q3 & q2 & q0), b0 = q3 & q0;
  const uint32_t H = ((hi | lo) & (B << 2)) | (b4 << 1) | b3, L = ((b2 & B) << 2) | ((b1 & B) << 1) | b0;
  c0 = (spread6(H & 0xFFFu) << 3) | spread6(L & 0xFFFu);
  c1 = (spread6((H >> 12) & 0xFFFu) << 3) | spread6((L >> 12) & 0xFFFu);
}
// The FP4 codes (sign above the chunk, 4 bits) of eight 3-bit fields.
__device__ __forceinline__ uint32_t fp4_of_chunks(uint32_t x) {
  x = (x & 0xFFFu) | ((x & 0xFFF000u) << 4);
  x = (x & 0x003F003Fu) | ((x & 0x0FC00FC0u) << 2);
  x = (x & 0x07070707u) | ((x & 0x38383838u) << 1);
  return (x & 0x33333333u) | ((x & 0x44444444u) << 1);
}
// 16 values' codes from four 24-bit pieces.
__device__ __forceinline__ u3_t join24(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return u3_t{a | (b << 24), (b >> 8) | (c << 16), (c >> 16) | (d << 8)};
}

// Packed storage to chunk planes at the stored width, one thread per group of
// 16.  NP: its 2-bit chunk planes.  Value by value this took 37 us on 8192 x
// 4096 at m = 4 (bound by its arithmetic and byte loads).
template <int NP>
__global__ __launch_bounds__(256) void k_unpack(const uint8_t* __restrict__ mant, const uint32_t* __restrict__ expw,
                                                int64_t ngroups, uint8_t* __restrict__ p0, uint8_t* __restrict__ p1,
                                                uint8_t* __restrict__ exps_out) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (gid >= ngroups) return;
  uint32_t a[NP], b[NP];  // fields of values 0..7 and 8..15
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    const uint16_t* src = reinterpret_cast<const uint16_t*>(mant + (c * ngroups + gid) * 6);
    const uint32_t w0 = src[0], w1 = src[1], w2 = src[2];
    a[c] = w0 | ((w1 & 0xFFu) << 16);
    b[c] = (w1 >> 8) | (w2 << 8);
  }
  if constexpr (NP == 1) {
    *reinterpret_cast<u2_t*>(p0 + gid * 8) = u2_t{fp4_of_chunks(a[0]), fp4_of_chunks(b[0])};
  } else {
    uint32_t c[4];
    fp6_of_chunks(a[0], a[1], c[0], c[1]);
    fp6_of_chunks(b[0], b[1], c[2], c[3]);
    *reinterpret_cast<u3_t*>(p0 + gid * 12) = join24(c[0], c[1], c[2], c[3]);
    if constexpr (NP == 3) {
      // Lo2: the FP6 codes of +-chunk/8 are the sign and the chunk as they are
      auto code = [](uint32_t f) { return (spread6(f & 0x924u) << 3) | spread6(f & 0x6DBu); };
      const u3_t t = join24(code(a[2] & 0xFFFu), code(a[2] >> 12), code(b[2] & 0xFFFu), code(b[2] >> 12));
      const uint2 d = lo2_pack(t.x, t.y, t.z);
      *reinterpret_cast<u2_t*>(p1 + gid * 8) = u2_t{d.x, d.y};
    } else if constexpr (NP == 4) {
      fp6_of_chunks(a[2], a[3], c[0], c[1]);
      fp6_of_chunks(b[2], b[3], c[2], c[3]);
      *reinterpret_cast<u3_t*>(p1 + gid * 12) = join24(c[0], c[1], c[2], c[3]);
    }
  }
  exps_out[gid] = (uint8_t)(packed_base(expw[0]) + packed_exponent_offset(expw, gid));
}

// Groups of G = 4 or 8 to 16-value units, one thread per source unit (16 / G
// groups): each group's codes, then zeros.  NCH planes of kinds K0, K1 are
// read and written.
template <int G, int NCH, int K0, int K1>
__global__ __launch_bounds__(256) void k_widen(const uint8_t* __restrict__ s0, const uint8_t* __restrict__ s1,
                                               const uint8_t* __restrict__ exps, int64_t nunits,
                                               uint8_t* __restrict__ p0, uint8_t* __restrict__ p1,
                                               uint8_t* __restrict__ exps_out) {
  constexpr int NG = 16 / G;
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (u >= nunits) return;
  auto plane = [&](auto kc, const uint8_t* s, uint8_t* p) {
    constexpr int K = decltype(kc)::value;
    if constexpr (K == kPlaneFP4) {
      const u2_t d = *reinterpret_cast<const u2_t*>(s + u * 8);
#pragma unroll
      for (int k = 0; k < NG; ++k) {
        const uint32_t w = G == 8 ? d[k] : (d[k / 2] >> (16 * (k & 1))) & 0xFFFFu;
        *reinterpret_cast<u2_t*>(p + (u * NG + k) * 8) = u2_t{w, 0u};
      }
    } else {
      uint32_t t[3];
      if constexpr (K == kPlaneLo2) {
        const u2_t d = *reinterpret_cast<const u2_t*>(s + u * 8);
        lo2_unpack(d.x, d.y, t[0], t[1], t[2]);
      } else {
        const u3_t d = *reinterpret_cast<const u3_t*>(s + u * 12);
        t[0] = d.x, t[1] = d.y, t[2] = d.z;
      }
#pragma unroll
      for (int k = 0; k < NG; ++k) {
        // bits 6 G k .. 6 G (k + 1) - 1 of the unit
        uint32_t w0, w1 = 0u;
        if constexpr (G == 8) {
          w0 = k == 0 ? t[0] : (t[1] >> 16) | (t[2] << 16);
          w1 = k == 0 ? t[1] & 0xFFFFu : t[2] >> 16;
        } else {
          w0 = (k == 0 ? t[0] : k == 1 ? (t[0] >> 24) | (t[1] << 8) : k == 2 ? (t[1] >> 16) | (t[2] << 16) : t[2] >> 8) &
               0xFFFFFFu;
        }
        if constexpr (K == kPlaneLo2) {
          const uint2 d = lo2_pack(w0, w1, 0u);
          *reinterpret_cast<u2_t*>(p + (u * NG + k) * 8) = u2_t{d.x, d.y};
        } else {
          *reinterpret_cast<u3_t*>(p + (u * NG + k) * 12) = u3_t{w0, w1, 0u};
        }
      }
    }
  };
  plane(std::integral_constant<int, K0>{}, s0, p0);
  if constexpr (NCH == 2) plane(std::integral_constant<int, K1>{}, s1, p1);
#pragma unroll
  for (int k = 0; k < NG; ++k) exps_out[u * NG + k] = exps[u * NG + k];
}

// Groups of 64 to groups of 32: every exponent twice.
__global__ __launch_bounds__(256) void k_exps_twice(const uint8_t* __restrict__ exps, int64_t n,
                                                    uint8_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) {
    const uint8_t e = exps[i];
    out[2 * i] = e;
    out[2 * i + 1] = e;
  }
}

template <int G>
hipError_t widen(const uint8_t* mant, const uint8_t* exps, int64_t nunits, int m, uint8_t* out, uint8_t* out_exps,
                 hipStream_t s) {
  const dim3 grid((unsigned)((nunits + 255) / 256));
  const uint8_t* s1 = mant + nunits * (plane_kind(m, 0) == kPlaneFP6 ? 12 : 8);
  uint8_t* p1 = out + nunits * (16 / G) * 12;  // (two planes: plane 0 holds FP6 codes)
#define FASTBFP_WIDEN(NCH, K0, K1)                                                                                  \
  hipLaunchKernelGGL((k_widen<G, NCH, K0, K1>), grid, dim3(256), 0, s, mant, s1, exps, nunits, out, p1, out_exps)
  if (m <= 2) FASTBFP_WIDEN(1, kPlaneFP4, kPlaneFP6);
  else if (m <= 4) FASTBFP_WIDEN(1, kPlaneFP6, kPlaneFP6);
  else if (m <= 6) FASTBFP_WIDEN(2, kPlaneFP6, kPlaneLo2);
  else FASTBFP_WIDEN(2, kPlaneFP6, kPlaneFP6);
#undef FASTBFP_WIDEN
  return hipGetLastError();
}

}  // namespace

hipError_t launch_exps_twice(const uint8_t* exps, int64_t n, uint8_t* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_exps_twice, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, exps, n, out);
  return hipGetLastError();
}

void repack_shape(int64_t len, int g, int64_t* len_out, int* g_out) {
  *len_out = g < 16 ? len * (16 / g) : len;
  *g_out = g <= 16 ? 16 : 32;
}

hipError_t launch_repack(const uint8_t* mant, const uint8_t* exps, int64_t rows, int64_t len, int g, int m, int m_use,
                         bool packed, uint8_t* out_mant, uint8_t* out_exps, hipStream_t s) {
  int64_t len_out;
  int g_out;
  repack_shape(len, g, &len_out, &g_out);
  const int64_t units_out = len_out / 16, total = rows * units_out;
  if (total == 0) return hipSuccess;
  if (packed && m_use == m) {
    const uint32_t* expw = reinterpret_cast<const uint32_t*>(exps);
    const dim3 grid((unsigned)((total + 255) / 256));
    uint8_t* q1 = out_mant + total * 12;  // (two planes: plane 0 holds FP6 codes)
    switch ((m + 1) / 2) {
      case 1: hipLaunchKernelGGL(k_unpack<1>, grid, dim3(256), 0, s, mant, expw, total, out_mant, q1, out_exps); break;
      case 2: hipLaunchKernelGGL(k_unpack<2>, grid, dim3(256), 0, s, mant, expw, total, out_mant, q1, out_exps); break;
      case 3: hipLaunchKernelGGL(k_unpack<3>, grid, dim3(256), 0, s, mant, expw, total, out_mant, q1, out_exps); break;
      default: hipLaunchKernelGGL(k_unpack<4>, grid, dim3(256), 0, s, mant, expw, total, out_mant, q1, out_exps); break;
    }
    return hipGetLastError();
  }
  if (g < 16 && m_use == m) {
    const int64_t nunits = rows * (len / 16);
    return g == 4 ? widen<4>(mant, exps, nunits, m, out_mant, out_exps, s)
                  : widen<8>(mant, exps, nunits, m, out_mant, out_exps, s);
  }
  const Opnd src = make_opnd(mant, exps, rows, len, g, m, m_use, packed);
  uint8_t* p1 = out_mant + total * (plane_kind(m_use, 0) == kPlaneFP6 ? 12 : 8);
  const dim3 grid((unsigned)((total + 255) / 256));
  switch (g) {
    case 4: hipLaunchKernelGGL(k_repack<4>, grid, dim3(256), 0, s, src, units_out, total, m_use, out_mant, p1, out_exps);
      break;
    case 8: hipLaunchKernelGGL(k_repack<8>, grid, dim3(256), 0, s, src, units_out, total, m_use, out_mant, p1, out_exps);
      break;
    case 16: hipLaunchKernelGGL(k_repack<16>, grid, dim3(256), 0, s, src, units_out, total, m_use, out_mant, p1,
                                out_exps);
      break;
    case 32: hipLaunchKernelGGL(k_repack<32>, grid, dim3(256), 0, s, src, units_out, total, m_use, out_mant, p1,
                                out_exps);
      break;
    default: hipLaunchKernelGGL(k_repack<64>, grid, dim3(256), 0, s, src, units_out, total, m_use, out_mant, p1,
                                out_exps);
      break;
  }
  return hipGetLastError();
}

}  // namespace fastbfp
