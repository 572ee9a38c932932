// gemm_parts.hip -- adds up the partial sums of a GEMM whose K was taken in
// parts (gemm_mx.h), into FP32 C or straight into BFP by the converter of
// section V-C.
//
// Bound by the latency of reading the parts (they sit in L2 or the Infinity
// Cache: a few MB just written), so with many parts the parts of one output
// are spread over the threads of a block.  The order is fixed: with more than
// kFlat parts, kGroups runs of consecutive parts, each added in order, then
// the runs in order; both kernels add in that order, so the converted output is
// the conversion of the FP32 one.
#include "bfp_quant.h"

namespace fastbfp {

namespace {

constexpr int kFlat = 8, kGroups = 8;

// The sum of parts [p0, p1) at `src`, `stride` values apart.
__device__ __forceinline__ v4f sum_run(const float* src, int64_t stride, int p0, int p1) {
  v4f v = v4f{0.f, 0.f, 0.f, 0.f};
  int p = p0;
  for (; p + 4 <= p1; p += 4) {  // four loads in flight
    v4f t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = *reinterpret_cast<const v4f*>(src + (p + k) * stride);
#pragma unroll
    for (int k = 0; k < 4; ++k) v += t[k];
  }
  for (; p < p1; ++p) v += *reinterpret_cast<const v4f*>(src + p * stride);
  return v;
}

// Z threads per four outputs (1, or kGroups: thread z adds run z).
template <int Z>
__global__ __launch_bounds__(256) void k_parts_sum(const float* __restrict__ src, int parts, int64_t quads, int N,
                                                   int ld, float* __restrict__ C, int64_t ldc) {
  constexpr int Q = 256 / Z;  // outputs / 4 per block
  __shared__ v4f run[Z > 1 ? Z : 1][Q];
  const int z = threadIdx.x / Q, i = threadIdx.x % Q;
  const int64_t q = (int64_t)blockIdx.x * Q + i, stride = 4 * quads;
  v4f v = v4f{0.f, 0.f, 0.f, 0.f};
  if (q < quads) {
    const int per = (parts + Z - 1) / Z;
    v = sum_run(src + 4 * q, stride, min(parts, z * per), min(parts, (z + 1) * per));
  }
  if constexpr (Z > 1) {
    run[z][i] = v;
    __syncthreads();
    if (z > 0) return;
#pragma unroll
    for (int k = 1; k < Z; ++k) v += run[k][i];
  }
  if (q >= quads) return;
  const int64_t row = 4 * q / ld;
  const int col = (int)(4 * q - row * ld);
  float* p = C + row * ldc + col;
  if ((ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0 && col + 3 < N) {
    *reinterpret_cast<v4f*>(p) = v;
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (col + t < N) p[t] = v[t];
  }
}

// One thread per group of 16 outputs.
template <int MODE, int NCH, int P0, int P1>
__global__ __launch_bounds__(256) void k_parts_convert(const float* __restrict__ src, int parts, int64_t ngroups,
                                                       uint32_t m, uint32_t key0, uint32_t key1,
                                                       uint8_t* __restrict__ mant0, uint8_t* __restrict__ mant1,
                                                       uint8_t* __restrict__ exps, uint32_t* status) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (gid >= ngroups) return;
  const int64_t stride = 16 * ngroups;
  uint32_t b[16];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float* s = src + 16 * gid + 4 * k;
    v4f v;
    if (parts <= kFlat) {
      v = sum_run(s, stride, 0, parts);
    } else {
      const int per = (parts + kGroups - 1) / kGroups;
      v = sum_run(s, stride, 0, per);
      for (int z = 1; z < kGroups; ++z) v += sum_run(s, stride, min(parts, z * per), min(parts, (z + 1) * per));
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) b[4 * k + t] = __float_as_uint(v[t]);
  }
  uint32_t w[NCH][3], E, s_lo, s_hi;
  bool nonfinite;
  quantize_group<16, MODE, NCH, false, P0, P1>(b, m, (uint64_t)gid, key0, key1, w, E, nonfinite, s_lo, s_hi);
  exps[gid] = (uint8_t)E;
  store_plane<16, P0 != kPlaneFP6>(mant0, gid, w[0]);
  if (NCH == 2) store_plane<16, P1 != kPlaneFP6>(mant1, gid, w[NCH - 1]);
  if (status && nonfinite) atomicOr(status, 1u);
}

template <int MODE, int NCH, int P0, int P1>
hipError_t convert_t(const float* p, int parts, int64_t ngroups, int m, uint64_t seed, uint8_t* mant, uint8_t* exps,
                     uint32_t* status, hipStream_t s) {
  hipLaunchKernelGGL((k_parts_convert<MODE, NCH, P0, P1>), dim3((unsigned)((ngroups + 255) / 256)), dim3(256), 0, s, p,
                     parts, ngroups, (uint32_t)m, (uint32_t)seed, (uint32_t)(seed >> 32), mant,
                     mant + ngroups * plane_group_bytes(16, m, 0), exps, status);
  return hipGetLastError();
}

template <int MODE>
hipError_t convert_mode(const float* p, int parts, int64_t ngroups, int m, uint64_t seed, uint8_t* mant,
                        uint8_t* exps, uint32_t* status, hipStream_t s) {
  if (m <= 2) return convert_t<MODE, 1, kPlaneFP4, kPlaneFP6>(p, parts, ngroups, m, seed, mant, exps, status, s);
  if (m <= 4) return convert_t<MODE, 1, kPlaneFP6, kPlaneFP6>(p, parts, ngroups, m, seed, mant, exps, status, s);
  if (m <= 6) return convert_t<MODE, 2, kPlaneFP6, kPlaneLo2>(p, parts, ngroups, m, seed, mant, exps, status, s);
  return convert_t<MODE, 2, kPlaneFP6, kPlaneFP6>(p, parts, ngroups, m, seed, mant, exps, status, s);
}

}  // namespace

hipError_t launch_parts_sum(const float* p, int parts, int64_t M, int64_t N, float* C, int64_t ldc, hipStream_t s) {
  const int64_t ld = gemm_plan_ld(N), quads = M * ld / 4;
  if (parts <= kFlat)
    hipLaunchKernelGGL(k_parts_sum<1>, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, p, parts, quads, (int)N,
                       (int)ld, C, ldc);
  else
    hipLaunchKernelGGL(k_parts_sum<kGroups>, dim3((unsigned)((quads + 256 / kGroups - 1) / (256 / kGroups))), dim3(256),
                       0, s, p, parts, quads, (int)N, (int)ld, C, ldc);
  return hipGetLastError();
}

// N a multiple of 16 (so that a part's rows are N apart).
hipError_t launch_parts_convert(const float* p, int parts, int64_t M, int64_t N, int c_m, int mode, uint64_t seed,
                                uint8_t* c_mant, uint8_t* c_exp, uint32_t* status, hipStream_t s) {
  const int64_t ngroups = M * (N / 16);
  if (mode == kStochastic)
    return convert_mode<kStochastic>(p, parts, ngroups, c_m, seed, c_mant, c_exp, status, s);
  if (mode == kNearest) return convert_mode<kNearest>(p, parts, ngroups, c_m, seed, c_mant, c_exp, status, s);
  return convert_mode<kTruncate>(p, parts, ngroups, c_m, seed, c_mant, c_exp, status, s);
}

}  // namespace fastbfp
