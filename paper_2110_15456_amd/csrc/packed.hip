// packed.hip -- the paper's packed BFP storage (section V-D): every 2-bit
// chunk of a mantissa stored with its value's sign in 3 bits, chunk planes
// most significant first, and a 3-bit exponent per group of 16 above one
// base for the tensor.  Conversion (FP32 -> packed) and the inverse; the GEMM
// on packed operands runs on the general kernel (gemm_general.hip).
//
// Layout (include/fastbfp.h): NP = ceil(m / 2) planes; plane c holds chunk c
// of every value (q >> 2 (NP - 1 - c) & 3) as a 3-bit field -- the sign at bit 2
// (only for a nonzero chunk), the chunk at bits 0-1 -- value t of group gid at
// bits 3t .. 3t + 2 of the group's 6 bytes, group gid at byte offset
// (c * ngroups + gid) * 6.  The exponent array starts with a 32-bit word
// holding the tensor's largest exponent field E_max; base B = max(E_max - 7,
// 0); then group gid's offset e = E - B in bits 3 gid .. 3 gid + 2 of the
// stream that follows (64 groups per 24 bytes).  Group gid is converted with
// the shared exponent E = max(its largest exponent field, B).
#include "bfp_quant.h"

namespace fastbfp {

namespace {

__global__ void k_packed_header_clear(uint32_t* hdr) { *hdr = 0u; }

// hdr = max(hdr, the largest exponent field of x[0 .. 4 n4)).  At most
// kExpMaxBlocks blocks, each a contiguous run of rounds of 1024 16-byte granules
// (four independent loads per thread and round).  Two blocks a CU: with 2048
// blocks (64 KB each) the conversion of 8192 x 4096 at m = 4 took 74 us, with
// 1024 62, 512 57, 256 66 (and 62, 58, 60 with 1024-thread blocks at 512, 256,
// 128); on 2048^2 25 us with 1024 blocks, 16 with 512 or 256.  At least two rounds
// a block: below 1024 rounds the time goes with the number of blocks, each with an
// access to the one word.  The conversion of 1536 x 1024 took 12.8 us with single
// rounds, 10.1 with two, 10.8 with four; of 2048 x 1024 14.6, 10.9 and 11.8; of
// 512 x 1024 9.1, 8.8, 9.1.
constexpr int kExpMaxBlocks = 512, kExpMaxRounds = 2;
__global__ __launch_bounds__(256) void k_exponent_max(const u32x4* __restrict__ x, int64_t n4, int64_t rounds,
                                                      uint32_t* hdr) {
  uint32_t e = 0;
  for (int64_t r = blockIdx.x * rounds; r < (blockIdx.x + 1) * rounds; ++r) {
    u32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t i = 1024 * r + 256 * j + threadIdx.x;
      v[j] = i < n4 ? stream_load(x + i) : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      e = max(max(e, (v[j].x >> 23) & 0xFFu), (v[j].y >> 23) & 0xFFu);
      e = max(max(e, (v[j].z >> 23) & 0xFFu), (v[j].w >> 23) & 0xFFu);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) e = max(e, (uint32_t)__shfl_xor((int)e, off));
  __shared__ uint32_t red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t bmax = max(max(red[0], red[1]), max(red[2], red[3]));
    if (bmax > __atomic_load_n(hdr, __ATOMIC_RELAXED)) atomicMax(hdr, bmax);
  }
}

// One lane per group of 16 values along the rows, a wave per 64 groups.  The
// wave's 4 KB of input come into its LDS region by four direct global->LDS
// loads of 1 KB contiguous each; chunk c (16 bytes) of lane l's group lands in
// slot 4 l + (c ^ ((l / 4) % 4)), so that the 16 lanes served together on the
// read-back hit all 64 banks.  NP = ceil(m / 2) chunk planes.
template <int MODE, int NP>
__global__ __launch_bounds__(256) void k_quantize_packed(const float* __restrict__ x, int64_t ngroups, uint32_t m,
                                                         uint32_t key0, uint32_t key1, uint8_t* __restrict__ mant,
                                                         uint32_t* __restrict__ expw, uint32_t* status) {
  __shared__ __attribute__((aligned(16))) uint32_t stage[4][64 * 16];
  __shared__ uint32_t e3s[256];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t g0 = ((int64_t)blockIdx.x * 4 + wave) * 64;  // the wave's first group
  const int64_t gid = g0 + lane;
  const int nvalid = (int)max((int64_t)0, min((int64_t)64, ngroups - g0));
  const uint32_t base = packed_base(expw[0]);
  uint32_t e3 = 0;
  if (nvalid > 0) {
    typedef __attribute__((address_space(3))) void lds_void;
    const uint8_t* src = reinterpret_cast<const uint8_t*>(x) + g0 * 64;
    const int last = nvalid * 4 - 1;  // chunks of groups past the end reread the last valid one (unused)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int slot = 64 * k + lane, l = slot / 4, c = (slot % 4) ^ ((l / 4) % 4);
      __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(src + min(4 * l + c, last) * 16),
                                       (lds_void*)&stage[wave][64 * 4 * k], 16, 0, kStreamPolicy);
    }
    __builtin_amdgcn_s_waitcnt(0);  // the wave reads back what its own loads wrote
  }
  if (lane < nvalid) {
    uint32_t b[16];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(&stage[wave][4 * (4 * lane + (c ^ ((lane / 4) % 4)))]);
      b[4 * c] = v.x;
      b[4 * c + 1] = v.y;
      b[4 * c + 2] = v.z;
      b[4 * c + 3] = v.w;
    }
    // (a) the group's exponent, raised to the tensor base
    const uint32_t Eg = group_exponent<16>(b);
    const uint32_t E = max(Eg, base);
    if (status && Eg == 255u) atomicOr(status, 1u);
    uint32_t noise[4] = {0u, 0u, 0u, 0u};
    if (MODE == kStochastic) group_noise<16>((uint64_t)gid, key0, key1, noise);
    // (b)-(d) the magnitudes, split into 2-bit chunks with the sign
    const int align = magnitude_align<MODE>(m, E);
    const uint32_t qmax = (1u << m) - 1u;
    // Fields of values 0..7 and 8..15 of every plane, and the signs at bit 2 of
    // each field; a field takes its sign only if its chunk is nonzero.  (The
    // kernel is bound by this arithmetic beside its reads: with each field
    // made and shifted into 64 bits by itself the conversion of 8192^2 at m = 4
    // took 116 us, now 108.)
    uint32_t plane[NP][2], sgn[2] = {0u, 0u};
#pragma unroll
    for (int c = 0; c < NP; ++c) plane[c][0] = plane[c][1] = 0u;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const uint32_t q = value_magnitude<MODE, true>(b[t], align, noise[t >> 2], t, qmax);
      const int h = t >> 3, sh = 3 * (t & 7);
      sgn[h] |= (b[t] >> 31) << (sh + 2);
#pragma unroll
      for (int c = 0; c < NP; ++c) plane[c][h] |= ((q >> (2 * (NP - 1 - c))) & 3u) << sh;
    }
#pragma unroll
    for (int c = 0; c < NP; ++c) {
      uint16_t* dst = reinterpret_cast<uint16_t*>(mant + (c * ngroups + gid) * 6);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t p = plane[c][h];
        plane[c][h] = p | (sgn[h] & (((p << 1) | (p << 2)) & 0x924924u));
      }
      dst[0] = (uint16_t)plane[c][0];
      dst[1] = (uint16_t)((plane[c][0] >> 16) | (plane[c][1] << 8));
      dst[2] = (uint16_t)(plane[c][1] >> 8);
    }
    e3 = E - base;
  }
  // The wave's 64 exponent offsets, 192 bits: lane d < 6 assembles dword d
  // from the fields of lanes 32d/3 .. (32d + 31)/3.
  e3s[threadIdx.x] = e3;
  __syncthreads();
  if (lane < 6 && nvalid > 0) {
    uint32_t w = 0;
    for (int l = (32 * lane) / 3; l <= (32 * lane + 31) / 3; ++l) {
      const int sh = 3 * l - 32 * lane;  // -2 .. 31
      const uint32_t f = e3s[wave * 64 + l];
      w |= sh >= 0 ? f << sh : f >> -sh;
    }
    expw[1 + (g0 / 64) * 6 + lane] = w;
  }
}

// y = +-q * 2^(E - 127 - (m - 1)), a lane per four consecutive values (so that
// a wave stores 1 KB in one piece; a lane per group took 110 us on 64M values
// at m = 4), Q of them per lane: four where the tensor fills the card, so that as
// many loads are in flight; one on small tensors (kFewQuads, launch.h), whose time
// is one lane's.
template <int NP, int Q>
__global__ __launch_bounds__(256) void k_dequantize_packed(const uint8_t* __restrict__ mant,
                                                           const uint32_t* __restrict__ expw, int64_t ngroups, int m,
                                                           float* __restrict__ y) {
  const int64_t q0 = (int64_t)blockIdx.x * (256 * Q) + threadIdx.x, nquads = 4 * ngroups;
  const uint32_t base = packed_base(expw[0]);
  int q[Q][4], e[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int64_t at = min(q0 + 256 * i, nquads - 1), gid = at >> 2;  // (quads past the end reread the last one)
    const int k = (int)(at & 3);
    e[i] = (int)(base + packed_exponent_offset(expw, gid)) - 127 - (m - 1);
    uint32_t f[NP], neg = 0u;
#pragma unroll
    for (int c = 0; c < NP; ++c) {
      // fields 4k .. 4k + 3: 12 bits from bit 12 k of the group's 48
      const uint16_t* src = reinterpret_cast<const uint16_t*>(mant + (c * ngroups + gid) * 6);
      const int h = (3 * k) >> 2;
      const uint32_t w = (uint32_t)src[h] | ((uint32_t)src[min(h + 1, 2)] << 16);
      f[c] = (w >> (12 * k - 16 * h)) & 0xFFFu;
      neg |= f[c];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      int v = 0;
#pragma unroll
      for (int c = 0; c < NP; ++c) v = 4 * v + (int)((f[c] >> (3 * t)) & 3u);
      q[i][t] = (neg >> (3 * t + 2)) & 1u ? -v : v;
    }
  }
  typedef float f4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int64_t at = q0 + 256 * i;
    if (at < nquads)
      stream_store(reinterpret_cast<f4*>(y) + at, f4{ldexpf((float)q[i][0], e[i]), ldexpf((float)q[i][1], e[i]),
                                                     ldexpf((float)q[i][2], e[i]), ldexpf((float)q[i][3], e[i])});
  }
}

template <int MODE>
hipError_t quantize_packed_mode(const float* x, int64_t ngroups, int m, uint64_t seed, uint8_t* mant, uint32_t* expw,
                                uint32_t* status, hipStream_t s) {
  const dim3 grid((unsigned)((ngroups + 255) / 256));
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  switch ((m + 1) / 2) {
    case 1: hipLaunchKernelGGL((k_quantize_packed<MODE, 1>), grid, dim3(256), 0, s, x, ngroups, (uint32_t)m, k0, k1,
                               mant, expw, status); break;
    case 2: hipLaunchKernelGGL((k_quantize_packed<MODE, 2>), grid, dim3(256), 0, s, x, ngroups, (uint32_t)m, k0, k1,
                               mant, expw, status); break;
    case 3: hipLaunchKernelGGL((k_quantize_packed<MODE, 3>), grid, dim3(256), 0, s, x, ngroups, (uint32_t)m, k0, k1,
                               mant, expw, status); break;
    default: hipLaunchKernelGGL((k_quantize_packed<MODE, 4>), grid, dim3(256), 0, s, x, ngroups, (uint32_t)m, k0, k1,
                                mant, expw, status); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_quantize_packed(const float* x, int64_t rows, int64_t len, int m, int mode, uint64_t seed,
                                  uint8_t* mant, uint8_t* exps, uint32_t* status, hipStream_t s) {
  const int64_t n = rows * len, ngroups = n / 16;
  uint32_t* expw = reinterpret_cast<uint32_t*>(exps);
  // E_max of the tensor first (the base every group's exponent is stored above)
  hipLaunchKernelGGL(k_packed_header_clear, dim3(1), dim3(1), 0, s, expw);
  const int64_t n4 = n / 4;
  const int64_t all = (n4 + 1023) / 1024, even = (all + kExpMaxBlocks - 1) / kExpMaxBlocks;
  const int64_t rounds = even < kExpMaxRounds ? kExpMaxRounds : even;
  hipLaunchKernelGGL(k_exponent_max, dim3((unsigned)((all + rounds - 1) / rounds)), dim3(256), 0, s,
                     reinterpret_cast<const u32x4*>(x), n4, rounds, expw);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (mode == kStochastic) return quantize_packed_mode<kStochastic>(x, ngroups, m, seed, mant, expw, status, s);
  if (mode == kNearest) return quantize_packed_mode<kNearest>(x, ngroups, m, seed, mant, expw, status, s);
  return quantize_packed_mode<kTruncate>(x, ngroups, m, seed, mant, expw, status, s);
}

hipError_t launch_dequantize_packed(const uint8_t* mant, const uint8_t* exps, int64_t rows, int64_t len, int m,
                                    float* y, hipStream_t s) {
  const int64_t ngroups = rows * len / 16;
  const uint32_t* expw = reinterpret_cast<const uint32_t*>(exps);
  const int64_t nquads = 4 * ngroups;
#define FASTBFP_PDQ(NP, Q)                                                                                          \
  hipLaunchKernelGGL((k_dequantize_packed<NP, Q>), dim3((unsigned)((nquads + 256 * Q - 1) / (256 * Q))), dim3(256), \
                     0, s, mant, expw, ngroups, m, y)
#define FASTBFP_PDQ_Q(NP)                     \
  if (nquads < kFewQuads) FASTBFP_PDQ(NP, 1); \
  else FASTBFP_PDQ(NP, 4);                    \
  break
  switch ((m + 1) / 2) {
    case 1: FASTBFP_PDQ_Q(1);
    case 2: FASTBFP_PDQ_Q(2);
    case 3: FASTBFP_PDQ_Q(3);
    default: FASTBFP_PDQ_Q(4);
  }
#undef FASTBFP_PDQ_Q
#undef FASTBFP_PDQ
  return hipGetLastError();
}

}  // namespace fastbfp
