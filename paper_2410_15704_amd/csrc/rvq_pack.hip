// Packed code storage (Section 3.2: the compression rate counts log2(K) bits per code): the
// depth codes of one (token, group) become a record of ceil(depth * b / 8) bytes, b = bits per
// code, code i in bits [b i, b i + b) of the record taken as a little-endian integer.
#include "rvq_internal.h"

namespace {

// the general case: one thread per record; a record is at most 16 * 15 bits = 30 bytes
__global__ __launch_bounds__(256) void pack_kernel(const int16_t *__restrict__ codes, int64_t V,
                                                   int depth, int bits, int rec, int K,
                                                   uint8_t *__restrict__ packed) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= V) return;
  const int16_t *c = codes + e * depth;
  uint8_t *o = packed + e * rec;
  unsigned long long acc = 0;  // bits not yet written, low end first
  int have = 0, w = 0;
  for (int i = 0; i < depth; ++i) {
    int k = c[i];
    k = k < 0 ? 0 : (k >= K ? K - 1 : k);
    acc |= (unsigned long long)(unsigned)k << have;
    have += bits;
    while (have >= 8) {
      o[w++] = (uint8_t)(acc & 0xffu);
      acc >>= 8;
      have -= 8;
    }
  }
  if (have > 0) o[w++] = (uint8_t)(acc & 0xffu);
}

// Records of eight codes end on a byte, so all records together are one stream of b-bit codes.  A workgroup
// takes 256 records: a thread fetches one as a 16-byte word, and then every thread makes whole 32-bit words of
// the stream from the codes in LDS (256 records are 64 b words).  One record after the other in 2-byte
// loads and 1-byte stores, a thread's loads one round trip each, it was 4.2 million records 55 us, now 28
// (110 MB: 4 TB/s), and 1 us more of an append of one row (31.4 -> 30.5 with the encode).
// B: bits per code, 0: `bits`.
constexpr int PACK_RECORDS = 256;
template <int B>
__global__ __launch_bounds__(PACK_RECORDS) void pack8_kernel(const int16_t *__restrict__ codes, int64_t V, int bits,
                                                             int K, uint8_t *__restrict__ packed) {
  __shared__ __align__(16) uint16_t sm[PACK_RECORDS * 8 + 40];  // (the last word may look 32 codes ahead)
  const int b = B ? B : bits;
  const int64_t e0 = (int64_t)blockIdx.x * PACK_RECORDS;
  const int n = (int)min((int64_t)PACK_RECORDS, V - e0);
  uint4 w = {0u, 0u, 0u, 0u};
  if ((int)threadIdx.x < n) {
    w = reinterpret_cast<const uint4 *>(codes)[e0 + threadIdx.x];
    uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int lo = min(max((int)(int16_t)(u[i] & 0xffffu), 0), K - 1), hi = min(max((int)u[i] >> 16, 0), K - 1);
      u[i] = (uint32_t)lo | ((uint32_t)hi << 16);
    }
    w = make_uint4(u[0], u[1], u[2], u[3]);
  }
  reinterpret_cast<uint4 *>(sm)[threadIdx.x] = w;
  if (threadIdx.x < 20) reinterpret_cast<uint32_t *>(sm + PACK_RECORDS * 8)[threadIdx.x] = 0u;
  __syncthreads();
  const int bytes = n * b;
  uint32_t *out = reinterpret_cast<uint32_t *>(packed + e0 * b);
  const uint32_t inv = (1u << 20) / (uint32_t)b + 1u;  // bit / b for bit < 2^15, b <= 15
  for (int i = threadIdx.x; i * 4 < bytes; i += PACK_RECORDS) {
    const uint32_t bit = 32u * (uint32_t)i, c0 = (bit * inv) >> 20;
    int have = (int)(c0 * (uint32_t)b) - (int)bit;  // where code c0 starts, <= 0
    unsigned long long acc = 0;
#pragma unroll
    for (int t = 0; t < (B ? 31 / B + 2 : 1); ++t) {
      const unsigned long long c = sm[c0 + t];
      acc |= have < 0 ? c >> -have : c << have;
      have += b;
    }
    if (!B)
      for (int t = 1; have < 32; ++t, have += b) acc |= (unsigned long long)sm[c0 + t] << have;
    const uint32_t word = (uint32_t)acc;
    if (i * 4 + 4 <= bytes) {
      out[i] = word;
    } else {
      for (int t = 0; t < bytes - i * 4; ++t) reinterpret_cast<uint8_t *>(out + i)[t] = (uint8_t)(word >> (8 * t));
    }
  }
}

__global__ __launch_bounds__(256) void unpack_kernel(const uint8_t *__restrict__ packed, int64_t V,
                                                     int depth, int bits, int rec,
                                                     int16_t *__restrict__ codes) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= V) return;
  const uint8_t *p = packed + e * rec;
  int16_t *c = codes + e * depth;
  unsigned long long acc = 0;
  int have = 0, r = 0;
  for (int i = 0; i < depth; ++i) {
    while (have < bits) {
      acc |= (unsigned long long)p[r++] << have;
      have += 8;
    }
    c[i] = (int16_t)(acc & ((1u << bits) - 1u));
    acc >>= bits;
    have -= bits;
  }
}

}  // namespace

hipError_t rvq_launch_pack(const rvq_ctx *ctx, const int16_t *dCodes, int64_t N, uint8_t *dPacked,
                           hipStream_t s) {
  const rvq_config &c = ctx->cfg;
  const int64_t V = N * ctx->G;
  const int64_t grid64 = (V + 255) / 256;
  if (grid64 > 0x7fffffffLL) return hipErrorInvalidValue;
  if (c.depth == 8) {
    static_assert(PACK_RECORDS == 256, "the grid is that of 256 records a workgroup");
#define RVQ_PACK8(B)                                                                                        \
  hipLaunchKernelGGL(pack8_kernel<B>, dim3((unsigned)grid64), dim3(PACK_RECORDS), 0, s, dCodes, V,            \
                     rvq_code_bits(c.K), c.K, dPacked)
    switch (rvq_code_bits(c.K)) {
      case 10: RVQ_PACK8(10); break;
      case 11: RVQ_PACK8(11); break;
      case 12: RVQ_PACK8(12); break;
      default: RVQ_PACK8(0); break;
    }
#undef RVQ_PACK8
    return hipGetLastError();
  }
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)grid64), dim3(256), 0, s, dCodes, V, c.depth,
                     rvq_code_bits(c.K), rvq_record_bytes(c.depth, c.K), c.K, dPacked);
  return hipGetLastError();
}

hipError_t rvq_launch_unpack(const rvq_ctx *ctx, const uint8_t *dPacked, int64_t N, int16_t *dCodes,
                             hipStream_t s) {
  const rvq_config &c = ctx->cfg;
  const int64_t V = N * ctx->G;
  const int64_t grid64 = (V + 255) / 256;
  if (grid64 > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(unpack_kernel, dim3((unsigned)grid64), dim3(256), 0, s, dPacked, V, c.depth,
                     rvq_code_bits(c.K), rvq_record_bytes(c.depth, c.K), dCodes);
  return hipGetLastError();
}
