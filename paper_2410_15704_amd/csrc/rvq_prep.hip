// Derived codebook data.
//   norms  : squared norms of the codewords, the constant term of ||c||^2 - 2 r.c
// and, for the matrix-core screen (dhat == 32), per stage:
//   perm   : the codewords ordered by norm (ties by index), -1 where a repeat would stand
//   perm16 : position pos = tile * 32 + row -> codeword: the same order with the repeats left out and
//            the others closed up, as uint16, 0xffff for the padding at the end (what the kernels keep
//            in LDS)
//   C16    : fp16(-2 c) of the codeword at each position, laid out exactly as the A operand of
//            v_mfma_f32_32x32x16_f16 is read, so the kernel copies it into LDS linearly and a
//            lane's operand is one 16-byte LDS read
//   groupA : for every (tile, lane half) group of 16 rows, the largest A = ||S 2c|| and the largest rounding error
//            ||fp16(S 2c) - S 2c||, in one word (rvq_bound_group)
//   normp  : S T ||c||^2 - kappa/8 * A^2, in the order a lane's 16 accumulator registers want (the term taken off
//            bounds the accumulation error of the group's scores)
//   stats  : per stage 8 floats: [1] usable flag (finite codebook); [3] S and [4] T, the powers of two the
//            codebook and the residuals are scaled by before rounding to fp16 (chosen so that the largest
//            |S a| lies in [2^13, 2^14) and T = S / 2); [5] the largest |a|
// A codeword that repeats an earlier one exactly can never win (ties go to the smallest index): it
// gets no position.
// Ordering by norm keeps the norms inside a group close to each other, which is what makes the
// per-group error bound of the screen tight when a few codewords are much longer than the rest.
#include "rvq_internal.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// one thread per codeword; the norm is summed in double and rounded once to float
__global__ void norms_kernel(const float *__restrict__ C, float *__restrict__ norms, int dhat,
                             int64_t first, int64_t count) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float *c = C + (first + i) * dhat;
  double acc = 0.0;
  for (int j = 0; j < dhat; ++j) acc += (double)c[j] * (double)c[j];
  norms[first + i] = (float)acc;
}

// dhat == 32, one lane per (codeword, channel); ema_finish32_kernel does the same for the codewords it makes
__global__ __launch_bounds__(256) void prep_rows32_kernel(const float *__restrict__ C, int stage_begin, int stage_end,
                                                          const RvqRows32 p) {
  const int64_t r = (int64_t)blockIdx.x * 8 + (threadIdx.x >> 5);  // row among the stages' rows
  const int j = threadIdx.x & 31;
  if (r >= (int64_t)(stage_end - stage_begin) * p.K) return;
  const int stage = stage_begin + (int)(r / p.K), k = (int)(r % p.K);
  rvq_prep_row32(p, stage, k, j, C[((int64_t)stage * p.K + k) * 32 + j]);
}

// Position of every codeword in the order (norm, index) of its stage, and whether it is an exact repeat of an
// earlier one (equal rows have equal norms).  A repeat leaves its position empty; screen_tile_kernel
// closes the ranks.  A workgroup takes RANK_CW codewords, a wavefront each at the end; the K norms are
// read once for all of them.
// Codewords of equal norm are mostly repeats of each other (dead ones are all zero), so a codeword is
// compared with the first one of its norm, in one round trip, and with the others only where that row differs.
// (One after the other, codebooks on the unit sphere, hundreds of codewords to a norm, took 372 us for eight
// stages of 2048, of -1 and 1 835; now 47 and 99.)
// (Compared by the threads that met the equal norm, element after element, each pair cost 32 round trips one
// after the other: 23 us for a stage of 2048 with some zero codewords, 4.8 now; eight
// stages 50 -> 15 us, of 4096 codewords 215 -> 38.)
constexpr int RANK_CW = 4;
__global__ __launch_bounds__(64 * RANK_CW) void rank_kernel(const float *__restrict__ C, const float *__restrict__ norms,
                                                            const float *__restrict__ rowmax, int K, int Kpad,
                                                            int stage_begin, int32_t *__restrict__ perm) {
  __shared__ int cnt_s[RANK_CW][RANK_CW], tie_s[RANK_CW][RANK_CW];  // [wavefront][codeword]
  const int per_stage = (K + RANK_CW - 1) / RANK_CW;
  const int stage = stage_begin + blockIdx.x / per_stage;
  const int k0 = blockIdx.x % per_stage * RANK_CW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float *n = norms + (int64_t)stage * K;
  float nk[RANK_CW];
  int cnt[RANK_CW], tie[RANK_CW];  // codewords in front; the first one of the same norm
#pragma unroll
  for (int i = 0; i < RANK_CW; ++i) {
    nk[i] = n[min(k0 + i, K - 1)];
    cnt[i] = 0;
    tie[i] = 0x7fffffff;
  }
#pragma unroll 8
  for (int j = threadIdx.x; j < K; j += 64 * RANK_CW) {
    const float nj = n[j];
#pragma unroll
    for (int i = 0; i < RANK_CW; ++i) {
      const bool same = nj == nk[i] && j < k0 + i;
      cnt[i] += (nj < nk[i] || same) ? 1 : 0;
      tie[i] = min(tie[i], same ? j : 0x7fffffff);
    }
  }
#pragma unroll
  for (int i = 0; i < RANK_CW; ++i) {
    for (int o = 32; o > 0; o >>= 1) {
      cnt[i] += __shfl_xor(cnt[i], o, 64);
      tie[i] = min(tie[i], __shfl_xor(tie[i], o, 64));
    }
    if (lane == 0) {
      cnt_s[wave][i] = cnt[i];
      tie_s[wave][i] = tie[i];
    }
  }
  __syncthreads();
  const int k = k0 + wave;
  if (k >= K) return;
  int pos = 0, first = 0x7fffffff;
#pragma unroll
  for (int w = 0; w < RANK_CW; ++w) {
    pos += cnt_s[w][wave];
    first = min(first, tie_s[w][wave]);
  }
  bool found = false;
  if (first < K) {  // uniform over the wavefront
    const float *Cs = C + (int64_t)stage * K * 32;
    const float c = Cs[(int64_t)k * 32 + (lane & 31)];
    found = __all(Cs[(int64_t)first * 32 + (lane & 31)] == c);
    // Different rows of equal norm (codebooks on a sphere, of few values): every later one of the norm that has the
    // same largest element too, a candidate per lane, until a piece of it differs.
    const float *m = rowmax + (int64_t)stage * K;
    const float nw = n[k], mw = m[k];
    const f32x4 *rows = reinterpret_cast<const f32x4 *>(Cs);
    constexpr int U = 4;
    for (int j0 = first + 1 + lane; !found && __any(j0 < k); j0 += 64 * U) {
      bool same[U], any = false;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = min(j0 + 64 * u, K - 1);
        same[u] = n[j] == nw && m[j] == mw && j0 + 64 * u < k;
        any = any || same[u];
      }
      for (int p = 0; p < 8 && __any(any); ++p) {
        const f32x4 own = rows[(int64_t)k * 8 + p];
        f32x4 c4[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c4[u] = rows[(int64_t)(same[u] ? j0 + 64 * u : k) * 8 + p];
        any = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          same[u] = same[u] && c4[u][0] == own[0] && c4[u][1] == own[1] && c4[u][2] == own[2] && c4[u][3] == own[3];
          any = any || same[u];
        }
      }
      found = __any(any);
    }
  }
  if (lane == 0) perm[(int64_t)stage * Kpad + pos] = found ? -1 : k;
}

// One workgroup per (stage, tile of 32 positions), one lane per (position, channel): the fp16
// operands, perm16, the error statistics, and per (tile, lane half) group normp and groupA.
// The repeats' empty positions are closed up here, by a prefix sum over the stage's order in every
// workgroup (one entry per thread and 1024 codewords).  Left open they move codewords of nearly equal norm
// into different groups: dead codewords repeat the zero vector, a short residual's candidates then
// lie in two groups instead of one, and the second ones overflow the search's queues (a stage of 1024
// codewords, 3 of them repeats: 62 us for 177441 vectors closed up, 207 us with the positions left empty).
// Operand order: tile t = pos / 32, row m = pos % 32; the lane (m, h) of matrix-core instruction
// q holds dims 16 h + 8 q .. + 7 of row m, as two 8-byte pieces at
// (((t * 2 + q) * 2 + piece) * 64 + h * 32 + m) * 8.
__global__ __launch_bounds__(1024) void screen_tile_kernel(
    const float *__restrict__ C, const int32_t *__restrict__ perm,
    const float *__restrict__ rowmax, int K, int Kpad, int stage_begin, float kappa,
    uint16_t *__restrict__ C16, uint16_t *__restrict__ C16s, uint16_t *__restrict__ perm16,
    float *__restrict__ normp,
    uint32_t *__restrict__ groupA, float *__restrict__ stats) {
  __shared__ float red[16];
  __shared__ int wave_held[16], here[32];  // codewords of the tile's rows, -1: none
  __shared__ float nrm[32], len[32], rnd[32];
  const int tiles = Kpad / 32;
  const int stage = stage_begin + blockIdx.x / tiles;
  const int t = blockIdx.x % tiles;
  const int m = threadIdx.x >> 5, j = threadIdx.x & 31;
  const int pos = t * 32 + m;
  // the stage's largest |2 c| (infinity: some element is not finite)
  float mxa = 0.f;
  for (int i = threadIdx.x; i < K; i += 1024) mxa = fmaxf(mxa, rowmax[(int64_t)stage * K + i]);
  for (int o = 32; o > 0; o >>= 1) mxa = fmaxf(mxa, __shfl_xor(mxa, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mxa;
  // this thread's entries of the order, and how many codewords they hold
  const int32_t *order = perm + (int64_t)stage * Kpad;
  const int per = (Kpad + 1023) / 1024;
  const int i0 = min((int)threadIdx.x * per, Kpad), i1 = min(i0 + per, Kpad);
  int held = 0;
  for (int i = i0; i < i1; ++i) held += order[i] >= 0 ? 1 : 0;
  int before = held;  // inclusive sum over the wavefront
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(before, o, 64);
    before += (int)(threadIdx.x & 63) >= o ? v : 0;
  }
  if ((threadIdx.x & 63) == 63) wave_held[threadIdx.x >> 6] = before;
  if (threadIdx.x < 32) here[threadIdx.x] = -1;
  __syncthreads();
  before -= held;  // codewords in front of this thread's
  for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) before += wave_held[w];
  if (before < t * 32 + 32 && before + held > t * 32)
    for (int i = i0; i < i1; ++i)
      if (order[i] >= 0) {
        if ((before >> 5) == t) here[before & 31] = order[i];
        ++before;
      }
  __syncthreads();
  mxa = red[0];
  for (int i = 1; i < 16; ++i) mxa = fmaxf(mxa, red[i]);
  const bool finite = mxa <= 1.0e30f;  // (and S at its best, see below)
  // S: power of two that brings the stage's largest |2c| into [2^13, 2^14); T = S / 2
  int ex = 0;
  if (mxa > 0.f && finite) (void)frexpf(mxa, &ex);  // mxa = f * 2^ex, f in [0.5, 1)
  ex = ex < -100 ? -100 : (ex > 100 ? 100 : ex);
  const float S = ldexpf(1.0f, 14 - ex);
  const float T = 0.5f * S;
  if (t == 0 && threadIdx.x == 0) {
    if (!finite) stats[stage * 8 + 1] = 0.0f;  // the screen cannot be used for this stage
    stats[stage * 8 + 3] = S;
    stats[stage * 8 + 4] = T;
    stats[stage * 8 + 5] = finite ? mxa : 0.f;
  }
  const int k = here[m];
  float a = 0.f;
  if (k >= 0) a = -2.0f * S * C[((int64_t)stage * K + k) * 32 + j];  // exact in fp32
  // values below the smallest normal half are dropped so that the error bound does not depend
  // on how the matrix cores treat subnormal inputs
  const bool flushed = fabsf(a) < 6.103515625e-5f;
  const __half hv = flushed ? __float2half_rn(0.f) : __float2half_rn(a);
  const double back = (double)__half2float(hv);
  const double a2 = rvq_row_sum32((double)a * a);
  const double e2 = rvq_row_sum32((back - a) * (back - a));  // rounding error, elements dropped among it
  // the 16-byte operand of a lane is stored as two 8-byte pieces 512 bytes apart, so that the
  // kernel fetches it with two conflict-free 8-byte LDS reads
  const int h = j >> 4, q = (j >> 3) & 1, e = j & 7;
  // row m of tile t sits in slot m ^ (t & 31): the sweep still reads a permutation of all
  // slots (no conflict), and lanes that fetch the same row of different tiles while re-scoring
  // no longer collide on one LDS bank
  uint16_t *dst = C16 + ((int64_t)stage * Kpad + (int64_t)t * 32) * 32;
  dst[((((q * 2 + (e >> 2)) * 64) + h * 32 + (m ^ (t & 31))) * 4) + (e & 3)] = __half_as_ushort(hv);
  // and as the two 16-row A operands of v_mfma_f32_16x16x32_f16: lane (channel group, row)
  C16s[((int64_t)stage * Kpad + (int64_t)t * 32) * 32 + (((m >> 4) * 64 + (j >> 3) * 16 + (m & 15)) * 8) + e] =
      __half_as_ushort(hv);
  if (j == 0) {
    perm16[(int64_t)stage * Kpad + pos] = k < 0 ? (uint16_t)0xffff : (uint16_t)k;
    if (k >= 0) {
      nrm[m] = (float)(a2 * 0.25 * ((double)T / (double)S));  // S T ||c||^2
      len[m] = (float)(sqrt(a2) * (1.0 + 1e-6));              // ||S 2c||, rounded up
      rnd[m] = (float)(sqrt(e2) * (1.0 + 1e-6));
    } else {
      nrm[m] = 1e30f;  // padding can never come near the minimum
      len[m] = 0.f;
      rnd[m] = 0.f;
    }
  }
  __syncthreads();
  if (threadIdx.x < 32) {
    // group hh of the tile: rows 8 b + 4 hh + i, b, i = 0..3, which are the 16 accumulator
    // registers rr = 4 b + i of the lanes of half hh
    const int hh = threadIdx.x >> 4, rr = threadIdx.x & 15;
    float A = 0.f, D = 0.f;
    for (int r2 = 0; r2 < 16; ++r2) {
      const int row = 8 * (r2 >> 2) + 4 * hh + (r2 & 3);
      A = fmaxf(A, len[row]);
      D = fmaxf(D, rnd[row]);
    }
    // kappa * (S T ||c||^2) = kappa / 4 * (T / S) * ||S 2c||^2 = kappa / 8 * A^2
    const float shift = 0.125f * kappa * A * A * 1.000001f;
    const int mm = 8 * (rr >> 2) + 4 * hh + (rr & 3);
    normp[(int64_t)stage * Kpad + (int64_t)t * 32 + hh * 16 + rr] = nrm[mm] - shift;
    if (rr == 0) groupA[(int64_t)stage * (Kpad / 16) + t * 2 + hh] = finite ? rvq_bound_group(A, D) : 0u;
  }
}

}  // namespace

hipError_t rvq_launch_prepare_codebook(const rvq_ctx *ctx, int stage_begin, int stage_end, bool rows_done,
                                       hipStream_t s) {
  const int64_t K = ctx->cfg.K;
  const int ns = stage_end - stage_begin;
  const int block = 256;
  auto blocks = [&](int64_t n) { return dim3((unsigned)((n + block - 1) / block)); };
  if (!ctx->C16) {  // dhat != 32: the norms are all that is derived
    hipLaunchKernelGGL(norms_kernel, blocks(ns * K), dim3(block), 0, s, ctx->C, ctx->norms,
                       ctx->cfg.dhat, (int64_t)stage_begin * K, (int64_t)ns * K);
    return hipGetLastError();
  }
  if (!rows_done)
    hipLaunchKernelGGL(prep_rows32_kernel, dim3((unsigned)((ns * K + 7) / 8)), dim3(256), 0, s, ctx->C,
                       stage_begin, stage_end, rvq_rows32(ctx));
  hipLaunchKernelGGL(rank_kernel, dim3((unsigned)(ns * ((K + RANK_CW - 1) / RANK_CW))), dim3(64 * RANK_CW), 0, s,
                     ctx->C, ctx->norms, ctx->rowmax, (int)K, ctx->Kpad, stage_begin, ctx->perm);
  hipLaunchKernelGGL(screen_tile_kernel, dim3((unsigned)(ns * (ctx->Kpad / 32))), dim3(1024), 0, s,
                     ctx->C, ctx->perm, ctx->rowmax, (int)K, ctx->Kpad, stage_begin, ctx->kappa,
                     ctx->C16, ctx->C16s, ctx->perm16, ctx->normp, ctx->groupA, ctx->stats);
  return hipGetLastError();
}
