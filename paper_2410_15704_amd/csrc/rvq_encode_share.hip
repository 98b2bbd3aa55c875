// Encode for calls between a few vectors and a full chip (dhat == 32): a workgroup's sixteen
// wavefronts share the CODEBOOK of a stage and all work on the same tokens.
//
// encode_screen_kernel gives every wavefront its own 64 or 128 tokens and lets it sweep the whole
// stage: whatever the number of tokens, a stage takes as long as one such sweep (23 us).  Here
// wavefront w keeps codewords [w K / 16, (w + 1) K / 16) of the stage in registers, as matrix-core A
// operands with their norms as accumulator inputs, and the tokens pass by in tiles of 16 (one
// 16-byte LDS read per lane and tile): a wavefront's part of a tile is 1/16 of the sweep, so the time
// follows the number of tokens.  Tokens per workgroup: ceil(vectors / CUs), up to SHR_TOKENS.
//
// Search, exact as in the other kernels (Algorithm 1: nearest codeword, smallest index on ties):
//  1. Sweep.  v_mfma_f32_16x16x32_f16 on fp16(S (-2c)) and fp16(T r) gives a lane four scores of one
//     token per instruction; per (32 codewords, lane) only the smallest of its eight is kept, in a
//     register.  With the error bound of the fp16 screen (|score - exact| <= e = gx B + k4 A^2, B and A the largest
//     of the wavefront's norm-sorted codewords, rvq_bound_group; the stored norms have the group's own k4 A^2
//     taken off) the smallest score gives an upper bound on the exact minimum;
//     the least over the wavefronts, found with lane exchanges and one LDS minimum per (wavefront,
//     token), is the token's threshold.
//  2. Pick.  A lane whose kept minimum reaches below its token's threshold marks those eight
//     codewords as candidates, one bit in LDS (1.03 groups per search).
//  3. Resolve.  Eight lanes own a token, four channels each: exact fp32 direct-form distances of the
//     marked codewords, added in the order of encode_exact_kernel, smallest index on ties; the
//     residual is updated in fp32 and turned into the next stage's fp16 operand.  The threshold
//     includes the rounding of those fp32 distances, so the codeword that the exact path
//     picks is always among the candidates and the codes, std and residuals equal the exact path's
//     bit for bit.  (In calls of more than SHR_FEW vectors, two distances closer than their rounding are
//     compared once more, summed in encode_screen_kernel's order, so that the two agree there.)
//  A token whose residual does not fit fp16 is searched exactly over the whole stage by the workgroup.
//
// What bounds it: up to 16 tokens per workgroup (FEW) a stage takes 4.1 us, a chain of latencies (the next
// stage's 128 KiB of operands through the CU's L1, the first rows of exact distances, four barriers
// and their LDS round trips).  With more tokens the general form: at 188 per workgroup the vector units
// issue in 59 % of the cycles (matrix cores 15 %, L1 address path 31 %); the rest is the sixteen
// wavefronts in step at a barrier per pair of tiles, and what a stage costs once.  At TPW = 4 its 128
// registers do not hold everything: 22 values per lane are spilled (9 at TPW = 2, 4 at TPW = 1).
// Measured, rows of 32 groups, K = 2048, depth 8, before (small-batch or one-token-per-lane kernel) and
// now: 32 rows 55 -> 34 us, 48 rows 83 -> 34, 128 rows 157 -> 37, 512 rows 203 -> 66, 1500 rows
// 217 -> 120, 2500 rows 217 -> 178 us; K = 4096, 32 rows of 128 groups 156 -> 71 us, 300 rows 192 us.
#include <algorithm>
#include <type_traits>

#include "rvq_internal.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int SHR_THREADS = 1024;
constexpr int SHR_WAVES = SHR_THREADS / 64;
constexpr int SHR_TOKENS = 512;               // most tokens of a workgroup (152 KB of LDS)
constexpr int SHR_PASS = SHR_THREADS / 8;     // tokens per pass of the resolve step
constexpr int SHR_ROWS = 64;                  // most rows whose std a workgroup computes itself
// Calls of at most this many vectors agree with the exact path bit for bit, never touch the caller's
// std scratch (what rvq_encode_static promises) and do not update the context's statistics; larger ones
// agree with encode_screen_kernel on near-ties.
constexpr int64_t SHR_FEW = 4096;
constexpr float SHR_BIG = 3.0e38f;

struct ShareArgs {
  const void *X;
  const float *std32;  // rows' std computed beforehand, or nullptr: computed here when scale is set
  const float *C32;
  const uint16_t *C16s;
  const float *normp;
  const uint32_t *groupA;
  const uint16_t *perm16;
  const float *stats;
  int16_t *codes;
  float *residual;
  void *std_out;
  unsigned long long *counters;  // nullptr: not counted
  int64_t N, ldx, V;
  int in_dtype, std_dtype, G, grouping, scale, ddof, vec_rows;
  int K, Kpad, depth, stage_begin, stage_end;
  int vpw;             // tokens per workgroup
  int tie_serial;      // near-ties are decided by distances summed channel after channel
  float kappa;
};

// LDS, in this order; T = tokens rounded up to whole tiles
struct ShareLds {
  size_t B, rs, best, info, bits, slow, nrm, perm, bytes;
};
__host__ __device__ inline ShareLds share_lds(int T, int piece) {
  ShareLds l;
  l.B = 0;                                   // [T / 16][64] 16-byte operands
  l.rs = l.B + (size_t)T * 64;               // [T][32] fp32 residuals
  l.info = l.rs + (size_t)T * 128;           // [T] {threshold as ordered bits, added to it, gx, -}
  l.bits = l.info + (size_t)T * 16;          // [T][8] candidate groups, one bit each
  l.best = l.bits + (size_t)T * 32;          // [T] (distance bits, codeword) found so far
  l.slow = l.best + (size_t)T * 8;           // [T] tokens for the exact search
  l.nrm = l.slow + (size_t)T * 2;            // [2][piece] norms in accumulator order
  l.perm = l.nrm + (size_t)2 * piece * 4;    // [2][piece] position -> codeword
  l.bytes = l.perm + (size_t)2 * piece * 2;
  return l;
}
// what no codeword beats (a NaN distance has larger bits): the exact path then keeps index 0
constexpr unsigned long long SHR_NONE = 0x7f800000ull << 32;

template <int CTRL>
__device__ __forceinline__ float shr_dpp(float v) {
  const int b = __float_as_int(v);
  return __int_as_float(__builtin_amdgcn_update_dpp(b, b, CTRL, 0xf, 0xf, false));
}
// sum over the eight lanes of a token, the balanced tree of the exact path; in all eight lanes
__device__ __forceinline__ float sum8(float v) {
  v += shr_dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v += shr_dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  v += shr_dpp<0x141>(v);  // mirrored half row: the other quad's sum
  return v;
}
__device__ __forceinline__ float max8(float v) {
  v = __builtin_fmaxf(v, shr_dpp<0xB1>(v));
  v = __builtin_fmaxf(v, shr_dpp<0x4E>(v));
  return __builtin_fmaxf(v, shr_dpp<0x141>(v));
}
// Workgroup barrier for what is passed on in LDS.  (__syncthreads also waits for the loads of the next
// stage's operands, which are meant to stay in flight: 1.7 us of each stage's 5.)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// floats as signed integers of the same order (and back)
__device__ __forceinline__ int order_bits(int b) { return b ^ ((b >> 31) & 0x7fffffff); }
__device__ __forceinline__ float min3f(float a, float b, float c) {
  return __builtin_fminf(__builtin_fminf(a, b), c);
}
__device__ __forceinline__ float min8(const f32x4 a, const f32x4 b) {
  return __builtin_fminf(min3f(min3f(min3f(a[0], a[1], a[2]), a[3], b[0]), b[1], b[2]), b[3]);
}
// smallest of the four lanes l, l ^ 16, l ^ 32, l ^ 48
__device__ __forceinline__ float min_rows16(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const float w = __builtin_fminf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const unsigned x = __float_as_uint(w);
  const auto b = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return __builtin_fminf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
template <int CTRL>
__device__ __forceinline__ uint32_t shr_dppu(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  v = min(v, shr_dppu<0xB1>(v));
  v = min(v, shr_dppu<0x4E>(v));
  v = min(v, shr_dppu<0x124>(v));  // row_ror 4
  v = min(v, shr_dppu<0x128>(v));  // row_ror 8
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32);
  const uint32_t r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
  return min(min(r0, r1), min(r2, r3));
}

typedef __attribute__((address_space(1))) const char glb_char;
typedef __attribute__((address_space(1))) const f32x4 glb_c4;
typedef __attribute__((address_space(3))) const f32x4 lds_c4;
typedef __attribute__((address_space(3))) const uint16_t lds_c16;
typedef __attribute__((address_space(3))) unsigned lds_u32;
typedef __attribute__((address_space(3))) unsigned long long lds_u64;
__device__ __forceinline__ void lds_min(lds_u64 *p, unsigned long long v) {
  (void)__hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Exact search over the whole stage for the `ns` tokens listed in `slow`, by all wavefronts: each holds
// 16 SLOTS codewords at a time and scores all of the tokens against them, so a codeword is fetched once
// for all and the caller needs one barrier.  (SLOTS = 8 costs the general form spills: one stage of K = 256
// for 32768 vectors 18.7 -> 19.4 us.)  K = 2048, sixteen tokens: 27 us a stage (one token after the other with
// two barriers each 48; the small-batch kernel, which this replaces there, 20).
template <int SLOTS>
__device__ __forceinline__ void search_slow(lds_c4 *res, lds_u64 *best, lds_c16 *slow, int ns, glb_char *Cs,
                                            int K, int wave, int lane) {
  // four lanes per codeword, eight channels each; the partial sums meet in the exact path's tree
  const int pc = (lane & 3) * 2;
  for (int k0 = wave * 16 * SLOTS; k0 < K; k0 += SHR_WAVES * 16 * SLOTS) {
    f32x4 c0[SLOTS], c1[SLOTS];
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
      const int k = min(k0 + 16 * j + (lane >> 2), K - 1);  // past the end: fetched, not scored
      glb_c4 *src = (glb_c4 *)(Cs + ((uint32_t)k * 128u + (uint32_t)pc * 16u));
      c0[j] = src[0];
      c1[j] = src[1];
    }
    for (int i = 0; i < ns; ++i) {
      const int tok = slow[i];
      const f32x4 r0 = res[tok * 8 + pc], r1 = res[tok * 8 + pc + 1];
      uint32_t bits = 0x7f800000u, idx = 0;
#pragma unroll
      for (int j = 0; j < SLOTS; ++j) {
        float p0 = 0.f, p1 = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float d0 = r0[e] - c0[j][e], d1 = r1[e] - c1[j][e];
          p0 = fmaf(d0, d0, p0);
          p1 = fmaf(d1, d1, p1);
        }
        float dist = p0 + p1;
        dist += shr_dpp<0xB1>(dist);
        dist += shr_dpp<0x4E>(dist);
        const uint32_t db = __float_as_uint(dist);
        const int k = k0 + 16 * j + (lane >> 2);
        if (k < K && db < bits) {  // a lane's later codewords have the larger indices
          bits = db;
          idx = (uint32_t)k;
        }
      }
      const uint32_t m = wave_min(bits);
      const uint32_t k = wave_min(bits == m ? idx : 0xffffffffu);
      if (lane == 0) lds_min(best + tok, ((unsigned long long)m << 32) | k);
    }
  }
}

// Exact distances of one token's marked groups, by a wavefront, eight groups at a time; the token's best
// codeword so far takes the place of its marks.  For few tokens with many candidates (codewords
// crowded into clusters): the kernel's own resolve step takes a token's groups one after the other, a
// round trip to L2 each, with most wavefronts idle.  600 vectors, K = 2048 in clusters of 64, depth 4: 44 us
// without it, 27 with it.  (Out of line: in line its registers are made room for on the common path, 48
// rows of 32 groups 37 us instead of 34.)
template <int TPW>
__device__ __noinline__ void resolve_crowded(lds_c4 *res, lds_u64 *best_p, lds_u32 *mark, lds_c16 *perm,
                                                glb_char *Cs, int K, int lane) {
  const int q = lane & 7, sub = lane >> 3;
  const unsigned word = mark[sub];
  const f32x4 r = res[q];
  // The marks of the eight words in order have ranks 0, 1, ...; in a round subgroup j of the wavefront takes
  // the mark of rank base + j.  rank0: rank of this word's first one.
  int rank0 = 0, total = 0;
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const int n = __popc((unsigned)__builtin_amdgcn_readlane((int)word, 8 * w));
    rank0 += w < sub ? n : 0;
    total += n;
  }
  unsigned long long best = SHR_NONE;
  unsigned left = word;
  int next = rank0;  // rank of the first mark left in the word
  for (int base = 0; base < total; base += 8) {
    int g = -1;
    for (int j = 0; j < 8; ++j) {
      const bool mine = left != 0 && next == base + j;
      const unsigned long long b = __ballot(mine);
      if (b != 0) {
        const int src = __ffsll((long long)b) - 1;
        const int bit = __ffs((unsigned)__builtin_amdgcn_readlane((int)left, src)) - 1;
        g = sub == j ? (src >> 3) * 32 + bit : g;
        if (mine) {
          left &= left - 1;
          ++next;
        }
      }
    }
    const int gc = g < 0 ? 0 : g;  // (no group: position 0, whose true distances may take part)
    const int pos = ((gc >> 4) * TPW + (gc & 3)) * 32 + (gc & 12);
    f32x4 c[8];
    unsigned k[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      k[e] = perm[pos + (e & 3) + 4 * (e & 4)];
      c[e] = *(glb_c4 *)(Cs + (min(k[e], (unsigned)(K - 1)) * 128u + (uint32_t)q * 16u));
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float p = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float d = r[i] - c[e][i];
        p = fmaf(d, d, p);
      }
      const unsigned long long key = ((unsigned long long)__float_as_uint(sum8(p)) << 32) | k[e];
      best = key < best ? key : best;
    }
  }
  if (q == 0) lds_min(best_p, best);
  if (q == 0) mark[sub] = 0u;
}

// TPW: tiles of 32 codewords per wavefront; a piece of 512 TPW codewords is in registers at a time
// (32 registers of operands and 32 of norms at TPW = 4, of the 128 that sixteen wavefronts leave
// each other).  K <= 2048 is one piece; larger codebooks are swept and resolved piece after piece, with
// the threshold and the best codeword carried over.
// FEW: at most SHR_FEW vectors in all and 16 in a workgroup, so one tile of tokens, a single step of the
// resolve loop, no near-ties to decide another way and nothing to count.  Without those branches the
// registers suffice, also with the rare paths in line (48 rows of 32 groups, K = 2048: 47 us in the
// general form, 34 here).
template <int TPW, bool FEW>
__global__ __launch_bounds__(SHR_THREADS) void encode_share_kernel(const ShareArgs a) {
  constexpr int PIECE = 512 * TPW;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ float row_sd[SHR_TOKENS + 2];
  __shared__ int slow_n[2];  // tokens for the exact search, stages of even and of odd number
  __shared__ unsigned stat[2];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lg = lane >> 4;     // which four rows of a 16 x 16 result this lane holds
  const int tcol = lane & 15;   // its token within the tile
  const int q = lane & 7;       // resolve: this lane's four channels, 4 q .. 4 q + 3
  const int64_t v0 = (int64_t)blockIdx.x * a.vpw;
  const int nvalid = (int)min((int64_t)a.vpw, a.V - v0);
  const int ntiles = FEW ? 1 : (a.vpw + 15) >> 4;
  const int T = ntiles * 16;
  const ShareLds L = share_lds(T, PIECE);
  uint4 *lds_B = reinterpret_cast<uint4 *>(smem + L.B);
  f32x4 *lds_r = reinterpret_cast<f32x4 *>(smem + L.rs);
  int4 *lds_i = reinterpret_cast<int4 *>(smem + L.info);
  unsigned *lds_h = reinterpret_cast<unsigned *>(smem + L.bits);
  unsigned long long *lds_b = reinterpret_cast<unsigned long long *>(smem + L.best);
  uint16_t *lds_slow = reinterpret_cast<uint16_t *>(smem + L.slow);
  float *lds_nrm = reinterpret_cast<float *>(smem + L.nrm);
  uint16_t *lds_perm = reinterpret_cast<uint16_t *>(smem + L.perm);
  int buf = 0;  // LDS half of the next piece

  const int ntc = a.Kpad >> 5;                        // tiles of 32 codewords in a stage
  const int pieces = (a.Kpad + PIECE - 1) / PIECE;
  const float k4 = 0.125f * a.kappa;
  const float k4u = 3.0f * k4;

  // ---- this wavefront's share of a piece, in registers
  half8 A[2 * TPW];
  f32x4 nrm[2 * TPW];
  uint32_t Wg = 0;  // the bounds of one of the groups, on their way
  float Bg = 0.f;   // the largest of the codewords' (they are sorted by norm: all alike)
  float Eg = 0.f;   // what their part of the bounds adds to a threshold
  float2 normw = {0.f, 0.f};  // two norms and two entries of the position -> codeword map of the piece,
  uint32_t permw = 0;         // on their way to LDS
  // (buffer loads: the bases stay in scalar registers and a lane's part of an address is one register;
  // with per-lane pointers the compiler kept, and spilled, sixteen of them)
  const int kall = a.Kpad * a.depth;
  const auto rsA = __builtin_amdgcn_make_buffer_rsrc((void *)a.C16s, 0, kall * 64, 0x00020000);
  const auto rsN = __builtin_amdgcn_make_buffer_rsrc((void *)a.normp, 0, kall * 4, 0x00020000);
  const auto rsP = __builtin_amdgcn_make_buffer_rsrc((void *)a.perm16, 0, kall * 2, 0x00020000);
  const auto rsC = __builtin_amdgcn_make_buffer_rsrc((void *)a.C32, 0, a.K * a.depth * 128, 0x00020000);
  const auto rsG = __builtin_amdgcn_make_buffer_rsrc((void *)a.groupA, 0, kall / 4, 0x00020000);
  auto load_piece = [&](int stage, int piece) {
    if (PIECE == 2048 || 2 * tid < PIECE) {
      const int p0 = stage * a.Kpad + piece * PIECE;
      // (what lies beyond the codebook is never looked at)
      const auto nw = __builtin_amdgcn_raw_buffer_load_b64(rsN, tid * 8, p0 * 4, 0);
      normw = make_float2(__int_as_float(nw[0]), __int_as_float(nw[1]));
      permw = __builtin_amdgcn_raw_buffer_load_b32(rsP, tid * 4, p0 * 2, 0);
    }
    // lane i of eight has the bound of one of the wavefront's 2 TPW groups (their maximum is taken
    // once they have arrived)
    const int gi = lane & (2 * TPW - 1);
    const int t0 = piece * (16 * TPW) + wave * TPW + (gi >> 1);
    Wg = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rsG, ((stage * ntc + min(t0, ntc - 1)) * 2 + (gi & 1)) * 4, 0, 0);
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
      const int t = piece * (16 * TPW) + wave * TPW + j;
      const int tc = stage * ntc + min(t, ntc - 1);
#pragma unroll
      for (int s = 0; s < 2; ++s)
        A[2 * j + s] = __builtin_bit_cast(
            half8, __builtin_amdgcn_raw_buffer_load_b128(rsA, lane * 16, tc * 2048 + s * 1024, 0));
    }
  };

  // ---- fp16 operand, error bound and bookkeeping of token `tok` for `stage`, from its residual
  // (eight lanes per token, four channels in each)
  struct StageConsts { float Tscale, tiny; bool usable; };
  auto stage_consts = [&](int stage) -> StageConsts {
    const float *st = a.stats + stage * 8;
    return {st[4], 6.103515625e-5f / st[4], st[1] != 0.0f};
  };
  auto convert = [&](int stage, const StageConsts &sc, int tok, const f32x4 r) {
    const float Tscale = sc.Tscale, tiny = sc.tiny;
    const bool usable = sc.usable;
    float s_q = 0.f, s_d = 0.f;
    half4 hx;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = r[e] * Tscale;  // exact: a power of two
      hx[e] = fabsf(r[e]) < tiny ? (_Float16)0.f : (_Float16)x;
      const float xr = (float)hx[e];
      const float dx = x - xr;
      s_q = fmaf(xr, xr, s_q);
      s_d = fmaf(dx, dx, s_d);
    }
    s_q = sum8(s_q);
    s_d = sum8(s_d);
    const bool valid = tok < nvalid;
    // an element beyond the half range turns s_q into infinity (or the sum into a NaN)
    const bool slow = !usable || (__float_as_uint(s_q) & 0x7fffffffu) >= 0x4f5693a4u /* 3.6e9f */;
    if (slow || !valid) hx = half4{0, 0, 0, 0};
    const float nq = sqrtf(s_q) * 1.000001f;
    const float nd = sqrtf(s_d) * 1.000001f;
    // channels 8 (q >> 1) .. of the tile's column tok % 16, this lane's half of the 16 bytes
    reinterpret_cast<uint2 *>(lds_B)[(((tok >> 4) * 64 + (q >> 1) * 16 + (tok & 15)) << 1) + (q & 1)] =
        __builtin_bit_cast(uint2, hx);
    lds_h[tok * 8 + q] = 0u;
    if (q == 0) {
      lds_b[tok] = SHR_NONE;
      int4 w = {0x7fffffff, 0, 0, 0};
      if (slow || !valid) {
        w.y = __float_as_int(-1e35f);  // below every score: no candidates are looked for
        if (valid) lds_slow[atomicAdd(&slow_n[stage & 1], 1)] = (uint16_t)tok;
      } else {
        // what the fp32 distances of two codewords can be off by rounding: 2 x 34 x 2^-24 of
        // (|r| + |c|)^2 <= 2 (|r|^2 + |c|^2), where S T |r|^2 = 2 nq^2 here (the |c|^2 part is
        // inside the spare third of the k4 term)
        w.y = __float_as_int(2e-5f * nq * nq);
        w.z = __float_as_int(fmaxf((nd + 1.0005f * a.kappa * nq) * 1.000001f, RVQ_BOUND_RHO * nq));
      }
      lds_i[tok] = w;
    }
  };

  load_piece(a.stage_begin, 0);
  if (tid < 2) slow_n[tid] = 0;
  if (tid < 2) stat[tid] = 0;
  // ---- the rows' std (the arithmetic of row_std_kernel), the tokens' channels, the first operands
  const int64_t n_first = v0 / a.G;
  if (a.scale && (FEW || !a.std32)) {
    const int nrows = (int)((v0 + nvalid - 1) / a.G - n_first) + 1;  // <= SHR_TOKENS + 1
    const int d = a.G * 32;
    for (int w = wave; w < nrows; w += SHR_WAVES) {
      const int64_t n = n_first + w, base = n * a.ldx;
      float sd;
      if (a.vec_rows) {
        sd = a.in_dtype == RVQ_F32    ? rvq_row_std<RVQ_F32, true>(a.X, base, d, a.ddof, lane)
             : a.in_dtype == RVQ_BF16 ? rvq_row_std<RVQ_BF16, true>(a.X, base, d, a.ddof, lane)
                                      : rvq_row_std<RVQ_F16, true>(a.X, base, d, a.ddof, lane);
      } else {
        sd = a.in_dtype == RVQ_F32    ? rvq_row_std<RVQ_F32, false>(a.X, base, d, a.ddof, lane)
             : a.in_dtype == RVQ_BF16 ? rvq_row_std<RVQ_BF16, false>(a.X, base, d, a.ddof, lane)
                                      : rvq_row_std<RVQ_F16, false>(a.X, base, d, a.ddof, lane);
      }
      if (lane == 0) {
        row_sd[w] = sd;
        // the workgroup that holds a row's group 0 stores the value
        if (a.std_out && n * a.G >= v0 && n * a.G < v0 + nvalid) {
          if (a.std_dtype == RVQ_F32) reinterpret_cast<float *>(a.std_out)[n] = sd;
          else reinterpret_cast<uint16_t *>(a.std_out)[n] = rvq_f32_to_f16_bits_sat(sd);
        }
      }
    }
  }
  lds_barrier();
  const StageConsts sc0 = stage_consts(a.stage_begin);
  for (int t0 = 0; t0 < T; t0 += SHR_PASS) {
    const int tok = t0 + (tid >> 3);
    if (tok >= T) break;  // uniform over a wavefront: T is a multiple of 16
    f32x4 r = {0.f, 0.f, 0.f, 0.f};
    if (tok < nvalid) {
      const int64_t v = v0 + tok, n = v / a.G;
      const int g = (int)(v - n * a.G);
      const float sd = !FEW && a.std32 ? a.std32[n] : (a.scale ? row_sd[n - n_first] : 1.0f);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 4 * q + e;
        const int64_t ch = a.grouping == RVQ_CONTIGUOUS ? (int64_t)g * 32 + j : (int64_t)j * a.G + g;
        const float x = rvq_load_in_rt(a.X, n * a.ldx + ch, a.in_dtype);
        r[e] = a.scale ? x / sd : x;
      }
    }
    lds_r[tok * 8 + q] = r;
    convert(a.stage_begin, sc0, tok, r);
  }

  unsigned n_exact = 0, n_slow = 0;  // wave-uniform
  for (int stage = a.stage_begin; stage < a.stage_end; ++stage) {
    const uint16_t *perm = nullptr;
    for (int piece = 0; piece < pieces; ++piece) {
      Bg = max8(rvq_bound_both(Wg));
      Eg = max8(rvq_bound_len(Wg));
      Eg = k4u * Eg * Eg;
      // (double buffers: the other half may still be read by a slower wavefront)
      float *nbuf = lds_nrm + buf * PIECE;
      uint16_t *pbuf = lds_perm + buf * PIECE;
      perm = pbuf;
      buf ^= 1;
      if (PIECE == 2048 || 2 * tid < PIECE) {
        reinterpret_cast<float2 *>(nbuf)[tid] = normw;
        reinterpret_cast<uint32_t *>(pbuf)[tid] = permw;
      }
      lds_barrier();  // operands, bounds, norms and map are in LDS
      // (every wavefront has read the previous stage's count; the next stage's tokens are counted
      // after at least one more barrier)
      if (piece == 0 && tid == 0) slow_n[(stage + 1) & 1] = 0;
#pragma unroll
      for (int j = 0; j < TPW; ++j)
#pragma unroll
        for (int s = 0; s < 2; ++s)  // rows 16 s + 4 lg .. + 3 of the tile
          nrm[2 * j + s] = *reinterpret_cast<const f32x4 *>(
              nbuf + (wave * TPW + j) * 32 + (lg & 1) * 16 + (2 * s + (lg >> 1)) * 4);
#pragma unroll
      for (int j = 0; j < TPW; ++j)
        if ((piece * 16 + wave) * TPW + j >= ntc)  // beyond the codebook: never near a minimum
          nrm[2 * j] = nrm[2 * j + 1] = f32x4{1e30f, 1e30f, 1e30f, 1e30f};

      // sweep of tiles 2 s and 2 s + 1: kept minima, and the tokens' thresholds
      auto sweep = [&](int s, float (&mm)[2][TPW]) {
        const int tile0 = 2 * s, tile1 = 2 * s + 1;
        const half8 B0 = __builtin_bit_cast(half8, lds_B[tile0 * 64 + lane]);
        const float g0 = __int_as_float(lds_i[tile0 * 16 + tcol].z);
        float ub0 = SHR_BIG;
        if (tile1 < ntiles) {
          const half8 B1 = __builtin_bit_cast(half8, lds_B[tile1 * 64 + lane]);
          const float g1 = __int_as_float(lds_i[tile1 * 16 + tcol].z);
          float ub1 = SHR_BIG;
#pragma unroll
          for (int j = 0; j < TPW; ++j) {
            const f32x4 d0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2 * j], B0, nrm[2 * j], 0, 0, 0);
            const f32x4 e0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2 * j], B1, nrm[2 * j], 0, 0, 0);
            const f32x4 d1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2 * j + 1], B0, nrm[2 * j + 1], 0, 0, 0);
            const f32x4 e1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2 * j + 1], B1, nrm[2 * j + 1], 0, 0, 0);
            mm[0][j] = min8(d0, d1);
            mm[1][j] = min8(e0, e1);
            ub0 = __builtin_fminf(ub0, mm[0][j]);
            ub1 = __builtin_fminf(ub1, mm[1][j]);
            __builtin_amdgcn_sched_barrier(0);  // (results of one step at a time: registers)
          }
          // the exact minimum is at most score + e + k4 A^2 (what the distances' rounding adds is added in `pick`),
          // with 2.5 % spare, for the rounding of this sum, on the 2 e above the scores' lower bound, score - e
          ub1 = min_rows16(fmaf(Bg, 1.05f * g1, ub1 + Eg));
          ub0 = min_rows16(fmaf(Bg, 1.05f * g0, ub0 + Eg));
          if (lane < 32) atomicMin(&lds_i[tile0 * 16 + lane].x, order_bits(__float_as_int(lane < 16 ? ub0 : ub1)));
        } else {
#pragma unroll
          for (int j = 0; j < TPW; ++j) {
            const f32x4 d0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2 * j], B0, nrm[2 * j], 0, 0, 0);
            const f32x4 d1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[2 * j + 1], B0, nrm[2 * j + 1], 0, 0, 0);
            mm[0][j] = min8(d0, d1);
            mm[1][j] = SHR_BIG;
            ub0 = __builtin_fminf(ub0, mm[0][j]);
          }
          ub0 = min_rows16(fmaf(Bg, 1.05f * g0, ub0 + Eg));
          if (lane < 16) atomicMin(&lds_i[tile0 * 16 + lane].x, order_bits(__float_as_int(ub0)));
        }
      };
      // candidate groups of tiles 2 s and 2 s + 1: a lane whose kept minimum is within its token's
      // threshold marks its eight codewords (rows 4 lg .. + 3 and 16 + 4 lg .. + 3 of the tile)
      auto pick = [&](int s, const float (&mm)[2][TPW]) {
#pragma unroll
        for (int u = 0; u < (FEW ? 1 : 2); ++u) {
          const int tile = 2 * s + u;
          if (u == 0 || tile < ntiles) {
            const int tok = tile * 16 + tcol;
            const int4 w = lds_i[tok];
            const float tadj = fmaf(__int_as_float(w.z), Bg, __int_as_float(order_bits(w.x)) + __int_as_float(w.y));
            float best = mm[u][0];
#pragma unroll
            for (int j = 1; j < TPW; ++j) best = __builtin_fminf(best, mm[u][j]);
            if (best <= tadj) {
              unsigned hits = 0;
#pragma unroll
              for (int j = 0; j < TPW; ++j) hits |= mm[u][j] <= tadj ? 1u << j : 0u;
              atomicOr(&lds_h[tok * 8 + (wave >> 1)], hits << ((wave & 1) * 16 + lg * 4));
            }
          }
        }
      };
      // (Sweeping the next pair before this one is picked from, to have work on both sides of the
      // barrier, costs eight more registers per wavefront: the compiler then spills operands, and 4096
      // rows took 365 us instead of 274.)
      const int nslow = slow_n[stage & 1];
      const int pairs = nslow < nvalid ? (ntiles + 1) >> 1 : 0;  // nothing to sweep when all of them are
      float mm[2][TPW];
      for (int s = 0; s < pairs; ++s) {
        sweep(s, mm);
        lds_barrier();
        pick(s, mm);
      }
      // What the operand registers hold next (at the end once more what they held) is requested when
      // this wavefront's first rows of exact distances have come back, ahead of the rest of the
      // resolve step: a wavefront's loads return in order, so requested earlier they would hold those
      // rows up.
      const bool last = piece + 1 == pieces;
      const int nstage = last ? min(stage + 1, a.stage_end - 1) : stage, npiece = last ? 0 : piece + 1;
      lds_barrier();  // all candidates are marked

      const int sC = stage * a.K * 128;
      auto row = [&](int k, int piece16) {  // four channels of codeword k
        return __builtin_bit_cast(
            f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsC, k * 128 + piece16 * 16, sC, 0));
      };
      // ---- exact search for the tokens that need it
      const int ns = piece == 0 ? nslow : 0;
      if (ns > 0) {
        search_slow<FEW ? 8 : 4>((lds_c4 *)lds_r, (lds_u64 *)lds_b, (lds_c16 *)lds_slow, ns,
                    (glb_char *)(a.C32 + (int64_t)stage * a.K * 32), a.K, wave, lane);
        lds_barrier();
        if (wave == 0) n_slow += (unsigned)ns;
      }
      // ---- many candidates: a wavefront to a token (otherwise 1.03 groups per token are marked, and the
      // resolve step has its wavefronts' tokens side by side).  Every wavefront counts all marks, two
      // words per lane: kept by an atomic add in the sweep instead, the count cost 0.7 us a stage.
      if constexpr (FEW) {
        const uint2 w = reinterpret_cast<const uint2 *>(lds_h)[lane];
        unsigned n = __popc(w.x) + __popc(w.y);
        n += shr_dppu<0xB1>(n);
        n += shr_dppu<0x4E>(n);
        if (__any(n > 5)) {
          if (wave < nvalid)
            resolve_crowded<TPW>((lds_c4 *)lds_r + wave * 8, (lds_u64 *)lds_b + wave, (lds_u32 *)lds_h + wave * 8,
                                 (lds_c16 *)perm, (glb_char *)(a.C32 + (int64_t)stage * a.K * 32), a.K, lane);
          lds_barrier();
        }
      }

      // ---- resolve
      const StageConsts scn = stage_consts(min(stage + 1, a.depth - 1));
      // First position of the first marked group of a token, whose mark is taken away.  (A token with no
      // more marks gets position 0 along with the others: true distances, which may take part.)
      auto next_group = [&](unsigned &marks, bool &has) -> int {
        unsigned g = marks ? (unsigned)(q * 32 + __ffs(marks) - 1) : 0xffffffffu;
        g = min(g, shr_dppu<0xB1>(g));
        g = min(g, shr_dppu<0x4E>(g));
        g = min(g, shr_dppu<0x141>(g));
        if ((int)(g >> 5) == q) marks &= marks - 1;
        has = g != 0xffffffffu;
        g = has ? g : 0u;
        return ((int)(g >> 4) * TPW + (int)(g & 3)) * 32 + (int)(g & 12);
      };
      auto resolve = [&](int t0, auto first) {
        const int tok = t0 + (tid >> 3);
        const bool valid = tok < nvalid;
        unsigned marks = lds_h[tok * 8 + q];  // wavefronts 2 q and 2 q + 1: bit (wave & 1, lane row, tile)
        const unsigned long long best0 = lds_b[tok];
        unsigned long long best = best0;
        float bd = __uint_as_float((uint32_t)(best0 >> 32)), second = INFINITY;  // two smallest distances
        f32x4 r = lds_r[tok * 8 + q];
        while (__any(marks != 0)) {
          bool has;
          const int pos = next_group(marks, has);
          n_exact += __popcll(__ballot(has));  // eight lanes, eight codewords
          const float second0 = second;
          const uint2 ka = *reinterpret_cast<const uint2 *>(perm + pos);
          const uint2 kb = *reinterpret_cast<const uint2 *>(perm + pos + 16);
          // A position of the padding holds 0xffff: it is scored as codeword K - 1 under that number,
          // which never wins, because the nearest codeword itself is always among the candidates.
          const unsigned k[8] = {ka.x & 0xffffu, ka.x >> 16, ka.y & 0xffffu, ka.y >> 16,
                                 kb.x & 0xffffu, kb.x >> 16, kb.y & 0xffffu, kb.y >> 16};
          f32x4 c[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) c[e] = row((int)min(k[e], (unsigned)(a.K - 1)), q);
          // (All eight in flight before the first is used: one round trip.  Left to itself the compiler
          // scores them four and four, 0.6 us a stage.  Later passes have no registers for it.)
          if constexpr (FEW || first)
            asm volatile("" : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]), "+v"(c[4]), "+v"(c[5]), "+v"(c[6]), "+v"(c[7]));
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float p = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float d = r[i] - c[e][i];
              p = fmaf(d, d, p);
            }
            const float dist = sum8(p);
            second = __builtin_amdgcn_fmed3f(bd, second, dist);
            bd = __builtin_fminf(bd, dist);
            // distances are >= +0: ordered like their bits; the smallest index among equals
            const unsigned long long key = ((unsigned long long)__float_as_uint(dist) << 32) | k[e];
            best = key < best ? key : best;
          }
          second = has ? second : second0;  // (position 0 may have been scored before)
        }
        // Two distances that differ by less than their rounding (34 + 9 roundings of 2^-24 on either
        // side), in a call that encode_screen_kernel took before: its order of summation decides, one
        // codeword of a group per lane.
        const bool near = !FEW && a.tie_serial && valid && second <= bd * 1.000006f;
        if (!FEW && __any(near)) {
          const int k0 = (int)(best0 & 0xffffffffull);
          unsigned long long sb = SHR_NONE;
          auto serial = [&](unsigned k) {
            float dist = 0.f;
            for (int c4 = 0; c4 < 8; ++c4) {
              const f32x4 c = row((int)min(k, (unsigned)(a.K - 1)), c4), x = lds_r[tok * 8 + c4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float d = x[e] - c[e];
                dist = fmaf(d, d, dist);
              }
            }
            const unsigned long long key = ((unsigned long long)__float_as_uint(dist) << 32) | k;
            sb = key < sb ? key : sb;
          };
          if (best0 != SHR_NONE) serial((unsigned)k0);
          unsigned again = lds_h[tok * 8 + q];
          while (__any(again != 0)) {
            bool has;
            const int pos = next_group(again, has);
            serial(perm[pos + (q & 3) + 4 * (q & 4)]);
          }
          // the nearest of the eight lanes, ties to the smallest index
          uint32_t sd = (uint32_t)(sb >> 32);
          sd = min(sd, shr_dppu<0xB1>(sd));
          sd = min(sd, shr_dppu<0x4E>(sd));
          sd = min(sd, shr_dppu<0x141>(sd));
          uint32_t sk = (uint32_t)(sb >> 32) == sd ? (uint32_t)sb : 0xffffffffu;
          sk = min(sk, shr_dppu<0xB1>(sk));
          sk = min(sk, shr_dppu<0x4E>(sk));
          sk = min(sk, shr_dppu<0x141>(sk));
          if (near) best = ((unsigned long long)__float_as_uint(bd) << 32) | sk;
        }
        if (!last) {
          if constexpr (first) load_piece(nstage, npiece);
          lds_h[tok * 8 + q] = 0u;
          if (q == 0) lds_b[tok] = best;
          return;
        }
        const int bestk = min((int)(best & 0xffffffffull), a.K - 1);
        const f32x4 bestc = row(bestk, q);
        if constexpr (first) load_piece(nstage, npiece);
        if (valid) {
          r -= bestc;
          if (q == 0) a.codes[(v0 + tok) * a.depth + stage] = (int16_t)bestk;
        }
        if (stage + 1 < a.stage_end) {
          lds_r[tok * 8 + q] = r;
          convert(stage + 1, scn, tok, r);
        } else if (a.residual && valid) {
          reinterpret_cast<f32x4 *>(a.residual + (v0 + tok) * 32)[q] = r;
        }
      };
      if (tid >> 3 < T) {  // uniform over a wavefront: T is a multiple of 16
        resolve(0, std::true_type());
        if constexpr (!FEW)
          for (int t0 = SHR_PASS; t0 + (tid >> 3) < T; t0 += SHR_PASS) resolve(t0, std::false_type());
      } else {
        // no token of its own: let the other wavefronts' rows go first
        __builtin_amdgcn_s_sleep(8);
        load_piece(nstage, npiece);
      }
    }
  }

  if (!FEW && a.counters) {  // one update per workgroup
    if (lane == 0) {
      atomicAdd(&stat[0], n_slow);
      atomicAdd(&stat[1], n_exact);
    }
    lds_barrier();
    if (tid < 2) atomicAdd(&a.counters[tid], (unsigned long long)stat[tid]);
    if (tid == 3)
      atomicAdd(&a.counters[3], (unsigned long long)nvalid * (unsigned)(a.stage_end - a.stage_begin));
  }
}

}  // namespace

// Where this kernel is used.  Times in us for all stages, depth 8, bf16 rows of 32 groups, "screen" is
// encode_screen_kernel, t / CU = tokens per CU.
//  below: with at most two vectors per CU the small-batch kernel's latency is lower (K = 2048, two: 33 : 33,
//    one: 28 : 33; three vectors per CU 55 : 33, K = 256 54 : 25, K = 4096 104 : 56).
//  up to 256 / CU: here encode_screen_kernel leaves half of the CUs free, so that keys and values of a layer,
//    a pair of calls on two streams, run side by side, while this kernel takes every CU and a pair takes
//    twice a call.  One call gains, a pair loses; the line is where the product of the two ratios is 1,
//    with pairs that follow each other without a join, which lose most.  One call; such a pair:
//    K = 256 at 128 / CU 84 : 61; 88 : 112, at 144 84 : 67; 86 : 125.  K = 512 at 160 98 : 71; 102 : 133, at 176
//    98 : 76; 101 : 144.  K = 1024 at 192 130 : 95; 138 : 186, at 208 132 : 102; 140 : 198.  K = 1536 at 208
//    172 : 128; 186 : 246, at 224 162 : 134; 174 : 267.  K = 2048 at 192 202 : 121; 208 : 229, at 240 209 : 145;
//    223 : 288, at 256 210 : 151; 219 : 301.  K = 3072 at 256 401 : 252; 444 : 504.
//  above 256 / CU: a pair no longer fits side by side, and encode_screen_kernel's wavefronts, which
//    re-use a token's operands for the whole stage, overtake once they are full, the later the larger the
//    codebook.  One call: K = 1536 at 288 168 : 163, at 304 166 : 171; K = 2048 at 352 214 : 194, at 384 213 : 216
//    (pair 416 : 429); K = 4096 (two pieces, each with its resolve step) at 384 563 : 408, at 500, key rows,
//    507 : 549; K = 8192, depth 4, at 512 717 : 470.
//  one stage (a step of codebook learning: nothing runs beside it, and encode_screen_kernel's first
//    copy of a stage's operands has nothing to hide under): up to 128 + K / 8.  fp32 vectors: K = 256 at
//    156 / CU 23 : 21; K = 1024 at 256 36 : 29; K = 2048 at 256 62 : 35, at 384 62 : 45.
bool rvq_share_fits(const rvq_ctx *ctx, int64_t V, int stages) {
  const int64_t cus = ctx->num_cus > 0 ? ctx->num_cus : 1;
  const int64_t K = ctx->Kpad;
  if (V <= RVQ_SMALL_PER_CU * cus) return false;
  // (promised for so few vectors: the exact path's codes, no use of the caller's std scratch; on a
  // partition of the chip with fewer CUs the lines below lie lower than that)
  if (V <= SHR_FEW) return V <= cus * SHR_TOKENS;
  if (stages > 1 && V <= 256 * cus) return V <= cus * std::min(96 + K / 8, 144 + 3 * K / 64);
  return V <= cus * (K > 2048 ? std::min<int64_t>(256 + K / 32, SHR_TOKENS)
                              : 128 + (stages > 1 ? 7 * K / 64 : K / 8));
}

// tokens per workgroup: the vectors spread evenly over the CUs (whole tiles of 16 where there are
// more than one); V <= CUs x SHR_TOKENS
static int share_tokens(const rvq_ctx *ctx, int64_t V) {
  const int64_t cus = ctx->num_cus > 0 ? ctx->num_cus : 1;
  int64_t vpw = (V + cus - 1) / cus;
  if (vpw > 16) vpw = (vpw + 15) / 16 * 16;
  return (int)vpw;
}

bool rvq_share_needs_std(const rvq_ctx *ctx, int64_t N) {
  const int64_t V = N * ctx->G;
  return ctx->cfg.scale && V > SHR_FEW && (share_tokens(ctx, V) - 1) / ctx->G + 2 > SHR_ROWS;
}

hipError_t rvq_launch_encode_share(const rvq_ctx *ctx, const void *dX, int64_t N, int64_t ldx,
                                   int stage_begin, int stage_end, int16_t *dCodes, float *dResidual,
                                   void *dStd, const float *std32, hipStream_t s) {
  const rvq_config &c = ctx->cfg;
  ShareArgs a;
  a.X = dX;
  a.std32 = c.scale && rvq_share_needs_std(ctx, N) ? std32 : nullptr;
  a.C32 = ctx->C;
  a.C16s = ctx->C16s;
  a.normp = ctx->normp;
  a.groupA = ctx->groupA;
  a.perm16 = ctx->perm16;
  a.stats = ctx->stats;
  a.codes = dCodes;
  a.residual = dResidual;
  a.std_out = dStd;
  a.N = N;
  a.ldx = ldx;
  a.V = N * ctx->G;
  if (a.V < 1) return hipSuccess;
  if (c.dhat != 32 || !rvq_share_fits(ctx, a.V, stage_end - stage_begin)) return hipErrorInvalidValue;
  a.counters = a.V > SHR_FEW ? ctx->counters : nullptr;
  a.in_dtype = c.in_dtype;
  a.std_dtype = c.std_dtype;
  a.G = ctx->G;
  a.grouping = c.grouping;
  a.scale = c.scale;
  a.ddof = c.std_ddof;
  a.vec_rows = rvq_rows_vectorizable(dX, ldx, c.d, c.in_dtype);
  a.K = c.K;
  a.Kpad = ctx->Kpad;
  a.depth = c.depth;
  a.stage_begin = stage_begin;
  a.stage_end = stage_end;
  a.vpw = share_tokens(ctx, a.V);
  a.tie_serial = a.V > SHR_FEW;
  a.kappa = ctx->kappa;
  const int T = (a.vpw + 15) / 16 * 16;
  const bool few = a.V <= SHR_FEW && T == 16;
  const int64_t grid64 = (a.V + a.vpw - 1) / a.vpw;
  if (grid64 > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)grid64), block(SHR_THREADS);
#define RVQ_LAUNCH_SHARE(TPW)                                                                    \
  do {                                                                                           \
    const size_t lds = share_lds(T, 512 * (TPW)).bytes;                                          \
    if (few) {                                                                                   \
      hipLaunchKernelGGL((encode_share_kernel<TPW, true>), grid, block, lds, s, a);              \
      break;                                                                                     \
    }                                                                                            \
    hipError_t e = hipFuncSetAttribute(                                                          \
        reinterpret_cast<const void *>(&encode_share_kernel<TPW, false>),                        \
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)share_lds(SHR_TOKENS, 512 * (TPW)).bytes); \
    if (e != hipSuccess) return e;                                                               \
    hipLaunchKernelGGL((encode_share_kernel<TPW, false>), grid, block, lds, s, a);               \
  } while (0)
  // as many codewords per wavefront as make one piece, up to 2048 per workgroup
  if (ctx->Kpad <= 512) RVQ_LAUNCH_SHARE(1);
  else if (ctx->Kpad <= 1024) RVQ_LAUNCH_SHARE(2);
  else RVQ_LAUNCH_SHARE(4);
#undef RVQ_LAUNCH_SHARE
  return hipGetLastError();
}
