// Attention of one query position over a cache that holds RVQ codes (Section 3: one quantizer on
// the key and one on the value projection of an attention block, keys quantized BEFORE the rotary
// embedding; the Conclusion names decoding inside attention as the open efficiency question).
// Keys and values are never written out: every (token, kv head) is decoded in registers, the key
// is rotated and scored against the query heads that share the kv head, and the value enters an
// online softmax accumulation.  HBM traffic per (token, kv head) is 2 x (64 B codes + 2 B std) and
// the token's 256 B of rotary tables (shared by its heads) instead of 2 x 256 B of fp16 K and V.
//
// Head vectors of 128 channels = 4 groups of 32 are the rows of both quantizers (row n * Hkv + h).
// Lane layout: 8 lanes own one (token, group), each a 16-byte quarter of every 128-byte codeword
// row (a row is one cache line, gathered from L2 like decode_rows32_kernel does); 32 lanes = one
// token, a wavefront works on two tokens at a time, a workgroup of four wavefronts on eight.
// The common case first scores a block of tokens and then adds up its values (attn_phases_kernel); the general
// one takes each token's key and value together (attn_partial_kernel).  Either leaves one partial result per
// (kv head, split of the cache), maximum, sum and weighted values in base 2, and a second small kernel
// merges the splits.
#include <type_traits>

#include "rvq_internal.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int ATT_WAVES = 4;
constexpr int ATT_HD = 128;            // channels per head
constexpr int ATT_G = 4;               // groups of 32 per head
constexpr int ATT_PART = ATT_HD + 2;   // floats of a partial result: maximum, sum, weighted values
constexpr float ATT_NEG = -1.0e30f;    // "no token yet": finite, so that differences stay finite

struct AttnArgs {
  const float *q;           // [Hq][128]
  const void *kcodes;       // int16 [N * Hkv][4][depth], or packed records [N * Hkv][4][PK bytes]
  const void *vcodes;
  const void *kstd;         // [N * Hkv] or nullptr
  const void *vstd;
  const float *Ck;          // [depth][Kk][32]
  const float *Cv;
  const float *cos;         // [N][64] or nullptr (no rotation)
  const float *sin;
  float *part;              // [Hkv][S][REP][ATT_PART]
  float *out;               // [Hq][128]
  int64_t N;
  int64_t tps;              // tokens per split (a multiple of 8)
  int Hkv, S, depth, k_depth_used, v_depth_used, Kk, Kv;
  int kstd_dtype, vstd_dtype, k_strided, v_strided;
  int alone;                // no CU has a second workgroup
  int per_xcd;              // workgroups per XCD
  float scale_log2e;        // softmax scale times log2(e): scores are kept in base 2
};

// The codes of one (row, group) as they come from memory: four 32-bit words.
//   PK == 0: up to eight int16, two per word.
//   PK == 11 / 12 (depth 8): a packed record of PK bytes with eight PK-bit codes, code i in bits
//   [PK i, PK i + PK), little endian (rvq_pack_codes), fetched as its first and its last eight
//   bytes (two unaligned 8-byte loads that never reach beyond the record).
struct AttCodes { i32x4 w; };
template <bool D8, int PK>
__device__ __forceinline__ AttCodes att_load_codes(const void *codes, uint32_t rec, int depth) {
  AttCodes r;  // rec = row * 4 + g, relative to the split's first record
  if constexpr (PK != 0) {
    const unsigned char *p = reinterpret_cast<const unsigned char *>(codes) + rec * (uint32_t)PK;
    typedef unsigned u32x2u __attribute__((ext_vector_type(2), aligned(1)));
    const u32x2u lo = *reinterpret_cast<const u32x2u *>(p);
    const u32x2u hi = *reinterpret_cast<const u32x2u *>(p + PK - 8);
    r.w = i32x4{(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
  } else {
    const int16_t *p = reinterpret_cast<const int16_t *>(codes) + rec * (uint32_t)depth;
    if constexpr (D8) {
      r.w = *reinterpret_cast<const i32x4 *>(p);  // depth 8: one aligned 16-byte word
    } else {
      int c[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) c[i] = i < depth ? (int)p[i] & 0xffff : 0;
      r.w = i32x4{c[0] | (c[1] << 16), c[2] | (c[3] << 16), c[4] | (c[5] << 16), c[6] | (c[7] << 16)};
    }
  }
  return r;
}
// code i of it, as an unsigned number (an int16 below 0 becomes a large one)
template <int PK>
__device__ __forceinline__ uint32_t att_code(const AttCodes &cd, int i) {
  const uint32_t w4[4] = {(uint32_t)cd.w.x, (uint32_t)cd.w.y, (uint32_t)cd.w.z, (uint32_t)cd.w.w};
  if constexpr (PK == 0) {
    return (i & 1) ? (w4[i >> 1] >> 16) : (w4[i >> 1] & 0xffffu);
  } else {
    // bits 0..63 are the first load, bits 64.. the tail of the second (which starts at byte PK - 8)
    const uint32_t W[3] = {w4[0], w4[1], w4[3] >> (8 * (12 - PK))};
    const int word = (PK * i) >> 5, sh = (PK * i) & 31;
    uint32_t v;
    if (sh + PK <= 32) v = W[word] >> sh;                          // a code lies in one word
    else v = __builtin_amdgcn_alignbit(W[word + 1], W[word], sh);  // or straddles two
    return v & ((1u << PK) - 1u);
  }
}

// This lane's quarter of the codeword rows that the eight codes select: the loads only.  Cb is
// the codebook (the same for all lanes), lane_off the lane's 16-byte offset inside a row; a
// load is (stage base, scalar) + (code * 128 + lane_off, 32 bits).  A code is read as an unsigned
// 16-bit number and limited to K - 1, so any stored value stays inside the codebook.
// FULL: all eight stages are used (no condition anywhere near the loads); otherwise stages beyond
// `used` fetch row 0 of stage 0 and later enter the sum with weight 0.
template <bool FULL, int PK>
__device__ __forceinline__ void att_issue(const char *Cb, uint32_t lane_off, int K, const AttCodes &cd,
                                          int used, f32x4 (&rows)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t raw = att_code<PK>(cd, i);
    const uint32_t code = min(raw, (uint32_t)(K - 1));
    const char *stage = Cb + (size_t)i * (size_t)K * 128u;  // scalar
    uint32_t off = code * 128u + lane_off;
    if (!FULL) {
      off = i < used ? off : lane_off;
      stage = i < used ? stage : Cb;
    }
    rows[i] = *reinterpret_cast<const f32x4 *>(stage + off);
  }
}
// their sum in stage order
template <bool FULL>
__device__ __forceinline__ f32x4 att_sum(const f32x4 (&rows)[8], int used) {
  f32x4 s = rows[0];
#pragma unroll
  for (int i = 1; i < 8; ++i) {
    if (FULL) {
      s += rows[i];
    } else {
      const float w = i < used ? 1.0f : 0.0f;  // (x * 1 + s rounds as x + s)
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] = fmaf(rows[i][e], w, s[e]);
    }
  }
  return s;
}

// sums over lanes without LDS traffic (data-parallel-primitive moves): within a row of 16 lanes
// by two quad permutes and two rotations
template <int CTRL>
__device__ __forceinline__ float att_mov_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float att_sum16(float s) {
  s += att_mov_dpp<0xB1>(s);   // quad_perm [1,0,3,2]
  s += att_mov_dpp<0x4E>(s);   // quad_perm [2,3,0,1]
  s += att_mov_dpp<0x124>(s);  // row_ror:4
  s += att_mov_dpp<0x128>(s);  // row_ror:8
  return s;
}

// The general case: any depth up to 8, no rotation or no std, fp32 std; those are run-time conditions, and the
// loop has branches around its loads.  attn_phases_kernel is for the others.
// KS / VS: strided grouping of the key / value quantizer.
// PK: 0 = int16 codes; 11 / 12 = packed records of that many bytes (depth 8 only).
template <int REP, bool KS, bool VS, int PK>
__global__ __launch_bounds__(64 * ATT_WAVES) void attn_partial_kernel(const AttnArgs a) {
  __shared__ float sm_m[2 * ATT_WAVES][REP];
  __shared__ float sm_l[2 * ATT_WAVES][REP];
  __shared__ float sm_acc[2 * ATT_WAVES][REP][ATT_HD];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int half = lane >> 5, g = (lane >> 3) & 3, q8 = lane & 7;
  const int h = blockIdx.x % a.Hkv;   // kv head
  const int sp = blockIdx.x / a.Hkv;  // split of the cache
  const int64_t nbeg = (int64_t)sp * a.tps;
  const int64_t nend = nbeg + a.tps < a.N ? nbeg + a.tps : a.N;
  const int hw = wave * 2 + half;     // this half-wavefront takes tokens nbeg + hw, + 8, + 16, ...

  // channels of this lane's four values: element j = 4 q8 + e of group g
  int ck[4], cv[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int j = 4 * q8 + e;
    ck[e] = KS ? j * ATT_G + g : g * 32 + j;
    cv[e] = VS ? j * ATT_G + g : g * 32 + j;
  }
  float qv[REP][4];
#pragma unroll
  for (int r = 0; r < REP; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e) qv[r][e] = a.q[(int64_t)(h * REP + r) * ATT_HD + ck[e]] * a.scale_log2e;

  float m[REP], l[REP], acc[REP][4];
#pragma unroll
  for (int r = 0; r < REP; ++r) {
    m[r] = ATT_NEG;
    l[r] = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[r][e] = 0.f;
  }

  // Everything of this workgroup's tokens is addressed with 32-bit offsets from bases that are
  // the same for the whole workgroup (the launcher checks that a split's rows fit).
  const int64_t row0 = nbeg * a.Hkv + h;                      // row of token nbeg
  const int64_t rec_bytes = PK ? PK : 2 * a.depth;           // bytes of one (row, group)
  const char *kcb = reinterpret_cast<const char *>(a.kcodes) + row0 * ATT_G * rec_bytes;
  const char *vcb = reinterpret_cast<const char *>(a.vcodes) + row0 * ATT_G * rec_bytes;
  const char *ksb = a.kstd ? (const char *)a.kstd + row0 * (a.kstd_dtype == RVQ_F32 ? 4 : 2) : nullptr;
  const char *vsb = a.vstd ? (const char *)a.vstd + row0 * (a.vstd_dtype == RVQ_F32 ? 4 : 2) : nullptr;
  const float *cosb = a.cos ? a.cos + nbeg * (ATT_HD / 2) : nullptr;
  const float *sinb = a.cos ? a.sin + nbeg * (ATT_HD / 2) : nullptr;
  const char *Ckb = reinterpret_cast<const char *>(a.Ck);
  const char *Cvb = reinterpret_cast<const char *>(a.Cv);
  const uint32_t lane_off = 16u * (uint32_t)q8;
  const uint32_t last = (uint32_t)(nend - nbeg) - 1u;         // last token of the split, relative
  const uint32_t row_recs = (uint32_t)(a.Hkv * ATT_G);        // (row, group) records between tokens

  // what a token needs from HBM; it is fetched one trip ahead (the gathers depend on the
  // codes)
  struct Pre {
    AttCodes kc, vc;
    float ks, vs, cs[4], sn[4];
  };
  auto fetch = [&](uint32_t t, Pre &p) {
    const uint32_t tc = t < last ? t : last;  // clamped: loads carry no branch
    const uint32_t rec = tc * row_recs + (uint32_t)g;
    p.kc = att_load_codes<false, PK>(kcb, rec, a.depth);
    p.vc = att_load_codes<false, PK>(vcb, rec, a.depth);
    const uint32_t ro = tc * (uint32_t)a.Hkv;
    p.ks = !ksb ? 1.0f : (a.kstd_dtype == RVQ_F32 ? ((const float *)ksb)[ro]
                                                  : rvq_f16_bits_to_f32(((const uint16_t *)ksb)[ro]));
    p.vs = !vsb ? 1.0f : (a.vstd_dtype == RVQ_F32 ? ((const float *)vsb)[ro]
                                                  : rvq_f16_bits_to_f32(((const uint16_t *)vsb)[ro]));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p.cs[e] = cosb ? cosb[tc * (ATT_HD / 2) + (ck[e] >> 1)] : 1.0f;
      p.sn[e] = cosb ? sinb[tc * (ATT_HD / 2) + (ck[e] >> 1)] : 0.0f;
    }
  };
  // A wavefront's loads come back in the order they were issued.  So a trip first issues the
  // gathers of its own token (L2), then the prefetch of the next one (HBM), and only then works on
  // the gathered rows: waiting for the gathers does not wait for HBM.
  struct Rows { f32x4 k[8], v[8]; };
  auto issue = [&](const Pre &p, Rows &R) {
    att_issue<false, PK>(Ckb, lane_off, a.Kk, p.kc, a.k_depth_used, R.k);
    att_issue<false, PK>(Cvb, lane_off, a.Kv, p.vc, a.v_depth_used, R.v);
  };
  auto work = [&](uint32_t t, const Pre &p, const Rows &R) {
    const bool valid = t <= last;
    f32x4 k4 = att_sum<false>(R.k, a.k_depth_used);
    f32x4 v4 = att_sum<false>(R.v, a.v_depth_used);
    k4 *= p.ks;
    v4 *= p.vs;
    // rotation: channel c and its partner c ^ 1 are one pair; the partner is element e ^ 1 of
    // this lane (contiguous groups) or the same element of the lane of group g ^ 1, eight lanes
    // away in the same row of 16 (strided)
    float kr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float mine = k4[e];
      const float other = KS ? att_mov_dpp<0x128>(mine) : k4[e ^ 1];
      // even channel: x0 cos - x1 sin; odd channel: x1 cos + x0 sin
      kr[e] = mine * p.cs[e] + ((ck[e] & 1) ? other : -other) * p.sn[e];
    }
#pragma unroll
    for (int r = 0; r < REP; ++r) {
      float s = kr[0] * qv[r][0];
#pragma unroll
      for (int e = 1; e < 4; ++e) s = fmaf(kr[e], qv[r][e], s);
      // the token's 32 lanes = two rows of 16: all of them end up with the whole score
      s = att_sum16(s);
      s += __shfl_xor(s, 16, 64);
      s = valid ? s : -3.0e38f;
      const float mn = fmaxf(m[r], s);
      const float corr = __builtin_amdgcn_exp2f(m[r] - mn);
      const float pw = __builtin_amdgcn_exp2f(s - mn);  // 0 for a token beyond the end
      m[r] = mn;
      l[r] = fmaf(l[r], corr, pw);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[r][e] = fmaf(acc[r][e], corr, pw * v4[e]);
    }
  };

  const int64_t span = nend - nbeg;
  const int trips = span > 0 ? (int)((span + 2 * ATT_WAVES - 1) / (2 * ATT_WAVES)) : 0;  // uniform
  constexpr uint32_t STEP = 2 * ATT_WAVES;
  Rows R;
  uint32_t t = (uint32_t)hw;  // token of this half-wavefront, relative to nbeg
  Pre pa, pb;
  if (trips > 0) fetch(t, pa);
  for (int it = 0; it < trips; it += 2) {
    issue(pa, R);
    fetch(t + STEP, pb);
    work(t, pa, R);
    t += STEP;
    if (it + 1 >= trips) break;
    issue(pb, R);
    fetch(t + STEP, pa);
    work(t, pb, R);
    t += STEP;
  }

  // merge the eight half-wavefronts of the workgroup
#pragma unroll
  for (int r = 0; r < REP; ++r) {
#pragma unroll
    for (int e = 0; e < 4; ++e) sm_acc[hw][r][cv[e]] = acc[r][e];
    if ((lane & 31) == 0) {
      sm_m[hw][r] = m[r];
      sm_l[hw][r] = l[r];
    }
  }
  __syncthreads();
  for (int idx = tid; idx < REP * ATT_HD; idx += 64 * ATT_WAVES) {
    const int r = idx / ATT_HD, c = idx % ATT_HD;
    float M = sm_m[0][r];
#pragma unroll
    for (int w = 1; w < 2 * ATT_WAVES; ++w) M = fmaxf(M, sm_m[w][r]);
    float tot = 0.f, L = 0.f;
#pragma unroll
    for (int w = 0; w < 2 * ATT_WAVES; ++w) {
      const float f = __builtin_amdgcn_exp2f(sm_m[w][r] - M);
      tot = fmaf(sm_acc[w][r][c], f, tot);
      L = fmaf(sm_l[w][r], f, L);
    }
    float *dst = a.part + (((int64_t)h * a.S + sp) * REP + r) * ATT_PART;
    dst[2 + c] = tot;
    if (c == 0) {
      dst[0] = M;
      dst[1] = L;
    }
  }
}

// sums of REP values over the 32 lanes of a token: every step that can hands half of the values to the partner
// lane and keeps the other half, so lane l ends up with the sum of value l % REP
template <int REP>
__device__ __forceinline__ float att_sum_token(float (&s)[REP], int lane) {
  float v;
  if constexpr (REP == 1) {
    v = s[0] + att_mov_dpp<0xB1>(s[0]);
  } else {
    float k[REP / 2];
#pragma unroll
    for (int i = 0; i < REP / 2; ++i) {
      const bool odd = (lane & 1) != 0;
      k[i] = (odd ? s[2 * i + 1] : s[2 * i]) + att_mov_dpp<0xB1>(odd ? s[2 * i] : s[2 * i + 1]);
    }
    if constexpr (REP == 2) {
      v = k[0];
    } else {
      float k2[REP / 4];
#pragma unroll
      for (int i = 0; i < REP / 4; ++i) {
        const bool up = (lane & 2) != 0;
        k2[i] = (up ? k[2 * i + 1] : k[2 * i]) + att_mov_dpp<0x4E>(up ? k[2 * i] : k[2 * i + 1]);
      }
      if constexpr (REP == 4) {
        v = k2[0];
      } else {
        const bool up = (lane & 4) != 0;  // (four lanes on, whatever the lane's bit 3: both are added below)
        v = (up ? k2[1] : k2[0]) + att_mov_dpp<0x124>(up ? k2[0] : k2[1]);
      }
    }
  }
  if constexpr (REP <= 2) v += att_mov_dpp<0x4E>(v);
  if constexpr (REP <= 4) v += att_mov_dpp<0x124>(v);
  v += att_mov_dpp<0x128>(v);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// op over the lanes of a wavefront that agree modulo REP (1, 2, 4 or 8), in every lane: by lane moves, none of
// which goes through LDS (six shuffles there are a quarter of a microsecond, twice per workgroup and merge)
template <int REP, class Op>
__device__ __forceinline__ float att_wave_reduce(float v, Op op) {
  {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  v = op(v, att_mov_dpp<0x128>(v));
  if constexpr (REP <= 4) v = op(v, att_mov_dpp<0x124>(v));
  if constexpr (REP <= 2) v = op(v, att_mov_dpp<0x4E>(v));
  if constexpr (REP <= 1) v = op(v, att_mov_dpp<0xB1>(v));
  return v;
}
__device__ __forceinline__ float att_max(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ float att_add(float a, float b) { return a + b; }

// The common case: depth 8 with all stages used, rotation tables given, both std buffers in half precision.  A
// workgroup takes ATT_BLOCK tokens at a time through two phases:
//   keys:   every token is decoded, rotated and scored; the scores stay in LDS;
//   (then the maxima of the wavefront's tokens, and the weights 2^(score - maximum) times the values' std, in place
//   of the scores: every wavefront by itself, there is no barrier before the end)
//   values: every token is decoded and added up under its weights.
// What bounds it is the gathers of 8 KiB of codeword rows per (token, kv head): L1 address path and L2.  Two
// phases because
//  - an XCD's L2 (4 MiB) holds one codebook (2 MiB at K = 2048) with room, not two: the workgroups of a launch
//    that is resident at once stay roughly in the same phase;
//  - a phase's rows take half the registers, so the next token's rows travel while this token's are worked on;
//  - a token's weight is computed once, not by its 32 lanes, and nothing is rescaled per token.
// The workgroups of the kv heads of one split sit on one XCD, or on two: rotary tables and the cache
// lines that several heads' codes share are fetched by one L2.  Every XCD gets as many workgroups as the next,
// whatever the numbers of heads and splits.
// Everything from HBM passes through LDS: the 64 lanes fetch the codes of eight trips of both half-wavefronts, a
// record each, and the 32 lanes of a token its tables, a piece each (per lane of use, 176 of a trip's 432
// L1 accesses would repeat another lane's).  A wavefront's own areas: its LDS operations run in order.
// Where every workgroup has a CU to itself and few trips to make, values are decoded along with the keys, both rows
// in one round trip, and their sums stay in LDS until the weights are there: what is left is a chain of
// round trips (1000 tokens x 8 kv heads, 4 queries each: 12.5 -> 11.9 us).  With a second workgroup on the CU to
// fill the waits, phases are faster (2000 tokens 15.4 : 16.4).
constexpr int ATT_BLOCK = 1024;
constexpr int ATT_BRIEF = 4;  // trips
template <int REP, bool KS, bool VS, int PK>
__global__ __launch_bounds__(64 * ATT_WAVES, 2) void attn_phases_kernel(const AttnArgs a) {
  constexpr int NT = 64 * ATT_WAVES;
  constexpr uint32_t STEP = 2 * ATT_WAVES;               // tokens per trip of the workgroup
  constexpr int BW = ATT_BLOCK / ATT_WAVES;              // tokens of a wavefront in a block
  constexpr int VPT = BW / 64;                           // value stds per lane
  __shared__ __align__(16) float sm_w[ATT_BLOCK * REP];  // scores, then weights: [wavefront][token][query head]
  __shared__ __align__(16) i32x4 sm_codes[2][ATT_WAVES][2][64];  // [K, V][eight trips, even / odd][half][trip][group]
  __shared__ float sm_std[ATT_WAVES][2][16];                  // [even / odd][half][trip]
  __shared__ __align__(16) float sm_tab[ATT_WAVES][2][ATT_HD];  // [half][64 cos, 64 sin]
  __shared__ __align__(16) f32x4 sm_v[ATT_BRIEF][NT];         // value sums of a short block
  __shared__ float sm_vs[ATT_WAVES][BW];                      // the values' std
  __shared__ float sm_m[ATT_WAVES][REP], sm_l[ATT_WAVES][REP], sm_corr[ATT_WAVES][REP];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, g = (lane >> 3) & 3, q8 = lane & 7;
  // An XCD (ids equal modulo eight) has every eighth split, or, if their number is no multiple of eight, an eighth of
  // the list of all (split, head).  Heads run fastest.
  const bool whole = (a.S & 7) == 0;
  const int xcd = blockIdx.x & 7, num = (whole ? 0 : xcd * a.per_xcd) + (int)(blockIdx.x >> 3);
  const int h = num % a.Hkv, sp = whole ? xcd + 8 * (num / a.Hkv) : num / a.Hkv;
  if (sp >= a.S) return;
  const int64_t nbeg = (int64_t)sp * a.tps;
  const int64_t nend = nbeg + a.tps < a.N ? nbeg + a.tps : a.N;
  const uint32_t span = (uint32_t)(nend - nbeg), last = span - 1u;  // tokens of the split (>= 1)
  const uint32_t hw = (uint32_t)(wave * 2 + half);

  int ck[4], cv[4];  // channels of this lane's four values: element j = 4 q8 + e of group g
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int j = 4 * q8 + e;
    ck[e] = KS ? j * ATT_G + g : g * 32 + j;
    cv[e] = VS ? j * ATT_G + g : g * 32 + j;
  }
  float qv[REP][4], acc[REP][4];
#pragma unroll
  for (int r = 0; r < REP; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      qv[r][e] = a.q[(int64_t)(h * REP + r) * ATT_HD + ck[e]] * a.scale_log2e;
      acc[r][e] = 0.f;
    }
  float m_run = ATT_NEG, l_run = 0.f;  // the wavefront's, of query head lane % REP; the sum of this lane's weights only

  // 32-bit offsets from bases that are the same for the whole workgroup (the launcher checks that they fit)
  const int64_t row0 = nbeg * a.Hkv + h;
  constexpr int64_t REC = PK ? PK : 16;  // bytes of one (row, group)
  const char *kcb = reinterpret_cast<const char *>(a.kcodes) + row0 * ATT_G * REC;
  const char *vcb = reinterpret_cast<const char *>(a.vcodes) + row0 * ATT_G * REC;
  const uint16_t *ksb = reinterpret_cast<const uint16_t *>(a.kstd) + row0;
  const uint16_t *vsb = reinterpret_cast<const uint16_t *>(a.vstd) + row0;
  const uint32_t hkv = (uint32_t)a.Hkv, row_recs = hkv * ATT_G;
  const uint32_t lane_off = 16u * (uint32_t)q8;
  // this lane's piece of a token's tables: lanes 0..15 of the half cos, 16..31 sin
  const int l32 = lane & 31;
  const float *tab_src = (l32 < 16 ? a.cos : a.sin) + nbeg * (ATT_HD / 2) + (l32 & 15) * 4;
  float *tab = sm_tab[wave][half];

  AttCodes cn;  // the next eight trips' record of this lane (trip q8, group g)
  auto fetch8 = [&](const char *base, uint32_t t0, int it) {
    const uint32_t tt = t0 + hw + STEP * (uint32_t)(it + q8), tc = tt < last ? tt : last;
    cn = att_load_codes<true, PK>(base, tc * row_recs + (uint32_t)g, 8);
  };
  auto store8 = [&](int kv, int it) { sm_codes[kv][wave][(it >> 3) & 1][half * 32 + q8 * 4 + g] = cn.w; };
  auto codes_of = [&](int kv, int i) {
    AttCodes c;
    c.w = sm_codes[kv][wave][(i >> 3) & 1][half * 32 + (i & 7) * 4 + g];
    return c;
  };

  for (uint32_t t0 = 0; t0 < span; t0 += ATT_BLOCK) {
    const uint32_t cnt = min(span - t0, (uint32_t)ATT_BLOCK);
    const int trips = (int)((cnt + STEP - 1) / STEP);  // >= 1
    const bool brief = a.alone && trips <= ATT_BRIEF;
    // token of the block that is number j of this wavefront: half j & 1, trip j >> 1
    auto token = [&](uint32_t j) { return (uint32_t)wave * 2u + (j & 1u) + STEP * (j >> 1); };
    float *wts = sm_w + wave * BW * REP;
    uint16_t vstd[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const uint32_t t = t0 + token((uint32_t)(lane + i * 64));
      vstd[i] = vsb[(t < last ? t : last) * hkv];
    }
    // ---- keys
    {
      float ksn;
      auto fetch_std = [&](int it) {
        const uint32_t tt = t0 + hw + STEP * (uint32_t)(it + q8), tc = tt < last ? tt : last;
        ksn = rvq_f16_bits_to_f32(ksb[tc * hkv]);
      };
      auto store_std = [&](int it) { sm_std[wave][(it >> 3) & 1][half * 8 + q8] = ksn; };
      auto fetch_tab = [&](int i) -> f32x4 {
        const uint32_t tt = t0 + hw + STEP * (uint32_t)i, tc = tt < last ? tt : last;
        typedef float f32x4a4 __attribute__((ext_vector_type(4), aligned(4)));
        return *reinterpret_cast<const f32x4a4 *>(tab_src + tc * (ATT_HD / 2));
      };
      fetch8(kcb, t0, 0);
      fetch_std(0);
      const AttCodes kn = cn;
      fetch8(vcb, t0, 0);
      const AttCodes vn = cn;
      cn = kn;
      f32x4 tabn = fetch_tab(0), tabm = fetch_tab(1);
      store8(0, 0);
      store_std(0);
      cn = vn;
      store8(1, 0);
      __builtin_amdgcn_wave_barrier();
      auto trip = [&](int i, f32x4 &tb, auto both) {
        f32x4 R[8], Rv[8];
        __builtin_amdgcn_wave_barrier();
        att_issue<true, PK>(reinterpret_cast<const char *>(a.Ck), lane_off, a.Kk, codes_of(0, i), 8, R);
        if constexpr (both) att_issue<true, PK>(reinterpret_cast<const char *>(a.Cv), lane_off, a.Kv, codes_of(1, i), 8, Rv);
        if (!both && (i & 7) == 0 && i + 8 < trips) {
          fetch8(kcb, t0, i + 8);
          fetch_std(i + 8);
        }
        const float ks = sm_std[wave][(i >> 3) & 1][half * 8 + (i & 7)];
        *reinterpret_cast<f32x4 *>(tab + l32 * 4) = tb;
        __builtin_amdgcn_wave_barrier();
        tb = fetch_tab(i + 2);
        float cs[4], sn[4];
        if constexpr (KS) {
          // pairs 8 q8 + 2 e + (g >> 1)
          const f32x4 *cp = reinterpret_cast<const f32x4 *>(tab + 8 * q8);
          const f32x4 *sp_ = reinterpret_cast<const f32x4 *>(tab + ATT_HD / 2 + 8 * q8);
          const f32x4 c0 = cp[0], c1 = cp[1], s0 = sp_[0], s1 = sp_[1];
          const bool hi = (g >> 1) != 0;
          cs[0] = hi ? c0[1] : c0[0]; cs[1] = hi ? c0[3] : c0[2];
          cs[2] = hi ? c1[1] : c1[0]; cs[3] = hi ? c1[3] : c1[2];
          sn[0] = hi ? s0[1] : s0[0]; sn[1] = hi ? s0[3] : s0[2];
          sn[2] = hi ? s1[1] : s1[0]; sn[3] = hi ? s1[3] : s1[2];
        } else {
          // the two pairs 16 g + 2 q8, + 1
          typedef float f32x2 __attribute__((ext_vector_type(2)));
          const f32x2 c2 = *reinterpret_cast<const f32x2 *>(tab + 16 * g + 2 * q8);
          const f32x2 s2 = *reinterpret_cast<const f32x2 *>(tab + ATT_HD / 2 + 16 * g + 2 * q8);
          cs[0] = cs[1] = c2[0]; cs[2] = cs[3] = c2[1];
          sn[0] = sn[1] = s2[0]; sn[2] = sn[3] = s2[1];
        }
        f32x4 k4 = att_sum<true>(R, 8);
        k4 *= ks;
        // rotation: the partner of channel c is c ^ 1, element e ^ 1 of this lane (contiguous groups) or the same
        // element of the lane of group g ^ 1, eight lanes away in the same row of 16 (strided)
        float kr[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float other = KS ? att_mov_dpp<0x128>(k4[e]) : k4[e ^ 1];
          kr[e] = k4[e] * cs[e] + ((ck[e] & 1) ? other : -other) * sn[e];
        }
        float s[REP];
#pragma unroll
        for (int r = 0; r < REP; ++r) {
          s[r] = kr[0] * qv[r][0];
#pragma unroll
          for (int e = 1; e < 4; ++e) s[r] = fmaf(kr[e], qv[r][e], s[r]);
        }
        const float v = att_sum_token<REP>(s, lane);
        if (l32 < REP) wts[(2 * i + half) * REP + l32] = v;  // (beyond the end: overwritten with weight 0)
        if constexpr (both) sm_v[i][tid] = att_sum<true>(Rv, 8);
        if (!both && (i & 7) == 5 && i + 3 < trips) {
          store8(0, i + 3);
          store_std(i + 3);
        }
      };
      if (brief) {
        for (int i = 0; i < trips; ++i) {
          trip(i, tabn, std::true_type());
          const f32x4 t = tabn;
          tabn = tabm;
          tabm = t;
        }
      } else {
        for (int i = 0; i < trips; i += 2) {
          trip(i, tabn, std::false_type());
          if (i + 1 < trips) trip(i + 1, tabm, std::false_type());
        }
      }
    }
    // ---- weights
    // the first trip's rows travel under the weights (also where a brief split has its values' sums in LDS: a condition
    // here gains a brief split nothing, 1000 tokens 11.6 us both, and costs the others 2 %, 2100 tokens 16.4 -> 16.65)
    f32x4 R[8];
    __builtin_amdgcn_wave_barrier();
    att_issue<true, PK>(reinterpret_cast<const char *>(a.Cv), lane_off, a.Kv, codes_of(1, 0), 8, R);
#pragma unroll
    for (int i = 0; i < VPT; ++i) sm_vs[wave][lane + i * 64] = rvq_f16_bits_to_f32(vstd[i]);
    __builtin_amdgcn_wave_barrier();
    {
      const int num = 2 * trips * REP;
      float mx = m_run;
      for (int idx = lane; idx < num; idx += 64)
        if (token((uint32_t)(idx / REP)) < cnt) mx = fmaxf(mx, wts[idx]);
      mx = att_wave_reduce<REP>(mx, att_max);
      const float corr = __builtin_amdgcn_exp2f(m_run - mx);
      l_run *= corr;
      m_run = mx;
      if (lane < REP) sm_corr[wave][lane] = corr;
      for (int idx = lane; idx < num; idx += 64) {
        const float pw = token((uint32_t)(idx / REP)) < cnt ? __builtin_amdgcn_exp2f(wts[idx] - mx) : 0.f;
        l_run += pw;
        wts[idx] = pw * sm_vs[wave][idx / REP];
      }
    }
    __builtin_amdgcn_wave_barrier();
    // ---- values
    {
#pragma unroll
      for (int r = 0; r < REP; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[r][e] *= sm_corr[wave][r];
      auto add = [&](int i, const f32x4 v4) {
        float w[REP];
#pragma unroll
        for (int r = 0; r < REP; ++r) w[r] = wts[(2 * i + half) * REP + r];
#pragma unroll
        for (int r = 0; r < REP; ++r)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[r][e] = fmaf(w[r], v4[e], acc[r][e]);
      };
      auto trip = [&](int i, bool first) {
        __builtin_amdgcn_wave_barrier();
        if (!first) att_issue<true, PK>(reinterpret_cast<const char *>(a.Cv), lane_off, a.Kv, codes_of(1, i), 8, R);
        if ((i & 7) == 0 && i + 8 < trips) fetch8(vcb, t0, i + 8);
        add(i, att_sum<true>(R, 8));
        if ((i & 7) == 5 && i + 3 < trips) store8(1, i + 3);
      };
      if (brief) {
        for (int i = 0; i < trips; ++i) add(i, sm_v[i][tid]);
      } else {
        trip(0, true);
        for (int i = 1; i < trips; ++i) trip(i, false);
      }
    }
    __builtin_amdgcn_wave_barrier();  // (the next block's scores overwrite the weights)
  }

  // ---- the workgroup's sums: the halves of a wavefront by a lane swap, the wavefronts, each with its own
  // maximum, through LDS (a wavefront's part of the weights' memory)
  static_assert(BW >= ATT_HD, "a wavefront's weights leave room for its sums");
#pragma unroll
  for (int r = 0; r < REP; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned u = __float_as_uint(acc[r][e]);
      const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
      if (half == 0) sm_w[(wave * REP + r) * BW + cv[e]] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
  l_run = att_wave_reduce<REP>(l_run, att_add);
  if (lane < REP) {
    sm_m[wave][lane] = m_run;
    sm_l[wave][lane] = l_run;
  }
  __syncthreads();
  float *dst = a.part + ((int64_t)h * a.S + sp) * REP * ATT_PART;
  for (int idx = tid; idx < REP * ATT_HD; idx += NT) {
    const int r = idx / ATT_HD, c = idx % ATT_HD;
    float M = sm_m[0][r], tot = 0.f, L = 0.f;
#pragma unroll
    for (int w = 1; w < ATT_WAVES; ++w) M = fmaxf(M, sm_m[w][r]);
#pragma unroll
    for (int w = 0; w < ATT_WAVES; ++w) {
      const float f = __builtin_amdgcn_exp2f(sm_m[w][r] - M);
      tot = fmaf(sm_w[(w * REP + r) * BW + c], f, tot);
      L = fmaf(sm_l[w][r], f, L);
    }
    dst[r * ATT_PART + 2 + c] = tot;
    if (c == 0) {
      dst[r * ATT_PART] = M;
      dst[r * ATT_PART + 1] = L;
    }
  }
}

// One workgroup per query head: merge the partial results of the splits and normalise.  Eight threads share a
// channel, an eighth of the splits each (one thread per channel took 16 us for 256 splits, 6 for 53: round trips).
constexpr int ATT_MAX_SPLITS = 2048;
constexpr int ATT_MERGE = 8 * ATT_HD;
__global__ __launch_bounds__(ATT_MERGE) void attn_merge_kernel(const float *__restrict__ part, int S, int REP,
                                                               float *__restrict__ out) {
  __shared__ float f[ATT_MAX_SPLITS];  // maxima of the splits, then their weights 2^(m_s - M)
  __shared__ float red[ATT_MERGE / 64][2];
  __shared__ float sums[8][ATT_HD];
  const int hq = blockIdx.x, c = threadIdx.x % ATT_HD, oct = threadIdx.x / ATT_HD;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = hq / REP, r = hq % REP;
  const float *base = part + ((int64_t)h * S * REP + r) * ATT_PART;
  const int64_t stride = (int64_t)REP * ATT_PART;
  // the first rounds of partial sums are requested along with the maxima
  constexpr int AHEAD = 8;
  float ps[AHEAD];
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) ps[i] = oct + 8 * i < S ? base[(oct + 8 * i) * stride + 2 + c] : 0.f;
  float ms[ATT_MAX_SPLITS / ATT_MERGE], ls[ATT_MAX_SPLITS / ATT_MERGE], M = ATT_NEG, L = 0.f;
#pragma unroll
  for (int i = 0; i < ATT_MAX_SPLITS / ATT_MERGE; ++i) {
    const int s = threadIdx.x + i * ATT_MERGE;
    ms[i] = s < S ? base[s * stride] : ATT_NEG;
    ls[i] = s < S ? base[s * stride + 1] : 0.f;
    M = fmaxf(M, ms[i]);
  }
  M = att_wave_reduce<1>(M, att_max);
  if (lane == 0) red[wave][0] = M;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < ATT_MERGE / 64; ++w) M = fmaxf(M, red[w][0]);
#pragma unroll
  for (int i = 0; i < ATT_MAX_SPLITS / ATT_MERGE; ++i) {
    const int s = threadIdx.x + i * ATT_MERGE;
    const float w = __builtin_amdgcn_exp2f(ms[i] - M);
    if (s < S) {
      f[s] = w;
      L = fmaf(ls[i], w, L);
    }
  }
  L = att_wave_reduce<1>(L, att_add);
  if (lane == 0) red[wave][1] = L;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int i = 0; i < AHEAD; ++i)
    if (oct + 8 * i < S) tot = fmaf(ps[i], f[oct + 8 * i], tot);
#pragma unroll 4
  for (int s = oct + 8 * AHEAD; s < S; s += 8) tot = fmaf(base[s * stride + 2 + c], f[s], tot);
  sums[oct][c] = tot;
  __syncthreads();
  if (oct == 0) {
    L = 0.f;
    tot = 0.f;
#pragma unroll
    for (int w = 0; w < ATT_MERGE / 64; ++w) L += red[w][1];
#pragma unroll
    for (int w = 0; w < 8; ++w) tot += sums[w][c];
    out[(int64_t)hq * ATT_HD + c] = tot / L;
  }
}

}  // namespace

// splits of a cache of N tokens over Hkv kv heads; the same rule sizes the workspace.  A long
// cache: about 2048 workgroups, at least 128 tokens each: what attn_partial_kernel wants and the most that a
// launch can have (attn_phases_kernel, the common case, takes two per CU, see below).  A short
// one is a matter of latency (a wavefront's trips are a chain of dependent loads): splits down to
// 32 tokens, four trips of a workgroup, as long as that makes no more than 512 workgroups
// (measured: 2048 tokens x 8 heads 32 -> 19 us; with 2048 workgroups of 32 tokens at 8192 tokens
// 43 -> 57 us, so not beyond 512).
static int attn_splits(int64_t N, int Hkv) {
  const int h = Hkv > 0 ? Hkv : 1;
  int64_t lng = (N + 127) / 128, cap = 2048 / h;
  if (cap < 1) cap = 1;
  if (lng > cap) lng = cap;
  int64_t shrt = (N + 31) / 32, cap_s = 512 / h;
  if (shrt > cap_s) shrt = cap_s;
  int64_t s = lng > shrt ? lng : shrt;
  if (s < 1) s = 1;
  return (int)s;
}

size_t rvq_attn_workspace_floats(int64_t N, int Hq, int Hkv) {
  return (size_t)attn_splits(N, Hkv) * (size_t)Hq * ATT_PART;
}

hipError_t rvq_launch_attn_decode(const rvq_ctx *kctx, const rvq_ctx *vctx, const float *dQ, int Hq,
                                  int Hkv, const void *dKCodes, const void *dKStd,
                                  const void *dVCodes, const void *dVStd, int packed_bytes, int64_t N,
                                  const float *dCos, const float *dSin, float scale, int k_depth_used,
                                  int v_depth_used, float *dOut, float *dWork, hipStream_t s) {
  AttnArgs a;
  a.q = dQ;
  a.kcodes = dKCodes;
  a.vcodes = dVCodes;
  a.kstd = dKStd;
  a.vstd = dVStd;
  a.Ck = kctx->C;
  a.Cv = vctx->C;
  a.cos = dCos;
  a.sin = dSin;
  a.part = dWork;
  a.out = dOut;
  a.N = N;
  a.Hkv = Hkv;
  a.S = attn_splits(N, Hkv);
  int64_t tps = (N + a.S - 1) / a.S;
  tps = (tps + 7) / 8 * 8;
  a.tps = tps;
  a.S = (int)((N + tps - 1) / tps);  // no empty split
  a.depth = kctx->cfg.depth;
  a.k_depth_used = k_depth_used;
  a.v_depth_used = v_depth_used;
  a.Kk = kctx->cfg.K;
  a.Kv = vctx->cfg.K;
  a.kstd_dtype = kctx->cfg.std_dtype;
  a.vstd_dtype = vctx->cfg.std_dtype;
  a.k_strided = kctx->cfg.grouping == RVQ_STRIDED;
  a.v_strided = vctx->cfg.grouping == RVQ_STRIDED;
  a.scale_log2e = scale * 1.4426950408889634f;
  const int rep = Hq / Hkv;
  const bool fast = a.depth == 8 && k_depth_used == 8 && v_depth_used == 8 && dCos && dKStd && dVStd &&
                    a.kstd_dtype == RVQ_F16 && a.vstd_dtype == RVQ_F16;
  if (fast) {
    // Two workgroups per CU, resident at once, so that their phases stay together.  131072 tokens x 8 kv heads, 4
    // queries each: one workgroup per CU 463 us, two 338, one and a half 464, two and a half 450, three 377
    // (blocks of 512), four 368: a CU's workgroups take the time of two, 338 / 256 of the whole per pair, an odd one
    // 463 / 512, and a few percent more where pairs follow each other.  Heads that do not divide two per CU well
    // (a kv head is the least a workgroup can have) get the number of rounds that leaves the least idle: 2^20 (token,
    // head), one query each, 36 heads 573 -> 322 us, 40 517 -> 328, 300 573 -> 317 (8: 309).
    const int64_t cus = kctx->num_cus > 0 ? kctx->num_cus : 1;
    if ((int64_t)a.S * Hkv > 2 * cus) {
      int64_t best = 0;
      double least = 0.0;
      for (int m = 2; m <= 8; ++m) {
        int64_t sm = m * cus / Hkv;
        if (sm < 1 || sm > a.S) continue;
        if (sm / 8 * 8 * 25 >= sm * 24) sm = sm / 8 * 8;  // (whole splits per XCD: 20 heads, 25 splits 346 us, 24 328)
        const double t = (338.0 * m + (m & 1 ? 125.0 : 0.0)) * (1.0 + 0.045 * (m - 2)) / (double)(sm * Hkv);
        if (best == 0 || t < least) {
          best = sm;
          least = t;
        }
      }
      const int64_t longer = best > 0 ? ((N + best - 1) / best + 7) / 8 * 8 : 0;
      if (longer > 0 && longer * Hkv * ATT_G * 16 < (int64_t)1 << 32) {  // (codes of a split are addressed with 32 bits)
        a.tps = longer;
        a.S = (int)((N + longer - 1) / longer);
      }
    }
  }
  a.alone = (int64_t)a.S * Hkv <= kctx->num_cus;
  a.per_xcd = (a.S * Hkv + 7) / 8;
  const dim3 grid((unsigned)(fast ? 8 * a.per_xcd : a.S * Hkv)), block(64 * ATT_WAVES);
  // (one and two queries per kv head leave room for a third workgroup on a CU: 10 KiB of LDS keep it out.  2^20 (token,
  // head), 200 heads 350 -> 319 us, 300 343 -> 317)
  const size_t lds = fast && rep <= 2 ? 10240 : 0;
#define RVQ_ATT_LAUNCH3(KERNEL, R, P)                                                                 \
  if (a.k_strided) {                                                                                 \
    if (a.v_strided) hipLaunchKernelGGL((KERNEL<R, true, true, P>), grid, block, lds, s, a);           \
    else hipLaunchKernelGGL((KERNEL<R, true, false, P>), grid, block, lds, s, a);                      \
  } else {                                                                                           \
    if (a.v_strided) hipLaunchKernelGGL((KERNEL<R, false, true, P>), grid, block, lds, s, a);          \
    else hipLaunchKernelGGL((KERNEL<R, false, false, P>), grid, block, lds, s, a);                     \
  }
#define RVQ_ATT_LAUNCH2(KERNEL, R)                   \
  if (packed_bytes == 11) {                          \
    RVQ_ATT_LAUNCH3(KERNEL, R, 11)                   \
  } else if (packed_bytes == 12) {                   \
    RVQ_ATT_LAUNCH3(KERNEL, R, 12)                   \
  } else {                                           \
    RVQ_ATT_LAUNCH3(KERNEL, R, 0)                    \
  }
#define RVQ_ATT_LAUNCH(R)                            \
  if (fast) {                                        \
    RVQ_ATT_LAUNCH2(attn_phases_kernel, R)           \
  } else {                                           \
    RVQ_ATT_LAUNCH2(attn_partial_kernel, R)          \
  }
  switch (rep) {
    case 1: RVQ_ATT_LAUNCH(1) break;
    case 2: RVQ_ATT_LAUNCH(2) break;
    case 4: RVQ_ATT_LAUNCH(4) break;
    default: RVQ_ATT_LAUNCH(8) break;
  }
#undef RVQ_ATT_LAUNCH
#undef RVQ_ATT_LAUNCH2
#undef RVQ_ATT_LAUNCH3
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(attn_merge_kernel, dim3((unsigned)Hq), dim3(ATT_MERGE), 0, s, dWork, a.S, rep, dOut);
  return hipGetLastError();
}
