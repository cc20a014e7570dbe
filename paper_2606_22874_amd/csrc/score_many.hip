// Selector scores of many query rows per sequence on the matrix cores (a
// prompt: one row per query block; paper Sections 2.1 and 2.3), for pooled
// keys (a score per key) and for per-token keys (the largest visible token
// score of every block of 16 or 64).  Any number of rows and keys, any key
// format.
//
// Row by row (the decode kernels), every row re-reads every key: 256 causal
// rows over 16384 tokens took 91 us, here 10.4 (2.1 GFLOP and 17 MB: bound
// by the latency of a workgroup's first loads and of each step's).  A workgroup
// takes 64 rows -- 16 per wave, their queries held in registers as B
// operands -- and streams a run of keys through LDS, 32 at a time, as the A
// operand of v_mfma_f32_16x16x32_bf16.  Lane l ends with the scores of keys
// 4(l/16) ..+3 for row l%16, so the ReLU, the row's w_h, the head sum and
// the maximum over keys need no exchange (two lane swaps finish a block's
// maximum).
//
// Quantized keys are staged as their codes in BF16 (INT4, INT8, E2M1 and
// E4M3 values are all exact there); one MFMA covers one 32-element group, and
// its FP32 sum is multiplied by the key's and (integer queries) the query's
// scale of the group, as in the row kernels.
#include <type_traits>

#include "mfma_core.h"
#include "score_core.h"

namespace spot {
namespace {

using mc::f32x4;
using mc::load_lds;
using mc::mfma;
using mc::pack2;

constexpr int kRows = 64;        // query rows per workgroup (16 per wave)
constexpr int kKeys = 32;        // keys per step
constexpr int kKeyB = 1024;      // bytes of one BF16 key (512 elements)

struct ManyArgs {
  const uint8_t *q, *q_scale;    // queries in format qfmt
  int qfmt;
  const float* w;
  const uint8_t *k, *k_scale;
  int n_seq, rows_per_seq, n_keys;
  const int32_t* see;            // row r sees keys below see[r] (NULL: all)
  float* scores;                 // [rows, n_keys / SB]
  int row_tiles, runs, steps;    // per sequence: row tiles, runs of `steps` steps of keys
};

// Physical 16-byte chunk of logical chunk c (of 64) of key or row r: the 16
// rows of a fragment read land in 16 different chunk slots.
__device__ __forceinline__ int swz(int r, int c) { return c ^ (r & 15); }

// The codes of a 16-byte piece (or 8 bytes, HALF) as BF16 pairs.
template <int KFMT>
__device__ __forceinline__ void codes_bf16(const uint32_t (&c)[4], uint32_t* o) {
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    if constexpr (KFMT == SPOT_KFMT_INT8_G32) {
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (float)((int)(c[x] << (24 - 8 * i)) >> 24);
      o[2 * x] = pack2(v[0], v[1]);
      o[2 * x + 1] = pack2(v[2], v[3]);
    } else if constexpr (KFMT == SPOT_KFMT_MXFP8_G32) {
      const f32x2 a = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c[x], 1.0f, false);
      const f32x2 b = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c[x], 1.0f, true);
      o[2 * x] = pack2(a[0], a[1]);
      o[2 * x + 1] = pack2(b[0], b[1]);
    } else if constexpr (KFMT == SPOT_KFMT_INT4_G32) {
      float v[8];
      int4_sixteenths(c[x], v);      // n / 16: the scale takes the 16
#pragma unroll
      for (int i = 0; i < 4; ++i) o[4 * x + i] = pack2(v[2 * i], v[2 * i + 1]);
    } else {
      const f32x2 v0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c[x], 1.0f, 0);
      const f32x2 v1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c[x], 1.0f, 1);
      const f32x2 v2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c[x], 1.0f, 2);
      const f32x2 v3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c[x], 1.0f, 3);
      o[4 * x] = pack2(v0[0], v0[1]);
      o[4 * x + 1] = pack2(v1[0], v1[1]);
      o[4 * x + 2] = pack2(v2[0], v2[1]);
      o[4 * x + 3] = pack2(v3[0], v3[1]);
    }
  }
}

// A key's (or integer query's) scale of one group; INT4 codes are n / 16.
template <int KFMT>
__device__ __forceinline__ float group_scale(const uint8_t* s, size_t at) {
  if constexpr (KFMT == SPOT_KFMT_INT4_G32)
    return 16.f * f16_to_f32(reinterpret_cast<const uint16_t*>(s)[at]);
  else if constexpr (KFMT == SPOT_KFMT_INT8_G32)
    return f16_to_f32(reinterpret_cast<const uint16_t*>(s)[at]);
  else
    return e8m0_to_f32(s[at]);
}

__device__ __forceinline__ float max_xor16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_xor32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// SB: keys per output value (1: pooled keys; 16 or 64: tokens of a block).
// QINT: INT4 / INT8 queries (a scale per row and group).
// (Two workgroups per CU, as the LDS allows: left alone, the 8-bit kernels of
// 128-dim heads take 258 registers and run one, 64 x 4 rows x 1024 keys 26 us
// instead of 15.)
template <int KFMT, int DS, int SB, bool QINT>
__global__ __launch_bounds__(256, 2) void score_many_kernel(ManyArgs a) {
  constexpr int HS = 512 / DS, KS = DS / 32;       // heads, groups per head
  constexpr bool KQ = KFMT != SPOT_KFMT_BF16;
  constexpr bool SCALED = KQ || QINT;
  constexpr bool C4 = KFMT == SPOT_KFMT_INT4_G32 || KFMT == SPOT_KFMT_MXFP4_G32;
  __shared__ __attribute__((aligned(16))) unsigned char sk0[kKeys * kKeyB], sk1[kKeys * kKeyB];
  __shared__ __attribute__((aligned(16))) float ss0[KQ ? 16 * kKeys : 4], ss1[KQ ? 16 * kKeys : 4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4;

  // The row tiles that read one run of keys get ids 8 apart (the same XCD's
  // L2); later rows, which see more keys, first.
  const int u = (blockIdx.x >> 3) / a.row_tiles * 8 + (blockIdx.x & 7);
  if (u >= a.n_seq * a.runs) return;
  const int rt = a.row_tiles - 1 - (blockIdx.x >> 3) % a.row_tiles;
  const int seq = u / a.runs, run = u % a.runs;
  const int k0 = run * a.steps * kKeys, k1 = min(k0 + a.steps * kKeys, a.n_keys);
  const int row_in = rt * kRows + wave * 16 + r16;            // this lane's row
  const bool row_ok = row_in < a.rows_per_seq;
  const size_t row = (size_t)seq * a.rows_per_seq + min(row_in, a.rows_per_seq - 1);
  int see = !row_ok ? 0 : a.see ? a.see[row] : a.n_keys;
  see = see < 0 ? 0 : (see > a.n_keys ? a.n_keys : see);
  const int see_wave = __builtin_amdgcn_readfirstlane((int)wave_max_u((uint32_t)see));
  __shared__ int s_see[4];
  if (lane == 0) s_see[wave] = see_wave;

  const size_t key0 = (size_t)seq * a.n_keys;
  const int n_out = a.n_keys / SB;
  float* const out = a.scores + row * n_out;

  // Keys [ks, ks + 32) into a buffer (past the end: the last key again, its
  // scores are masked): BF16 rows straight from global memory, codes by way
  // of the registers.
  constexpr int CP = C4 ? 2 : 4;   // 16-byte pieces of codes per thread
  u32x4 code[CP];
  float gsc[2];
  auto fetch = [&](unsigned char* buf, int ks) {
    if constexpr (!KQ) {
#pragma unroll
      for (int x = 0; x < kKeys / 4; ++x) {
        const int r = wave * (kKeys / 4) + x;
        load_lds(a.k + (key0 + min(ks + r, a.n_keys - 1)) * kKeyB + swz(r, lane) * 16,
                 buf + r * kKeyB);
      }
    } else {
      constexpr int PB = C4 ? 16 : 32;      // pieces per key
#pragma unroll
      for (int x = 0; x < CP; ++x) {
        const int p = x * 256 + tid, r = p / PB;
        code[x] = *reinterpret_cast<const u32x4*>(
            a.k + ((key0 + min(ks + r, a.n_keys - 1)) * PB + p % PB) * 16);
      }
      const size_t key = key0 + min(ks + (tid >> 3), a.n_keys - 1);
#pragma unroll
      for (int x = 0; x < 2; ++x) gsc[x] = group_scale<KFMT>(a.k_scale, key * 16 + (tid & 7) * 2 + x);
    }
  };
  auto put = [&](unsigned char* buf, float* sc) {
    if constexpr (KQ) {
      constexpr int PB = C4 ? 16 : 32, CH = C4 ? 4 : 2;   // chunks of 8 elements per piece
#pragma unroll
      for (int x = 0; x < CP; ++x) {
        const int p = x * 256 + tid, r = p / PB;
        const uint32_t c[4] = {code[x][0], code[x][1], code[x][2], code[x][3]};
        uint32_t o[CH * 4];
        codes_bf16<KFMT>(c, o);
#pragma unroll
        for (int y = 0; y < CH; ++y)
          *reinterpret_cast<u32x4*>(buf + r * kKeyB + swz(r, (p % PB) * CH + y) * 16) =
              u32x4{o[4 * y], o[4 * y + 1], o[4 * y + 2], o[4 * y + 3]};
      }
#pragma unroll
      for (int x = 0; x < 2; ++x) sc[((tid & 7) * 2 + x) * kKeys + (tid >> 3)] = gsc[x];
    }
  };

  // ---- this wave's queries: B operand fragments of all 16 groups, and w
  u32x4 qf[16];
  float qs[QINT ? 16 : 1], wh[HS];
#pragma unroll
  for (int h = 0; h < HS; ++h) wh[h] = a.w[row * HS + h];
  if (!QINT && a.qfmt == SPOT_KFMT_BF16) {
    // by way of the key buffers (64 rows = both of them): coalesced, where
    // fragment loads would touch four lines per four lanes
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const int rr = min(rt * kRows + wave * 16 + x, a.rows_per_seq - 1);
      load_lds(a.q + ((size_t)seq * a.rows_per_seq + rr) * kKeyB + swz(x, lane) * 16,
               (wave < 2 ? sk0 : sk1) + ((wave & 1) * 16 + x) * kKeyB);
    }
    mc::wait_loads<0>();
    const unsigned char* mine = (wave < 2 ? sk0 : sk1) + ((wave & 1) * 16 + r16) * kKeyB;
#pragma unroll
    for (int g = 0; g < 16; ++g)
      qf[g] = *reinterpret_cast<const u32x4*>(mine + swz(r16, g * 4 + kg) * 16);
  } else {
    // Elements 32 g + 8 kg ..+7 of the row, as load_query decodes lane
    // 4 g + kg of its row: MX values are exact in BF16, integer codes too.
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      uint4 raw;
      float f[8], sc;
      const int l = 4 * g + kg;
      if constexpr (QINT) {
        if (a.qfmt == SPOT_KFMT_INT4_G32)
          load_query<SPOT_KFMT_INT4_G32>(a.q, a.q_scale, (int)row, l, raw, f, sc);
        else
          load_query<SPOT_KFMT_INT8_G32>(a.q, a.q_scale, (int)row, l, raw, f, sc);
        qs[g] = sc;
        qf[g] = u32x4{pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7])};
      } else {
        if (a.qfmt == SPOT_KFMT_MXFP4_G32)
          load_query<SPOT_KFMT_MXFP4_G32>(a.q, a.q_scale, (int)row, l, raw, f, sc);
        else
          load_query<SPOT_KFMT_MXFP8_G32>(a.q, a.q_scale, (int)row, l, raw, f, sc);
        qf[g] = u32x4{raw.x, raw.y, raw.z, raw.w};
      }
    }
  }
  __syncthreads();   // s_see is there; the buffers are free for keys
  const int see_wg = max(max(s_see[0], s_see[1]), max(s_see[2], s_see[3]));
  const int kend = min(k1, see_wg);          // keys some row of the tile sees end here

  // A block's value: the largest of its visible scores that are no NaN.  Where
  // all of them are NaN (w or a key infinite or NaN), v is, and the value is
  // what the row kernels give: -inf from 4-bit keys, and for a 64-token block
  // of BF16 keys of which at most half is visible (one of its two waves saw
  // nothing); NaN otherwise.
  auto put_block = [&](int j, float v) {
    const bool low = C4 || (!KQ && SB == 64 && see <= j * SB + SB / 2);
    if (kg == 0 && row_ok) out[j] = j * SB >= see ? -INFINITY : low ? fmaxf(v, -INFINITY) : v;
  };

  // ---- scores of 32 keys against the wave's 16 rows (unseen keys of a block: NaN,
  // which no maximum takes)
  constexpr float kUnseen = SB == 1 ? -INFINITY : __builtin_nanf("");
  float m = kUnseen;                         // SB == 64: the block's maximum so far
  // (with two scales a group the body twice is more than the compiler unrolls,
  // and qf would go to scratch memory)
  constexpr int kUnrollT = KQ && QINT && DS == 64 ? 1 : kKeys / 16;
  auto score = [&](const unsigned char* buf, const float* sc, int ks) {
#pragma unroll kUnrollT
    for (int t = 0; t < kKeys / 16; ++t) {
      const int kt = ks + 16 * t;            // the 16 keys' first
      if (kt >= k1) break;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      if (kt < see_wave) {
        const unsigned char* kr = buf + (16 * t + r16) * kKeyB;
        // Groups of a head, then heads, are added pairwise (the error of the
        // row kernels' butterflies).
        f32x4 part[HS];
#pragma unroll
        for (int h = 0; h < HS; ++h) {
          f32x4 e[KS];
#pragma unroll
          for (int x = 0; x < KS; ++x) {
            const int g = h * KS + x;
            const u32x4 kf = *reinterpret_cast<const u32x4*>(kr + swz(r16, g * 4 + kg) * 16);
            if constexpr (SCALED) {
              // (the query's FP16 scale first: neither the product of the scales nor
              // a sum under the key's alone need be an FP32 number)
              e[x] = mfma(kf, qf[g], f32x4{0.f, 0.f, 0.f, 0.f});
              if constexpr (QINT) e[x] *= qs[g];
              if constexpr (KQ)
                e[x] *= *reinterpret_cast<const f32x4*>(sc + g * kKeys + 16 * t + 4 * kg);
            } else {
              e[x] = mfma(kf, qf[g], x & 1 ? e[x - 1] : f32x4{0.f, 0.f, 0.f, 0.f});
            }
          }
          f32x4 s;
          if constexpr (SCALED)
            s = KS == 2 ? e[0] + e[1] : (e[0] + e[1]) + (e[KS - 2] + e[KS - 1]);
          else
            s = KS == 2 ? e[1] : e[1] + e[KS - 1];
#pragma unroll
          for (int i = 0; i < 4; ++i) part[h][i] = wh[h] * fmaxf(s[i], 0.f);
        }
#pragma unroll
        for (int n = HS / 2; n >= 1; n /= 2)
#pragma unroll
          for (int h = 0; h < n; ++h) part[h] = part[2 * h] + part[2 * h + 1];
        acc = part[0];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (kt + 4 * kg + i >= see) acc[i] = kUnseen;
      if constexpr (SB == 1) {
        if (row_ok) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (kt + 4 * kg + i < a.n_keys) out[kt + 4 * kg + i] = acc[i];
        }
      } else {
        const float v = max_xor32(
            max_xor16(fmaxf(fmaxf(acc[0], acc[1]), fmaxf(acc[2], acc[3]))));
        if constexpr (SB == 16) {
          put_block(kt / 16, v);
        } else {
          m = fmaxf(m, v);
          if (kt % 64 == 48) {
            put_block(kt / 64, m);
            m = kUnseen;
          }
        }
      }
    }
  };

  // One step: keys in `cur`, the next step's on their way into `other`.
  auto step = [&](unsigned char* cur, float* scc, unsigned char* other, float* sco, int ks) {
    const bool more = ks + kKeys < kend;
    if (more) fetch(other, ks + kKeys);
    score(cur, scc, ks);
    if (more) put(other, sco);
    mc::wait_loads<0>();
    __syncthreads();
  };
  int ks = k0;
  if (ks < kend) {
    fetch(sk0, ks);
    put(sk0, ss0);
    mc::wait_loads<0>();
    __syncthreads();
    for (;;) {
      step(sk0, ss0, sk1, ss1, ks);
      ks += kKeys;
      if (ks >= kend) break;
      step(sk1, ss1, sk0, ss0, ks);
      ks += kKeys;
      if (ks >= kend) break;
    }
  }
  // Keys of the run that no row of the tile sees (the last 64-token block
  // may have been seen in part).
  for (; ks < k1; ks += kKeys) score(sk0, ss0, ks);
}

template <int KFMT, int DS, int SB, bool QINT>
hipError_t go(const ManyArgs& a, unsigned grid, hipStream_t s) {
  hipLaunchKernelGGL((score_many_kernel<KFMT, DS, SB, QINT>), dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int KFMT>
hipError_t go_fmt(const ManyArgs& a, int ds, int sb, unsigned grid, hipStream_t s) {
  const bool qint = a.qfmt == SPOT_KFMT_INT4_G32 || a.qfmt == SPOT_KFMT_INT8_G32;
  if (sb == 1 && qint) return ds == 64 ? go<KFMT, 64, 1, true>(a, grid, s)
                                       : go<KFMT, 128, 1, true>(a, grid, s);
  if (sb == 1) return ds == 64 ? go<KFMT, 64, 1, false>(a, grid, s)
                               : go<KFMT, 128, 1, false>(a, grid, s);
  if (sb == 16) return ds == 64 ? go<KFMT, 64, 16, false>(a, grid, s)
                                : go<KFMT, 128, 16, false>(a, grid, s);
  return ds == 64 ? go<KFMT, 64, 64, false>(a, grid, s) : go<KFMT, 128, 64, false>(a, grid, s);
}

}  // namespace

namespace {

// How a call is split: row tiles, and runs of `steps` steps of keys per sequence.
// As many steps per workgroup (at most 8) as leave two workgroups per CU (512)
// in one round, at least one 64-token block (256 rows x 16384 tokens: 2 / 4 / 8
// steps 12.9 / 10.4 / 13.9 us).
struct Plan {
  int row_tiles, runs, steps;
  long long wgs;
};
Plan plan_of(int n_seq, int rows_per_seq, int n_keys, bool tokens) {
  const int low = tokens ? 2 : 1, key_steps = (n_keys + kKeys - 1) / kKeys;
  const int most = key_steps >= 8 ? 8 : (key_steps + low - 1) / low * low;
  Plan p;
  p.row_tiles = (rows_per_seq + kRows - 1) / kRows;
  const long long tiles = (long long)n_seq * p.row_tiles, all = tiles * key_steps;
  const long long steps = ((all + 511) / 512 + low - 1) / low * low;
  p.steps = (int)(steps < low ? low : steps > most ? most : steps);
  while (p.steps < most && tiles * ((key_steps + p.steps - 1) / p.steps) > 512) p.steps += low;
  p.runs = (key_steps + p.steps - 1) / p.steps;
  p.wgs = tiles * p.runs;
  return p;
}

}  // namespace

// The row kernels read every key once per row but start at once; here a call
// costs two dependent trips to memory (queries, then keys) before its first
// product, and a tile of 64 rows costs the same for two.
//
// Token keys: the lines lie at these numbers of (row, key) pairs; us, row kernel /
// this one, replayed calls, (sequences x) rows x keys:
//   BF16: 64 x 1024 5.1 / 5.7, 8 x 16 x 512 5.0 / 5.6, 64 x 1536 7.1 / 5.7; where
//     the keys outgrow an XCD's L2 earlier: 8 x 8192 6.1 / 5.6, 8 x 4 x 2048
//     6.9 / 6.1, 4 x 131072 43 / 24 (8 x 3 x 2048 7.0 / 6.0 stays)
//   quantized: INT4 8 x 4 x 2048 5.7 / 7.7, 12 x 8192 8.3 / 7.7, 4 x 32768 8.6 /
//     9.4, 8 x 131072 44 / 26; INT8 2 x 131072 22 / 25, 12 x 8192 11.3 / 7.5
// Pooled keys: the smaller of two estimates, fitted to calls of 1 .. 1000
// sequences, 2 .. 512 rows and 33 .. 20000 keys.
//   This kernel: the steps of a workgroup, in rounds of 512 workgroups; integer and
//   MX queries come in small pieces.  (BF16 200 x 200 5.2, 64 x 4 x 512 8.0, x 2048
//   24.8; INT8 256 x 256 5.8, 64 x 4 x 512 9.1, x 2048 26.1; INT8 queries 9.6)
//   Row kernel: pairs; BF16 keys once they outgrow an XCD's L2 (4 MB) twice as slow,
//   but never below 32768 pairs.  (BF16 200 x 200 4.6, 8 x 5 x 1024 8.3, 64 x 4 x 2048
//   76; INT8 222 x 222 6.0, 64 x 2 x 2048 22.2, 64 x 4 x 2048 40.5)
bool score_many_takes(const void* k, int kfmt, int qfmt, int n_seq, int rows_per_seq, int n_keys,
                      bool tokens) {
  const bool quant = kfmt != SPOT_KFMT_BF16;
  // codes are read 16 bytes at a time here, 4 or 8 by the row kernels
  if (quant && (reinterpret_cast<uintptr_t>(k) & 15u) != 0) return false;
  const double pairs = (double)n_seq * rows_per_seq * n_keys;
  const double keys = (double)n_seq * n_keys;
  if (rows_per_seq < 2 || pairs <= 32768.) return false;
  const Plan p = plan_of(n_seq, rows_per_seq, n_keys, tokens);
  // grid size (padded to 8 runs): below 2^32 threads
  if ((p.wgs / p.row_tiles + 7) / 8 * 8 * p.row_tiles > 0x00ffffffLL) return false;
  if (tokens)
    return quant ? rows_per_seq >= 8 && pairs >= 98304.
                 : rows_per_seq >= 4 && pairs >= (keys >= 8192. ? 65536. : 98304.);
  const bool four_bit = kfmt == SPOT_KFMT_INT4_G32 || kfmt == SPOT_KFMT_MXFP4_G32;
  const double rounds = (double)((p.wgs + 511) / 512);
  const bool qint = qfmt == SPOT_KFMT_INT4_G32 || qfmt == SPOT_KFMT_INT8_G32;
  double here = p.wgs <= 256 && p.steps == 1 ? (quant ? 5.7 : 5.1)
                : rounds * (quant ? 3.8 + (qint ? 3.6 : 3.0) * p.steps : 2.9 + 2.9 * p.steps);
  if (qint)
    here += 3.9;
  else if (qfmt != SPOT_KFMT_BF16)
    here += 2.3;
  const double row = quant           ? 2.2 + (four_bit ? 6.4e-5 : 7.0e-5) * pairs
                     : keys > 4096. ? 2.0 + 1.5e-4 * pairs
                                    : 2.0 + 6.3e-5 * pairs;
  return here < row;
}

hipError_t launch_score_many(const void* q, const void* q_scale, int qfmt, const float* w,
                             const void* k, const void* k_scale, int kfmt, int n_seq,
                             int rows_per_seq, int n_keys, int ds, int sb, const int32_t* see,
                             float* scores, hipStream_t s) {
  ManyArgs a;
  a.q = static_cast<const uint8_t*>(q);
  a.q_scale = static_cast<const uint8_t*>(q_scale);
  a.qfmt = qfmt;
  a.w = w;
  a.k = static_cast<const uint8_t*>(k);
  a.k_scale = static_cast<const uint8_t*>(k_scale);
  a.n_seq = n_seq;
  a.rows_per_seq = rows_per_seq;
  a.n_keys = n_keys;
  a.see = see;
  a.scores = scores;
  const Plan p = plan_of(n_seq, rows_per_seq, n_keys, sb != 1);
  a.row_tiles = p.row_tiles;
  a.runs = p.runs;
  a.steps = p.steps;
  const unsigned grid = (unsigned)(((long long)n_seq * p.runs + 7) / 8 * 8 * p.row_tiles);
  switch (kfmt) {
    case SPOT_KFMT_BF16: return go_fmt<SPOT_KFMT_BF16>(a, ds, sb, grid, s);
    case SPOT_KFMT_INT4_G32: return go_fmt<SPOT_KFMT_INT4_G32>(a, ds, sb, grid, s);
    case SPOT_KFMT_INT8_G32: return go_fmt<SPOT_KFMT_INT8_G32>(a, ds, sb, grid, s);
    case SPOT_KFMT_MXFP8_G32: return go_fmt<SPOT_KFMT_MXFP8_G32>(a, ds, sb, grid, s);
    default: return go_fmt<SPOT_KFMT_MXFP4_G32>(a, ds, sb, grid, s);
  }
}

}  // namespace spot
