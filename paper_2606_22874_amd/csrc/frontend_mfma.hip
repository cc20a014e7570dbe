// Selector projections of many rows on the matrix cores (paper Section 2.1;
// Appendix A for the rotary split): [q^I, k^I, w] = [W_q; W_k; W_w] h for a
// prompt's tokens (or a large decode batch).  Both kernels take the weights
// as the A operand and the hidden rows as the B operand of
// v_mfma_f32_16x16x32_bf16, so that lane l ends with four consecutive output
// dims (4(l/16) ..+3 of a 16-dim tile) of token l%16, and both order the
// output dims so that a rotary pair sits in the same lane and register of two
// neighbouring tiles: pair P of W_q or W_k (256 of each; head P / (d_s/2),
// pp = P % (d_s/2)) is dims (a, b) = (pp, pp + rope/2) for pp < rope/2, and
// for the dims that do not rotate (rope + i, rope + (d_s - rope)/2 + i) with
// i = pp - rope/2.  Weight rows are gathered in that order when they are
// loaded, so the rotation costs no exchange.
//
//  * proj_tile_kernel: tiles of tokens x dims per workgroup (256 x 128 for
//    long prompts), operands staged through LDS.  Bound by LDS: a 256 x 128
//    step moves 176 KiB through it (reads of 64 x 64 wave tiles and the
//    staging writes) while its MFMAs need three quarters of that time; 8100
//    rows of 4096 take 81 us, 0.84 PFLOP/s (the row kernel: 2530 us).
//  * proj_skinny_kernel: 16 NT tokens x 32 dims per workgroup, its 8 waves
//    splitting d_model, operands straight from global memory to registers:
//    few rows, where tiles would leave the chip idle.  Bound by the address
//    unit (operand rows are spread over a quad's lanes: four lines a quad);
//    64 rows of 4096 take 14.3 us (the row kernel: 21.9).
#include <type_traits>

#include "frontend_core.h"
#include "mfma_core.h"

namespace spot {
namespace {

using namespace mc;

constexpr int kOut = 512;        // h_s * d_s

// First (B = false) or second dim of pair pp of a head.
template <bool B>
__device__ __forceinline__ int pair_dim(int pp, int d_s, int rope) {
  const int half = rope >> 1;
  if (pp < half) return B ? pp + half : pp;
  return rope + pp - half + (B ? (d_s - rope) >> 1 : 0);
}
// Row of W_q / W_k of pair P's first or second dim.
template <bool B>
__device__ __forceinline__ int pair_row(int P, int d_s, int rope) {
  const int sh = __builtin_ctz(d_s >> 1);
  return (P >> sh) * d_s + pair_dim<B>(P & ((d_s >> 1) - 1), d_s, rope);
}

// Stores four values of pairs pp0 .. pp0+3's first (or second) dims.  With
// vec (half a multiple of 4 and an 8-byte aligned destination) they are four
// consecutive, aligned dims.
template <bool B>
__device__ __forceinline__ void store_dims(uint16_t* head, int pp0, int d_s, int rope, bool vec,
                                           const f32x4& v) {
  if (vec) {
    *reinterpret_cast<u32x2*>(head + pair_dim<B>(pp0, d_s, rope)) =
        u32x2{pack2(v[0], v[1]), pack2(v[2], v[3])};
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) head[pair_dim<B>(pp0 + i, d_s, rope)] = f32_to_bf16_rne(v[i]);
  }
}

// Where row r's q or k goes: nullptr for a key outside the cache.
__device__ __forceinline__ uint16_t* out_row(const ProjectArgs& a, bool is_k, int r, int p) {
  if (!is_k) return a.q_out + (size_t)r * kOut;
  if (p < 0 || p >= a.l_cap) return nullptr;
  return a.k_cache + ((size_t)(r / a.rows_per_seq) * a.l_cap + p) * kOut;
}

// ------------------------------------------------- compensated FP32 sums
// w is an FP32 output: its 32-element products (one MFMA from zero each) are
// added with their rounding errors kept (2Sum), so that the long chain over
// d_model costs no accuracy.
struct CompSum {
  f32x4 s = {0.f, 0.f, 0.f, 0.f}, e = {0.f, 0.f, 0.f, 0.f};
  __device__ __forceinline__ void add(const f32x4& x) {
#pragma clang fp contract(off) reassociate(off)
    const f32x4 t = s + x, y = t - s;
    e += (s - (t - y)) + (x - y);
    s = t;
  }
  // (a sum that reached an infinity has none left to correct: its error terms
  // are inf - inf)
  __device__ __forceinline__ f32x4 value() const {
    f32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_isfinite(s[i]) ? s[i] + e[i] : s[i];
    return r;
  }
};

// ------------------------------------------------------------------ tiles
constexpr int kK = 64;           // d_model elements per step
constexpr int kRowB = kK * 2;    // bytes of one operand row of a step

// Physical 16-byte chunk of logical chunk c (of 8) of tile row r: two rows
// share a 256-byte LDS line, so the 16 rows of a fragment read (one chunk of
// each) land in 16 different chunk slots.
__device__ __forceinline__ int swz(int r, int c) { return c ^ ((r >> 1) & 7); }

__device__ __forceinline__ u32x4 frag(const unsigned char* t, int r, int c) {
  return *reinterpret_cast<const u32x4*>(t + r * kRowB + (swz(r, c) << 4));
}

// TT tokens x TD dims per workgroup of WT x WD waves.  S step buffers rotate:
// while step kt is computed, steps kt+1 .. kt+S-1 are on their way (16-byte
// direct global -> LDS loads, chunk-swizzled rows), because a load that
// misses L2 takes longer than a step (W_q and W_k, 8 MB, do not fit one XCD's
// L2).  One barrier a step: it says that step kt+1 has landed for every wave
// and that step kt's buffer is free.  W_w rides along: the workgroups of a
// token tile share out its tokens in groups of 16, one more MFMA per 32
// elements, which waves take in turn (four partial sums, added at the end).
// The workgroups of a token tile get ids 8 apart: the same XCD, whose L2 then
// holds the hidden rows for all of them.
template <int TT, int TD, int WT, int WD, int S>
__global__ __launch_bounds__(64 * WT * WD) void proj_tile_kernel(ProjectArgs a, int n_tiles,
                                                                 int vec) {
  constexpr int NW = WT * WD;                     // waves
  constexpr int J = 2 * kOut / TD;                // dim tiles (W_q's, then W_k's)
  constexpr int ND = TD / WD / 16, NT = TT / WT / 16;   // MFMA tiles per wave
  constexpr int L = (TT + TD) * kRowB / 1024 / NW;      // loads per wave and step
  constexpr int GW = NW / 4;                      // W_w token groups per workgroup
  static_assert(ND % 2 == 0 && (TT + TD) * kRowB % (1024 * NW) == 0 && (S == 3 || S == 4) &&
                    J * GW * 16 >= TT && NW % 4 == 0 && TT * 16 * 8 <= (TT + TD) * kRowB,
                "tile shape");
  // Each buffer is a variable of its own, named at compile time by every
  // access (the loop is unrolled by S), so that the compiler does not make
  // the reads of one wait for the direct-to-LDS loads into another.
  constexpr int kBuf = (TT + TD + 8) * kRowB;     // weight rows, tokens, rows of W_w
  __shared__ __attribute__((aligned(16))) unsigned char s0[kBuf], s1[kBuf], s2[kBuf];
  __shared__ __attribute__((aligned(16))) unsigned char s3[S == 4 ? kBuf : 16];
  __shared__ f32x4 s_w[NW][64];
  // (the wave's index as a scalar: LDS and base addresses stay scalar)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const int j = (blockIdx.x >> 3) & (J - 1);                           // dim tile
  const int tile = (int)(blockIdx.x / (8 * J)) * 8 + (blockIdx.x & 7);  // token tile
  if (tile >= n_tiles) return;
  const bool is_k = j >= J / 2;
  const int P0 = (j & (J / 2 - 1)) * (TD / 2);   // first pair of the dim tile
  const int t0 = tile * TT;                      // first token
  const int dm = a.d_model, steps = (dm + kK - 1) / kK, full = dm / kK;

  // This thread's 16-byte chunks of a step: rows 0 .. TD-1 are weight rows
  // (16 first dims, then the 16 second dims of each pair group), the rest
  // tokens (past the end: the last row again, its results are dropped).
  // One more load, of wave 0, brings 8 rows of W_w.
  constexpr int LW = TD * kRowB / 1024 / NW;      // loads 0 .. LW-1: weights, the rest: tokens
  static_assert(TD * kRowB % (1024 * NW) == 0, "a load is all weights or all tokens");
  const uint16_t* const wmat = is_k ? a.w_k : a.w_q;
  const uint16_t* const hmat = a.h + (size_t)t0 * dm;
  // 32-bit lane offsets from the scalar bases (bytes; the launcher bounds
  // d_model)
  uint32_t off[L + 1];
  int lc[L + 1];
#pragma unroll
  for (int u = 0; u <= L; ++u) {
    const int p = u == L ? (TT + TD) * 8 + lane : (u * NW + wave) * 64 + lane, r = p >> 3;
    lc[u] = swz(r, p & 7) * 8;
    int row;
    if (u == L) {
      row = min(r - TD - TT, a.h_s - 1);
    } else if (u < LW) {
      const int P = P0 + 16 * (r >> 5) + (r & 15);
      row = r & 16 ? pair_row<true>(P, a.d_s, a.rope_dim)
                   : pair_row<false>(P, a.d_s, a.rope_dim);
    } else {
      row = min(r - TD, a.rows - 1 - t0);
    }
    off[u] = ((uint32_t)row * (uint32_t)dm + (uint32_t)lc[u]) * 2u;
  }
  auto at = [&](int u, int kt) {
    const uint16_t* base = u == L ? a.w_w : u < LW ? wmat : hmat;
    return reinterpret_cast<const uint16_t*>(
        reinterpret_cast<const unsigned char*>(base + (size_t)kt * kK) + off[u]);
  };
  auto stage_full = [&](unsigned char* buf, int kt) {
    if (wave == 0) load_lds(at(L, kt), buf + (TT + TD) * kRowB);
#pragma unroll
    for (int u = 0; u < L; ++u)
      load_lds(at(u, kt), buf + (u * NW + wave) * 1024);
  };
  auto stage = [&](unsigned char* buf, int kt) {
    const int k0 = kt * kK;
    if (kt < full) {
      stage_full(buf, kt);
    } else if (kt < steps) {   // the last step of a d_model that is no multiple of 64
#pragma unroll
      for (int u = 0; u <= L; ++u) {
        if (u == L && wave != 0) break;
        u32x4 x = {0u, 0u, 0u, 0u};
        if (k0 + lc[u] < dm) x = *reinterpret_cast<const u32x4*>(at(u, kt));
        *reinterpret_cast<u32x4*>(buf + (u == L ? (TT + TD) * kRowB : (u * NW + wave) * 1024) +
                                  lane * 16) = x;
      }
    }
  };

  const int wd = (wave % WD) * (TD / WD), wt = (wave / WD) * (TT / WT);
  f32x4 acc[ND][NT];
#pragma unroll
  for (int d = 0; d < ND; ++d)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[d][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // W_w: this wave's group of 16 tokens and its turns, the 32-element parts
  // p = 2 kt + ks with p % 4 == wave % 4.
  const int grp = j * GW + wave / 4;
  const bool has_w = grp * 16 < TT;
  const int wks = wave & 1, wpar = (wave >> 1) & 1;
  CompSum sw;

  u32x4 fa[2][ND], fb[2][NT];   // fragments of a step's two 32-element parts
  auto read = [&](const unsigned char* buf, int ks) {
#pragma unroll
    for (int d = 0; d < ND; ++d) fa[ks][d] = frag(buf, wd + 16 * d + r16, ks * 4 + kg);
#pragma unroll
    for (int t = 0; t < NT; ++t) fb[ks][t] = frag(buf, TD + wt + 16 * t + r16, ks * 4 + kg);
  };
  auto multiply = [&](int ks) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int d = 0; d < ND; ++d) acc[d][t] = mfma(fa[ks][d], fb[ks][t], acc[d][t]);
  };

  // Step kt from buffer `cur`, part 0 already in registers: part 1 is read
  // while part 0 multiplies, the next step's part 0 while part 1 does, with
  // the barrier between the two.  STEADY: steps up to kt + S are full, so the
  // loads need no condition.
  auto step = [&](auto cur, auto steady, int kt) {
    constexpr int c = decltype(cur)::value, nx = (c + 1) % S;
    constexpr bool STEADY = decltype(steady)::value;
    unsigned char* buf = c == 0 ? s0 : c == 1 ? s1 : c == 2 ? s2 : s3;
    const unsigned char* next = nx == 0 ? s0 : nx == 1 ? s1 : nx == 2 ? s2 : s3;
    read(buf, 1);
    const bool w_turn = has_w && (kt & 1) == wpar;
    u32x4 fwa, fwb;
    f32x4 pw;
    if (w_turn) {   // (tile rows 8 .. 15 repeat the last W_w row and are never stored)
      fwa = frag(buf, TD + TT + min(r16, 7), wks * 4 + kg);
      fwb = frag(buf, TD + 16 * grp + r16, wks * 4 + kg);
    }
    __builtin_amdgcn_sched_barrier(0);
    multiply(0);
    if (w_turn) pw = mfma(fwa, fwb, f32x4{0.f, 0.f, 0.f, 0.f});
    __builtin_amdgcn_sched_barrier(0);
    // step kt + 1 has landed: at most the loads of the S - 2 full steps
    // after it may be outstanding (near the end: none)
    if (STEADY || kt + S - 1 < full)
      wait_loads<L*(S - 2)>();
    else
      wait_loads<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (STEADY) {
      stage_full(buf, kt + S);
      read(next, 0);
    } else {
      stage(buf, kt + S);
      if (kt + 1 < steps) read(next, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    multiply(1);
    if (w_turn) sw.add(pw);
  };

  stage(s0, 0);
  stage(s1, 1);
  stage(s2, 2);
  if constexpr (S == 4) stage(s3, 3);
  if (S - 1 < full)
    wait_loads<L*(S - 1)>();
  else
    wait_loads<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read(s0, 0);
  int kt = 0;
  const std::integral_constant<int, 0> c0;
  const std::integral_constant<int, 1> c1;
  const std::integral_constant<int, 2> c2;
  const std::integral_constant<int, 3> c3;
  for (; kt + 2 * S - 1 < full; kt += S) {
    step(c0, std::true_type(), kt);
    step(c1, std::true_type(), kt + 1);
    step(c2, std::true_type(), kt + 2);
    if constexpr (S == 4) step(c3, std::true_type(), kt + 3);
  }
  for (;; kt += S) {   // the last steps (at least one is left)
    step(c0, std::false_type(), kt);
    if (kt + 1 >= steps) break;
    step(c1, std::false_type(), kt + 1);
    if (kt + 2 >= steps) break;
    step(c2, std::false_type(), kt + 2);
    if (kt + 3 >= steps) break;
    if constexpr (S == 4) {
      step(c3, std::false_type(), kt + 3);
      if (kt + 4 >= steps) break;
    }
  }

  // ---- w of this workgroup's token groups: lane holds heads 4 kg ..+3 of
  // token r16 of group wave / 4
  s_w[wave][lane] = sw.value();
  __syncthreads();   // (also: every wave is done with the step buffers)
  if (wave % 4 == 0 && has_w) {
    const f32x4 s = (s_w[wave][lane] + s_w[wave + 1][lane]) +
                    (s_w[wave + 2][lane] + s_w[wave + 3][lane]);
    const int r = t0 + 16 * grp + r16;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (r < a.rows && 4 * kg + i < a.h_s) a.w_out[(size_t)r * a.h_s + 4 * kg + i] = s[i];
  }

  // ---- the rotations of the tile's tokens, then rotate and store.  A pass
  // covers pairs [32 c, 32 c + 32) of a head: (sin, cos) of 16 pairs each in
  // s0 and s1, [token][pair]; c beyond the rotary pairs has nothing to form.
  const int half = a.rope_dim >> 1;
  for (int c = 0; 32 * c < a.d_s >> 1; ++c) {
    if (c) __syncthreads();
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int pp = 32 * c + 16 * g + (tid & 15);
      if (32 * c + 16 * g >= half) break;
      unsigned char* buf = g ? s1 : s0;
      for (int t = tid >> 4; t < TT; t += NW * 4) {
        f32x2 sc = {0.f, 1.f};
        if (pp < half) {
          float sn, cs;
          rope_sincos(a.pos[min(t0 + t, a.rows - 1)], a.freq.f[pp], sn, cs);
          sc = f32x2{sn, cs};
        }
        *reinterpret_cast<f32x2*>(buf + (t * 16 + (tid & 15)) * 8) = sc;
      }
    }
    __syncthreads();
#pragma unroll
    for (int gg = 0; gg < ND / 2; ++gg) {
      const int P = P0 + (wd >> 1) + 16 * gg;       // the pair group's first pair
      const int pg = P & ((a.d_s >> 1) - 1);        // within its head
      if (pg >> 5 != c) continue;
      const int pp0 = pg + 4 * kg;
      const unsigned char* buf = pg & 16 ? s1 : s0;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int tt = wt + 16 * t + r16, r = t0 + tt;
        if (r >= a.rows) continue;
        uint16_t* dst = out_row(a, is_k, r, a.pos[r]);
        if (!dst) continue;
        f32x4 A = acc[2 * gg][t], B = acc[2 * gg + 1][t];
        if (pg < half) {
          const f32x2* sc = reinterpret_cast<const f32x2*>(buf + (tt * 16 + 4 * kg) * 8);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const f32x2 x = sc[i];
            const float ra = A[i] * x[1] - B[i] * x[0], rb = B[i] * x[1] + A[i] * x[0];
            if (pp0 + i < half) {
              A[i] = ra;
              B[i] = rb;
            }
          }
        }
        uint16_t* head = dst + (P >> __builtin_ctz(a.d_s >> 1)) * a.d_s;
        store_dims<false>(head, pp0, a.d_s, a.rope_dim, vec, A);
        store_dims<true>(head, pp0, a.d_s, a.rope_dim, vec, B);
      }
    }
  }
}

// ------------------------------------------------------------- few rows
constexpr int kSkWaves = 8;

// Workgroup (x, y): pairs 16x .. 16x+15 of [W_q; W_k] (x == 32: the rows of
// W_w) for tokens 16 NT y ..  Wave w takes every 8th 64-element run of
// d_model (a whole line of each row), kU 32-element parts in flight together; the waves' partial sums meet
// in LDS and are added pairwise, then waves 0 .. NT-1 rotate and store.
template <int NT>
__global__ __launch_bounds__(64 * kSkWaves) void proj_skinny_kernel(ProjectArgs a, int vec) {
  __shared__ f32x4 part[kSkWaves][2][NT][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, kg = lane >> 4;
  const bool is_w = blockIdx.x == 32, is_k = blockIdx.x >= 16;
  const int P0 = (blockIdx.x & 15) * 16;
  const int t0 = blockIdx.y * 16 * NT;
  const int dm = a.d_model;
  const uint16_t *pa, *pb, *ph[NT];
  if (is_w) {
    pa = pb = a.w_w + (size_t)min(r16, a.h_s - 1) * dm;
  } else {
    const uint16_t* w = is_k ? a.w_k : a.w_q;
    pa = w + (size_t)pair_row<false>(P0 + r16, a.d_s, a.rope_dim) * dm;
    pb = w + (size_t)pair_row<true>(P0 + r16, a.d_s, a.rope_dim) * dm;
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) ph[t] = a.h + (size_t)min(t0 + 16 * t + r16, a.rows - 1) * dm;

  f32x4 acc[2][NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[0][t] = acc[1][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  CompSum sw[NT];
  constexpr int kU = NT == 1 ? 8 : 4;   // (parts in flight; 16 and 8 measured the same)
  // element of part u of a pass (a wave's parts come in pairs: a whole
  // 128-byte line of each row)
  auto part_k = [](int u) { return (u >> 1) * kSkWaves * 64 + (u & 1) * 32; };
  for (int k0 = wave * 64; k0 < dm; k0 += kU * kSkWaves * 32) {
    u32x4 fa[kU], fb[kU], fh[kU][NT];
    const bool full = k0 + part_k(kU - 1) + 32 <= dm;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int k = min(k0 + part_k(u) + kg * 8, dm - 8);
      fa[u] = *reinterpret_cast<const u32x4*>(pa + k);
      fb[u] = *reinterpret_cast<const u32x4*>(pb + k);
#pragma unroll
      for (int t = 0; t < NT; ++t) fh[u][t] = *reinterpret_cast<const u32x4*>(ph[t] + k);
    }
    if (!full) {   // elements past d_model are zeros on both sides
      const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const bool ok = k0 + part_k(u) + kg * 8 < dm;
        fa[u] = ok ? fa[u] : z;
        fb[u] = ok ? fb[u] : z;
#pragma unroll
        for (int t = 0; t < NT; ++t) fh[u][t] = ok ? fh[u][t] : z;
      }
    }
    if (is_w) {
#pragma unroll
      for (int u = 0; u < kU; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          sw[t].add(mfma(fa[u], fh[u][t], f32x4{0.f, 0.f, 0.f, 0.f}));
    } else {
#pragma unroll
      for (int u = 0; u < kU; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          acc[0][t] = mfma(fa[u], fh[u][t], acc[0][t]);
          acc[1][t] = mfma(fb[u], fh[u][t], acc[1][t]);
        }
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    part[wave][0][t][lane] = is_w ? sw[t].value() : acc[0][t];
    part[wave][1][t][lane] = acc[1][t];
  }
  __syncthreads();
  if (wave >= NT) return;
  const int r = t0 + 16 * wave + r16;
  if (r >= a.rows) return;
  static_assert(kSkWaves == 8, "the sum below");
  auto sum = [&](int ab) {
    f32x4 x[8];
#pragma unroll
    for (int w = 0; w < 8; ++w) x[w] = part[w][ab][wave][lane];
    return ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
  };
  f32x4 A = sum(0), B = sum(1);
  if (is_w) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * kg + i < a.h_s) a.w_out[(size_t)r * a.h_s + 4 * kg + i] = A[i];
    return;
  }
  const int p = a.pos[r];
  uint16_t* dst = out_row(a, is_k, r, p);
  if (!dst) return;
  const int half = a.rope_dim >> 1;
  const int pp0 = (P0 & ((a.d_s >> 1) - 1)) + 4 * kg;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (pp0 + i < half) {
      float s, c;
      rope_sincos(p, a.freq.f[pp0 + i], s, c);
      const float ra = A[i] * c - B[i] * s, rb = B[i] * c + A[i] * s;
      A[i] = ra;
      B[i] = rb;
    }
  }
  uint16_t* head = dst + (P0 >> __builtin_ctz(a.d_s >> 1)) * a.d_s;
  store_dims<false>(head, pp0, a.d_s, a.rope_dim, vec, A);
  store_dims<true>(head, pp0, a.d_s, a.rope_dim, vec, B);
}

}  // namespace

bool project_mfma_takes(int rows, int d_model) {
  // Up to two 16-row passes of the row kernel are as fast (13.8 against
  // 14.1 us for 32 rows of 4096), three where d_model is large (33 / 48 rows of
  // 8192 25.4 / 27.5 against 25.3, of 16384 40 / 42 against 46, of 32768 69 / 74
  // against 87; 64 rows of 32768 96 against 87); tile offsets are 32-bit (512 rows
  // of d_model BF16).
  return rows > (d_model <= 8192 ? 32 : 48) && d_model <= 1 << 21;
}

// Which kernel: the skinny one while its grid is at most one workgroup per
// CU (256 CUs, 33 workgroups per token tile), then the smallest tiles whose
// grid is at most two resident workgroups per CU (512), then the largest.  Replayed, us for d_model 4096 (the
// row kernel first, then the one taken): 64 rows 21.9 / 14.3, 192 rows
// 51.8 / 18.2, 256 rows 65 / 23.4 (skinny 32.1), 1024 rows 232 / 25.3 (128 x
// 64 tiles 35.4), 4096 rows 1280 / 49.9 (64 x 64: 61.5, 256 x 128: 70.3),
// 8100 rows 2530 / 80.7 (128 x 64: 104).
hipError_t launch_project_mfma(const ProjectArgs& a, hipStream_t s) {
  const uintptr_t at = reinterpret_cast<uintptr_t>(a.q_out) | reinterpret_cast<uintptr_t>(a.k_cache);
  const int vec = (a.rope_dim >> 1) % 4 == 0 && (at & 7u) == 0;
  if (a.rows <= 224) {
    const int nt = a.rows <= 112 ? 1 : 2;
    const dim3 grid(33, (a.rows + 16 * nt - 1) / (16 * nt));
    if (nt == 1)
      hipLaunchKernelGGL((proj_skinny_kernel<1>), grid, dim3(64 * kSkWaves), 0, s, a, vec);
    else
      hipLaunchKernelGGL((proj_skinny_kernel<2>), grid, dim3(64 * kSkWaves), 0, s, a, vec);
    return hipGetLastError();
  }
  auto tiles = [&](auto kern, int tt, int td, int threads) {
    const int n = (int)(((long long)a.rows + tt - 1) / tt);
    hipLaunchKernelGGL(kern, dim3((unsigned)((n + 7) / 8) * 8u * (2 * kOut / td)), dim3(threads),
                       0, s, a, n, vec);
    return hipGetLastError();
  };
  if (a.rows <= 2048) return tiles(proj_tile_kernel<64, 64, 2, 2, 4>, 64, 64, 256);
  if (a.rows <= 4096) return tiles(proj_tile_kernel<128, 64, 2, 2, 3>, 128, 64, 256);
  return tiles(proj_tile_kernel<256, 128, 4, 2, 3>, 256, 128, 512);
}

}  // namespace spot
