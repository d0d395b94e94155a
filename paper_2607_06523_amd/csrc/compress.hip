// Append/compress (Sec. 3, the storage half of Eq. 1) on gfx950: dense
// key/value vectors of new tokens become their coefficient rows, routed
// residual entries and gate-folded scales, written in place into the cache.
//
// Two kernels with the same results bit for bit:
//  * compress_kernel, for a few tokens: one wave takes one token (its arithmetic
//    is in compress_dev.h).
//  * compress_tile_kernel, for prompts: one wave takes 16 tokens, the
//    projection and the basis term as products on v_mfma_f32_16x16x4_f32.
//    That instruction adds its four products to the accumulator one after
//    the other, each rounded as a fused multiply-add would, so a chain of them
//    is the left-to-right sum the results are defined by (fp16 products are
//    exact in float32).  Bound by its instructions, the products and after them
//    the selection of the entries, and by their chains: with one token in three
//    holding entries the matrix cores are busy 25 % and vector instructions issue
//    38 % of a SIMD's cycles, and a wave waits on a dependency for 37 % of its
//    own.  A layer of 32K tokens and 8 KV heads (r_b 48) takes 129, 190 and 359
//    us with one token in twenty, one in four and every token holding entries
//    (100, 68 and 36 TFLOP/s of the two products, tokens without entries counted
//    in full); one token per wave, four waves to 64 tokens, took 629, 702 and 875.
#include <algorithm>

#include "compress_dev.h"

namespace dwkv {
namespace {

using namespace cdev;

constexpr int kCW = 4;                   // waves of the one-wave-per-token kernel's workgroup
struct Smem {
  uint16_t bas[kMaxRB * kBRow];          // basis rows of (sequence, window, head, Z)
  float xs[kCW][D];                      // the wave's input vector
  float as[kCW][kMaxRB];                 // its fp16-rounded coefficients
  uint8_t ech[kCW][D];                   // entries in storage order: channel
  uint8_t ecode[kCW][D];                 //                          int4 nibble
};

// Largest b with cu[b] <= t (t < cu[batch]): the sequence holding packed token t.
__device__ __forceinline__ int sequence_of(const int32_t* cu, int batch, int64_t t) {
  int lo = 0, hi = batch;                // invariant: cu[lo] <= t < cu[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)cu[mid] <= t) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ TokenIn load_token(const CompressArgs& a, const Slab& sl, int lane, int h, int z,
                                              int64_t t) {
  const int64_t k = t - a.t0;
  const uint16_t* X = (z ? a.xv : a.xk) + (k * a.n_kv_heads + h) * D;
  TokenIn in;
  in.xw = reinterpret_cast<const uint32_t*>(X)[lane];
  in.lvl = sl.code[t];
  in.e0 = sl.off[t];
  in.e1 = sl.off[t + 1];
  in.g = a.gate ? a.gate[(int64_t)(z * a.n_kv_heads + h) * a.gate_ld + a.gate_k0 + k] : 1.0f;
  return in;
}

__device__ __forceinline__ Slab make_slab(const CompressArgs& a, int h, int z) {
  const int64_t slab = (int64_t)z * a.n_kv_heads + h;
  Slab sl;
  sl.code = a.code + (int64_t)h * a.T;
  sl.off = a.off + (int64_t)h * (a.T + 1);
  sl.coef = (z == 0 ? a.coef_k : a.coef_v) + (int64_t)h * a.T16 * a.rb;
  sl.coef8 = reinterpret_cast<uint8_t*>(z == 0 ? a.coef_k : a.coef_v) + (int64_t)h * a.T16 * a.rb;
  sl.cscale = a.c8 ? (z == 0 ? a.cscale_k : a.cscale_v) + (int64_t)h * (a.rb / 16) * a.T : nullptr;
  sl.res_idx = a.res_idx + slab * a.res_stride;
  sl.res_val = a.res_val + slab * (a.res_stride / 2);
  sl.res_scale = a.res_scale + slab * a.T;
  return sl;
}

// grid (ceil(n / 4), Hkv, 2): a wave takes one token
__global__ __launch_bounds__(kCW * 64) void compress_kernel(const CompressArgs a) {
  __shared__ __align__(16) Smem sm;
  const int h = blockIdx.y, z = blockIdx.z;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const Slab sl = make_slab(a, h, z);
  const int64_t c0 = a.t0 + (int64_t)blockIdx.x * kCW, end = min(c0 + kCW, a.t0 + a.n), t = c0 + wv;
  const int rb = a.rb;
  TokenIn in = {};
  if (t < end) in = load_token(a, sl, lane, h, z, t);     // in flight while the basis loads
  for (int b = sequence_of(a.cu, a.batch, c0); b < a.batch && (int64_t)a.cu[b] < end; ++b) {
    const int64_t s0 = max(c0, (int64_t)a.cu[b]), s1 = min(end, (int64_t)a.cu[b + 1]);
    if (s1 <= s0) continue;              // empty sequence (uniform over the workgroup)
    __syncthreads();                     // every wave is done with the previous basis
    const uint16_t* src = a.basis + (int64_t)b * a.basis_b_stride + (int64_t)(h * 2 + z) * rb * D;
    for (int e = threadIdx.x; e < rb * (D / 8); e += kCW * 64) {
      const int i = e / (D / 8), q = e % (D / 8);
      *reinterpret_cast<uint4*>(sm.bas + i * kBRow + 8 * q) =
          *reinterpret_cast<const uint4*>(src + (int64_t)i * D + 8 * q);
    }
    __syncthreads();
    if (t >= s0 && t < s1)
      compress_token(a, sl, CWave{sm.bas, sm.xs[wv], sm.as[wv], sm.ech[wv], sm.ecode[wv]}, lane, z, t, in);
  }
}

// ---- the tile kernel ----------------------------------------------------------------

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kPT = 16;                  // tokens of a wave's tile
constexpr int kRRow = D + 4;             // residual row in LDS (floats)
constexpr int kERow = D + 8;             // entry row in LDS; slot D takes what is not kept

// Basis and input rows lie in LDS with their channels dealt by channel % 4
// (channel j at position (j % 4) * 32 + j / 4): lane group kk of a product's
// k-step u reads channel 4 u + kk, so 8 consecutive halves are its next 8 steps.
//
// A wave's rows are a ring of 2 x 16: `n` tokens whose entries are still to be
// formed start at `head`, the tile at hand follows them.  Tokens without
// entries leave the ring after the projection; once 16 are waiting, their basis
// term and entries are formed together, so neither the products nor the
// entries' instructions run for absent tokens.
constexpr int kRing = 2 * kPT;

template <int RB, bool C8>
struct TileWave {
  // coefficient row: fp16 dealt by index % 4 like the channels, or int8 codes
  // and then the block scales
  static constexpr int AB = C8 ? RB + 16 : 2 * RB + 16;
  alignas(16) uint16_t x[kRing][kBRow];
  alignas(16) unsigned char a[kRing][AB];
  alignas(16) float res[4][kRRow];       // residuals of four tokens
  alignas(16) uint16_t ent[4][kERow];    // their entries in storage order: channel | code << 8
  int rho[kRing];
  uint32_t e0[kRing];                    // first entry
  float g[kRing];
  int tok[kRing];                        // token - the workgroup's first, bit 31: no room for its entries
  uint8_t list[kPT];
};

// Waves of a workgroup: two per SIMD where their rows and the basis fit the LDS.
template <int RB>
constexpr int kTileWaves = RB <= 64 ? 8 : 6;

template <int RB, bool C8>
struct TileSmem {
  alignas(16) uint16_t bas[RB][kBRow];
  TileWave<RB, C8> w[kTileWaves<RB>];
};

// What a wave loads ahead for its next 16 tokens: input rows (16-byte chunk
// lane + 64 i: row / 16, chunk % 16) and, in lanes 0-15, a token's metadata.
struct TileIn {
  uint4 x[4];
  uint32_t lvl, e0, e1;
  float g;
};

__device__ __forceinline__ uint32_t half_at(const uint4& v, int i) {
  const uint32_t w = i < 2 ? v.x : i < 4 ? v.y : i < 6 ? v.z : v.w;
  return (i & 1) ? w >> 16 : w & 0xffffu;
}

__device__ __forceinline__ float half_f(const uint4& v, int i) { return half_bits_to_float((uint16_t)half_at(v, i)); }

// 8 channels j0 .. j0 + 7 (j0 a multiple of 8) into a dealt row.
__device__ __forceinline__ void store_dealt(uint16_t* row, int j0, const uint4& v) {
#pragma unroll
  for (int k = 0; k < 4; ++k)
    *reinterpret_cast<uint32_t*>(row + 32 * k + (j0 >> 2)) = half_at(v, k) | half_at(v, k + 4) << 16;
}

// Reductions and scans over a row of 16 lanes; every lane gets the result.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t row_sum(uint32_t v) {
  v += dpp_u<0xB1>(v);                   // quad_perm(1,0,3,2)
  v += dpp_u<0x4E>(v);                   // quad_perm(2,3,0,1)
  v += dpp_u<0x141>(v);                  // row_half_mirror
  return v + dpp_u<0x140>(v);            // row_mirror
}
__device__ __forceinline__ uint32_t row_max(uint32_t v) {
  v = max(v, dpp_u<0xB1>(v));
  v = max(v, dpp_u<0x4E>(v));
  v = max(v, dpp_u<0x141>(v));
  return max(v, dpp_u<0x140>(v));
}
__device__ __forceinline__ float row_fmax(float v) {
  v = fmaxf(v, __uint_as_float(dpp_u<0xB1>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(dpp_u<0x4E>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(dpp_u<0x141>(__float_as_uint(v))));
  return fmaxf(v, __uint_as_float(dpp_u<0x140>(__float_as_uint(v))));
}
__device__ __forceinline__ uint32_t row_prefix(uint32_t v) {   // sum of the row's lower lanes
  uint32_t s = v;
  s += dpp_u<0x111>(s);                  // row_shr by 1, 2, 4, 8 (zeros shift in)
  s += dpp_u<0x112>(s);
  s += dpp_u<0x114>(s);
  s += dpp_u<0x118>(s);
  return s - v;
}

// Field v (0..7) of the byte counters lo (0..3), hi (4..7).
__device__ __forceinline__ uint32_t field(uint32_t lo, uint32_t hi, int v) {
  return ((v & 4 ? hi : lo) >> (8 * (v & 3))) & 255u;
}

__device__ __forceinline__ void tile_load(TileIn& in, const CompressArgs& a, const Slab& sl, int64_t base, int h,
                                          int z, int lane) {
  const int64_t end = a.t0 + a.n;
  const uint16_t* X = (z ? a.xv : a.xk) + (int64_t)h * D;
  const int64_t xs = (int64_t)a.n_kv_heads * D;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t t = base + ((lane + 64 * i) >> 4);
    in.x[i] = make_uint4(0u, 0u, 0u, 0u);
    if (t >= a.t0 && t < end) in.x[i] = *reinterpret_cast<const uint4*>(X + (t - a.t0) * xs + 8 * (lane & 15));
  }
  const int64_t t = base + (lane & 15);
  in.lvl = 255u;
  in.e0 = in.e1 = 0u;
  in.g = 1.0f;
  if (t >= a.t0 && t < end) {
    in.lvl = sl.code[t];
    in.e0 = sl.off[t];
    in.e1 = sl.off[t + 1];
    if (a.gate) in.g = a.gate[(int64_t)(z * a.n_kv_heads + h) * a.gate_ld + a.gate_k0 + (t - a.t0)];
  }
}

// Loaded inputs into the ring rows from `tile` on; `off0`: the tile's first
// token - the workgroup's first.
template <int RB, bool C8>
__device__ __forceinline__ void tile_stage(TileWave<RB, C8>& w, const CompressArgs& a, const TileIn& in, int tile,
                                           int off0, int lane) {
  wave_lds_sync();                       // the rows' previous tokens are done with
#pragma unroll
  for (int i = 0; i < 4; ++i) store_dealt(w.x[(tile + ((lane + 64 * i) >> 4)) % kRing], 8 * (lane & 15), in.x[i]);
  if (lane < kPT) {
    const int rho = in.lvl < (uint32_t)a.n_levels ? a.levels[in.lvl] : -1;
    const bool ok = (int64_t)in.e1 - (int64_t)in.e0 == rho && (int64_t)in.e1 <= a.res_stride && (in.e0 & 1u) == 0;
    const int at = (tile + lane) % kRing;
    w.rho[at] = rho;
    w.e0[at] = in.e0;
    w.tok[at] = (off0 + lane) | (ok ? 0 : (int)0x80000000);
    w.g[at] = in.g;
  }
  wave_lds_sync();
}

// The residual entries of up to four tokens, one per row of 16 lanes (ring row
// `at`, idle rows with act false), from their residuals in w.res: lane r of a
// row owns channels 8 r .. 8 r + 7.
//
// The codes come first (|code| never decreases with |r|): with their counts,
// every channel whose |code| lies above the level v that the rho-th largest
// falls into is kept, and only within level v a search over the |r| bits
// separates the kept from the rest.  Storage positions are the counts of the
// higher levels plus a prefix over the kept channels of the same level.
template <int RB, bool C8>
__device__ __forceinline__ void tile_entries(const Slab& sl, TileWave<RB, C8>& w, int64_t first, int at, bool act,
                                             int lane) {
#pragma clang fp contract(off)
  const int row = lane >> 4, r = lane & 15;
  const int rho = act ? w.rho[at] : 1;
  const float* rr = &w.res[row][8 * r];
  const f4 ra = *reinterpret_cast<const f4*>(rr), rb4 = *reinterpret_cast<const f4*>(rr + 4);
  const float rv[8] = {ra.x, ra.y, ra.z, ra.w, rb4.x, rb4.y, rb4.z, rb4.w};
  uint32_t ab[8], top = 0;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    ab[u] = __float_as_uint(rv[u]) & 0x7fffffffu;
    top = max(top, ab[u]);
  }
  top = row_max(top);
  float mx = __uint_as_float(top);
  const bool odd = __ballot(top > 0x7f800000u) != 0;     // a NaN somewhere: the maximum ignores it
  if (odd) {
    mx = fabsf(rv[0]);
#pragma unroll
    for (int u = 1; u < 8; ++u) mx = fmaxf(mx, fabsf(rv[u]));
    mx = row_fmax(mx);
  }
  const float S = mx / 7.0f;
  float gS = w.g[at] * S;
  asm volatile("" : "+v"(gS));           // rounded to float32 before the fp16 conversion
  const int tk = w.tok[at];
  if (act && r == 0) sl.res_scale[first + (tk & 0x7fffffff)] = float_to_half_bits(gS);

  // codes: rint(r / S) from r * (1 / S), whose error stays below 4e-6 of a code,
  // unless it lies within 2e-5 of a tie between two codes (or is not a number)
  int q[8];
  {
    const float inv = __builtin_amdgcn_rcpf(S);
    bool near = false;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float v = rv[u] * inv, rn = __builtin_rintf(v);
      near |= !(fabsf(v - rn) < 0.49998f);
      q[u] = (int)fminf(fmaxf(rn, -7.f), 7.f);
    }
    if (__ballot(near) != 0) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
        q[u] = S > 0.f ? (int)fminf(fmaxf(__builtin_rintf(rv[u] / S), -7.f), 7.f) : 0;
    }
  }
  int m[8];
  uint32_t lo = 0, hi = 0;               // channels of this lane per |code|, a byte each
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    m[u] = q[u] < 0 ? -q[u] : q[u];
    const uint32_t one = 1u << (8 * (m[u] & 3));
    lo += m[u] < 4 ? one : 0u;
    hi += m[u] < 4 ? 0u : one;
  }
  // ch, cl: per level, the row's channels at or above it (at most 128: no carries)
  uint32_t ch = row_sum(hi), cl = row_sum(lo);
  ch += ch >> 8;
  ch += ch >> 16;
  cl += cl >> 8;
  cl += cl >> 16;
  cl += (ch & 255u) * 0x01010101u;
  int lev = 0;                           // the level of the rho-th largest
#pragma unroll
  for (int v = 1; v < 8; ++v) lev += field(cl, ch, v) >= (uint32_t)rho ? 1 : 0;
  const uint32_t upl = cl >> 8 | ch << 24, uph = ch >> 8;   // per level, the channels above it
  const uint32_t above = field(upl, uph, lev);
  const uint32_t need = (uint32_t)rho - above;              // kept channels of level lev
  uint32_t clo = field(cl, ch, lev) - above, chi = 0, tlo = 0, thi = 0x80000000u;
  if (__ballot(act && clo != need) != 0) {
    // bits in [tlo, thi): clo channels reach tlo (>= need), chi reach thi (< need)
    uint32_t mk[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) mk[u] = m[u] == lev ? ab[u] : 0u;
    if (!odd && S > 1e-30f && S < 1e30f) {                  // the level's own interval, widened
      tlo = lev > 0 ? __float_as_uint(((float)lev - 0.500002f) * S) : 0u;
      thi = __float_as_uint(((float)lev + 0.500002f) * S) + 1u;
    }
    while (true) {
      const bool go = clo != need && thi - tlo > 1u;
      if (__ballot(act && go) == 0) break;
      const uint32_t mid = tlo + ((thi - tlo) >> 1);
      uint32_t c = 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) c += mk[u] >= mid ? 1u : 0u;
      c = row_sum(c);
      if (go) {
        if (c >= need) { tlo = mid; clo = c; } else { thi = mid; chi = c; }
      }
    }
  }
  uint32_t keep = 0;                     // bit u: channel 8 r + u is kept
#pragma unroll
  for (int u = 0; u < 8; ++u) keep |= (m[u] > lev || (m[u] == lev && ab[u] >= tlo)) ? 1u << u : 0u;
  if (__ballot(act && clo != need) != 0) {
    // more than need channels hold the exact threshold: the lowest of them are kept
    uint32_t tie = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) tie |= (clo != need && m[u] == lev && ab[u] == tlo) ? 1u << u : 0u;
    uint32_t before = row_prefix(__popc(tie));
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (tie >> u & 1u) {
        if (before >= need - chi) keep &= ~(1u << u);
        ++before;
      }
    }
  }
  // storage positions
  lo = hi = 0;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const uint32_t one = (keep >> u & 1u) << (8 * (m[u] & 3));
    lo += m[u] < 4 ? one : 0u;
    hi += m[u] < 4 ? 0u : one;
  }
  lo = row_prefix(lo) + upl;
  hi = row_prefix(hi) + uph;
  wave_lds_sync();                       // the previous tokens' entries are stored
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const uint32_t one = (keep >> u & 1u) << (8 * (m[u] & 3));
    const uint32_t pos = keep >> u & 1u ? field(lo, hi, m[u]) : (uint32_t)D;
    w.ent[row][pos] = (uint16_t)((8 * r + u) | (q[u] & 15) << 8);
    lo += m[u] < 4 ? one : 0u;
    hi += m[u] < 4 ? 0u : one;
  }
  wave_lds_sync();
  if (act && tk >= 0) {                  // else the offsets disagree with the rank: leave the slab alone
    const int64_t e0 = w.e0[at];
    for (int j = r; j < rho / 2; j += 16) {
      const uint32_t e = *reinterpret_cast<const uint32_t*>(&w.ent[row][2 * j]);
      *reinterpret_cast<uint16_t*>(sl.res_idx + e0 + 2 * j) = (uint16_t)((e & 255u) | (e >> 8 & 0xff00u));
      sl.res_val[(e0 >> 1) + j] = (uint8_t)((e >> 8 & 15u) | (e >> 20 & 0xf0u));
    }
  }
}

// Product operands: lane (r, kk) = (lane % 16, lane / 16) holds row r (A) or
// column r (B) at depth kk; the result's rows 4 kk .. 4 kk + 3 of column r.

// Basis term, residuals and entries of the first nv (at most 16) waiting
// tokens.  Row 4 kk + j of the product is waiting token 4 j + kk, so that step j
// forms the entries of tokens 4 j .. 4 j + 3.
template <int RB, bool C8>
__device__ __forceinline__ void tile_residuals(const Slab& sl, const TileSmem<RB, C8>& sm, TileWave<RB, C8>& w,
                                               int64_t first, int head, int nv, int lane) {
#pragma clang fp contract(off)
  constexpr int NS = RB / 16;
  const int r = lane & 15, kk = lane >> 4;
  // tokens x channels, left to right over the basis rows; column r of product
  // u is the channel at position 8 r + u of a dealt row
  f4 p[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) p[u] = f4{-0.f, -0.f, -0.f, -0.f};
  if constexpr (C8) {
    // int8 rows code * S carry up to 18 significant bits: their products with
    // the fp16 basis are not exact in float32, so each product is rounded on
    // its own before the sum
    const unsigned char* ar[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) ar[j] = w.a[(head + 4 * j + kk) % kRing];
    for (int s = 0; s < NS; ++s) {
      float S[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) S[j] = half_bits_to_float(reinterpret_cast<const uint16_t*>(ar[j] + RB)[s]);
#pragma unroll 2
      for (int i4 = 0; i4 < 4; ++i4) {
        uint32_t cw[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) cw[j] = *reinterpret_cast<const uint32_t*>(ar[j] + 16 * s + 4 * i4);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const uint4 bw = *reinterpret_cast<const uint4*>(&sm.bas[16 * s + 4 * i4 + v][8 * r]);
          float av[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) av[j] = (float)(int8_t)(cw[j] >> (8 * v)) * S[j];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const float b = half_f(bw, u);
#pragma unroll
            for (int j = 0; j < 4; ++j) p[u][j] = p[u][j] + av[j] * b;
          }
        }
      }
    }
  } else {
    const uint16_t* ar =
        reinterpret_cast<const uint16_t*>(w.a[(head + 4 * (r & 3) + (r >> 2)) % kRing]) + kk * (RB / 4);
#pragma unroll
    for (int b4 = 0; b4 < NS; ++b4) {
      const uint2 aw = *reinterpret_cast<const uint2*>(ar + 4 * b4);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float av = half_bits_to_float((uint16_t)((v < 2 ? aw.x : aw.y) >> (16 * (v & 1))));
        const uint4 bw = *reinterpret_cast<const uint4*>(&sm.bas[16 * b4 + 4 * v + kk][8 * r]);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          p[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, half_f(bw, u), p[u], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (4 * j >= nv) break;              // uniform
    const int at = (head + 4 * j + kk) % kRing;
    // position 8 r + u is channel 4 (8 (r % 4) + u) + r / 4; a row's 16 lanes
    // write and read their own token only
    const uint4 xw = *reinterpret_cast<const uint4*>(&w.x[at][8 * r]);
#pragma unroll
    for (int u = 0; u < 8; ++u) w.res[kk][32 * (r & 3) + 4 * u + (r >> 2)] = half_f(xw, u) - p[u][j];
    wave_lds_sync();
    tile_entries<RB, C8>(sl, w, first, at, 4 * j + kk < nv, lane);
  }
}

// The tile in the ring rows from `tile` on, tokens base .. base + 15, of which
// [s0, s1) belong to the sequence whose basis is in LDS: projects and stores
// their coefficients and lets those with entries join the waiting tokens,
// which end at ring row `tail` (at or before the tile).  Returns how many.
template <int RB, bool C8>
__device__ __forceinline__ int tile_project(const CompressArgs& a, const Slab& sl, const TileSmem<RB, C8>& sm,
                                            TileWave<RB, C8>& w, int64_t base, int64_t s0, int64_t s1, int tile,
                                            int tail, int z, int lane) {
#pragma clang fp contract(off)
  constexpr int NS = RB / 16;
  const int r = lane & 15, kk = lane >> 4;
  const int tlo = (int)(max(s0, base) - base), thi = (int)(min(s1, base + kPT) - base);   // valid tokens

  // ---- coefficients: tokens x basis rows, left to right over the channels
  f4 ca[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) ca[s] = f4{-0.f, -0.f, -0.f, -0.f};
  const uint16_t* xr = w.x[(tile + r) % kRing];
#pragma unroll
  for (int qd = 0; qd < 4; ++qd) {
    const uint4 xw = *reinterpret_cast<const uint4*>(xr + 32 * kk + 8 * qd);
    uint4 bw[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) bw[s] = *reinterpret_cast<const uint4*>(&sm.bas[16 * s + r][32 * kk + 8 * qd]);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float av = half_f(xw, u);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        ca[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, half_f(bw[s], u), ca[s], 0, 0, 0);
    }
  }
  // lane (r, kk) holds coefficient 16 s + r of tokens 4 kk .. 4 kk + 3
  unsigned char* ar[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) ar[i] = w.a[(tile + 4 * kk + i) % kRing];
  if constexpr (C8) {
    // 8-bit blockwise: the 16 lanes of coefficient block s share, per token,
    // S = fp16(max |A| / 127); code = rne(A / S) in [-127, 127] (0 when S is
    // 0); the residual uses the rebuilt code * S
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      uint32_t cb = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint16_t sb = float_to_half_bits(row_fmax(fabsf(ca[s][i])) / 127.0f);
        const float S = half_bits_to_float(sb);
        int q = 0;
        if (S > 0.f) q = (int)fminf(fmaxf(__builtin_rintf(ca[s][i] / S), -127.f), 127.f);
        ar[i][16 * s + r] = (uint8_t)(int8_t)q;
        cb |= (uint32_t)(q & 255) << (8 * i);
        const int tl = 4 * kk + i;
        if (r == 0) {
          reinterpret_cast<uint16_t*>(ar[i] + RB)[s] = sb;
          if (tl >= tlo && tl < thi) sl.cscale[(int64_t)s * a.T + base + tl] = sb;
        }
      }
      if (z == 1) {                      // value blocks: 16 tokens of one coefficient
        uint8_t* dst = sl.coef8 + (((base >> 4) * RB + 16 * s + r) << 4) + 4 * kk;
        if (4 * kk >= tlo && 4 * kk + 4 <= thi) {
          *reinterpret_cast<uint32_t*>(dst) = cb;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (4 * kk + i >= tlo && 4 * kk + i < thi) dst[i] = (uint8_t)(cb >> (8 * i));
        }
      }
    }
    wave_lds_sync();
    if (z == 0) {                        // key tiles: 16 codes of one token and block
#pragma unroll
      for (int e = lane; e < kPT * NS; e += 64) {
        const int tl = e & 15, s = e >> 4;
        if (tl >= tlo && tl < thi)
          *reinterpret_cast<uint4*>(sl.coef8 + (((base >> 4) * NS + s) << 8) + (tl << 4)) =
              *reinterpret_cast<const uint4*>(w.a[(tile + tl) % kRing] + 16 * s);
      }
    }
  } else {
    // rounded to fp16; rows dealt by index % 4 (index i at (i % 4) * RB/4 + i / 4)
    uint2 vb[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      uint16_t hb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        hb[i] = float_to_half_bits(ca[s][i]);
        reinterpret_cast<uint16_t*>(ar[i])[(r & 3) * (RB / 4) + 4 * s + (r >> 2)] = hb[i];
      }
      vb[s] = make_uint2(hb[0] | (uint32_t)hb[1] << 16, hb[2] | (uint32_t)hb[3] << 16);
    }
    if (z == 1) {                        // value blocks: 8 tokens of one coefficient, this lane's 4 of them
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        uint16_t* dst = sl.coef + value_index(base + 4 * kk, 16 * s + r, RB);
        if (4 * kk >= tlo && 4 * kk + 4 <= thi) {
          *reinterpret_cast<uint2*>(dst) = vb[s];
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (4 * kk + i >= tlo && 4 * kk + i < thi)
              dst[i] = (uint16_t)((i < 2 ? vb[s].x : vb[s].y) >> (16 * (i & 1)));
        }
      }
    }
    wave_lds_sync();
    if (z == 0) {                        // key tiles: 8 coefficients of one token
#pragma unroll
      for (int e = lane; e < kPT * (RB / 8); e += 64) {
        const int tl = e & 15, m8 = e >> 4;
        if (tl >= tlo && tl < thi) {
          const uint16_t* ae = reinterpret_cast<const uint16_t*>(w.a[(tile + tl) % kRing]) + 2 * m8;
          uint32_t p[4];                 // index 8 m8 + k, 8 m8 + 4 + k
#pragma unroll
          for (int k = 0; k < 4; ++k) p[k] = *reinterpret_cast<const uint32_t*>(ae + k * (RB / 4));
          uint4 o;
          o.x = (p[0] & 0xffffu) | p[1] << 16;
          o.y = (p[2] & 0xffffu) | p[3] << 16;
          o.z = p[0] >> 16 | (p[1] & 0xffff0000u);
          o.w = p[2] >> 16 | (p[3] & 0xffff0000u);
          *reinterpret_cast<uint4*>(sl.coef + key_index(base + tl, 8 * m8, RB)) = o;
        }
      }
    }
  }

  // ---- rank-0 tokens get scale 0; the others move up to the waiting ones, in
  // order, four rows at a time (a row never moves down, and each step reads
  // before it writes)
  const bool mine = kk == 0 && r >= tlo && r < thi;
  const int at = (tile + r) % kRing, rho = w.rho[at];
  const uint32_t act = (uint32_t)__ballot(mine && rho > 0);
  const int n = __popc(act);
  if (mine) {
    if (rho <= 0) sl.res_scale[base + r] = 0;
    else w.list[__popc(act & ((1u << r) - 1u))] = (uint8_t)r;
  }
  wave_lds_sync();
  for (int k = 0; k < n; k += 4) {
    const bool go = k + kk < n;
    const int from = (tile + w.list[go ? k + kk : 0]) % kRing, to = (tail + k + kk) % kRing;
    const uint4 xw = *reinterpret_cast<const uint4*>(&w.x[from][8 * r]);
    constexpr int AU = TileWave<RB, C8>::AB / 16;            // 16-byte pieces of a coefficient row
    const uint4 a0 = *reinterpret_cast<const uint4*>(w.a[from] + 16 * min(r, AU - 1));
    uint4 a1 = a0;
    if constexpr (AU > 16) a1 = *reinterpret_cast<const uint4*>(w.a[from] + 16 * (AU - 1));
    const int f_rho = w.rho[from], f_tok = w.tok[from];
    const uint32_t f_e0 = w.e0[from];
    const float f_g = w.g[from];
    wave_lds_sync();
    if (go && from != to) {
      *reinterpret_cast<uint4*>(&w.x[to][8 * r]) = xw;
      if (r < AU) *reinterpret_cast<uint4*>(w.a[to] + 16 * r) = a0;
      if constexpr (AU > 16) {
        if (r == 0) *reinterpret_cast<uint4*>(w.a[to] + 16 * (AU - 1)) = a1;
      }
      if (r == 0) {
        w.rho[to] = f_rho;
        w.tok[to] = f_tok;
        w.e0[to] = f_e0;
        w.g[to] = f_g;
      }
    }
    wave_lds_sync();
  }
  return n;
}

// grid (workgroups of `groups` consecutive token groups, Hkv, 2); a group is
// one 16-token tile for each wave.  Groups start at multiples of 16 tokens, so
// a tile is one block of the coefficient layouts.
template <int RB, bool C8>
__global__ __launch_bounds__(kTileWaves<RB> * 64) void compress_tile_kernel(const CompressArgs a, int groups) {
  constexpr int NW = kTileWaves<RB>, WT = NW * kPT;
  __shared__ TileSmem<RB, C8> sm;
  const int h = blockIdx.y, z = blockIdx.z;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const Slab sl = make_slab(a, h, z);
  TileWave<RB, C8>& w = sm.w[wv];
  const int64_t end = a.t0 + a.n;
  const int64_t c0 = (a.t0 & ~(int64_t)15) + (int64_t)blockIdx.x * groups * WT;
  const int64_t c1 = min(c0 + (int64_t)groups * WT, end);
  if (c0 >= c1) return;
  int b = sequence_of(a.cu, a.batch, max(c0, a.t0)), held = -1;
  int head = 0, n = 0;                   // waiting tokens: ring rows head .. head + n - 1, n <= 15 between tiles
  TileIn in;
  tile_load(in, a, sl, c0 + kPT * wv, h, z, lane);
  for (int64_t g0 = c0; g0 < c1; g0 += WT) {
    const int64_t base = g0 + kPT * wv, g1 = min(g0 + (int64_t)WT, c1);
    const int tile = (head + n) % kRing;
    tile_stage<RB, C8>(w, a, in, tile, (int)(base - c0), lane);
    if (g0 + WT < c1) tile_load(in, a, sl, base + WT, h, z, lane);   // the next tile's inputs
    for (; b < a.batch && (int64_t)a.cu[b] < g1; ++b) {
      const int64_t s0 = max(max(g0, a.t0), (int64_t)a.cu[b]), s1 = min(g1, (int64_t)a.cu[b + 1]);
      if (s1 > s0) {                     // uniform over the workgroup
        if (held != b) {
          if (n > 0) tile_residuals<RB, C8>(sl, sm, w, c0, head, n, lane);   // under the basis they wait for
          head = (head + n) % kRing;
          n = 0;
          __syncthreads();               // every wave is done with the previous basis
          const uint16_t* src = a.basis + (int64_t)b * a.basis_b_stride + (int64_t)(h * 2 + z) * RB * D;
          for (int e = threadIdx.x; e < RB * (D / 8); e += NW * 64)
            store_dealt(sm.bas[e >> 4], 8 * (e & 15), reinterpret_cast<const uint4*>(src)[e]);
          held = b;
          __syncthreads();
        }
        if (base < s1 && base + kPT > s0) {
          n += tile_project<RB, C8>(a, sl, sm, w, base, s0, s1, tile, (head + n) % kRing, z, lane);
          if (n >= kPT) {
            tile_residuals<RB, C8>(sl, sm, w, c0, head, kPT, lane);
            head = (head + kPT) % kRing;
            n -= kPT;
          }
        }
      }
      if ((int64_t)a.cu[b + 1] > g1) break;   // the next group goes on in this sequence
    }
  }
  if (n > 0) tile_residuals<RB, C8>(sl, sm, w, c0, head, n, lane);
}

template <int RB>
void launch_tile(const CompressArgs& a, hipStream_t s) {
  constexpr int WT = kTileWaves<RB> * kPT;
  const int64_t n16 = a.n + (a.t0 & 15), ng = (n16 + WT - 1) / WT;
  // groups per workgroup (each loads the basis once and ends with a partly
  // filled batch of waiting tokens): as many as leave two rounds of the one
  // workgroup a compute unit holds, up to 64.  128K tokens of 8 KV heads (r_b 48)
  // take 774 us, with one round 763 and with four 803; at r_b 96 1739, 2105 and
  // 1728.  512K tokens take 2.54 ms with up to 64 groups, 2.67 with up to 16 and
  // 2.51 with no limit.
  const int64_t per = std::max<int64_t>(1, std::min<int64_t>(64, ng * a.n_kv_heads * 2 / 512));
  const dim3 grid((unsigned)((ng + per - 1) / per), a.n_kv_heads, 2);
  if (a.c8) hipLaunchKernelGGL((compress_tile_kernel<RB, true>), grid, dim3(WT * 4), 0, s, a, (int)per);
  else hipLaunchKernelGGL((compress_tile_kernel<RB, false>), grid, dim3(WT * 4), 0, s, a, (int)per);
}

// Short ranges keep the one-wave-per-token kernel, whose time holds as long as
// its workgroups run at once, 8.4 us at r_b 48 and 13.8 at r_b 128.  A tile's
// products take the same time for 1 token and 16: 12 and 21 us from 5 tokens on
// in fp16, 20 to 22 and 41 to 43 us in int8, whose basis term runs on the vector
// units.  The line is where tiles overtook a workgroup of four waves that took
// the range's tokens in turn: 13.9 and 24 us for 5 fp16 tokens; in int8 14.6 and
// 25 us for 5, 20 and 37 for 12, 26 and 47 for 16.
constexpr int64_t kFewTokens = 4, kFewTokensI8 = 15;

}  // namespace

hipError_t launch_compress(const CompressArgs& a, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  if (a.n <= (a.c8 ? kFewTokensI8 : kFewTokens)) {
    const unsigned nb = (unsigned)((a.n + kCW - 1) / kCW);
    hipLaunchKernelGGL(compress_kernel, dim3(nb, a.n_kv_heads, 2), dim3(kCW * 64), 0, s, a);
    return hipGetLastError();
  }
  switch (a.rb) {
    case 16: launch_tile<16>(a, s); break;
    case 32: launch_tile<32>(a, s); break;
    case 48: launch_tile<48>(a, s); break;
    case 64: launch_tile<64>(a, s); break;
    case 80: launch_tile<80>(a, s); break;
    case 96: launch_tile<96>(a, s); break;
    case 112: launch_tile<112>(a, s); break;
    case 128: launch_tile<128>(a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace dwkv
