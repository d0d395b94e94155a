// Router (Eq. 2) with its residual-offset scan (over the whole packed axis or a
// token range that continues an existing table), the residual-map test hook and
// the layout validator (gfx950).
#include "entry.h"
#include "internal.h"

namespace dwkv {
namespace {

constexpr int D = kHeadDim;
constexpr int kRT = 256;                                  // route block threads
constexpr int kPerThread = kRouteTokensPerBlock / kRT;   // 4 tokens per thread

// Router score, float32, left to right, each product and sum rounded on its own
// (no fused multiply-add), so it reproduces bit for bit on any IEEE machine.
__device__ __forceinline__ float router_score(const float4 u, const float4 f) {
#pragma clang fp contract(off)
  float z = u.x * f.x;
  z = z + u.y * f.y;
  z = z + u.z * f.z;
  z = z + u.w * f.w;
  return z;
}

__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) red[wv] = v;
  __syncthreads();
  uint32_t t = 0;
  for (int i = 0; i < kRT / 64; ++i) t += red[i];
  return t;
}

// Exclusive prefix over the block's threads (kRT threads); returns the block total in *total.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* red, uint32_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t inc = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t n = __shfl_up(inc, o);
    if (lane >= o) inc += n;
  }
  if (lane == 63) red[wv] = inc;
  __syncthreads();
  uint32_t before = 0, all = 0;
  for (int i = 0; i < kRT / 64; ++i) {
    if (i < wv) before += red[i];
    all += red[i];
  }
  *total = all;
  return before + inc - v;
}

// Level codes of this thread's tokens of block `blk`, written to a.code; the
// routed ranks go to rho[] (0 past the range).  Returns their sum.
__device__ __forceinline__ uint32_t route_block_tokens(const RouteArgs& a, int mh, int blk,
                                                       uint32_t (&rho)[kPerThread]) {
  const int m = mh / a.n_kv_heads;
  const float4 u = *reinterpret_cast<const float4*>(a.u + 4 * m);
  const int nth = a.n_levels - 1;
  float th[DWKV_MAX_LEVELS - 1];
#pragma unroll
  for (int j = 0; j < DWKV_MAX_LEVELS - 1; ++j) th[j] = j < nth ? a.theta[m * nth + j] : 0.f;
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    const int64_t t = a.t0 + (int64_t)blk * kRouteTokensPerBlock + threadIdx.x * kPerThread + i;
    rho[i] = 0u;
    if (t < a.t0 + a.n) {
      const float4 f = *reinterpret_cast<const float4*>(a.phi + ((int64_t)mh * a.T + t) * 4);
      const float z = router_score(u, f);
      int k = 0;
#pragma unroll
      for (int j = 0; j < DWKV_MAX_LEVELS - 1; ++j) k += (j < nth && z > th[j]) ? 1 : 0;
      a.code[(int64_t)mh * a.T + t] = (uint8_t)k;
      rho[i] = (uint32_t)a.levels[k];
      sum += rho[i];
    }
  }
  return sum;
}

// Offsets of this thread's tokens: off[t+1] = carry + (ranks of earlier tokens) + rho_t,
// with `carry` the offset of the block's first token.
__device__ __forceinline__ void route_write_offsets(const RouteArgs& a, int mh, int blk, uint32_t carry,
                                                    const uint32_t (&rho)[kPerThread], uint32_t* red) {
  uint32_t mine = 0;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) mine += rho[i];
  uint32_t total;
  uint32_t run = carry + block_exclusive_scan(mine, red, &total);
  uint32_t* off = a.off + (int64_t)mh * (a.T + 1);
  if (a.t0 == 0 && blk == 0 && threadIdx.x == 0) off[0] = 0u;
  const int64_t end = a.t0 + a.n;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    const int64_t t = a.t0 + (int64_t)blk * kRouteTokensPerBlock + threadIdx.x * kPerThread + i;
    run += rho[i];
    if (t < end) off[t + 1] = run;
  }
}

// A range of at most one block of tokens in one launch: codes, scan, offsets.  grid (M*Hkv)
__global__ __launch_bounds__(kRT) void route_small_kernel(const RouteArgs a) {
  __shared__ uint32_t red[kRT / 64];
  const int mh = blockIdx.x;
  uint32_t rho[kPerThread];
  route_block_tokens(a, mh, 0, rho);
  const uint32_t carry = a.t0 == 0 ? 0u : a.off[(int64_t)mh * (a.T + 1) + a.t0];
  route_write_offsets(a, mh, 0, carry, rho, red);
}

// Level codes and per-block rank sums.  grid (nblk, M*Hkv)
__global__ __launch_bounds__(kRT) void route_codes_kernel(const RouteArgs a) {
  __shared__ uint32_t red[kRT / 64];
  const int mh = blockIdx.y;
  uint32_t rho[kPerThread];
  const uint32_t sum = route_block_tokens(a, mh, blockIdx.x, rho);
  const uint32_t tot = block_sum(sum, red);
  if (threadIdx.x == 0) a.bsum[(int64_t)mh * a.nblk + blockIdx.x] = tot;
}

// Exclusive scan of the block sums of one (window, head).  grid (M*Hkv)
__global__ __launch_bounds__(kRT) void route_block_scan_kernel(const RouteArgs a) {
  __shared__ uint32_t red[kRT / 64];
  const int mh = blockIdx.x;
  uint32_t carry = 0;
  for (int b0 = 0; b0 < a.nblk; b0 += kRT) {
    const int b = b0 + threadIdx.x;
    const uint32_t v = b < a.nblk ? a.bsum[(int64_t)mh * a.nblk + b] : 0u;
    uint32_t total;
    const uint32_t ex = block_exclusive_scan(v, red, &total);
    if (b < a.nblk) a.bpre[(int64_t)mh * a.nblk + b] = carry + ex;
    carry += total;
    __syncthreads();
  }
}

// Offsets of a multi-block range from the codes and the scanned block sums.
__global__ __launch_bounds__(kRT) void route_offsets_kernel(const RouteArgs a) {
  __shared__ uint32_t red[kRT / 64];
  const int mh = blockIdx.y;
  const int64_t end = a.t0 + a.n;
  uint32_t rho[kPerThread];
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    const int64_t t = a.t0 + (int64_t)blockIdx.x * kRouteTokensPerBlock + threadIdx.x * kPerThread + i;
    rho[i] = t < end ? (uint32_t)a.levels[a.code[(int64_t)mh * a.T + t]] : 0u;
  }
  // carry-in: the offset of the range's first token (0 for a table that starts here)
  const uint32_t base = a.t0 == 0 ? 0u : a.off[(int64_t)mh * (a.T + 1) + a.t0];
  route_write_offsets(a, mh, blockIdx.x, base + a.bpre[(int64_t)mh * a.nblk + blockIdx.x], rho, red);
}

// Budget routing (two levels, Eq. 2 with tau chosen for a memory budget): the
// n = floor((E - N rho_min) / (rho_max - rho_min)) tokens of largest score z
// get level 1, ties to the lower token.  The n-th largest of the scores'
// order-preserving bits is found from the top in digits of 11, 11 and 10 bits
// (a histogram of the scores that match the digits fixed so far); every score
// above it is kept, and of those equal to it the first ones that complete n.
// The offsets then follow from running counts of both.
//
// Ranges of up to kBudgetOne tokens run in one workgroup per (window, head),
// the scores held in registers.  Longer ones spread over the chip in six
// launches (clear 3 us, three digits 16, 12 and 6, counts 7, write 11): 64
// pairs of 64K tokens take 52 to 55 us (their 88 MB of features and results alone 18
// at the copy rate) and are bound by the launches and by the histograms'
// atomics.  One workgroup per pair with eight passes over 64-bit keys in memory
// took 540 us.  For 1024 and 16384 tokens the single launch takes 12 and 18 us,
// the six take 25 and 29.
constexpr int kBins = 2048;
constexpr int kBT = 1024;                                 // threads of the one-workgroup form
constexpr int kBudgetPer = 16;                            // its scores per thread
constexpr int64_t kBudgetOne = (int64_t)kBT * kBudgetPer;
constexpr int kBudgetRounds = kBudgetTokensPerBlock / kRT;

// The kept tokens: score bits above thr, and the first `tie` of those equal.
struct BudgetCut {
  uint32_t thr, tie;
};

// Level-1 tokens of one (window, head).
__device__ __forceinline__ int64_t budget_count(const RouteArgs& a, int mh) {
  const int64_t N = a.n, rmin = a.levels[0], rmax = a.levels[1];
  const int64_t room = a.entries[mh] - N * rmin;
  const int64_t n = rmax > rmin && room >= 0 ? room / (rmax - rmin) : 0;
  return min(max(n, (int64_t)0), N);
}

__device__ __forceinline__ uint32_t budget_bits(const float4 u, const float4 f) {
  const float z = router_score(u, f) + 0.0f;              // -0 -> +0: equal scores tie
  const uint32_t b = __float_as_uint(z);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Bin (from the top) in which the rem-th largest of `hist` lies, and how many
// of that bin complete it.  NT threads, kBins / NT bins each; the histogram is
// complete and visible, and holds at least rem >= 1.
template <int NT>
__device__ __forceinline__ void budget_pick(const uint32_t* hist, uint32_t rem, uint32_t* red, uint32_t* pick) {
  constexpr int P = kBins / NT;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t c[P], mine = 0;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    c[i] = hist[kBins - 1 - (threadIdx.x * P + i)];
    mine += c[i];
  }
  uint32_t inc = mine;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(inc, o);
    if (lane >= o) inc += v;
  }
  if (lane == 63) red[wv] = inc;
  __syncthreads();
  uint32_t above = inc - mine;
  for (int i = 0; i < wv; ++i) above += red[i];
  if (above < rem && rem <= above + mine) {               // one thread
#pragma unroll
    for (int i = 0; i < P; ++i) {
      if (above < rem && rem <= above + c[i]) {
        pick[0] = kBins - 1 - (threadIdx.x * P + i);
        pick[1] = rem - above;
      }
      above += c[i];
    }
  }
  __syncthreads();
}

// Code and offset of token j of the range, given the kept tokens before and at it.
__device__ __forceinline__ void budget_write(const RouteArgs& a, int mh, int64_t j, uint32_t carry, bool keep,
                                             uint32_t kept) {
  a.code[(int64_t)mh * a.T + a.t0 + j] = keep ? 1 : 0;
  a.off[(int64_t)mh * (a.T + 1) + a.t0 + j + 1] =
      carry + (uint32_t)a.levels[0] * (uint32_t)(j + 1) + (uint32_t)(a.levels[1] - a.levels[0]) * kept;
}

// Counts of the tokens above and at the threshold over R rounds of NT tokens
// in token order (gt, eq: this thread's flags, a bit per round): per round, the
// counts before this thread.  cnt: [R NT / 64 + 4][2] in LDS.
template <int NT, int R>
__device__ __forceinline__ void budget_scan(uint32_t gt, uint32_t eq, uint32_t (*cnt)[2], uint32_t (&bg)[R],
                                            uint32_t (&be)[R]) {
  constexpr int W = NT / 64, E = R * W;                   // a wave's share of a round per entry
  static_assert(E <= NT, "one entry per thread");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const unsigned long long mg = __ballot(gt >> i & 1u), me = __ballot(eq >> i & 1u);
    bg[i] = __builtin_amdgcn_mbcnt_hi((uint32_t)(mg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mg, 0u));
    be[i] = __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0u));
    if (lane == 0) {
      cnt[i * W + wv][0] = __popcll(mg);
      cnt[i * W + wv][1] = __popcll(me);
    }
  }
  __syncthreads();
  uint32_t g = tid < E ? cnt[tid][0] : 0u, e = tid < E ? cnt[tid][1] : 0u;
  const uint32_t g0 = g, e0 = e;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t vg = __shfl_up(g, o), ve = __shfl_up(e, o);
    if (lane >= o) { g += vg; e += ve; }
  }
  if (lane == 63 && wv < 4) { cnt[E + wv][0] = g; cnt[E + wv][1] = e; }
  __syncthreads();
  for (int v = 0; v < min(wv, 4); ++v) { g += cnt[E + v][0]; e += cnt[E + v][1]; }
  if (tid < E) { cnt[tid][0] = g - g0; cnt[tid][1] = e - e0; }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < R; ++i) {
    bg[i] += cnt[i * W + wv][0];
    be[i] += cnt[i * W + wv][1];
  }
}

// The one-workgroup form, N <= kBudgetOne.  grid (M*Hkv)
__global__ __launch_bounds__(kBT) void route_budget_one_kernel(const RouteArgs a) {
  __shared__ uint32_t hist[kBins], red[kBT / 64], pick[2];
  __shared__ uint32_t cnt[kBudgetPer * kBT / 64 + 4][2];
  const int mh = blockIdx.x, tid = threadIdx.x;
  const int64_t N = a.n, n = budget_count(a, mh);
  const float4 u = *reinterpret_cast<const float4*>(a.u + 4 * (mh / a.n_kv_heads));
  const float4* phi = reinterpret_cast<const float4*>(a.phi) + (int64_t)mh * a.T + a.t0;
  const uint32_t carry = a.t0 == 0 ? 0u : a.off[(int64_t)mh * (a.T + 1) + a.t0];
  uint32_t o[kBudgetPer];
#pragma unroll
  for (int i = 0; i < kBudgetPer; ++i) {
    const int64_t j = (int64_t)i * kBT + tid;
    o[i] = j < N ? budget_bits(u, phi[j]) : 0u;
  }
  BudgetCut cut{n == 0 ? ~0u : 0u, n == 0 ? 0u : ~0u};    // nothing, or everything
  if (n > 0 && n < N) {
    uint32_t prefix = 0, rem = (uint32_t)n;
#pragma unroll
    for (int lv = 0; lv < 3; ++lv) {
      const int sh = lv == 0 ? 21 : lv == 1 ? 10 : 0, dig = lv == 2 ? 1023 : 2047;
      for (int i = tid; i < kBins; i += kBT) hist[i] = 0u;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kBudgetPer; ++i) {
        const bool in = (int64_t)i * kBT + tid < N && (lv == 0 || (o[i] >> (lv == 1 ? 21 : 10)) == prefix);
        if (in) atomicAdd(&hist[(o[i] >> sh) & dig], 1u);
      }
      __syncthreads();
      budget_pick<kBT>(hist, rem, red, pick);
      prefix = lv == 2 ? prefix << 10 | pick[0] : prefix << 11 | pick[0];
      rem = pick[1];
      __syncthreads();
    }
    cut = BudgetCut{prefix, rem};
  }
  uint32_t gt = 0, eq = 0, bg[kBudgetPer], be[kBudgetPer];
#pragma unroll
  for (int i = 0; i < kBudgetPer; ++i) {
    const bool in = (int64_t)i * kBT + tid < N;
    gt |= in && o[i] > cut.thr ? 1u << i : 0u;
    eq |= in && o[i] == cut.thr ? 1u << i : 0u;
  }
  budget_scan<kBT, kBudgetPer>(gt, eq, cnt, bg, be);
  if (a.t0 == 0 && tid == 0) a.off[(int64_t)mh * (a.T + 1)] = 0u;
#pragma unroll
  for (int i = 0; i < kBudgetPer; ++i) {
    const int64_t j = (int64_t)i * kBT + tid;
    if (j < N) {
      const uint32_t ig = gt >> i & 1u, ie = eq >> i & 1u;
      const bool keep = ig || (ie && be[i] < cut.tie);
      budget_write(a, mh, j, carry, keep, bg[i] + ig + min(be[i] + ie, cut.tie));
    }
  }
}

// The spread form.  Per (window, head) in the workspace: the scores' bits, one
// histogram per digit, and the state the launches hand on (digits found so
// far, how many the rest still has to give).
__global__ __launch_bounds__(kRT) void route_budget_clear_kernel(const RouteArgs a) {
  a.hist[(int64_t)blockIdx.x * kBins * 3 + blockIdx.y * kRT + threadIdx.x] = 0u;
}

// Digit LV of the scores: LV 0 also forms the bits from the features.
// grid (nblk, M*Hkv)
template <int LV>
__global__ __launch_bounds__(kRT) void route_budget_digit_kernel(const RouteArgs a) {
  __shared__ uint32_t hist[kBins], red[kRT / 64], pick[2];
  const int mh = blockIdx.y, tid = threadIdx.x;
  const int64_t N = a.n, n = budget_count(a, mh), c0 = (int64_t)blockIdx.x * kBudgetTokensPerBlock;
  uint32_t* bits = a.keys + (int64_t)mh * a.T;
  uint32_t* gh = a.hist + (int64_t)mh * kBins * 3;
  uint32_t* st = a.state + 4 * mh;
  const bool search = n > 0 && n < N;
  for (int i = tid; i < kBins; i += kRT) hist[i] = 0u;
  uint32_t prefix = 0;
  if constexpr (LV > 0) {
    if (!search) return;
    const uint32_t rem = LV == 1 ? (uint32_t)n : st[1];
    budget_pick<kRT>(gh + (LV - 1) * kBins, rem, red, pick);
    prefix = LV == 1 ? pick[0] : st[0] << 11 | pick[0];
    if (blockIdx.x == 0 && tid == 0) {                    // for the next launch
      st[2 * (LV - 1)] = prefix;
      st[2 * (LV - 1) + 1] = pick[1];
    }
  } else {
    __syncthreads();
  }
  const float4 u = *reinterpret_cast<const float4*>(a.u + 4 * (mh / a.n_kv_heads));
  const float4* phi = reinterpret_cast<const float4*>(a.phi) + (int64_t)mh * a.T + a.t0;
#pragma unroll
  for (int i = 0; i < kBudgetRounds; ++i) {
    const int64_t j = c0 + i * kRT + tid;
    if (j < N) {
      uint32_t o;
      if constexpr (LV == 0) {
        o = budget_bits(u, phi[j]);
        bits[j] = o;
        atomicAdd(&hist[o >> 21], 1u);
      } else {
        o = bits[j];
        if (o >> (LV == 1 ? 21 : 10) == prefix) atomicAdd(&hist[LV == 1 ? (o >> 10) & 2047u : o & 1023u], 1u);
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < kBins; i += kRT)
    if (hist[i]) atomicAdd(&gh[LV * kBins + i], hist[i]);
}

// Per block, the tokens above and at the threshold.  grid (nblk, M*Hkv)
__global__ __launch_bounds__(kRT) void route_budget_count_kernel(const RouteArgs a) {
  __shared__ uint32_t red[kRT / 64], pick[2], cnt[2];
  const int mh = blockIdx.y, tid = threadIdx.x;
  const int64_t N = a.n, n = budget_count(a, mh), c0 = (int64_t)blockIdx.x * kBudgetTokensPerBlock;
  const uint32_t* bits = a.keys + (int64_t)mh * a.T;
  uint32_t* st = a.state + 4 * mh;
  BudgetCut cut{n == 0 ? ~0u : 0u, n == 0 ? 0u : ~0u};
  if (tid < 2) cnt[tid] = 0u;
  if (n > 0 && n < N) {
    const uint32_t prefix = st[2], rem = st[3];
    budget_pick<kRT>(a.hist + (int64_t)mh * kBins * 3 + 2 * kBins, rem, red, pick);
    cut = BudgetCut{prefix << 10 | pick[0], pick[1]};
  }
  __syncthreads();
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int i = 0; i < kBudgetRounds; ++i) {
    const int64_t j = c0 + i * kRT + tid;
    const uint32_t o = j < N ? bits[j] : 0u;
    gt += __popcll(__ballot(j < N && o > cut.thr));
    eq += __popcll(__ballot(j < N && o == cut.thr));
  }
  if ((tid & 63) == 0) {
    atomicAdd(&cnt[0], gt);
    atomicAdd(&cnt[1], eq);
  }
  __syncthreads();
  if (tid < 2) a.bsum[((int64_t)mh * a.nblk + blockIdx.x) * 2 + tid] = cnt[tid];
  if (blockIdx.x == 0 && tid == 0) {                      // the cut, for the last launch
    st[0] = cut.thr;
    st[1] = cut.tie;
  }
}

// Codes and offsets.  grid (nblk, M*Hkv)
__global__ __launch_bounds__(kRT) void route_budget_write_kernel(const RouteArgs a) {
  __shared__ uint32_t cnt[kBudgetRounds * kRT / 64 + 4][2], before[2];
  const int mh = blockIdx.y, tid = threadIdx.x;
  const int64_t N = a.n, c0 = (int64_t)blockIdx.x * kBudgetTokensPerBlock;
  const uint32_t* bits = a.keys + (int64_t)mh * a.T;
  const BudgetCut cut{a.state[4 * mh], a.state[4 * mh + 1]};
  const uint32_t carry = a.t0 == 0 ? 0u : a.off[(int64_t)mh * (a.T + 1) + a.t0];
  if (tid < 2) before[tid] = 0u;
  __syncthreads();
  uint32_t g = 0, e = 0;
  for (int i = tid; i < (int)blockIdx.x; i += kRT) {
    g += a.bsum[((int64_t)mh * a.nblk + i) * 2];
    e += a.bsum[((int64_t)mh * a.nblk + i) * 2 + 1];
  }
  for (int o = 32; o > 0; o >>= 1) {
    g += __shfl_xor(g, o);
    e += __shfl_xor(e, o);
  }
  if ((tid & 63) == 0 && (g | e)) {
    atomicAdd(&before[0], g);
    atomicAdd(&before[1], e);
  }
  uint32_t gt = 0, eq = 0, bg[kBudgetRounds], be[kBudgetRounds];
#pragma unroll
  for (int i = 0; i < kBudgetRounds; ++i) {
    const int64_t j = c0 + i * kRT + tid;
    const uint32_t o = j < N ? bits[j] : 0u;
    gt |= j < N && o > cut.thr ? 1u << i : 0u;
    eq |= j < N && o == cut.thr ? 1u << i : 0u;
  }
  budget_scan<kRT, kBudgetRounds>(gt, eq, cnt, bg, be);   // its barriers also publish `before`
  if (a.t0 == 0 && blockIdx.x == 0 && tid == 0) a.off[(int64_t)mh * (a.T + 1)] = 0u;
#pragma unroll
  for (int i = 0; i < kBudgetRounds; ++i) {
    const int64_t j = c0 + i * kRT + tid;
    if (j < N) {
      const uint32_t ig = gt >> i & 1u, ie = eq >> i & 1u, eb = be[i] + before[1];
      const bool keep = ig || (ie && eb < cut.tie);
      budget_write(a, mh, j, carry, keep, bg[i] + before[0] + ig + min(eb + ie, cut.tie));
    }
  }
}

// One thread per token: dense g*R row of the token.
__global__ __launch_bounds__(256) void residual_map_kernel(const uint32_t* off, const uint8_t* idx,
                                                           const uint8_t* val, const uint16_t* scale,
                                                           int64_t t0, int64_t t1, int64_t slab_len,
                                                           float* dense) {
  const int64_t t = t0 + (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= t1) return;
  float* row = dense + (t - t0) * D;
  for (int c = 0; c < D; ++c) row[c] = 0.f;
  const float s = half_bits_to_float(scale[t]);
  const int64_t e0 = off[t], e1 = off[t + 1];
  const int64_t end = min(min(e1, e0 + D), slab_len);   // bounded even for a corrupt table
  for (int64_t e = e0; e < end; ++e)
    row[idx[e] & (D - 1)] = s * (float)entry_code(val[e >> 1], e);
}

struct ValidateArgs {
  const uint8_t* code;
  const uint32_t* off;
  const uint8_t* idx;
  const uint8_t* val;
  unsigned long long* bad;
  int64_t T, res_stride;
  int32_t n_kv_heads, window, n_levels;
  int32_t levels[DWKV_MAX_LEVELS];
};

__device__ __forceinline__ void report(unsigned long long* bad, int64_t mh, int64_t T, int64_t t, int kind) {
  atomicMin(bad, (unsigned long long)(((mh * (T + 1) + t) << 3) | kind));
}

__global__ void fill_u64_kernel(unsigned long long* p, unsigned long long v) { *p = v; }

// grid (ceil((T+1)/256), M*Hkv)
__global__ __launch_bounds__(256) void validate_kernel(const ValidateArgs a) {
  const int64_t mh = blockIdx.y;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t > a.T) return;
  const uint32_t* off = a.off + mh * (a.T + 1);
  if (t == a.T) {              // global checks ride on the extra thread
    if (off[0] != 0u || (int64_t)off[a.T] + kResTailPad > a.res_stride) report(a.bad, mh, a.T, t, 7);
    return;
  }
  const uint32_t o0 = off[t], o1 = off[t + 1];
  const uint32_t k = a.code[mh * a.T + t];
  if (k >= (uint32_t)a.n_levels) { report(a.bad, mh, a.T, t, 2); return; }
  if (o1 < o0 || o1 - o0 != (uint32_t)a.levels[k]) { report(a.bad, mh, a.T, t, 1); return; }
  if ((int64_t)o1 > a.res_stride) { report(a.bad, mh, a.T, t, 7); return; }
  const int m = (int)(mh / a.n_kv_heads), h = (int)(mh % a.n_kv_heads);
  for (int li = 0; li < a.window; ++li) {
    const int l = m * a.window + li;
    for (int z = 0; z < 2; ++z) {
      const int64_t slab = ((int64_t)(l * 2 + z) * a.n_kv_heads + h);
      const uint8_t* ix = a.idx + slab * a.res_stride;
      const uint8_t* vl = a.val + slab * (a.res_stride / 2);
      uint32_t seen[4] = {0u, 0u, 0u, 0u};
      int prev_abs = 8, prev_c = -1;
      for (uint32_t e = o0; e < o1; ++e) {
        const int c = ix[e];
        if (c >= D) { report(a.bad, mh, a.T, t, 3); return; }
        if (seen[c >> 5] & (1u << (c & 31))) { report(a.bad, mh, a.T, t, 4); return; }
        seen[c >> 5] |= 1u << (c & 31);
        const int code = entry_code(vl[e >> 1], e);
        if (code == -8) { report(a.bad, mh, a.T, t, 5); return; }
        const int ab = code < 0 ? -code : code;
        if (ab > prev_abs || (ab == prev_abs && c < prev_c)) { report(a.bad, mh, a.T, t, 6); return; }
        prev_abs = ab;
        prev_c = c;
      }
    }
  }
}

}  // namespace

hipError_t launch_route(const RouteArgs& a, int n_mh, hipStream_t s) {
  if (a.nblk <= 1) {                     // one block per (window, head): a single launch
    hipLaunchKernelGGL(route_small_kernel, dim3(n_mh), dim3(kRT), 0, s, a);
  } else {
    hipLaunchKernelGGL(route_codes_kernel, dim3(a.nblk, n_mh), dim3(kRT), 0, s, a);
    hipLaunchKernelGGL(route_block_scan_kernel, dim3(n_mh), dim3(kRT), 0, s, a);
    hipLaunchKernelGGL(route_offsets_kernel, dim3(a.nblk, n_mh), dim3(kRT), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_route_budget(const RouteArgs& a, int n_mh, hipStream_t s) {
  if (a.n <= kBudgetOne) {
    hipLaunchKernelGGL(route_budget_one_kernel, dim3(n_mh), dim3(kBT), 0, s, a);
    return hipGetLastError();
  }
  const dim3 grid(a.nblk, n_mh);
  hipLaunchKernelGGL(route_budget_clear_kernel, dim3(n_mh, 3 * kBins / kRT), dim3(kRT), 0, s, a);
  hipLaunchKernelGGL(route_budget_digit_kernel<0>, grid, dim3(kRT), 0, s, a);
  hipLaunchKernelGGL(route_budget_digit_kernel<1>, grid, dim3(kRT), 0, s, a);
  hipLaunchKernelGGL(route_budget_digit_kernel<2>, grid, dim3(kRT), 0, s, a);
  hipLaunchKernelGGL(route_budget_count_kernel, grid, dim3(kRT), 0, s, a);
  hipLaunchKernelGGL(route_budget_write_kernel, grid, dim3(kRT), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_residual_map(const uint32_t* off, const uint8_t* idx, const uint8_t* val,
                               const uint16_t* scale, int64_t t0, int64_t t1, int64_t slab_len,
                               float* dense, hipStream_t s) {
  const int64_t n = t1 - t0;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(residual_map_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, off,
                     idx, val, scale, t0, t1, slab_len, dense);
  return hipGetLastError();
}

hipError_t launch_validate(const dwkv_dims* d, const dwkv_cache* c, unsigned long long* bad,
                           hipStream_t s) {
  ValidateArgs a;
  a.code = c->rank_code;
  a.off = c->res_off;
  a.idx = c->res_idx;
  a.val = c->res_val;
  a.bad = bad;
  a.T = d->total_tokens;
  a.res_stride = d->res_stride;
  a.n_kv_heads = d->n_kv_heads;
  a.window = d->window;
  a.n_levels = d->n_levels;
  for (int i = 0; i < DWKV_MAX_LEVELS; ++i) a.levels[i] = d->levels[i];
  const int n_mh = (d->n_layers / d->window) * d->n_kv_heads;
  hipLaunchKernelGGL(fill_u64_kernel, dim3(1), dim3(1), 0, s, bad, ~0ull);
  hipLaunchKernelGGL(validate_kernel, dim3((unsigned)((a.T + 1 + 255) / 256), n_mh), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace dwkv
