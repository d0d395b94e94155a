// Materialization of the rebuilt cache (Eq. 1 written out to HBM) on gfx950:
// K_hat = A^K B^K + g R^K and V_hat = A^V B^V + g R^V for every token and KV
// head of one layer, rounded once to fp16.  It exists for the unfused
// comparison path (rebuild, then dense attention over the rebuilt cache), the
// design the fused decode avoids.
//
// Bound by HBM: a 64K layer of 8 KV heads (r_b 48) reads 108 MB and writes 268
// in 84 to 94 us, 4.0 to 4.5 TB/s where torch's copy kernel reaches 4.8.
// A workgroup of 4 waves stages the basis of each sequence its tokens belong to
// in LDS, transposed (channel-major, so an MFMA fragment is one 8-byte read);
// the waves take its 16-token blocks in turn, each [16 tokens x 128 channels]
// on v_mfma_f32_16x16x16f16.  The operands are chosen so that a result is
// stored from the registers it ends in (keys row-major, values in the 16-token
// blocked layout, padding tokens of the last block zeroed); only the routed
// residual codes go through LDS, as bytes, and are added to the float32 product
// before the one rounding.  They are added at every channel, 0 where there is no
// entry, which holds for finite scales only: entries of other scales follow
// behind the wave's blocks (mat_odd).  A block's coefficients and entries are
// loaded one block ahead, its offsets two, and 4 waves fit a SIMD up to r_b 64.
// Measured at that layer: the materialize + dense decode pair takes 145 us,
// against 208 us when two-wave workgroups passed a float32 tile through LDS and
// waited for every block's entries.
#include "entry.h"
#include "internal.h"

namespace dwkv {
namespace {

constexpr int D = kHeadDim;
constexpr int kMW = 4;                   // waves per workgroup
constexpr int kMBlocks = 16;             // 16-token blocks per wave of a large launch (64K tokens of 8 KV heads at
                                         // r_b 48 and 128: 94.7 and 146.8 us; 8: 100.9 and 154.1; 32: 94.8 and 148.5)
constexpr int kMWaves = 4096;            // 4 waves on each of 1024 SIMDs
constexpr int kMRegRank = 32;            // bases up to this rank keep their fragments in registers (at 48
                                         // they no longer fit the 128 registers of 4 waves per SIMD)
constexpr int kMaxEnt = 16;              // entries of a token read in one batch (4 per lane of its column)

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));   // not uint4, whose copies stay in scratch

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int seq_of(const int32_t* cu, int batch, int64_t t) {
  int lo = 0, hi = batch;                // cu[lo] <= t < cu[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)cu[mid] <= t) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ uint32_t pack_half2(float lo, float hi) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)lo) |
         ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)hi) << 16);
}

template <int RB>
struct MSmem {
  static constexpr int BT = RB + 4;      // transposed basis row (halves); the pad spreads the
                                         // 16 lanes of a fragment read over distinct banks
  static constexpr int ST = RB * 8 + 8;  // 8 tokens' value coefficients; the pad keeps the block's
                                         // two halves on distinct banks
  static constexpr int KROW = D + 8;     // key codes of one token, padded the same way
  alignas(16) uint16_t bt[D * BT];       // bt[c][k] = B[k][c]
  alignas(16) uint8_t codes[kMW][16 * KROW];    // int4 codes of a block: keys [token][c], values [c][token]
  alignas(16) uint16_t stage[kMW][2 * ST];      // a block's value coefficients as stored
};

// Fragment (output tile nt, k-step s) of the basis in LDS.
template <int RB, int Z>
__device__ __forceinline__ h4 mat_frag(const MSmem<RB>& sm, int nt, int s, int lane) {
  const int grp = lane >> 4, r = lane & 15;
  const int c = Z == 0 ? 32 * (nt >> 1) + 8 * (r >> 2) + 4 * (nt & 1) + (r & 3) : 16 * nt + r;
  return *reinterpret_cast<const h4*>(&sm.bt[c * MSmem<RB>::BT + 16 * s + 4 * grp]);
}

// Offsets and scale of token w0 + r of a 16-token block.
struct MHead {
  uint32_t e0, rho, sbits;
};

__device__ __forceinline__ void mat_head(MHead& m, const MatArgs& a, int w0, int s0, int s1, int r,
                                         const uint32_t* off, const uint16_t* scale) {
  const int t = min(w0 + r, (int)a.T - 1);
  const uint32_t e0 = off[t], e1 = off[t + 1];
  m.sbits = scale[t];
  m.e0 = e0;
  m.rho = w0 + r >= s0 && w0 + r < s1 && e1 > e0 ? min(e1 - e0, (uint32_t)D) : 0u;
  if (e0 + m.rho > (uint64_t)a.res_stride) m.rho = 0;   // a malformed table adds nothing
}

__device__ __forceinline__ bool scale_finite(const MHead& m) { return (m.sbits & 0x7c00u) != 0x7c00u; }

// Coefficients and residual entries of a block.  The four lanes of a token's
// column share its entries: lane group grp takes entries grp, grp + 4, ...
template <int RB, int Z>
struct MBlock {
  static constexpr int NV = (2 * RB + 63) / 64;
  u4 raw[Z ? NV : 1];                    // values: 16-byte pieces lane, lane + 64, ... of the block
  h4 af[Z ? 1 : RB / 16];                // keys: fragments of token w0 + r
  uint32_t chs[kMaxEnt / 4], cbs[kMaxEnt / 4];
};

template <int RB, int Z>
__device__ __forceinline__ void mat_load(MBlock<RB, Z>& m, const MHead& hd, int w0, int lane,
                                         const uint16_t* coef, const uint8_t* idx, const uint8_t* val) {
  const int grp = lane >> 4, r = lane & 15;
  if constexpr (Z == 0) {
#pragma unroll
    for (int s = 0; s < RB / 16; ++s)
      m.af[s] = *reinterpret_cast<const h4*>(coef + (int64_t)w0 * RB + key_index(r, 16 * s + 4 * grp, RB));
  } else {
    const u4* src = reinterpret_cast<const u4*>(coef + (int64_t)w0 * RB);
#pragma unroll
    for (int u = 0; u < MBlock<RB, Z>::NV; ++u) m.raw[u] = src[min(lane + 64 * u, 2 * RB - 1)];
  }
#pragma unroll
  for (int u = 0; u < kMaxEnt / 4; ++u) {
    const uint32_t j = grp + 4u * u;
    m.chs[u] = m.cbs[u] = 0u;
    if (j < hd.rho) {
      m.chs[u] = idx[hd.e0 + j];
      m.cbs[u] = val[(hd.e0 + j) >> 1];
    }
  }
}

// One wave, one 16-token block [w0, w0+16): the rows [a0, a1) of it that
// belong to the sequence whose basis is in LDS are computed, completed with
// their residual channels, rounded once to fp16 and stored.  Keys take the
// basis as the A operand, so a lane ends with 8 consecutive channels of one
// token (row i of tile nt is channel 32 (nt / 2) + 8 (i / 4) + 4 (nt % 2) +
// i % 4); values take the coefficients as A, so a lane ends with 4 consecutive
// tokens of one channel: both store whole 64-byte and longer segments from
// registers.
template <int RB, int Z>
__device__ __forceinline__ void mat_block(MSmem<RB>& sm, const h4 (&bf)[RB <= kMRegRank ? D / 16 : 1][RB / 16],
                                          int wv, int w0, int a0, int a1, int lane,
                                          const MBlock<RB, Z>& m, const MHead& hd, const uint8_t* idx,
                                          const uint8_t* val, uint16_t* out) {
  constexpr int NS = RB / 16;
  constexpr int KROW = MSmem<RB>::KROW, ST = MSmem<RB>::ST;
  const int grp = lane >> 4, r = lane & 15;
  uint8_t* codes = sm.codes[wv];
  const bool any = __any(hd.rho > 0);    // uniform
  wave_lds_sync();                       // the previous block's reads are done
  h4 af[NS];
  if constexpr (Z == 0) {
#pragma unroll
    for (int s = 0; s < NS; ++s) af[s] = m.af[s];
  } else {
#pragma unroll
    for (int u = 0; u < MBlock<RB, Z>::NV; ++u) {
      const int p = lane + 64 * u;
      if (p < 2 * RB) *reinterpret_cast<u4*>(&sm.stage[wv][8 * p + (p >= RB ? 8 : 0)]) = m.raw[u];
    }
  }
  if (any) {
    if constexpr (Z == 0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) *reinterpret_cast<uint2*>(codes + r * KROW + 32 * grp + 8 * u) = make_uint2(0u, 0u);
    } else {
#pragma unroll
      for (int u = 0; u < 2; ++u) *reinterpret_cast<uint4*>(codes + 32 * lane + 16 * u) = make_uint4(0u, 0u, 0u, 0u);
    }
  }
  wave_lds_sync();
  if (any) {                             // the channels of a token are distinct: no two lanes meet
    auto put = [&](uint32_t ch, int q) __attribute__((always_inline)) {
      ch &= D - 1;
      codes[Z == 0 ? r * KROW + ch : ch * 16 + r] = (uint8_t)q;
    };
#pragma unroll
    for (int u = 0; u < kMaxEnt / 4; ++u) {
      const uint32_t j = (uint32_t)grp + 4u * u;
      if (j < hd.rho) put(m.chs[u], entry_code(m.cbs[u], (int64_t)(hd.e0 + j)));
    }
    for (uint32_t j = kMaxEnt + grp; j < hd.rho; j += 4) {   // ranks above 16
      const uint32_t e = hd.e0 + j;
      put(idx[e], entry_code(val[e >> 1], (int64_t)e));
    }
  }
  if constexpr (Z == 1) {
    const uint16_t* st = sm.stage[wv] + (r >> 3) * ST + (r & 7);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const uint16_t* p = st + (16 * s + 4 * grp) * 8;
      af[s] = __builtin_bit_cast(h4, make_uint2(p[0] | ((uint32_t)p[8] << 16), p[16] | ((uint32_t)p[24] << 16)));
    }
  }
  wave_lds_sync();
  // channels without an entry take code 0, so the scale has to be finite here
  const float gs = scale_finite(hd) ? half_bits_to_float((uint16_t)hd.sbits) : 0.f;
  // the product of output tile nt; the basis fragments of wide bases stay in LDS
  auto product = [&](int nt) __attribute__((always_inline)) {
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const h4 b = RB <= kMRegRank ? bf[RB <= kMRegRank ? nt : 0][s] : mat_frag<RB, Z>(sm, nt, s, lane);
      acc = Z == 0 ? __builtin_amdgcn_mfma_f32_16x16x16f16(b, af[s], acc, 0, 0, 0)
                   : __builtin_amdgcn_mfma_f32_16x16x16f16(af[s], b, acc, 0, 0, 0);
    }
    return acc;
  };
  auto code = [](uint32_t w, int j) __attribute__((always_inline)) { return (float)(int8_t)(w >> (8 * j)); };
  if constexpr (Z == 0) {
    const bool mine = w0 + r >= a0 && w0 + r < a1;
    uint16_t* dst = out + (int64_t)w0 * D + (r * D + 8 * grp);
#pragma unroll
    for (int q = 0; q < D / 32; ++q) {
      f4 lo = product(2 * q), hi = product(2 * q + 1);
      if (any) {
        const uint2 w = *reinterpret_cast<const uint2*>(codes + r * KROW + 32 * q + 8 * grp);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          lo[j] += gs * code(w.x, j);
          hi[j] += gs * code(w.y, j);
        }
      }
      if (mine)
        *reinterpret_cast<uint4*>(dst + 32 * q) = make_uint4(pack_half2(lo[0], lo[1]), pack_half2(lo[2], lo[3]),
                                                             pack_half2(hi[0], hi[1]), pack_half2(hi[2], hi[3]));
    }
  } else {
    const bool full = a0 == w0 && a1 == w0 + 16;
    float g4[4];                         // scales of tokens 4 grp ..
#pragma unroll
    for (int j = 0; j < 4; ++j) g4[j] = __shfl(gs, 4 * grp + j);
#pragma unroll
    for (int nt = 0; nt < D / 16; ++nt) {
      const int c = 16 * nt + r;
      f4 x = product(nt);
      if (any) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(codes + 16 * c + 4 * grp);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] += g4[j] * code(w, j);
      }
      uint16_t* dst = out + (int64_t)w0 * D + (c * 16 + 4 * grp);
      if (full) {
        *reinterpret_cast<uint2*>(dst) = make_uint2(pack_half2(x[0], x[1]), pack_half2(x[2], x[3]));
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int t = w0 + 4 * grp + j;
          if (t >= a0 && t < a1) dst[j] = __builtin_bit_cast(uint16_t, (_Float16)x[j]);
        }
      }
    }
  }
}

// Entries of a block's tokens whose scale is not finite, which mat_block leaves
// out: each one's product again (all that matters of it is whether it is finite),
// the sum stored over what the wave stored before.  Lanes share a token's
// entries as in MBlock.
template <int RB, int Z>
__device__ __forceinline__ void mat_odd(const MSmem<RB>& sm, int w0, int lane, const MHead& hd, const uint16_t* coef,
                                        const uint8_t* idx, const uint8_t* val, uint16_t* out) {
  const int r = lane & 15;
  if (scale_finite(hd)) return;
  const float gs = half_bits_to_float((uint16_t)hd.sbits);
  for (uint32_t j = lane >> 4; j < hd.rho; j += 4) {
    const uint32_t e = hd.e0 + j;
    const int c = idx[e] & (D - 1);
    float x = 0.f;
#pragma unroll 1
    for (int k = 0; k < RB; ++k)
      x += half_bits_to_float(coef[(int64_t)w0 * RB + (Z == 0 ? key_index(r, k, RB) : value_index(r, k, RB))]) *
           half_bits_to_float(sm.bt[c * MSmem<RB>::BT + k]);
    x += gs * (float)entry_code(val[e >> 1], (int64_t)e);
    out[(int64_t)w0 * D + (Z == 0 ? r * D + c : c * 16 + r)] = __builtin_bit_cast(uint16_t, (_Float16)x);
  }
}

// Blocks i0..i1 of the workgroup (16 tokens from g0 + 16 i), dealt to the waves
// in turn; block i's coefficients and entries are loaded one turn ahead and its
// offsets, which the entries wait for, two.
template <int RB, int Z>
__device__ __forceinline__ void mat_rows(const MatArgs& a, MSmem<RB>& sm, int wv, int lane, int g0, int s0, int s1,
                                         const uint16_t* coef, const uint32_t* off, const uint16_t* scale,
                                         const uint8_t* idx, const uint8_t* val, uint16_t* out) {
  const int r = lane & 15;
  const int b0 = (s0 - g0) >> 4, b1 = (s1 - 1 - g0) >> 4;
  const int first = b0 + ((wv - b0) % kMW + kMW) % kMW;
  int i = first;
  if (i > b1) return;
  h4 bf[RB <= kMRegRank ? D / 16 : 1][RB / 16];
  if constexpr (RB <= kMRegRank) {
#pragma unroll
    for (int nt = 0; nt < D / 16; ++nt)
#pragma unroll
      for (int s = 0; s < RB / 16; ++s) bf[nt][s] = mat_frag<RB, Z>(sm, nt, s, lane);
  }
  // past the wave's last block the loads repeat it
  const int last = i + (b1 - i) / kMW * kMW;
  auto tok = [&](int b) __attribute__((always_inline)) { return g0 + 16 * min(b, last); };
  bool odd = false;                      // uniform
  MHead h0, h1;
  MBlock<RB, Z> cur;
  mat_head(h0, a, tok(i), s0, s1, r, off, scale);
  mat_head(h1, a, tok(i + kMW), s0, s1, r, off, scale);
  mat_load<RB, Z>(cur, h0, tok(i), lane, coef, idx, val);
  for (; i <= b1; i += kMW) {
    MHead h2;
    MBlock<RB, Z> nxt;
    mat_head(h2, a, tok(i + 2 * kMW), s0, s1, r, off, scale);
    mat_load<RB, Z>(nxt, h1, tok(i + kMW), lane, coef, idx, val);
    const int w0 = g0 + 16 * i;
    mat_block<RB, Z>(sm, bf, wv, w0, max(s0, w0), min(s1, w0 + 16), lane, cur, h0, idx, val, out);
    odd |= __any(h0.rho > 0 && !scale_finite(h0));
    cur = nxt;
    h0 = h1;
    h1 = h2;
  }
  if (odd) {                             // behind the loop, whose registers are full: the lane is taken anew
    const int ln = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    for (i = first; i <= b1; i += kMW) {
      mat_head(h0, a, g0 + 16 * i, s0, s1, ln & 15, off, scale);
      mat_odd<RB, Z>(sm, g0 + 16 * i, ln, h0, coef, idx, val, out);
    }
  }
}

// grid (ceil(T16 / tokens per workgroup), Hkv, 2)
template <int RB>
__global__ __launch_bounds__(kMW * 64, RB <= 64 ? 4 : RB < 128 ? 3 : 2) void materialize_kernel(const MatArgs a) {
  constexpr int BT = MSmem<RB>::BT;
  __shared__ MSmem<RB> sm;
  const int h = blockIdx.y, z = blockIdx.z;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int T = (int)a.T;                // below 2^31: cu_seqlens are 32-bit
  const int g0 = blockIdx.x * a.wg_tokens;                // a multiple of 16
  const int gend = (int)min((int64_t)g0 + a.wg_tokens, a.T);
  const int64_t slab = (int64_t)z * a.n_kv_heads + h;
  const uint16_t* coef = (z ? a.coef_v : a.coef_k) + (int64_t)h * a.T16 * RB;
  const uint32_t* off = a.off + (int64_t)h * (a.T + 1);
  const uint8_t* idx = a.idx + slab * a.res_stride;
  const uint8_t* val = a.val + slab * (a.res_stride / 2);
  const uint16_t* scale = a.scale + slab * a.T;
  uint16_t* out = z ? a.v_out + (int64_t)h * a.T16 * D : a.k_out + (int64_t)h * a.T * D;

  if (g0 < T) {
    for (int b = seq_of(a.cu, a.batch, g0); b < a.batch && a.cu[b] < gend; ++b) {
      const int s0 = max(g0, a.cu[b]), s1 = min(gend, a.cu[b + 1]);
      if (s1 <= s0) continue;            // empty sequence (uniform)
      __syncthreads();                   // every wave is done with the previous basis
      const uint16_t* src = a.basis + (int64_t)b * a.basis_b_stride + (int64_t)(h * 2 + z) * RB * D;
      for (int e = threadIdx.x; e < RB * (D / 8); e += kMW * 64) {
        const int k = e % RB, c8 = e / RB;   // lanes along k: the 2-byte writes of a wave are contiguous
        const uint4 w = *reinterpret_cast<const uint4*>(src + (int64_t)k * D + 8 * c8);
        const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int u = 0; u < 8; ++u)
          sm.bt[(8 * c8 + u) * BT + k] = (uint16_t)(ws[u >> 1] >> (16 * (u & 1)));
      }
      __syncthreads();
      if (z == 0)
        mat_rows<RB, 0>(a, sm, wv, lane, g0, s0, s1, coef, off, scale, idx, val, out);
      else
        mat_rows<RB, 1>(a, sm, wv, lane, g0, s0, s1, coef, off, scale, idx, val, out);
    }
  }
  // value padding of the last block: tokens [T, T16) are zero
  if (z == 1 && T < a.T16 && wv == 0) {
    const int64_t wl = a.T16 - 16;
    if (wl >= g0 && wl < (int64_t)g0 + a.wg_tokens) {
      for (int c = lane; c < D; c += 64) {
        uint16_t* dst = out + ((wl >> 4) * D + c) * 16;
        for (int64_t tt = a.T; tt < wl + 16; ++tt) dst[tt - wl] = 0;
      }
    }
  }
}

template <int RB>
hipError_t launch_mat(const MatArgs& in, hipStream_t s) {
  MatArgs a = in;
  // Each wave takes kMBlocks blocks, fewer where that would leave the chip's
  // kMWaves resident waves idle: staging the basis then costs less than idle waves.
  const int64_t blocks = a.T16 / 16 * a.n_kv_heads * 2;
  a.wg_tokens = 16 * kMW * (int32_t)max((int64_t)1, min((int64_t)kMBlocks, blocks / kMWaves));
  const unsigned nb = (unsigned)((a.T16 + a.wg_tokens - 1) / a.wg_tokens);
  hipLaunchKernelGGL(materialize_kernel<RB>, dim3(nb, a.n_kv_heads, 2), dim3(kMW * 64), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_materialize(const MatArgs& a, hipStream_t s) {
  if (a.T16 <= 0) return hipSuccess;
  switch (a.rb) {
    case 16: return launch_mat<16>(a, s);
    case 32: return launch_mat<32>(a, s);
    case 48: return launch_mat<48>(a, s);
    case 64: return launch_mat<64>(a, s);
    case 80: return launch_mat<80>(a, s);
    case 96: return launch_mat<96>(a, s);
    case 112: return launch_mat<112>(a, s);
    case 128: return launch_mat<128>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace dwkv
