// Online basis initialization (Sec. 3): a window's shared bases from a small
// randomized sketch of its prefill keys and values, per head and per Z.
// Y = Omega X, with X the window's prefill vectors of one head ((w T_b) x d)
// and Omega (r_b x (w T_b)) a caller-drawn random matrix; the basis is the
// Gram-Schmidt orthonormalization of Y's rows, rounded to fp16.
//
// Three launches:
//  1. split-K sketch partials on v_mfma_f64_16x16x4_f64 (fp16 products are
//     exact in float64), one workgroup per (4096-row chunk, head, Z),
//     each of its 4 waves owning 32 channels and every row of Omega.  Bound by
//     the float64 matrix rate where the workgroups fill the chip: the 51.5 GFLOP
//     of a 4 x 64K window (r_b 48, 8 heads; 1024 workgroups) take 0.91 ms, 57
//     TFLOP/s of the published 78.6, the matrix cores busy 77 % of the cycles; one
//     thread per channel on float64 FMAs, converting Omega's row in every thread,
//     took 6.1 ms.  Below a workgroup for each of the 256 compute units (4 x 16K
//     tokens of 8 heads) the call takes 265 to 290 us from 4096 rows on: one
//     chunk's rows in turn, and the Gram-Schmidt.
//  2. the chunk partials summed in chunk order, one thread per element (50 MB
//     read once in 10 us; inside the orthonormalization one compute unit would
//     pull each head's share).
//  3. the orthonormalization, one 16-wave workgroup per (head, Z): modified
//     Gram-Schmidt from the left, every later row updated as soon as a row is
//     final, rows dealt to the waves in turn.  Bound by its serial chain
//     (r_b steps of a normalization, a barrier and a dot product): 40 us at
//     r_b 48, against 1.1 ms for one wave that also summed the partials.
#include "entry.h"
#include "internal.h"

namespace dwkv {
namespace {

constexpr int D = kHeadDim;
constexpr int kSkWaves = 4;                     // waves of a partial workgroup
constexpr int kSkRowsPerChunk = 4096;           // sketch rows of a partial (the workspace holds one per 4096)
constexpr int kSkU = 8;                         // 4-row MFMA steps per load group
constexpr int kSkGroup = 4 * kSkU;              // rows per load group
constexpr int kOrthWaves = 16;

typedef double d4 __attribute__((ext_vector_type(4)));

// Loads of one group of kSkGroup rows: step u of lane (r, kk) is row 4 u + kk.
template <int NS>
struct SkRows {
  uint32_t x[kSkU];                             // channels 2 r, 2 r + 1 of the wave's 32
  uint32_t om[kSkU][NS % 2 ? NS : NS / 2];      // Omega entries NS r .. NS r + NS - 1
};

template <int NS, bool EDGE>
__device__ __forceinline__ void sk_load(SkRows<NS>& f, const uint16_t* x, const uint16_t* om, int row0, int rows,
                                        int64_t xstride, int kk) {
#pragma unroll
  for (int u = 0; u < kSkU; ++u) {
    const int row = row0 + 4 * u + kk;
    const int rc = EDGE ? min(row, rows - 1) : row;
    const uint16_t* o = om + (int64_t)rc * (16 * NS);
    f.x[u] = *reinterpret_cast<const uint32_t*>(x + rc * xstride);
    if constexpr (NS % 2) {
#pragma unroll
      for (int s = 0; s < NS; ++s) f.om[u][s] = o[s];
    } else {
#pragma unroll
      for (int s = 0; s < NS / 2; ++s) f.om[u][s] = reinterpret_cast<const uint32_t*>(o)[s];
    }
    if (EDGE && row >= rows) {                  // rows past the chunk add nothing
      f.x[u] = 0u;
#pragma unroll
      for (int s = 0; s < (NS % 2 ? NS : NS / 2); ++s) f.om[u][s] = 0u;
    }
  }
}

template <int NS>
__device__ __forceinline__ void sk_mma(d4 (&acc)[NS][2], const SkRows<NS>& f) {
#pragma unroll
  for (int u = 0; u < kSkU; ++u) {
    const double b0 = (double)half_bits_to_float((uint16_t)(f.x[u] & 0xffffu));
    const double b1 = (double)half_bits_to_float((uint16_t)(f.x[u] >> 16));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const uint32_t w = NS % 2 ? f.om[u][s] : f.om[u][s / 2] >> (16 * (s & 1));
      const double a = (double)half_bits_to_float((uint16_t)(w & 0xffffu));
      acc[s][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b0, acc[s][0], 0, 0, 0);
      acc[s][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b1, acc[s][1], 0, 0, 0);
    }
  }
}

// grid (chunks, Hkv, 2); a chunk runs over the layers that its rows lie in.  Of
// the MFMA operands, lane (r, kk) = (lane % 16, lane / 16) holds row r (A) or
// column r (B) at depth kk, and the result's rows 4 i + kk of column r.  Operand
// rows and columns are dealt so that a lane's loads are contiguous: A row r of
// tile s is Omega entry NS r + s, B column r of tile c is channel 2 r + c of the
// wave's 32.
template <int RB>
__global__ __launch_bounds__(64 * kSkWaves) void sketch_partial_kernel(const SketchArgs a) {
  constexpr int NS = RB / 16;
  const int chunk = blockIdx.x, h = blockIdx.y, z = blockIdx.z;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r = lane & 15, kk = lane >> 4;
  const int64_t n = a.n_tokens, xstride = (int64_t)a.n_kv_heads * D;
  const int64_t first = (int64_t)chunk * kSkRowsPerChunk, end = min(first + kSkRowsPerChunk, a.w * n);
  d4 acc[NS][2];
#pragma unroll
  for (int s = 0; s < NS; ++s) acc[s][0] = acc[s][1] = d4{0.0, 0.0, 0.0, 0.0};
  for (int64_t row = first; row < end;) {
    const int64_t l = row / n, t0 = row - l * n;
    const int rows = (int)min(end - row, n - t0);
    const uint16_t* x = a.x + ((l * 2 + z) * n + t0) * xstride + (int64_t)h * D + 32 * wv + 2 * r;
    const uint16_t* om = a.omega + row * RB + NS * r;
    const int full = rows / kSkGroup;           // the next group's loads run under this one's products
    SkRows<NS> cur, nxt;
    if (full > 0) sk_load<NS, false>(cur, x, om, 0, rows, xstride, kk);
    for (int g = 0; g + 1 < full; ++g) {
      sk_load<NS, false>(nxt, x, om, (g + 1) * kSkGroup, rows, xstride, kk);
      sk_mma<NS>(acc, cur);
      cur = nxt;
    }
    if (full > 0) sk_mma<NS>(acc, cur);
    if (rows % kSkGroup) {
      sk_load<NS, true>(cur, x, om, full * kSkGroup, rows, xstride, kk);
      sk_mma<NS>(acc, cur);
    }
    row += rows;
  }
  double* out = a.part + (((int64_t)chunk * a.n_kv_heads + h) * 2 + z) * RB * D + 32 * wv + 2 * r;
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<double2*>(out + (int64_t)(NS * (4 * i + kk) + s) * D) = make_double2(acc[s][0][i], acc[s][1][i]);
}

// Y: the chunk partials summed in chunk order, one thread per element.
__global__ __launch_bounds__(256) void sketch_sum_kernel(const SketchArgs a) {
  const int64_t n = (int64_t)a.n_kv_heads * 2 * a.rb * D, e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  double y = 0.0;
#pragma unroll 8
  for (int ch = 0; ch < a.n_chunks; ++ch) y += a.part[ch * n + e];
  a.q[e] = y;
}

// Sum over the wave: DPP inside each row of 16 lanes, then the four rows'
// sums read into scalar registers.  Every lane returns the same bits.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ double lane_d(double v, int l) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, l);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ double wave_sum_d(double v) {
  v += dpp_d<0xB1>(v);                          // quad_perm(1,0,3,2)
  v += dpp_d<0x4E>(v);                          // quad_perm(2,3,0,1)
  v += dpp_d<0x141>(v);                         // row_half_mirror
  v += dpp_d<0x140>(v);                         // row_mirror
  return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}

// grid (Hkv, 2): row i belongs to wave i % 16, lane l owns channels 2l, 2l+1.
// Step i: the owner of row i (by now free of the rows before it) normalizes
// and publishes it, then every wave takes its component out of its later rows
// -- for each row the subtractions of modified Gram-Schmidt, in their order.
// The published row alternates between two buffers, so one barrier per step
// is enough: a wave that writes a buffer again has passed the barrier that
// every reader of its old content reached afterwards.
template <int RB>
__global__ __launch_bounds__(64 * kOrthWaves) void sketch_orth_kernel(const SketchArgs a) {
  constexpr int NR = RB / kOrthWaves;
  __shared__ double2 qrow[2][D / 2];
  __shared__ double nmax[kOrthWaves];
  const int h = blockIdx.x, z = blockIdx.y, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double2* y = reinterpret_cast<const double2*>(a.q + ((int64_t)h * 2 + z) * RB * D);
  uint32_t* bout = reinterpret_cast<uint32_t*>(a.basis + ((int64_t)h * 2 + z) * RB * D);
  double2 v[NR];
  double ymax = 0.0;
#pragma unroll
  for (int j = 0; j < NR; ++j) v[j] = y[(kOrthWaves * j + wv) * (D / 2) + lane];
#pragma unroll
  for (int j = 0; j < NR; ++j) ymax = fmax(ymax, sqrt(wave_sum_d(v[j].x * v[j].x + v[j].y * v[j].y)));
  if (lane == 0) nmax[wv] = ymax;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kOrthWaves; ++w) ymax = fmax(ymax, nmax[w]);
  const double floor_n = 1e-9 * ymax;
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    for (int o = 0; o < kOrthWaves; ++o) {      // row 16 j + o
      const int buf = o & 1;
      if (wv == o) {
        const double n = sqrt(wave_sum_d(v[j].x * v[j].x + v[j].y * v[j].y));
        if (n > floor_n && n > 0.0) {
          v[j].x /= n;
          v[j].y /= n;
        } else {
          v[j] = make_double2(0.0, 0.0);
        }
        qrow[buf][lane] = v[j];
        const uint32_t lo = __builtin_bit_cast(uint16_t, (_Float16)(float)v[j].x);
        const uint32_t hi = __builtin_bit_cast(uint16_t, (_Float16)(float)v[j].y);
        bout[(kOrthWaves * j + o) * (D / 2) + lane] = lo | hi << 16;
      }
      __syncthreads();
      const double2 q = qrow[buf][lane];
#pragma unroll
      for (int k = j; k < NR; ++k) {
        if (k == j && wv <= o) continue;        // rows up to this one are final
        const double dot = wave_sum_d(v[k].x * q.x + v[k].y * q.y);
        v[k].x -= dot * q.x;
        v[k].y -= dot * q.y;
      }
    }
  }
}

template <int RB>
hipError_t launch_sketch_rb(const SketchArgs& a, hipStream_t s) {
  const unsigned n = (unsigned)a.n_kv_heads * 2 * RB * D;
  hipLaunchKernelGGL(sketch_partial_kernel<RB>, dim3(a.n_chunks, a.n_kv_heads, 2), dim3(64 * kSkWaves), 0, s, a);
  hipLaunchKernelGGL(sketch_sum_kernel, dim3((n + 255) / 256), dim3(256), 0, s, a);
  hipLaunchKernelGGL(sketch_orth_kernel<RB>, dim3(a.n_kv_heads, 2), dim3(64 * kOrthWaves), 0, s, a);
  return hipGetLastError();
}

}  // namespace

int sketch_chunks(int64_t rows) { return (int)((rows + kSkRowsPerChunk - 1) / kSkRowsPerChunk); }

hipError_t launch_sketch(const SketchArgs& a, hipStream_t s) {
  switch (a.rb) {
    case 16: return launch_sketch_rb<16>(a, s);
    case 32: return launch_sketch_rb<32>(a, s);
    case 48: return launch_sketch_rb<48>(a, s);
    case 64: return launch_sketch_rb<64>(a, s);
    case 80: return launch_sketch_rb<80>(a, s);
    case 96: return launch_sketch_rb<96>(a, s);
    case 112: return launch_sketch_rb<112>(a, s);
    case 128: return launch_sketch_rb<128>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace dwkv
