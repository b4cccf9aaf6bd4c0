// Float64 reductions (loss, gradient norm, out-of-band data energy), the
// per-frequency power iteration for the largest singular value of the kernel, and
// the small helpers: the reciprocity average (z + z^T) / 2, per-frequency maxima of
// D_k, the list of every source.  Every sum runs in a fixed order (no atomics), so
// results are bitwise reproducible run to run.
#include <algorithm>

#include "device_common.h"
#include "mdd_internal.h"

namespace mdd {
namespace {

constexpr int RED_THREADS = 1024;

// loss = scale * sum(loss partials) + sum_b oob[idx[b]] (oob[b] for staged data, every
// source's for the full gradient, idx NULL); gnorm2 = sum(gnorm partials).
// The per-source constants are gathered by one thread each (no serial chain of
// dependent loads) and added in batch order.
__global__ __launch_bounds__(RED_THREADS) void k_reduce(ReduceArgs a) {
  __shared__ double red[RED_THREADS / 64];
  __shared__ double s_oob[NB_LIMIT];
  if (threadIdx.x < a.nb) {
    double o = 0.0;
    if (a.oob) {
      const int s = a.idx[threadIdx.x];
      if (s >= 0 && s < a.ns) o = a.oob[a.oob_pos ? threadIdx.x : s];
    }
    s_oob[threadIdx.x] = o;
  }
  const double l = block_fixed_sum<RED_THREADS>(a.loss_part, a.n_loss, red);
  const double g = block_fixed_sum<RED_THREADS>(a.gn_part, a.n_gn, red);
  const double all = a.oob && !a.idx ? block_fixed_sum<RED_THREADS>(a.oob, a.ns, red) : 0.0;
  if (threadIdx.x == 0) {
    double o = all;
    for (int b = 0; b < a.nb; ++b) o += s_oob[b];
    if (a.loss_out) a.loss_out[0] = l * a.loss_scale + o;
    if (a.gnorm2_out) a.gnorm2_out[0] = g;
  }
}

// First level of a two-level sum for long partial arrays: block j of row y adds
// slice j of array y (y = 0: loss partials, 1: gradient-norm partials) in a fixed
// order.  The second level is k_reduce over the 2 * RED_SLICES results.
constexpr int RED_SLICES = 256;
__global__ __launch_bounds__(256) void k_presum(const double* loss_part, int n_loss, const double* gn_part,
                                                int n_gn, double* stage) {
  __shared__ double red[4];
  const double* p = blockIdx.y == 0 ? loss_part : gn_part;
  const int n = blockIdx.y == 0 ? n_loss : n_gn;
  const int per = (n + RED_SLICES - 1) / RED_SLICES;
  const int lo = min(n, (int)blockIdx.x * per), hi = min(n, lo + per);
  const double v = block_fixed_sum<256>(p + lo, hi - lo, red);
  if (threadIdx.x == 0) stage[blockIdx.y * RED_SLICES + blockIdx.x] = v;
}

__global__ void k_row_sum(const double* part, int rows, int cols, double scale, double* out) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < rows) {
    double s = 0.0;
    for (int c = 0; c < cols; ++c) s += part[(size_t)r * cols + c];
    out[r] = s * scale;
  }
}

// Sum of one double per lane over the wavefront, in every lane: rotations within 16 lanes,
// then the four rows' sums through scalar registers (no LDS traffic).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const int2 x = __builtin_bit_cast(int2, v);
  int2 y;
  y.x = __builtin_amdgcn_update_dpp(0, x.x, CTRL, 0xf, 0xf, false);
  y.y = __builtin_amdgcn_update_dpp(0, x.y, CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, y);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  const int2 x = __builtin_bit_cast(int2, v);
  int2 y;
  y.x = __builtin_amdgcn_readlane(x.x, lane);
  y.y = __builtin_amdgcn_readlane(x.y, lane);
  return __builtin_bit_cast(double, y);
}
__device__ __forceinline__ double row16_sum(double v) {  // in every lane of each 16
  v += dpp_move<0x128>(v);  // row_ror 8, 4, 2, 1
  v += dpp_move<0x124>(v);
  v += dpp_move<0x122>(v);
  v += dpp_move<0x121>(v);
  return v;
}
__device__ __forceinline__ double wave_sum_all(double v) {
  v = row16_sum(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
// a + b with halves (HALF 32) or odd and even 16-lane rows (HALF 16) exchanged between the
// two: the lower half (the even rows) of the result sums a over the exchanged pairs of
// lanes, the upper half (the odd rows) sums b.
template <int HALF>
__device__ __forceinline__ double swap_add(double a, double b) {
  const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
  uint2 p, q;
  if constexpr (HALF == 32) {
    const auto lo = __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false);
    p = make_uint2(lo[0], hi[0]);
    q = make_uint2(lo[1], hi[1]);
  } else {
    const auto lo = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    p = make_uint2(lo[0], hi[0]);
    q = make_uint2(lo[1], hi[1]);
  }
  return __builtin_bit_cast(double, p) + __builtin_bit_cast(double, q);
}
// Sums over the wavefront of two complex values at once: the four parts share the steps.
__device__ __forceinline__ void wave_sum_pair(double2& a, double2& b) {
  const double v = row16_sum(swap_add<16>(swap_add<32>(a.x, a.y), swap_add<32>(b.x, b.y)));
  a = make_double2(lane_value(v, 0), lane_value(v, 32));
  b = make_double2(lane_value(v, 16), lane_value(v, 48));
}

// One power iteration on D_k^H D_k (all ns sources), float64: the workgroup of row group p
// of frequency k normalises v = sum of the previous iteration's group partials (or the
// start vector), and for each of its rows s forms y_s = D_k[s, :] v and, the row still in
// registers, adds conj(D_k[s, :]) y_s to its partial of z = D_k^H D_k v.  The last
// iteration writes the group's part of the Rayleigh quotient ||D_k v||^2 instead.
//
// Bound by the bytes of D_k, which is read once per iteration, by P workgroups: 86 MB in
// 20 us at 201 x 201 and 257 bins (4.3 TB/s, from the last-level cache), 188 MB in 38 us at
// 301 x 301.  Before, one workgroup per frequency read D_k twice an iteration and reduced
// row by row: 129 us at the first size.  Two rows share the steps of their sums
// (wave_sum_pair), the row base is a scalar, and two groups of rows are in flight.
//
// SPLIT: the row is spread over the workgroup's wavefronts (more than 512 receivers) and
// each pair of rows is reduced across them through LDS; otherwise every wavefront holds
// whole rows, and the wavefronts' partials are added once at the end.
template <int MQ, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? 512 : 256) void k_sigma_pass(const float2* Df, int ns, int nr, int nrp,
                                                                  int P, int first, int last, const double2* zin,
                                                                  double2* zout, double* lamp) {
  constexpr int RB = 2;                            // rows per group, two groups in flight
  extern __shared__ double2 s_z[];                 // !SPLIT: [wavefronts][MQ * 128]
  __shared__ double2 s_y[2][RB][8];
  __shared__ double s_n[8];
  const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int total = gridDim.x, bid = blockIdx.x, full = (total / 8) * 8;
  const int logical = bid < full ? (bid % 8) * (total / 8) + bid / 8 : bid;  // one XCD per frequency
  const int k = logical / P, p = logical % P;
  const int npair = nrp / 2, q0 = (SPLIT ? wave * MQ * 64 : 0) + lane;
  const char* D = reinterpret_cast<const char*>(Df) + (long long)k * ns * nrp * 8;

  const int i0 = (int)((long long)ns * p / P), i1 = (int)((long long)ns * (p + 1) / P);
  const int stride = SPLIT ? RB : RB * nw;
  const int ifirst = i0 + (SPLIT ? 0 : RB * wave);
  unsigned qoff[MQ];                               // byte offsets of the lane's pairs in a row
#pragma unroll
  for (int m = 0; m < MQ; ++m) qoff[m] = 16u * min(q0 + 64 * m, npair - 1);
  float4 d0[RB][MQ], d1[RB][MQ];
  auto load_rows = [&](float4 (&d)[RB][MQ], int i) {
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const char* row = D + (long long)min(i + b, i1 - 1) * nrp * 8;
#pragma unroll
      for (int m = 0; m < MQ; ++m) d[b][m] = *reinterpret_cast<const float4*>(row + qoff[m]);
    }
  };
  load_rows(d0, ifirst);                           // in flight while v is formed
  load_rows(d1, ifirst + stride);

  // v: receivers 2 q, 2 q + 1 for q = q0 + 64 m (zero past nr).  The group partials are
  // requested GB at a time and added in group order.
  double2 v[MQ][2], z[MQ][2];
#pragma unroll
  for (int m = 0; m < MQ; ++m)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 2 * (q0 + 64 * m) + h;
      v[m][h] = z[m][h] = make_double2(0.0, 0.0);
      if (first && r < nr)                         // deterministic, non-degenerate start
        v[m][h] = make_double2(1.0 + 0.25 * (double)((r * 37) % 11), 0.1 * (double)((r * 17) % 7));
    }
  if (!first) {
    constexpr int GB = MQ <= 2 ? 4 : 2;
    const double2* part = zin + (long long)k * P * nr;
#pragma unroll 1
    for (int g0 = 0; g0 < P; g0 += GB) {
      double2 t[GB][MQ][2];
#pragma unroll
      for (int g = 0; g < GB; ++g)
#pragma unroll
        for (int m = 0; m < MQ; ++m)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            t[g][m][h] = part[(long long)min(g0 + g, P - 1) * nr + min(2 * (q0 + 64 * m) + h, nr - 1)];
#pragma unroll
      for (int g = 0; g < GB; ++g)
#pragma unroll
        for (int m = 0; m < MQ; ++m)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            if (g0 + g < P && 2 * (q0 + 64 * m) + h < nr) {
              v[m][h].x += t[g][m][h].x;
              v[m][h].y += t[g][m][h].y;
            }
    }
  }
  double n2 = 0.0;
#pragma unroll
  for (int m = 0; m < MQ; ++m)
#pragma unroll
    for (int h = 0; h < 2; ++h) n2 += v[m][h].x * v[m][h].x + v[m][h].y * v[m][h].y;
  n2 = wave_sum_all(n2);
  if constexpr (SPLIT) {
    if (lane == 0) s_n[wave] = n2;
    __syncthreads();
    n2 = 0.0;
    for (int w = 0; w < nw; ++w) n2 += s_n[w];
    __syncthreads();
  }
  const double inv = n2 > 0.0 ? 1.0 / sqrt(n2) : 0.0;
#pragma unroll
  for (int m = 0; m < MQ; ++m)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v[m][h].x *= inv;
      v[m][h].y *= inv;
    }

  double lam = 0.0;
  auto group = [&](int i, int par, float4 (&d)[RB][MQ]) {
    double2 y[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      double re = 0.0, im = 0.0;
#pragma unroll
      for (int m = 0; m < MQ; ++m) {
        const double a0 = d[b][m].x, b0 = d[b][m].y, a1 = d[b][m].z, b1 = d[b][m].w;
        re += a0 * v[m][0].x - b0 * v[m][0].y;
        im += a0 * v[m][0].y + b0 * v[m][0].x;
        re += a1 * v[m][1].x - b1 * v[m][1].y;
        im += a1 * v[m][1].y + b1 * v[m][1].x;
      }
      y[b] = make_double2(re, im);
    }
    wave_sum_pair(y[0], y[1]);
    if constexpr (SPLIT) {
      if (lane == 0)
        for (int b = 0; b < RB; ++b) s_y[par][b][wave] = y[b];
      __syncthreads();  // the other buffer (par ^ 1) is free again after this barrier
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        y[b] = make_double2(0.0, 0.0);
        for (int w = 0; w < nw; ++w) {
          y[b].x += s_y[par][b][w].x;
          y[b].y += s_y[par][b][w].y;
        }
      }
    }
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      if constexpr (MQ > 2) {  // converted again: the float64 values would take the registers
#pragma unroll                 // of the rows in flight
        for (int m = 0; m < MQ; ++m)
          asm volatile("" : "+v"(d[b][m].x), "+v"(d[b][m].y), "+v"(d[b][m].z), "+v"(d[b][m].w));
      }
      if (i + b >= i1) y[b] = make_double2(0.0, 0.0);
      lam += y[b].x * y[b].x + y[b].y * y[b].y;
#pragma unroll
      for (int m = 0; m < MQ; ++m) {
        const double a0 = d[b][m].x, b0 = d[b][m].y, a1 = d[b][m].z, b1 = d[b][m].w;
        z[m][0].x += a0 * y[b].x + b0 * y[b].y;
        z[m][0].y += a0 * y[b].y - b0 * y[b].x;
        z[m][1].x += a1 * y[b].x + b1 * y[b].y;
        z[m][1].y += a1 * y[b].y - b1 * y[b].x;
      }
    }
    load_rows(d, i + 2 * stride);
  };
#pragma unroll 1
  for (int i = ifirst; i < i1; i += 2 * stride) {
    group(i, 0, d0);
    if (i + stride >= i1) break;
    group(i + stride, 1, d1);
  }

  if (last) {
    if constexpr (!SPLIT) {
      if (lane == 0) s_n[wave] = lam;
      __syncthreads();
      lam = 0.0;
      for (int w = 0; w < nw; ++w) lam += s_n[w];
    }
    if (tid == 0) lamp[(long long)k * P + p] = lam;
    return;
  }
  double2* out = zout + ((long long)k * P + p) * nr;
  if constexpr (SPLIT) {
#pragma unroll
    for (int m = 0; m < MQ; ++m)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = 2 * (q0 + 64 * m) + h;
        if (r < nr) out[r] = z[m][h];
      }
  } else {
#pragma unroll
    for (int m = 0; m < MQ; ++m)
#pragma unroll
      for (int h = 0; h < 2; ++h) s_z[wave * MQ * 128 + 2 * (lane + 64 * m) + h] = z[m][h];
    __syncthreads();
    for (int r = tid; r < nr; r += blockDim.x) {
      double2 x = s_z[r];
      for (int w = 1; w < nw; ++w) {
        const double2 t = s_z[w * MQ * 128 + r];
        x.x += t.x;
        x.y += t.y;
      }
      out[r] = x;
    }
  }
}

// Largest |Re| or |Im| of D_k over all sources and receivers, per frequency (the fp16 split
// form scales D_{b,k} by a power of two derived from it): of the first `count` entries of
// each frequency's block (blocks `stride` entries apart, both even).  One workgroup per
// frequency, whose memory latency is what bounds it on a staged batch: sixteen wavefronts
// with four 16-byte loads in flight each (48 rows of 400, 200 bins: with four wavefronts
// and one 8-byte load 21 us, now 8 us).  A maximum does not depend on the order.
constexpr int ABSMAX_THREADS = 1024;
__global__ __launch_bounds__(ABSMAX_THREADS) void k_freq_absmax(const float2* Df, long long count,
                                                                long long stride, float* out) {
  const float4* x = reinterpret_cast<const float4*>(Df + (long long)blockIdx.x * stride);
  const long long n = count / 2;
  auto amax = [](float4 v) { return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))); };
  float m = 0.f;
  long long i = threadIdx.x;
  for (; i + 3 * ABSMAX_THREADS < n; i += 4 * ABSMAX_THREADS) {
    const float4 a = x[i], b = x[i + ABSMAX_THREADS], c = x[i + 2 * ABSMAX_THREADS], d = x[i + 3 * ABSMAX_THREADS];
    m = fmaxf(fmaxf(m, fmaxf(amax(a), amax(b))), fmaxf(amax(c), amax(d)));
  }
  for (; i < n; i += ABSMAX_THREADS) m = fmaxf(m, amax(x[i]));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  __shared__ float s_m[ABSMAX_THREADS / 64];
  if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < ABSMAX_THREADS / 64; ++w) m = fmaxf(m, s_m[w]);
    out[blockIdx.x] = m;
  }
}

// C_r z = (z + z^T) / 2 over the first two axes of [n][n][nt]: the workgroup of
// pair (r, vs), r <= vs, reads both traces and writes the average to both, so the
// call may run in place.
__global__ __launch_bounds__(256) void k_reciprocity(const float* z, float* out, int n, int nt) {
  const int vs = blockIdx.x, r = blockIdx.y;
  if (vs < r) return;
  const long long ta = ((long long)r * n + vs) * nt, tb = ((long long)vs * n + r) * nt;
  for (int i = threadIdx.x * 4; i < nt; i += 256 * 4) {
    const float4 a = *reinterpret_cast<const float4*>(z + ta + i);
    const float4 b = *reinterpret_cast<const float4*>(z + tb + i);
    const float4 m = make_float4((a.x + b.x) * 0.5f, (a.y + b.y) * 0.5f, (a.z + b.z) * 0.5f,
                                 (a.w + b.w) * 0.5f);
    *reinterpret_cast<float4*>(out + ta + i) = m;
    *reinterpret_cast<float4*>(out + tb + i) = m;
  }
}

// C_r on blocked spectra (nr = nvs = n): X(r, vs, k) <- (X(r, vs, k) + X(vs, r, k)) / 2 for
// every retained bin k, which equals the spectra of C_r applied to the traces (the time
// transform acts on each trace alone).  Element (r, vs, k) sits at
// r * s_row + (vs / 16) * s_cb + k * 16 + vs % 16.  Workgroup (pair, k) takes the 16 x 16
// tiles (I, J) and (J, I), I <= J, of bin k: both are read, transposed through LDS, and
// the average is written to both (a diagonal tile is its own mirror).  Receivers and
// columns at or beyond n are left alone.
__global__ __launch_bounds__(256) void k_spec_reciprocity(float2* X, int n, long long s_row,
                                                          long long s_cb, int ntile) {
  __shared__ float2 s_b[16][17];
  int p = blockIdx.x, I = 0;
  while (p >= ntile - I) {  // pair index -> (I, J), I <= J, row-major over the triangle
    p -= ntile - I;
    ++I;
  }
  const int J = I + p;
  const int k = blockIdx.y;
  const int i = threadIdx.x >> 4, j = threadIdx.x & 15;
  const int ra = I * 16 + i, ca = J * 16 + j;  // element of tile (I, J)
  const int rb = J * 16 + i, cb = I * 16 + j;  // element of tile (J, I)
  const bool oka = ra < n && ca < n, okb = rb < n && cb < n;
  float2* pa = X + (oka ? ra : 0) * s_row + (long long)J * s_cb + (long long)k * 16 + j;
  float2* pb = X + (okb ? rb : 0) * s_row + (long long)I * s_cb + (long long)k * 16 + j;
  const float2 a = oka ? *pa : make_float2(0.f, 0.f);
  const float2 b = okb ? *pb : make_float2(0.f, 0.f);
  s_b[i][j] = b;
  __syncthreads();
  // mirror of (ra, ca) = (I*16 + i, J*16 + j) is (J*16 + j, I*16 + i): element (j, i) of tile (J, I)
  const float2 m = s_b[j][i];
  const float2 v = make_float2((a.x + m.x) * 0.5f, (a.y + m.y) * 0.5f);
  __syncthreads();
  s_b[j][i] = v;  // the same value, as seen from tile (J, I)
  __syncthreads();
  if (oka) *pa = v;
  if (okb && I != J) *pb = s_b[i][j];
}

// out[i] = i: the list of every source, batched in order by the full gradient.
__global__ void k_iota(int32_t* out, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = i;
}

}  // namespace

hipError_t launch_reduce(const ReduceArgs& a, hipStream_t s) {
  if (a.stage && (a.n_loss > RED_TWO_LEVEL || a.n_gn > RED_TWO_LEVEL)) {
    hipLaunchKernelGGL(k_presum, dim3(RED_SLICES, 2), dim3(256), 0, s, a.loss_part, a.n_loss,
                       a.gn_part, a.n_gn, a.stage);
    ReduceArgs b = a;
    b.loss_part = a.stage;
    b.n_loss = a.n_loss > 0 ? RED_SLICES : 0;
    b.gn_part = a.stage + RED_SLICES;
    b.n_gn = a.n_gn > 0 ? RED_SLICES : 0;
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(RED_THREADS), 0, s, b);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(RED_THREADS), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_reciprocity(const float* z, float* out, int n, int nt, hipStream_t s) {
  hipLaunchKernelGGL(k_reciprocity, dim3(n, n), dim3(256), 0, s, z, out, n, nt);
  return hipGetLastError();
}

hipError_t launch_spec_reciprocity(float2* X, int n, int nf, long long s_row, long long s_cb,
                                   hipStream_t s) {
  const int ntile = (n + 15) / 16;
  const int npair = ntile * (ntile + 1) / 2;
  if (n < 1 || nf < 1 || nf > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_spec_reciprocity, dim3(npair, nf), dim3(256), 0, s, X, n, s_row, s_cb, ntile);
  return hipGetLastError();
}

hipError_t launch_iota(int32_t* out, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_iota, dim3((n + 255) / 256), dim3(256), 0, s, out, n);
  return hipGetLastError();
}

hipError_t launch_freq_absmax(const float2* Df, int nf, long long count, long long stride,
                              float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_freq_absmax, dim3(nf), dim3(ABSMAX_THREADS), 0, s, Df, count, stride, out);
  return hipGetLastError();
}

hipError_t launch_row_sum(const double* part, int rows, int cols, double scale, double* out,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_row_sum, dim3((rows + 255) / 256), dim3(256), 0, s, part, rows, cols, scale,
                     out);
  return hipGetLastError();
}

int sigma_groups(int nf, int ns, int nr, int nvb) {
  const int want = (3 * 256 + nf / 2) / nf;        // about three workgroups per CU,
  const int most = (ns + 15) / 16;                 // at least 16 rows each,
  const int room = std::min(4 * nvb - 1, 4 * nr);  // and 32 P nr + 8 P <= 128 nr nvb bytes
  return std::max(1, std::min(want, std::min(most, room)));
}

hipError_t launch_sigma(const float2* Df, int nf, int ns, int nr, int nrp, int iters, int P,
                        void* scratch, double* lam_out, hipStream_t s) {
  double2* z[2] = {static_cast<double2*>(scratch), static_cast<double2*>(scratch) + (size_t)nf * P * nr};
  double* lamp = reinterpret_cast<double*>(z[1] + (size_t)nf * P * nr);
  const int npair = nrp / 2;
  auto go = [&](auto kernel, int nw, size_t sm) {
    for (int it = 0; it < iters; ++it) {
      hipLaunchKernelGGL(kernel, dim3(nf * P), dim3(64 * nw), sm, s, Df, ns, nr, nrp, P, it == 0,
                         it == iters - 1, z[(it + 1) & 1], z[it & 1], lamp);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  };
  auto whole = [&](auto kernel, int mq) { return go(kernel, 4, sizeof(double2) * 4 * mq * 128); };
  hipError_t e;
  if (npair <= 64) e = whole(k_sigma_pass<1, false>, 1);
  else if (npair <= 128) e = whole(k_sigma_pass<2, false>, 2);
  else if (npair <= 192) e = whole(k_sigma_pass<3, false>, 3);
  else if (npair <= 256) e = whole(k_sigma_pass<4, false>, 4);
  else e = go(k_sigma_pass<4, true>, (npair + 255) / 256, 0);
  return e == hipSuccess ? launch_row_sum(lamp, nf, P, 1.0, lam_out, s) : e;
}

}  // namespace mdd
