// Products for a single virtual source (nvs = 1): at each retained frequency the
// operator's matrix-matrix product reduces to a matrix-vector product (cost analysis,
// Appendix A), so D_b is the only large operand and the work is bound by its bytes.
//
//   k_gemv<GK_FUSED>  res_i = D_{b,k}[i, :] . r_k - U_{b,k}[i]  (float64 loss partials),
//                     g_k += conj(D_{b,k}[i, :]) res_i  over the rows i of the workgroup
//   k_gemv<GK_FWD>    P_k[i] = D_{b,k}[i, :] . r_k  -> batch spectra
//   k_gemv<GK_ADJ>    g_k = sum_i conj(D_{b,k}[i, :]) V_k[i], V from batch spectra
//
// One pass over D_b: each row of D_{b,k} is loaded once into registers, reduced to
// res_i and, still in registers, multiplied into the adjoint sum.  k_gemv gives each row to
// one wavefront; k_gemv_wide, for more than 1664 receivers and where rows are few, to the
// workgroup.  The rows of one frequency are split into P groups (one workgroup each) so that
// the grid covers the chip; with P > 1 the group partials of g_k go to a scratch buffer and
// are added in group order by the trace kernel that transforms them, or (the full gradient)
// by k_gemv_sum.
//
// Layout at nvs = 1 (the trace kernels see one row of nr columns): model and gradient
// spectra hold receiver j at frequency k at ((j / 16) * nf + k) * 16 + j % 16; batch
// spectra hold batch row i at ((i / 16) * nf + k) * 16 + i % 16.  Arithmetic is float32
// on the vector units for every precision setting: the product is bound by D_b's bytes.
#include "device_common.h"
#include "mdd_internal.h"

namespace mdd {
namespace {

constexpr int GV_THREADS = 256;
constexpr int GV_GR = 2;   // k_gemv_wide: rows reduced per workgroup barrier
constexpr int GV_MQ = 13;  // k_gemv: receiver pairs per lane at most

__device__ __forceinline__ float2 wave_sum2(float2 v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    v.x += __shfl_xor(v.x, off, 64);
    v.y += __shfl_xor(v.y, off, 64);
  }
  return v;
}

// g += conj(d) * s for the two complex values of d.
__device__ __forceinline__ void cmac_conj(float4& g, float4 d, float2 s) {
  g.x += d.x * s.x + d.y * s.y;
  g.y += d.x * s.y - d.y * s.x;
  g.z += d.z * s.x + d.w * s.y;
  g.w += d.z * s.y - d.w * s.x;
}

// Adjoint product for receivers 2q, 2q + 1 at frequency k: written over R_k in F (Gout
// NULL), or into Gout, or added to Gout (gacc), in the one-row spectra layout.
__device__ __forceinline__ void store_pair(const GemmArgs& a, int k, int q, float4 v) {
  const int c = 2 * q;
  float4* dst = reinterpret_cast<float4*>(a.Gout ? a.Gout : a.F) +
                ((((long long)(c >> 4) * a.nf + k) * CB + (c & 15)) >> 1);
  if (a.gacc) {
    const float4 o = *dst;
    v.x += o.x;
    v.y += o.y;
    v.z += o.z;
    v.w += o.w;
  }
  *dst = v;
}

template <int KIND, int MQ>
__global__ __launch_bounds__(GV_THREADS) void k_gemv_wide(GemmArgs a) {
  __shared__ float2 s_red[2][GV_GR][GV_THREADS / 64];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // The P groups of one frequency run on one XCD (dispatch is round-robin over the 8).
  const int total = a.nf * a.P;
  const int bid = blockIdx.x;
  const int full = (total / 8) * 8;
  const int logical = bid < full ? (bid % 8) * (total / 8) + bid / 8 : bid;
  const int k = logical / a.P, p = logical % a.P;
  const int rpg = (a.nb + a.P - 1) / a.P;
  const int i0 = p * rpg;
  const int i1 = min(a.nb, i0 + rpg);
  const int npair = a.nrp / 2;  // receiver pairs (2q, 2q + 1), zero-padded to nrp
  const double wk = (k == 0 || 2 * k == a.nt) ? 1.0 : 2.0;

  const float4* D4 = reinterpret_cast<const float4*>(a.Df);
  // Spectra element (column c, frequency k) of the one-row layout, c even -> float4 index.
  auto spec4 = [&](int c) -> long long { return (((long long)(c >> 4) * a.nf + k) * CB + (c & 15)) >> 1; };
  auto spec2 = [&](int c) -> long long { return ((long long)(c >> 4) * a.nf + k) * CB + (c & 15); };

  // Model spectra r_k: pairs q = tid + 256 m (zero beyond the padded receivers).
  float4 rv[MQ];
  float4 gv[MQ];
#pragma unroll
  for (int m = 0; m < MQ; ++m) {
    const int q = tid + GV_THREADS * m;
    gv[m] = make_float4(0.f, 0.f, 0.f, 0.f);
    rv[m] = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (KIND != GK_ADJ) {
      const int qc = q < npair ? q : npair - 1;
      const float4 v = reinterpret_cast<const float4*>(a.F)[spec4(2 * qc)];
      rv[m] = q < npair ? v : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }

  double lpart = 0.0;
  int par = 0;
#pragma unroll 1
  for (int i = i0; i < i1; i += GV_GR, par ^= 1) {
    int src[GV_GR];
    float4 dv[GV_GR][MQ];
#pragma unroll
    for (int r = 0; r < GV_GR; ++r) {
      const int ii = i + r;
      int s = ii < i1 ? a.idx[ii] : -1;
      if (s < 0 || s >= a.ns) s = -1;
      src[r] = s;
      const long long row = ((long long)k * a.dns + (s < 0 ? 0 : drow_of(a, ii, s))) * (a.nrp / 2);
#pragma unroll
      for (int m = 0; m < MQ; ++m) {
        const int q = tid + GV_THREADS * m;
        dv[r][m] = D4[row + (q < npair ? q : npair - 1)];
      }
    }
    float2 res[GV_GR];
    if constexpr (KIND == GK_ADJ) {
#pragma unroll
      for (int r = 0; r < GV_GR; ++r) {
        const int ii = i + r;
        const float2 v = a.Bsp[spec2(ii < i1 ? ii : i)];
        res[r] = src[r] >= 0 ? v : make_float2(0.f, 0.f);
      }
    } else {
#pragma unroll
      for (int r = 0; r < GV_GR; ++r) {
        float2 acc = make_float2(0.f, 0.f);
#pragma unroll
        for (int m = 0; m < MQ; ++m) {
          const float4 d = dv[r][m], x = rv[m];
          acc.x += d.x * x.x - d.y * x.y;
          acc.y += d.x * x.y + d.y * x.x;
          acc.x += d.z * x.z - d.w * x.w;
          acc.y += d.z * x.w + d.w * x.z;
        }
        acc = wave_sum2(acc);
        if (lane == 0) s_red[par][r][wave] = acc;
      }
      __syncthreads();  // the other buffer (par ^ 1) is free again after this barrier
#pragma unroll
      for (int r = 0; r < GV_GR; ++r) {
        float2 z = s_red[par][r][0];
#pragma unroll
        for (int w = 1; w < GV_THREADS / 64; ++w) z = cadd(z, s_red[par][r][w]);
        const int ii = i + r;
        if constexpr (KIND == GK_FUSED) {
          if (src[r] >= 0) {
            z = csub(z, a.Uf[urow_off(a, k, ii, src[r])]);
            lpart += wk * ((double)z.x * z.x + (double)z.y * z.y);
          } else {
            z = make_float2(0.f, 0.f);
          }
        } else {
          if (tid == 0 && ii < i1) a.Bsp[spec2(ii)] = src[r] >= 0 ? z : make_float2(0.f, 0.f);
        }
        res[r] = z;
      }
    }
    if constexpr (KIND != GK_FWD) {
#pragma unroll
      for (int r = 0; r < GV_GR; ++r) {
        if (src[r] < 0) continue;  // its loads read a row that is not its own
#pragma unroll
        for (int m = 0; m < MQ; ++m) cmac_conj(gv[m], dv[r][m], res[r]);
      }
    }
  }

  if constexpr (KIND == GK_FUSED) {
    if (tid == 0) a.loss_part[logical] = lpart;
  }
  if constexpr (KIND == GK_FWD) return;

  // Adjoint product of this group's rows -> G (P == 1) or the group partial.
#pragma unroll
  for (int m = 0; m < MQ; ++m) {
    const int q = tid + GV_THREADS * m;
    if (q >= npair) continue;
    if (a.P == 1)
      store_pair(a, k, q, gv[m]);
    else
      a.gpart[((long long)k * a.P + p) * npair + q] = gv[m];
  }
}

// Sum over the wavefront of one complex value per lane, for one row or two at once: the
// parts share the steps (lane halves, then 16-lane rows exchanged between them), and the
// results are scalars.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row16_sum(float v) {  // in every lane of each 16
  v = dpp_add<0x128>(v);  // row_ror 8, 4, 2, 1
  v = dpp_add<0x124>(v);
  v = dpp_add<0x122>(v);
  return dpp_add<0x121>(v);
}
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ float swap32_add(float a, float b) {  // lower half: a's sums, upper: b's
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_add(float a, float b) {  // even 16-lane rows: a's, odd: b's
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ void wave_sums(float2 (&z)[1]) {
  const float v = row16_sum(swap32_add(z[0].x, z[0].y));
  z[0] = make_float2(lane_value(v, 0) + lane_value(v, 16), lane_value(v, 32) + lane_value(v, 48));
}
__device__ __forceinline__ void wave_sums(float2 (&z)[2]) {
  const float v = row16_sum(swap16_add(swap32_add(z[0].x, z[0].y), swap32_add(z[1].x, z[1].y)));
  z[0] = make_float2(lane_value(v, 0), lane_value(v, 32));
  z[1] = make_float2(lane_value(v, 16), lane_value(v, 48));
}
__device__ __forceinline__ void wave_sums(float2 (&z)[4]) {
  float2 lo[2] = {z[0], z[1]}, hi[2] = {z[2], z[3]};
  wave_sums(lo);
  wave_sums(hi);
  z[0] = lo[0];
  z[1] = lo[1];
  z[2] = hi[0];
  z[3] = hi[1];
}

// One wavefront per row (up to 1664 receivers, MQ pairs of them a lane): no barrier between
// a row's dot product and its use in the adjoint sum, and the next RB rows are in flight
// while RB are reduced.  The four wavefronts of a workgroup take every fourth group of its
// rows and add their parts of g_k once at the end.  Bound by the bytes of D_b: at 1600
// receivers, 64 rows, 200 bins 164 MB in 33 us (5.0 TB/s); at 201 receivers, 32 rows, 257
// bins 13.5 MB in 8 us, where the workgroup-per-row kernel took 11.7 us and, with four
// groups per frequency instead of one, 4.1 us more to add them.
template <int KIND, int MQ, int RB>
__global__ __launch_bounds__(GV_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_gemv(GemmArgs a) {
  constexpr int NW = GV_THREADS / 64;
  // r_k during the rows, then g_k of the wavefronts 1 .. NW - 1
  __shared__ float4 s_x[(KIND == GK_FWD ? 1 : NW - 1) * MQ * 64];
  __shared__ double s_l[NW];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // The P groups of one frequency run on one XCD (dispatch is round-robin over the 8).
  const int total = a.nf * a.P;
  const int bid = blockIdx.x;
  const int full = (total / 8) * 8;
  const int logical = bid < full ? (bid % 8) * (total / 8) + bid / 8 : bid;
  const int k = logical / a.P, p = logical % a.P;
  const int i0 = p * a.nb / a.P, i1 = (p + 1) * a.nb / a.P;  // at most 64 rows
  const int npair = a.nrp / 2;  // receiver pairs (2q, 2q + 1), zero-padded to nrp
  auto spec2 = [&](int c) -> long long { return ((long long)(c >> 4) * a.nf + k) * CB + (c & 15); };

  // Lane b: source, row of D_k and data (or adjoint operand) entry of batch row i0 + b.
  int src = -1;
  if (i0 + lane < i1) {
    src = a.idx[i0 + lane];
    if (src < 0 || src >= a.ns) src = -1;
  }
  const int drow = src >= 0 ? drow_of(a, i0 + lane, src) : 0;
  float2 entry = make_float2(0.f, 0.f);
  if (KIND != GK_FWD && src >= 0)
    entry = KIND == GK_ADJ ? a.Bsp[spec2(i0 + lane)] : a.Uf[urow_off(a, k, i0 + lane, src)];

  const char* dk = reinterpret_cast<const char*>(a.Df + (long long)k * a.dns * a.nrp);
  unsigned qoff[MQ];
#pragma unroll
  for (int m = 0; m < MQ; ++m) qoff[m] = 16u * min(lane + 64 * m, npair - 1);
  float4 d0[RB][MQ], d1[RB][MQ];
  auto load_rows = [&](float4 (&d)[RB][MQ], int i) {  // rows past the group's last read that one
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const int row = __builtin_amdgcn_readlane(drow, min(i + b, i1 - 1) - i0);
      const char* at = dk + (long long)row * a.nrp * 8;
#pragma unroll
      for (int m = 0; m < MQ; ++m) d[b][m] = *reinterpret_cast<const float4*>(at + qoff[m]);
    }
  };
  const int ifirst = i0 + RB * wave, stride = RB * NW;
  load_rows(d0, ifirst);
  load_rows(d1, ifirst + stride);
  if constexpr (KIND != GK_ADJ) {  // model spectra r_k (zero beyond the padded receivers)
    for (int q = tid; q < MQ * 64; q += GV_THREADS)
      s_x[q] = q < npair ? reinterpret_cast<const float4*>(a.F)[spec2(2 * q) >> 1] : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
  }

  float4 gv[MQ];
#pragma unroll
  for (int m = 0; m < MQ; ++m) gv[m] = make_float4(0.f, 0.f, 0.f, 0.f);
  double lpart = 0.0;
  auto group = [&](int i, float4 (&d)[RB][MQ]) {
    float2 z[RB];
    if constexpr (KIND != GK_ADJ) {
#pragma unroll
      for (int b = 0; b < RB; ++b) z[b] = make_float2(0.f, 0.f);
#pragma unroll
      for (int m = 0; m < MQ; ++m) {
        const float4 x = s_x[lane + 64 * m];
#pragma unroll
        for (int b = 0; b < RB; ++b) {
          const float4 v = d[b][m];
          z[b].x += v.x * x.x - v.y * x.y;
          z[b].y += v.x * x.y + v.y * x.x;
          z[b].x += v.z * x.z - v.w * x.w;
          z[b].y += v.z * x.w + v.w * x.z;
        }
      }
      wave_sums(z);
    }
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const int at = min(i + b, i1 - 1) - i0;
      const bool ok = i + b < i1 && __builtin_amdgcn_readlane(src, at) >= 0;  // uniform
      const float2 u = make_float2(lane_value(entry.x, at), lane_value(entry.y, at));
      if constexpr (KIND == GK_ADJ) z[b] = u;
      if constexpr (KIND == GK_FUSED) z[b] = csub(z[b], u);
      if (!ok) z[b] = make_float2(0.f, 0.f);
      if constexpr (KIND == GK_FUSED) lpart += (double)z[b].x * z[b].x + (double)z[b].y * z[b].y;
      if constexpr (KIND == GK_FWD) {
        if (lane == 0 && i + b < i1) a.Bsp[spec2(i + b)] = z[b];
      } else if (ok) {  // (the loads of a rejected or missing row read another one)
#pragma unroll
        for (int m = 0; m < MQ; ++m) cmac_conj(gv[m], d[b][m], z[b]);
      }
    }
    load_rows(d, i + 2 * stride);
  };
#pragma unroll 1
  for (int i = ifirst; i < i1; i += 2 * stride) {
    group(i, d0);
    if (i + stride >= i1) break;
    group(i + stride, d1);
  }
  if constexpr (KIND == GK_FWD) return;

  // This group's loss partial and adjoint product: G (P == 1) or the group partial.
  __syncthreads();
  if (lane == 0) s_l[wave] = lpart;
  if (wave > 0) {
#pragma unroll
    for (int m = 0; m < MQ; ++m) s_x[((wave - 1) * MQ + m) * 64 + lane] = gv[m];
  }
  __syncthreads();
  if (wave > 0) return;
  if (KIND == GK_FUSED && lane == 0) {
    double l = 0.0;
    for (int w = 0; w < NW; ++w) l += s_l[w];
    a.loss_part[logical] = l * (k == 0 || 2 * k == a.nt ? 1.0 : 2.0);
  }
#pragma unroll
  for (int m = 0; m < MQ; ++m) {
    const int q = lane + 64 * m;
    float4 g = gv[m];
#pragma unroll
    for (int w = 0; w < NW - 1; ++w) {
      const float4 t = s_x[(w * MQ + m) * 64 + lane];
      g.x += t.x;
      g.y += t.y;
      g.z += t.z;
      g.w += t.w;
    }
    if (q >= npair) continue;
    if (a.P == 1)
      store_pair(a, k, q, g);
    else
      a.gpart[((long long)k * a.P + p) * npair + q] = g;
  }
}

// G_k for receiver pairs q: the P group partials added in group order.
__global__ __launch_bounds__(GV_THREADS) void k_gemv_sum(GemmArgs a) {
  const int npair = a.nrp / 2;
  const int nqb = (npair + GV_THREADS - 1) / GV_THREADS;
  const int k = blockIdx.x / nqb;
  const int q = (blockIdx.x % nqb) * GV_THREADS + threadIdx.x;
  if (q >= npair) return;
  const float4* part = a.gpart + (long long)k * a.P * npair + q;
  float4 s = part[0];
  for (int g = 1; g < a.P; ++g) {
    const float4 v = part[(long long)g * npair];
    s.x += v.x;
    s.y += v.y;
    s.z += v.z;
    s.w += v.w;
  }
  store_pair(a, k, q, s);
}

// Row groups per frequency, at least 8 rows each.  One wavefront per row: about one
// workgroup per CU, since every group's partial of g_k is written and read once more (3D
// patch with one virtual source, products + update: 49.5 us with 2 groups, 56 with 3, 60
// with 4).  The wide kernel waits at a barrier per two rows and wants about three
// workgroups per CU, and at least four groups.
int row_groups(int nb, int nf, bool wide) {
  const int most = (nb + 7) / 8;
  int want = ((wide ? 3 : 1) * 256 + nf - 1) / nf;
  if (wide && want < 4) want = 4;
  return want < most ? want : most;
}

// A workgroup per row beats a wavefront per row (us, a wavefront -> a workgroup)
//   where most wavefronts would have no row: 1664 receivers, 257 bins, 2 rows fused 10.2 ->
//     7.4, 600 receivers 8.3 -> 6.2, but 8 rows 13.4 -> 14.2; adjoint alone, with no dot product
//     to wait for, 8 rows 10.3 -> 8.3;
//   where the registers of the long rows allow two workgroups a CU and there are more than
//     that: 513 bins, 8 rows 22.4 -> 17.0;
//   in the forward kind with long rows: 257 bins, 64 rows 40 -> 35 (8 rows 9.4 -> 10.9).
// The forward kind leaves no partials: with many rows at least two groups (1100 receivers, 257
// bins, 64 rows 28.8 -> 26.7).
template <int KIND>
hipError_t launch_rows(GemmArgs a, hipStream_t s) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(a.nf * a.P), dim3(GV_THREADS), 0, s, a);
    return hipGetLastError();
  };
  const int mq = (a.nrp / 2 + 63) / 64;            // receiver pairs per lane
  const bool long_forward = KIND == GK_FWD && mq > 10 && a.nf > 256 && a.nb > 8;
  if (long_forward) a.P = row_groups(a.nb, a.nf, true);
  else if (KIND == GK_FWD && a.nb >= 32 && a.P < 2) a.P = 2;
  if (mq > GV_MQ || long_forward || (mq > 4 && a.nb <= 4) || (mq > 8 && a.nb <= 8 && (KIND == GK_ADJ || a.nf > 512))) {
    if (mq <= 8) return go(k_gemv_wide<KIND, 2>);
    if (mq <= 16) return go(k_gemv_wide<KIND, 4>);
    return go(k_gemv_wide<KIND, 8>);
  }
  if (mq <= 1) return go(k_gemv<KIND, 1, 4>);
  if (mq <= 2) return go(k_gemv<KIND, 2, 4>);
  if (mq <= 3) return go(k_gemv<KIND, 3, 2>);
  if (mq <= 4) return go(k_gemv<KIND, 4, 2>);
  if (mq <= 6) return go(k_gemv<KIND, 6, 2>);
  if (mq <= 8) return go(k_gemv<KIND, 8, 1>);
  if (mq <= 10) return go(k_gemv<KIND, 10, 1>);
  return go(k_gemv<KIND, 13, 1>);                  // (16 pairs a lane: 76 registers spilled)
}

template <int KIND>
hipError_t launch_kind(const GemmArgs& a, bool sum, hipStream_t s) {
  const hipError_t e = launch_rows<KIND>(a, s);
  if (e != hipSuccess || KIND == GK_FWD || a.P == 1 || !sum) return e;
  const int nqb = (a.nrp / 2 + GV_THREADS - 1) / GV_THREADS;
  hipLaunchKernelGGL(k_gemv_sum, dim3(a.nf * nqb), dim3(GV_THREADS), 0, s, a);
  return hipGetLastError();
}

}  // namespace

int gemv_groups(int nb, int nf, int nr) { return row_groups(nb, nf, round16(nr) / 2 > 64 * GV_MQ); }

hipError_t launch_gemv(int kind, const GemmArgs& a, bool sum, hipStream_t s) {
  if (a.nb < 1 || a.nb > NB_LIMIT || a.nvs != 1 || a.P < 1) return hipErrorInvalidValue;
  if (a.P > 1 && !a.gpart) return hipErrorInvalidValue;
  switch (kind) {
    case GK_FUSED: return launch_kind<GK_FUSED>(a, sum, s);
    case GK_FWD: return launch_kind<GK_FWD>(a, sum, s);
    case GK_ADJ: return launch_kind<GK_ADJ>(a, sum, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mdd
