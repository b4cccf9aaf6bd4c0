// Split-precision (bf16x3, fp16x3) and bf16 (diagnostic) per-frequency products, one
// wavefront per 16-column block (every kind, every batch size):
//
//   Res_k = D_{b,k} R_k - U_{b,k},   G_k = D_{b,k}^H Res_k written over R_k
//
// Every complex operand is split into hi + lo halves of bf16 or fp16 and the three
// significant products hi*hi + hi*lo + lo*hi are accumulated in float32 on
// v_mfma_f32_16x16x32_{bf16,f16}; the bf16 form has the hi halves alone.
//
// As in the float32 kernel, the wavefronts of a workgroup share the rows of D_{b,k} in LDS
// and nothing else: each streams its own block of R_k from HBM into registers, splits it
// there, and keeps the residual in registers as the right operand of the adjoint product.
// A forward product leaves batch row 4 q + e of a tile in lane quarter q, element e; the
// adjoint's k-slots are given to the batch rows in that order (slots 0-3 of quarter q are
// rows 4 q .. 4 q + 3 of one tile, slots 4-7 the same rows of the next), so no value
// changes lanes.  D is split once per element and workgroup, while it is staged: for the
// forward product as [row][receiver], for the adjoint as [receiver][row] in the order
// above, so that each operand is one 16-byte LDS read per plane (re hi, re lo, and hi, lo of
// the negated imaginary part).  fp16 carries power-of-two scales so that the low halves stay
// normal: one per column for each receiver chunk of R_k and for the residual, and for
// D_{b,k} at up to 16 batch rows one per batch row (forward) and per receiver (adjoint) of a
// chunk, found while it is staged, so that weak sources keep their bits beside a strong one;
// with more rows one per frequency (from the largest |D| of all sources, found when the kernel
// is set).
//
// What bounds it: the traffic of R_k and G_k in pieces of 16 columns (128 bytes, a whole
// spectra row apart), 3.4 to 3.9 TB/s for the forward and adjoint kinds alone; the bf16 form,
// with a third of the matrix work, takes as long as bf16x3.  More chunks of R_k or D in flight,
// other orders of the workgroups and a schedule with the splitting between the products all
// measured the same or slower.  HIP events; before: a kernel with loader and compute
// wavefronts (fused, over 32 rows), a tiled one and a persistent one:
//   nr = nvs   nb   nf   form        fused             forward          adjoint
//      1600    64  200   bf16x3   2101 -> 2040 us   3134 -> 1055 us   2038 -> 1212 us
//      1600    64  200   fp16x3   2520 -> 2095 us   3540 -> 1105 us   2160 -> 1240 us
//      1600    64  200   bf16     4160 -> 2036 us   1896 -> 1041 us   2194 -> 1278 us
//       400    48  200   fp16x3    235 -> 170 us     268 -> 83 us      197 -> 93 us
//       301    64  257   bf16x3    161 -> 136 us     190 -> 68 us      147 -> 78 us
//       301    32  257   bf16x3    178 -> 110 us      86 -> 45 us       77 -> 66 us
//       201    16  257   fp16x3     58 -> 53 us       48 -> 26 us       62 -> 35 us
// Errors against 64 bits: fp16x3 gradient 2.4e-7 (before 2.6e-7), bf16x3 unchanged.
#include <type_traits>

#include "device_common.h"
#include "mdd_internal.h"

namespace mdd {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

template <int PREC>
struct SplitT {
  static constexpr bool F16 = PREC == MDD_PREC_FP16X3;
  static constexpr bool LO = PREC != MDD_PREC_BF16;  // the low halves count
  using E = std::conditional_t<F16, _Float16, __bf16>;
  using V = std::conditional_t<F16, halfx8, bf16x8>;
  using V2 = std::conditional_t<F16, halfx2, bf16x2>;
  static __device__ __forceinline__ floatx4 mma(V a, V b, floatx4 c) {
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ void split(float x, E& hi, E& lo) {
    hi = (E)x;
    lo = (E)(x - (float)hi);
  }
};

// Two values split at once (one packed conversion for the two hi halves and one for
// the two lo halves), bf16 only.
typedef float floatx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split2_bf16(float x0, float x1, bf16x2& hi, bf16x2& lo) {
  const floatx2 x = {x0, x1};
  hi = __builtin_convertvector(x, bf16x2);
  lo = __builtin_convertvector(x - __builtin_convertvector(hi, floatx2), bf16x2);
}

// acc += A * B with the imaginary part of A given negated (nai = -Im A, which the operand
// staging supplies at no cost): Re += ar br + nai bi and Im += ar bi, while the remaining
// imaginary term nai br goes into u, subtracted once at the end (Im = im - u).  The terms
// with a low half come first where the sums start from zero: their rounding is then 2^-11
// of what it is beside the full sum.
template <typename T, typename V>
__device__ __forceinline__ void cmma_lo(const V (&a)[4], const V& brh, const V& brl, const V& bih,
                                        const V& bil, floatx4& re, floatx4& im, floatx4& u) {
  re = T::mma(a[0], brl, re);
  im = T::mma(a[0], bil, im);
  u = T::mma(a[2], brl, u);
  re = T::mma(a[1], brh, re);
  im = T::mma(a[1], bih, im);
  u = T::mma(a[3], brh, u);
  re = T::mma(a[2], bil, re);
  re = T::mma(a[3], bih, re);
}
template <typename T, typename V>
__device__ __forceinline__ void cmma_hi(const V (&a)[4], const V& brh, const V& bih, floatx4& re,
                                        floatx4& im, floatx4& u) {
  re = T::mma(a[0], brh, re);
  im = T::mma(a[0], bih, im);
  u = T::mma(a[2], brh, u);
  re = T::mma(a[2], bih, re);
}

// Power-of-two scale bringing max |x| to [2^13, 2^14), and its inverse, from the exponent
// bits; clamped so that both stay finite (1 where the maximum is not).  A zero maximum takes
// the largest scale, which its zeros ignore.
__device__ __forceinline__ float2 pow2_scale_pair(float amax) {
  const int e = __float_as_int(amax) >> 23;  // amax = m 2^(e - 126), m in [0.5, 1)
  const int sh = e == 255 ? 0 : min(140 - e, 120);
  return make_float2(__int_as_float((127 + sh) << 23), __int_as_float((127 - sh) << 23));
}

template <int PREC, typename V>
__device__ __forceinline__ void split8(const float (&x)[8], V& hi, V& lo) {
  if constexpr (SplitT<PREC>::F16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      _Float16 h, l;
      SplitT<PREC>::split(x[e], h, l);
      hi[e] = h;
      lo[e] = l;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      bf16x2 h, l;
      split2_bf16(x[e], x[e + 1], h, l);
      hi[e] = h[0];
      hi[e + 1] = h[1];
      lo[e] = l[0];
      lo[e + 1] = l[1];
    }
  }
}

// Maximum over the four lanes of a column (lane quarters).
__device__ __forceinline__ float column_max(float m) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  m = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

template <int NBT>
struct SplitCfg {
  static constexpr int KC = 32;                     // receivers per chunk: one forward k-step
  static constexpr int MB = 16 * NBT;
  static constexpr int NK = (NBT + 1) / 2;          // adjoint k-steps of 32 rows (an odd last
                                                    // one half empty: see the kernel)
  // Row pitches (elements): a 16-byte read is served 16 lanes at a time, lanes 0-3, 12-15
  // and 20-27 first; with pitches of 6 or 10 times 16 bytes these touch 16 different banks.
  static constexpr int FP = KC + 16;
  static constexpr int AP = 32 * NK + 16;
  static constexpr int FPL = MB * FP, APL = KC * AP;              // one plane
  static constexpr int SLOT = 4 * (FPL > APL ? FPL : APL);        // elements per chunk of D
  static constexpr size_t SMEM = 2 * 2 * (size_t)SLOT;            // two chunks of 2-byte elements
};

// Largest magnitude among 8 complex values (a tree: it is in the way of their use).
__device__ __forceinline__ float amax8(const float (&x)[8], const float (&y)[8]) {
  float m[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    m[i] = fmaxf(fmaxf(fabsf(x[2 * i]), fabsf(y[2 * i])), fmaxf(fabsf(x[2 * i + 1]), fabsf(y[2 * i + 1])));
  return fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
}
// Maximum over four neighbouring lanes.
__device__ __forceinline__ float quad_max(float m) {
  m = fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0xb1, 0xf, 0xf, false)));  // 1, 0, 3, 2
  return fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x4e, 0xf, 0xf, false)));  // 2, 3, 0, 1
}

// Eight values of a row (or receiver): real parts x and the negated imaginary parts y, split
// into the planes at p.
template <int PREC, typename E>
__device__ __forceinline__ void put_planes(E* p, int plane, const float (&x)[8], const float (&y)[8]) {
  using T = SplitT<PREC>;
  using V = typename T::V;
  V h, l;
  split8<PREC>(x, h, l);
  *reinterpret_cast<V*>(p) = h;
  if constexpr (T::LO) *reinterpret_cast<V*>(p + plane) = l;
  split8<PREC>(y, h, l);
  *reinterpret_cast<V*>(p + 2 * plane) = h;
  if constexpr (T::LO) *reinterpret_cast<V*>(p + 3 * plane) = l;
}

// The residual as the adjoint's right operand (k-step kk: tiles 2 kk and 2 kk + 1).
template <int PREC, int NBT, typename V>
__device__ __forceinline__ void residual_operand(const floatx4 (&re)[NBT], const floatx4 (&im)[NBT], float scale,
                                                 V* srh, V* srl, V* sih, V* sil) {
#pragma unroll
  for (int kk = 0; kk < SplitCfg<NBT>::NK; ++kk) {
    float x[8], y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int t = 2 * kk + (e >> 2);
      x[e] = t < NBT ? re[t < NBT ? t : 0][e & 3] * scale : 0.f;
      y[e] = t < NBT ? im[t < NBT ? t : 0][e & 3] * scale : 0.f;
    }
    split8<PREC>(x, srh[kk], srl[kk]);
    split8<PREC>(y, sih[kk], sil[kk]);
  }
}

// One 16 x 16 tile of D^H Res; p: this lane's receiver and row group in the adjoint's planes.
template <int PREC, int NBT, typename E, typename V>
__device__ __forceinline__ void adjoint_tile(const E* p, const V* srh, const V* srl, const V* sih, const V* sil,
                                             floatx4& gr, floatx4& gi) {
  using C = SplitCfg<NBT>;
  using T = SplitT<PREC>;
  V av[C::NK][4];
  floatx4 gu = {0.f, 0.f, 0.f, 0.f};
  gr = gi = gu;
#pragma unroll
  for (int kk = 0; kk < C::NK; ++kk)
#pragma unroll
    for (int i = 0; i < 4; i += T::LO ? 1 : 2)
      av[kk][i] = *reinterpret_cast<const V*>(p + i * C::APL + kk * 32);
  if constexpr (T::LO) {
#pragma unroll
    for (int kk = 0; kk < C::NK; ++kk) cmma_lo<T>(av[kk], srh[kk], srl[kk], sih[kk], sil[kk], gr, gi, gu);
  }
#pragma unroll
  for (int kk = 0; kk < C::NK; ++kk) cmma_hi<T>(av[kk], srh[kk], sih[kk], gr, gi, gu);
  gi -= gu;
}

// OUT: G written (plainly, or with streaming stores), or added to what is there.
enum { OUT_WRITE, OUT_ADD, OUT_STREAM };

// NP = 2 (few column blocks): eight wavefronts on four blocks.  The two that share a block take
// the receiver chunks in turn, forward and adjoint, with LDS slots of their own half; between
// the two products they add their sums through LDS, so that both hold the residual.  D is
// read and split as often as before, and each wavefront's chain of chunks is half as long.
template <int PREC, int NBT, int KIND, int OUT, int NP>
__global__ __launch_bounds__(256 * NP) __attribute__((amdgpu_waves_per_eu(NBT >= 3 || NP > 1 ? 2 : 3)))
void k_gemm_split(GemmArgs a) {
  using C = SplitCfg<NBT>;
  using T = SplitT<PREC>;
  using E = typename T::E;
  using V = typename T::V;
  constexpr int KC = C::KC, MB = C::MB, NK = C::NK, NW = 4;
  constexpr bool F16 = T::F16, FWD = KIND != GK_ADJ;
  // fp16, up to 16 rows: one wavefront stages whole rows of a chunk (forward) or whole receivers
  // (adjoint), and so finds their scales itself
  constexpr bool OWN = F16 && NBT == 1;
  extern __shared__ __align__(16) char s_raw[];
  __shared__ __align__(16) float s_inv[OWN ? NP : 1][2][KC];  // OWN: the inverse scales, by slot

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & (NW - 1);
  const int part = __builtin_amdgcn_readfirstlane(tid >> 6) / NW;  // which chunks: part + NP v
  E* const s_d = reinterpret_cast<E*>(s_raw) + part * 2 * C::SLOT;
  const int lr = lane & 15, lq = lane >> 4;
  // the column groups of one frequency share an XCD, whose L2 then serves D_k once; the
  // blocks of a frequency are spread evenly over its groups
  const int ncg = (a.nvb + NW - 1) / NW;
  const int total = a.nf * ncg;
  const int bid = blockIdx.x, full = (total / 8) * 8;
  const int logical = bid < full ? (bid % 8) * (total / 8) + bid / 8 : bid;
  const int k = logical / ncg, cg = logical % ncg;
  const int blk0 = (int)((long long)cg * a.nvb / ncg), blk1 = (int)((long long)(cg + 1) * a.nvb / ncg);
  const bool active = blk0 + wave < blk1;
  const int blk = active ? blk0 + wave : blk0;
  const long long rowstride = (long long)a.nvb * a.nf * CB;
  const unsigned rs32 = (unsigned)rowstride;
  const int nr = a.nr, nc = (nr + KC - 1) / KC, nv = (nc + NP - 1) / NP;

  // R_k: receivers 8 lq .. 8 lq + 7 of a chunk, column lr; past nr out of bounds: zeros (32
  // rows of at most 256 blocks x 513 bins fit 32 bits).
  const long long col = ((long long)blk * a.nf + k) * CB;
  auto rows_at = [&](float2* base, int r0, int rows) {
    const int n = max(min(nr - r0, rows), 0);
    return buffer_at(base + r0 * rowstride + col, n ? (unsigned)n * rs32 * 8u - (unsigned)col * 8u : 0u);
  };
  unsigned roff[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) roff[e] = ((unsigned)(8 * lq + e) * rs32 + lr) * 8u;
  auto load_r = [&](float2 (&dst)[8], int c) {
    const auto rb = rows_at(a.F, c * KC, KC);
#pragma unroll
    for (int e = 0; e < 8; ++e) dst[e] = buffer_get2(rb, roff[e]);
  };
  float2 rbuf[2][8];
  if constexpr (FWD) load_r(rbuf[0], part);            // in flight while the batch is looked up

  // Batch rows: lane b of every wavefront holds the source of batch entry b, or -1.
  int src = -1;
  if (lane < a.nb) {
    src = a.idx[lane];
    if (src < 0 || src >= a.ns) src = -1;
  }
  const int drow = src >= 0 ? drow_of(a, lane, src) : -1;
  float2 sd = make_float2(1.f, 1.f);                // D's scale and its inverse (fp16, not OWN)
  if constexpr (F16 && !OWN) sd = pow2_scale_pair(a.dmax[k]);

  // D_{b,k} for the forward product: staging wavefront w takes rows 16 w .. 16 w + 15, a lane
  // eight receivers of one row (the last wavefront is the first to stage: with few column
  // blocks it has no block of its own); rows without a source and receivers past the padded row are out of
  // bounds: zeros.
  const char* dbase = reinterpret_cast<const char*>(a.Df + (long long)k * a.dns * a.nrp);
  const unsigned dbytes = (unsigned)a.dns * (unsigned)a.nrp * 8u;
  auto chunk_at = [&](int c) {
    return buffer_at(dbase + (long long)c * KC * 8, dbytes - (unsigned)(c * KC) * 8u);
  };
  const int sw = NW - 1 - wave;
  const int frow = 16 * sw + (lane >> 2), fg = 8 * (lane & 3);
  const int fsrc = __shfl(drow, frow, 64);
  const unsigned foff = ((unsigned)fsrc * (unsigned)a.nrp + fg) * 8u;
  auto load_f = [&](float4 (&d)[4], int c) {
    const auto db = chunk_at(c);
    const bool in = fsrc >= 0 && fg < a.nrp - c * KC;
#pragma unroll
    for (int q = 0; q < 4; ++q) d[q] = buffer_get4(db, in ? foff + 16u * q : PAST_END);
  };
  auto stage_f = [&](int slot, float4 (&d)[4]) {
    if (sw < NBT) {
      float x[8], y[8];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // used here and not before: hoisted above the step's products, the split would wait
        // there for these loads
        asm volatile("" : "+v"(d[q].x), "+v"(d[q].y), "+v"(d[q].z), "+v"(d[q].w));
        x[2 * q] = d[q].x;
        y[2 * q] = -d[q].y;
        x[2 * q + 1] = d[q].z;
        y[2 * q + 1] = -d[q].w;
      }
      float sc = sd.x;
      if constexpr (OWN) {
        const float2 sp = pow2_scale_pair(quad_max(amax8(x, y)));
        sc = sp.x;
        if ((lane & 3) == 0) s_inv[part][slot][frow] = sp.y;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        x[e] *= sc;
        y[e] *= sc;
      }
      put_planes<PREC>(s_d + slot * C::SLOT + frow * C::FP + fg, C::FPL, x, y);
    }
  };
  // For the adjoint: a lane takes one receiver and eight rows, 4 lq .. 4 lq + 3 of tiles 2 w'
  // and 2 w' + 1 (zeros where the second is past the batch); the left operand is conj(D),
  // whose negated imaginary part is Im D.  A half-empty k-step keeps the 16x16x32 shape:
  // with 16x16x16 products at the end of the same sums, two of a tile's four result registers
  // were wrong by 1e-4, and not the same from run to run, in one of the instances (fp16, 48
  // rows).  That is not explained: staging, barriers and scaling were those of this kernel, and
  // in the assembly of that form, built again, every read of a product's result comes 8 or more
  // issue slots after it, which the 4 passes of these products ask for.
  const int akk = sw >> 1, ar = 16 * (sw & 1) + lr;
  unsigned aoff[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int row = __shfl(drow, (32 * akk + 4 * lq + (e & 3) + 16 * (e >> 2)) & 63, 64);
    aoff[e] = row >= 0 ? ((unsigned)row * (unsigned)a.nrp + ar) * 8u : PAST_END;
  }
  auto load_a = [&](float2 (&d)[8], int chunk) {
    const int c = max(chunk, 0);
    const auto db = chunk_at(c);
    const bool in = ar < a.nrp - c * KC;
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = buffer_get2(db, in ? aoff[e] : PAST_END);
  };
  auto stage_a = [&](int slot, float2 (&d)[8]) {
    if (2 * akk < NBT) {
      float x[8], y[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        asm volatile("" : "+v"(d[e].x), "+v"(d[e].y));
        x[e] = d[e].x;
        y[e] = d[e].y;
      }
      float sc = sd.x;
      if constexpr (OWN) {
        const float2 sp = pow2_scale_pair(column_max(amax8(x, y)));
        sc = sp.x;
        if (lq == 0) s_inv[part][slot][ar] = sp.y;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        x[e] *= sc;
        y[e] *= sc;
      }
      put_planes<PREC>(s_d + slot * C::SLOT + ar * C::AP + akk * 32 + 8 * lq, C::APL, x, y);
    }
  };

  // Inverses of D's scales for the lane's four results of a tile, rows (receivers) at + 4 lq on.
  auto inv_scales = [&](int slot, int at) -> floatx4 {
    if constexpr (OWN) return *reinterpret_cast<const floatx4*>(&s_inv[part][slot][at + 4 * lq]);
    else return floatx4{sd.y, sd.y, sd.y, sd.y};
  };

  // Data (or the adjoint's operand) entries of the lane: batch row 16 t + 4 lq + e.
  unsigned okrow = 0;                               // bit 4 t + e: the entry counts
  float2 upre[NBT][4];
  auto load_u = [&]() {
#pragma unroll
    for (int t = 0; t < NBT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = t * 16 + lq * 4 + e;
        const int s = __shfl(src, row, 64), rowc = min(row, a.nb - 1);
        if (s >= 0 && blk * CB + lr < a.nvs) okrow |= 1u << (4 * t + e);
        if constexpr (KIND == GK_ADJ)
          upre[t][e] = a.Bsp[(((size_t)rowc * a.nvb + blk) * a.nf + k) * CB + lr];
        else if constexpr (KIND == GK_FUSED)
          upre[t][e] = a.Uf[urow_off(a, k, rowc, max(s, 0)) + blk * CB + lr];
      }
  };

  floatx4 re[NBT], im[NBT], un[NBT];                // un: what Im lacks (cmma_lo)
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
  if constexpr (FWD) {
#pragma unroll
    for (int t = 0; t < NBT; ++t) re[t] = im[t] = un[t] = zero;
    float4 dv[4];
    load_f(dv, part);
    stage_f(0, dv);
    load_f(dv, part + NP);
    __syncthreads();
    auto step = [&](int v, float2 (&cur)[8], float2 (&nxt)[8]) {
      load_r(nxt, part + NP * (v + 1));  // past the last chunk: zeros
      if (active) {
        float x[8], y[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          x[e] = cur[e].x;
          y[e] = cur[e].y;
        }
        float2 sr = make_float2(1.f, 1.f);
        if constexpr (F16) {
          sr = pow2_scale_pair(column_max(amax8(x, y)));
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            x[e] *= sr.x;
            y[e] *= sr.x;
          }
        }
        V brh, brl, bih, bil;
        split8<PREC>(x, brh, brl);
        split8<PREC>(y, bih, bil);
        const E* p = s_d + (v & 1) * C::SLOT + lr * C::FP + 8 * lq;
        V av[2][4];
        auto read_a = [&](int t) {
#pragma unroll
          for (int i = 0; i < 4; i += T::LO ? 1 : 2)
            av[t & 1][i] = *reinterpret_cast<const V*>(p + i * C::FPL + t * 16 * C::FP);
        };
        read_a(0);
        const floatx4 si = inv_scales(v & 1, 0);
#pragma unroll
        for (int t = 0; t < NBT; ++t) {
          if (t + 1 < NBT) read_a(t + 1);
          __builtin_amdgcn_sched_barrier(0);
          floatx4 cr = F16 ? zero : re[t], ci = F16 ? zero : im[t], cu = F16 ? zero : un[t];
          if constexpr (T::LO) cmma_lo<T>(av[t & 1], brh, brl, bih, bil, cr, ci, cu);
          cmma_hi<T>(av[t & 1], brh, bih, cr, ci, cu);
          if constexpr (F16) {
            re[t] += (cr * si) * sr.y;
            im[t] += ((ci - cu) * si) * sr.y;
          } else {
            re[t] = cr;
            im[t] = ci;
            un[t] = cu;
          }
        }
      }
      stage_f((v + 1) & 1, dv);
      load_f(dv, part + NP * (v + 2));
      __syncthreads();
    };
    int v = 0;
    while (true) {
      step(v, rbuf[0], rbuf[1]);
      if (++v == nv) break;
      step(v, rbuf[1], rbuf[0]);
      if (++v == nv) break;
    }
  }

  float2 da[8];
  if constexpr (KIND != GK_FWD) load_a(da, nc - 1 - part);
  if (active) load_u();
  if constexpr (FWD && NP > 1) {
    float2* const s_sum = reinterpret_cast<float2*>(s_raw) + wave * MB * 16;  // [NP][NW][MB][16]
    static_assert(NW * MB * 16 * sizeof(float2) <= C::SMEM, "sums fit the slots");
#pragma unroll
    for (int t = 0; t < NBT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        s_sum[(part * NW * MB + t * 16 + lq * 4 + e) * 16 + lr] = make_float2(re[t][e], im[t][e] - un[t][e]);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NBT; ++t) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2* p = s_sum + (t * 16 + lq * 4 + e) * 16 + lr;
        const float2 z = cadd(p[0], p[NW * MB * 16]);
        re[t][e] = z.x;
        im[t][e] = z.y;
      }
      un[t] = zero;
    }
    __syncthreads();
  }
  // residual and float64 loss partial (or predicted data, or the adjoint's operand)
  double lpart = 0.0;
  float zm = 0.f;
  if (active) {
#pragma unroll
    for (int t = 0; t < NBT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = t * 16 + lq * 4 + e;
        float2 z = KIND == GK_ADJ ? upre[t][e] : make_float2(re[t][e], im[t][e] - un[t][e]);
        if constexpr (KIND == GK_FUSED) z = csub(z, upre[t][e]);
        if (!((okrow >> (4 * t + e)) & 1)) z = make_float2(0.f, 0.f);
        if constexpr (KIND == GK_FUSED) lpart += (double)z.x * z.x + (double)z.y * z.y;
        if constexpr (KIND == GK_FWD) {
          if (row < a.nb && part == 0) a.Bsp[(((size_t)row * a.nvb + blk) * a.nf + k) * CB + lr] = z;
        }
        zm = fmaxf(zm, fmaxf(fabsf(z.x), fabsf(z.y)));
        re[t][e] = z.x;
        im[t][e] = z.y;
      }
    if constexpr (KIND == GK_FUSED) {
      lpart = wave_sum(lpart);
      if (lane == 0 && part == 0) a.loss_part[k * a.nvb + blk] = lpart * (k == 0 || 2 * k == a.nt ? 1.0 : 2.0);
    }
  }
  if constexpr (KIND == GK_FWD) return;

  // adjoint: G_k = D_b^H Res, 16 receivers at a time, written over R_k (or into Gout)
  stage_a(0, da);
  load_a(da, nc - 1 - part - NP);
  float2 ss = make_float2(1.f, 1.f);
  if constexpr (F16) ss = pow2_scale_pair(column_max(zm));
  V srh[NK], srl[NK], sih[NK], sil[NK];
  residual_operand<PREC, NBT>(re, im, ss.x, srh, srl, sih, sil);
  __syncthreads();
  float2* gbase = a.Gout ? a.Gout : a.F;
  unsigned goff[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) goff[e] = active ? ((unsigned)(4 * lq + e) * rs32 + lr) * 8u : PAST_END;
  auto visit = [&](int v) {
    const int slot = v & 1, c = nc - 1 - part - NP * v;  // below 0: no chunk
    const E* p = s_d + slot * C::SLOT + lr * C::AP;
#pragma unroll
    for (int m = 0; m < KC / 16; ++m) {
      const auto gb = rows_at(gbase, c * KC + m * 16, c >= 0 ? 16 : 0);
      float2 old[4];
      if constexpr (OUT == OUT_ADD) {
#pragma unroll
        for (int e = 0; e < 4; ++e) old[e] = buffer_get2(gb, goff[e]);
      }
      floatx4 gr = zero, gi = zero;
      const floatx4 si = inv_scales(slot, m * 16);
      if (active) adjoint_tile<PREC, NBT>(p + m * 16 * C::AP + 8 * lq, srh, srl, sih, sil, gr, gi);
      if constexpr (F16) {
        gr = (gr * si) * ss.y;
        gi = (gi * si) * ss.y;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float2 z = make_float2(gr[e], gi[e]);
        if constexpr (OUT == OUT_ADD) z = cadd(z, old[e]);
        buffer_put2<OUT == OUT_STREAM>(gb, goff[e], z);
      }
    }
    stage_a(slot ^ 1, da);
    load_a(da, c - 2 * NP);
    __syncthreads();
  };
#pragma unroll 1
  for (int v = 0; v < nv; ++v) visit(v);
}

template <int PREC, int NBT, int NP>
hipError_t launch_np(int kind, const GemmArgs& a, hipStream_t s) {
  const dim3 grid(a.nf * ((a.nvb + 3) / 4)), block(256 * NP);
  constexpr size_t sm = NP * SplitCfg<NBT>::SMEM;
  auto go = [&](auto kernel) {
    if (sm > 65536)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
    hipLaunchKernelGGL(kernel, grid, block, sm, s, a);
    return hipGetLastError();
  };
  switch (kind) {
    case GK_FUSED:
      if (a.gacc) return go(k_gemm_split<PREC, NBT, GK_FUSED, OUT_ADD, NP>);
      // Spectra past the last-level cache (256 MB): with streaming stores D stays in L2 (1600
      // receivers, 64 rows: the step 8970 -> 8850 us).  Smaller ones the trace kernel finds in
      // the cache (201 receivers, 32 rows, float32 kernel: 198 -> 208 us with them).
      if constexpr (NP == 1) {
        if (8.0 * CB * a.nr * a.nvb * a.nf > 256e6) return go(k_gemm_split<PREC, NBT, GK_FUSED, OUT_STREAM, NP>);
      }
      return go(k_gemm_split<PREC, NBT, GK_FUSED, OUT_WRITE, NP>);
    case GK_FWD: return go(k_gemm_split<PREC, NBT, GK_FWD, OUT_WRITE, NP>);
    case GK_ADJ: return go(k_gemm_split<PREC, NBT, GK_ADJ, OUT_WRITE, NP>);
    default: return hipErrorInvalidValue;
  }
}

template <int PREC, int NBT>
hipError_t launch_nbt(int kind, const GemmArgs& a, hipStream_t s) {
  // fewer workgroups than CUs: two wavefronts per block (fused, 300 receivers, 64 rows, 100
  // bins: 33 columns 29 -> 25 us; 258 workgroups of 100 receivers lose with it, 25 -> 34 us)
  if (a.nf * ((a.nvb + 3) / 4) < 256) return launch_np<PREC, NBT, 2>(kind, a, s);
  return launch_np<PREC, NBT, 1>(kind, a, s);
}

template <int PREC>
hipError_t launch_prec(int kind, const GemmArgs& a, hipStream_t s) {
  if (a.nb <= 16) return launch_nbt<PREC, 1>(kind, a, s);
  if (a.nb <= 32) return launch_nbt<PREC, 2>(kind, a, s);
  if (a.nb <= 48) return launch_nbt<PREC, 3>(kind, a, s);
  return launch_nbt<PREC, 4>(kind, a, s);
}

}  // namespace

hipError_t launch_gemm_split(int kind, int precision, const GemmArgs& a, hipStream_t s) {
  if (a.nb < 1 || a.nb > NB_LIMIT) return hipErrorInvalidValue;
  switch (precision) {
    case MDD_PREC_BF16X3: return launch_prec<MDD_PREC_BF16X3>(kind, a, s);
    case MDD_PREC_FP16X3: return launch_prec<MDD_PREC_FP16X3>(kind, a, s);
    case MDD_PREC_BF16: return launch_prec<MDD_PREC_BF16>(kind, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mdd
