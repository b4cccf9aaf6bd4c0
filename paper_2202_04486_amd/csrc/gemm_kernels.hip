// Per-frequency complex products of the MDC operator on MFMA (Theory section,
// matrix form P-_f = P+_f R_f; Appendix A "batched matrix-matrix
// multiplication"), with the residual, the float64 loss partials and the
// adjoint product fused for the mini-batch gradient:
//
//   Res_k = D_{b,k} R_k - U_{b,k}      ([nb x nr] [nr x nvs])
//   G_k   = D_{b,k}^H Res_k            ([nr x nb] [nb x nvs]), written over R_k
//
// k_gemm<prec, NBT, TNB, kind>  tiled: a workgroup owns one frequency k and TNB column
//     blocks (16 virtual sources each); the batch rows of D_k are gathered by index into
//     LDS in receiver chunks and the residual block stays in LDS between the two
//     products.  The bf16 diagnostic, and the split forms at up to 16 batch rows except
//     for the fused kind over few receivers.  The other split-precision kernels are in
//     gemm_split.hip, the float32 ones in gemm_rows.hip.
// R_k is read and G_k written exactly once.  G_k goes over R_k, or (the full
// gradient) into, or added to, a second spectra buffer.
//
// There is no complex MFMA: a complex product is four real products
// (Re = Ar Br - Ai Bi, Im = Ar Bi + Ai Br) on v_mfma_f32_16x16x32_{bf16,f16}, in the
// split forms with each operand split into hi + lo and hi*hi + hi*lo + lo*hi accumulated
// in fp32.
#include "device_common.h"
#include "mdd_internal.h"

namespace mdd {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));

// Operand of a 16x16x32 split-precision MFMA: 8 consecutive k values of one
// row (A) or one column (B), real and imaginary parts, hi and lo.
template <int PREC>
struct SplitOp;

template <>
struct SplitOp<MDD_PREC_BF16X3> {
  using V = bf16x8;
  V rh, rl, ih, il;
  __device__ __forceinline__ void set(int e, float2 z) {
    const __bf16 a = (__bf16)z.x, b = (__bf16)z.y;
    rh[e] = a;
    ih[e] = b;
    rl[e] = (__bf16)(z.x - (float)a);
    il[e] = (__bf16)(z.y - (float)b);
  }
  static __device__ __forceinline__ floatx4 mma(V a, V b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

template <>
struct SplitOp<MDD_PREC_BF16> {
  using V = bf16x8;
  V rh, rl, ih, il;
  __device__ __forceinline__ void set(int e, float2 z) {
    rh[e] = (__bf16)z.x;
    ih[e] = (__bf16)z.y;
    rl[e] = (__bf16)0.f;
    il[e] = (__bf16)0.f;
  }
  static __device__ __forceinline__ floatx4 mma(V a, V b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

template <>
struct SplitOp<MDD_PREC_FP16X3> {
  using V = halfx8;
  V rh, rl, ih, il;
  __device__ __forceinline__ void set(int e, float2 z) {  // operands are pre-scaled
    const _Float16 a = (_Float16)z.x, b = (_Float16)z.y;
    rh[e] = a;
    ih[e] = b;
    rl[e] = (_Float16)(z.x - (float)a);
    il[e] = (_Float16)(z.y - (float)b);
  }
  static __device__ __forceinline__ floatx4 mma(V a, V b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};

// acc += A * B (complex), or A^H-style when the caller passes conj(A).
template <int PREC, typename Op>
__device__ __forceinline__ void split_cmma(const Op& A, const Op& B, floatx4& re, floatx4& im) {
  using V = typename Op::V;
  const V nih = -A.ih, nil = -A.il;
  if constexpr (PREC == MDD_PREC_BF16) {
    re = Op::mma(A.rh, B.rh, re);
    re = Op::mma(nih, B.ih, re);
    im = Op::mma(A.rh, B.ih, im);
    im = Op::mma(A.ih, B.rh, im);
  } else {
    re = Op::mma(A.rh, B.rh, re);
    re = Op::mma(A.rh, B.rl, re);
    re = Op::mma(A.rl, B.rh, re);
    re = Op::mma(nih, B.ih, re);
    re = Op::mma(nih, B.il, re);
    re = Op::mma(nil, B.ih, re);
    im = Op::mma(A.rh, B.ih, im);
    im = Op::mma(A.rh, B.il, im);
    im = Op::mma(A.rl, B.ih, im);
    im = Op::mma(A.ih, B.rh, im);
    im = Op::mma(A.ih, B.rl, im);
    im = Op::mma(A.il, B.rh, im);
  }
}

// Power-of-two scale bringing max |x| near 2^14 (fp16 split keeps 22 bits
// for entries down to ~2^-8 of the tile maximum).
__device__ __forceinline__ float pow2_scale(float amax) {
  if (!(amax > 0.f) || !(amax < 3.0e38f)) return 1.f;
  int e;
  frexpf(amax, &e);  // amax = m 2^e, m in [0.5, 1)
  return ldexpf(1.f, 14 - e);
}

template <int PREC, int NBT, int TNB>
struct GemmCfg {
  static constexpr int MB = NBT * 16;                 // padded batch rows
  static constexpr int NW = TNB * 16;                 // columns per workgroup
  static constexpr int TILES = NBT * TNB;             // 16x16 output tiles of the forward product
  static constexpr int S = TILES >= 4 ? 1 : 4 / TILES;  // waves splitting K
  static constexpr int G = 4 / S;                     // wave groups over tiles
  static constexpr int TPWV = TILES / G;              // tiles per wave
  static constexpr int KSTEP = 32;                    // receivers per MFMA
  static constexpr int KCMAX = NBT == 1 ? 256 : (NBT == 2 ? 128 : 64);  // receiver chunk
  static constexpr int KSW = KCMAX / KSTEP / S;       // k-steps per wave per chunk
  static constexpr int BREG = 8;                      // right-operand values per lane per k-step
  static constexpr int DST = KCMAX + 2;               // LDS row stride of D (16-byte aligned)
  static constexpr int RST = NW + 1;                  // LDS row stride of the residual
  static constexpr int RED_SZ = S > 1 ? S * MB * NW : 0;
  static constexpr size_t SMEM = sizeof(float2) * ((size_t)MB * DST + RED_SZ + (size_t)MB * RST);
  static_assert(TILES % G == 0 && KCMAX % (KSTEP * S) == 0, "tiling");
  // Tiles of one wave share their column tile when TILES >= 4 (tile = g + t * G).
  static_assert(S > 1 || G % TNB == 0, "a wave's tiles must share one column tile");
};

template <int PREC, int NBT, int TNB, int KIND>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs a) {
  using C = GemmCfg<PREC, NBT, TNB>;
  constexpr int MB = C::MB, NW = C::NW, KCMAX = C::KCMAX, KSTEP = C::KSTEP;
  extern __shared__ float2 smem[];
  float2* s_d = smem;                       // D_{b,k} chunk [MB][DST]
  float2* s_part = s_d + MB * C::DST;       // split-K partials [S][MB][NW] (S > 1)
  float2* s_res = s_part + C::RED_SZ;       // residual [MB][RST]
  __shared__ int s_idx[MB];
  __shared__ long long s_drow[MB];          // element offset of row idx[b] of D_k (or -1)
  __shared__ double s_red[4];
  __shared__ float s_scale[4];              // fp16 split: per-chunk max-abs exchange

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;

  // Map the linear workgroup id so that the column groups of one frequency run
  // on the same XCD (dispatch is round-robin over the 8 XCDs): they share D_k.
  const int ncg = (a.nvb + TNB - 1) / TNB;
  const int total = a.nf * ncg;
  const int bid = blockIdx.x;
  const int full = (total / 8) * 8;
  const int logical = bid < full ? (bid % 8) * (total / 8) + bid / 8 : bid;
  const int k = logical / ncg, cg = logical % ncg;
  const int blk0 = cg * TNB;
  const int nchunks = (a.nr + KCMAX - 1) / KCMAX;
  const double wk = (k == 0 || 2 * k == a.nt) ? 1.0 : 2.0;
  // F element (r, blk, k, c) is at r * rowstride + (blk * nf + k) * CB + c.
  const long long rowstride = (long long)a.nvb * a.nf * CB;

  auto fill_idx = [&]() {
    for (int b = tid; b < MB; b += 256) {
      int s = -1;
      if (b < a.nb) {
        s = a.idx[b];
        if (s < 0 || s >= a.ns) s = -1;
      }
      s_idx[b] = s;
      s_drow[b] = s >= 0 ? ((long long)k * a.dns + drow_of(a, b, s)) * a.nrp : -1;
    }
    __syncthreads();
  };
  if constexpr (KIND == GK_ADJ) fill_idx();

  // Rows r0 .. r0 + lenp of D_{b,k} -> s_d (zero beyond nr and for bad indices).
  auto load_d_chunk = [&](int r0, int lenp) {
    constexpr int PAIRS = KCMAX / 2;
    for (int i = tid; i < MB * PAIRS; i += 256) {
      const int b = i / PAIRS, rr = 2 * (i % PAIRS);
      if (rr >= lenp) continue;
      const long long off = s_drow[b];
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (off >= 0 && r0 + rr < a.nr) v = *reinterpret_cast<const float4*>(a.Df + off + r0 + rr);
      s_d[b * C::DST + rr] = make_float2(v.x, v.y);
      s_d[b * C::DST + rr + 1] = make_float2(v.z, v.w);
    }
  };

  auto block_amax_scale = [&](float m) -> float {  // fp16 split: power-of-two scale of a block
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if (lane == 0) s_scale[wave] = m;
    __syncthreads();
    const float amax = fmaxf(fmaxf(s_scale[0], s_scale[1]), fmaxf(s_scale[2], s_scale[3]));
    __syncthreads();
    return pow2_scale(amax);
  };
  auto lds_amax = [&](const float2* base, int rows, int stride, int cols) -> float {
    float m = 0.f;
    for (int i = tid; i < rows * cols; i += 256) {
      const float2 z = base[(i / cols) * stride + (i % cols)];
      m = fmaxf(m, fmaxf(fabsf(z.x), fabsf(z.y)));
    }
    return m;
  };

  int last_r0 = -1;  // receiver chunk resident in s_d

  // ------------------------------------------------------------ forward
  if constexpr (KIND != GK_ADJ) {
    const int g = wave % C::G, ks = wave / C::G;
    const int nt_w = g % TNB;                       // column tile of this wave (S == 1)
    // Right operand (R_k rows of this wave's k-steps), straight from HBM into
    // registers: each load instruction reads 4 rows x 16 columns = 4 x 128 B.
    // With S > 1 every wave uses the single column tile 0.
    float2 bfr[C::KSW][C::BREG];
    const int ncol_blk = blk0 + (C::S == 1 ? nt_w : 0);
    auto load_b = [&](int r0, int len) {
      const int rr0 = ks * KSTEP + lq * 8;
      const float2* fb =
          a.F + (r0 + rr0) * rowstride + ((long long)ncol_blk * a.nf + k) * CB + lr;
      const bool colok = ncol_blk < a.nvb;
#pragma unroll
      for (int q = 0; q < C::KSW; ++q) {
#pragma unroll
        for (int e = 0; e < C::BREG; ++e) {
          const int dr = q * C::S * KSTEP + e;     // row offset from rr0
          float2 v = make_float2(0.f, 0.f);
          if (colok && rr0 + dr < len) v = fb[dr * rowstride];
          bfr[q][e] = v;
        }
      }
    };
    load_b(0, min(KCMAX, a.nr));   // issued before the batch indices are known
    fill_idx();
    float2 upre[C::TPWV][4];                        // data entries subtracted later (S == 1)
    float2 upre_s[(MB * NW + 255) / 256];           // the same for S > 1
    if constexpr (KIND == GK_FUSED && C::S > 1) {
#pragma unroll
      for (int q = 0; q < (MB * NW + 255) / 256; ++q) {
        const int i = tid + 256 * q;
        const int row = i / NW, col = i % NW;
        const int vs = blk0 * CB + col;
        upre_s[q] = make_float2(0.f, 0.f);
        if (i < MB * NW && row < a.nb && vs < a.nvs && s_idx[row] >= 0)
          upre_s[q] = a.Uf[urow_off(a, k, row, s_idx[row]) + vs];
      }
    }
    if constexpr (KIND == GK_FUSED && C::S == 1) {
#pragma unroll
      for (int t = 0; t < C::TPWV; ++t) {
        const int mt = (g + t * C::G) / TNB;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = mt * 16 + lq * 4 + e, vs = (blk0 + nt_w) * CB + lr;
          upre[t][e] = make_float2(0.f, 0.f);
          if (row < a.nb && vs < a.nvs && s_idx[row] >= 0)
            upre[t][e] = a.Uf[urow_off(a, k, row, s_idx[row]) + vs];
        }
      }
    }
    floatx4 acc_re[C::TPWV], acc_im[C::TPWV];
#pragma unroll
    for (int t = 0; t < C::TPWV; ++t) {
      acc_re[t] = floatx4{0.f, 0.f, 0.f, 0.f};
      acc_im[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    for (int r0 = 0; r0 < a.nr; r0 += KCMAX) {
      const int len = min(KCMAX, a.nr - r0);
      const int lenp = (len + 31) & ~31;
      if (r0 > 0) {
        load_b(r0, len);
        __syncthreads();
      }
      load_d_chunk(r0, lenp);
      last_r0 = r0;
      __syncthreads();
      float fp16_sd = 1.f, fp16_sr = 1.f;
      floatx4 cre[C::TPWV], cim[C::TPWV];             // fp16 split: per-chunk accumulators
      if constexpr (PREC == MDD_PREC_FP16X3) {
        fp16_sd = block_amax_scale(lds_amax(s_d, MB, C::DST, lenp));
        float m = 0.f;
#pragma unroll
        for (int q = 0; q < C::KSW; ++q)
#pragma unroll
          for (int e = 0; e < C::BREG; ++e)
            m = fmaxf(m, fmaxf(fabsf(bfr[q][e].x), fabsf(bfr[q][e].y)));
        fp16_sr = block_amax_scale(m);
#pragma unroll
        for (int t = 0; t < C::TPWV; ++t) {
          cre[t] = floatx4{0.f, 0.f, 0.f, 0.f};
          cim[t] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
      }
#pragma unroll
      for (int q = 0; q < C::KSW; ++q) {
        const int kk = ks + q * C::S;
        if (kk * KSTEP >= lenp) break;
        using Op = SplitOp<PREC>;
        Op B;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float2 rv = bfr[q][e];
          if constexpr (PREC == MDD_PREC_FP16X3) rv = cscale(rv, fp16_sr);
          B.set(e, rv);
        }
#pragma unroll
        for (int t = 0; t < C::TPWV; ++t) {
          const int mt = (g + t * C::G) / TNB;
          Op A;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float2 dv = s_d[(mt * 16 + lr) * C::DST + kk * 32 + lq * 8 + e];
            if constexpr (PREC == MDD_PREC_FP16X3) dv = cscale(dv, fp16_sd);
            A.set(e, dv);
          }
          if constexpr (PREC == MDD_PREC_FP16X3) split_cmma<PREC>(A, B, cre[t], cim[t]);
          else split_cmma<PREC>(A, B, acc_re[t], acc_im[t]);
        }
      }
      if constexpr (PREC == MDD_PREC_FP16X3) {
        const float inv = 1.f / (fp16_sd * fp16_sr);
#pragma unroll
        for (int t = 0; t < C::TPWV; ++t) {
          acc_re[t] += cre[t] * inv;
          acc_im[t] += cim[t] * inv;
        }
      }
    }

    // Residual (or predicted data) and the loss partial.
    double lpart = 0.0;
    if constexpr (C::S == 1) {
#pragma unroll
      for (int t = 0; t < C::TPWV; ++t) {
        const int mt = (g + t * C::G) / TNB;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = mt * 16 + lq * 4 + e, col = nt_w * 16 + lr;
          const int vs = blk0 * CB + col;
          const bool ok = row < a.nb && vs < a.nvs && s_idx[row] >= 0;
          float2 z = make_float2(acc_re[t][e], acc_im[t][e]);
          if constexpr (KIND == GK_FUSED) {
            if (ok) {
              z = csub(z, upre[t][e]);
              lpart += wk * ((double)z.x * z.x + (double)z.y * z.y);
            } else {
              z = make_float2(0.f, 0.f);
            }
            s_res[row * C::RST + col] = z;
          } else {
            if (row < a.nb && blk0 + nt_w < a.nvb)
              a.Bsp[(((size_t)row * a.nvb + blk0 + nt_w) * a.nf + k) * CB + lr] =
                  ok ? z : make_float2(0.f, 0.f);
          }
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < C::TPWV; ++t) {
        const int tile = g + t * C::G;
        const int mt = tile / TNB, nt = tile % TNB;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = mt * 16 + lq * 4 + e, col = nt * 16 + lr;
          s_part[(ks * MB + row) * NW + col] = make_float2(acc_re[t][e], acc_im[t][e]);
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < (MB * NW + 255) / 256; ++q) {
        const int i = tid + 256 * q;
        if (i >= MB * NW) break;
        const int row = i / NW, col = i % NW;
        float2 z = s_part[row * NW + col];
#pragma unroll
        for (int s = 1; s < C::S; ++s) z = cadd(z, s_part[(s * MB + row) * NW + col]);
        const int vs = blk0 * CB + col;
        const bool ok = row < a.nb && vs < a.nvs && s_idx[row] >= 0;
        if constexpr (KIND == GK_FUSED) {
          if (ok) {
            z = csub(z, upre_s[q]);
            lpart += wk * ((double)z.x * z.x + (double)z.y * z.y);
          } else {
            z = make_float2(0.f, 0.f);
          }
          s_res[row * C::RST + col] = z;
        } else {
          const int blk = blk0 + col / 16;
          if (row < a.nb && blk < a.nvb)
            a.Bsp[(((size_t)row * a.nvb + blk) * a.nf + k) * CB + (col & 15)] =
                ok ? z : make_float2(0.f, 0.f);
        }
      }
    }
    if constexpr (KIND == GK_FUSED) {
      const double tot = block_sum256(lpart, s_red);
      if (tid == 0) a.loss_part[logical] = tot;
    }
    if constexpr (KIND == GK_FWD) return;
  } else {
    // Adjoint only: the batch spectra V_k are the right-hand operand.
    for (int i = tid; i < MB * NW; i += 256) {
      const int row = i / NW, col = i % NW;
      const int blk = blk0 + col / 16;
      float2 z = make_float2(0.f, 0.f);
      if (row < a.nb && blk < a.nvb && s_idx[row] >= 0)
        z = a.Bsp[(((size_t)row * a.nvb + blk) * a.nf + k) * CB + (col & 15)];
      s_res[row * C::RST + col] = z;
    }
  }
  __syncthreads();

  // ------------------------------------------------------------ adjoint
  float fp16_ss = 1.f;
  if constexpr (PREC == MDD_PREC_FP16X3)
    fp16_ss = block_amax_scale(lds_amax(s_res, MB, C::RST, NW));
  for (int r0 = 0; r0 < a.nr; r0 += KCMAX) {
    const int len = min(KCMAX, a.nr - r0);
    const int lenp = (len + 31) & ~31;
    if (!(nchunks == 1 && last_r0 == r0)) {   // the single chunk is still resident
      if (r0 > 0) __syncthreads();
      load_d_chunk(r0, lenp);
      __syncthreads();
    }
    float fp16_sd = 1.f;
    if constexpr (PREC == MDD_PREC_FP16X3) fp16_sd = block_amax_scale(lds_amax(s_d, MB, C::DST, lenp));
    for (int mt = wave; mt * 16 < len; mt += 4) {
#pragma unroll
      for (int nt = 0; nt < TNB; ++nt) {
        floatx4 re = floatx4{0.f, 0.f, 0.f, 0.f}, im = floatx4{0.f, 0.f, 0.f, 0.f};
        using Op = SplitOp<PREC>;
#pragma unroll
        for (int kk = 0; kk < (MB + 31) / 32; ++kk) {
          Op A, B;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int b = kk * 32 + lq * 8 + e;
            float2 dv = make_float2(0.f, 0.f), sv = make_float2(0.f, 0.f);
            if (b < MB) {
              dv = cconj(s_d[b * C::DST + mt * 16 + lr]);
              sv = s_res[b * C::RST + nt * 16 + lr];
            }
            if constexpr (PREC == MDD_PREC_FP16X3) {
              dv = cscale(dv, fp16_sd);
              sv = cscale(sv, fp16_ss);
            }
            A.set(e, dv);
            B.set(e, sv);
          }
          split_cmma<PREC>(A, B, re, im);
        }
        if constexpr (PREC == MDD_PREC_FP16X3) {
          const float inv = 1.f / (fp16_sd * fp16_ss);
          re *= inv;
          im *= inv;
        }
        const int blk = blk0 + nt;
        if (blk < a.nvb) {
          const int rb = r0 + mt * 16 + lq * 4;
          float2* fw = a.F + rb * rowstride + ((long long)blk * a.nf + k) * CB + lr;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (rb + e < a.nr) store_g(a, (fw - a.F) + e * rowstride, make_float2(re[e], im[e]));
        }
      }
    }
  }
}

template <int PREC, int NBT, int TNB>
hipError_t launch_cfg(int kind, const GemmArgs& a, hipStream_t s) {
  using C = GemmCfg<PREC, NBT, TNB>;
  const int ncg = (a.nvb + TNB - 1) / TNB;
  const dim3 grid(a.nf * ncg), block(256);
  const size_t sm = C::SMEM;
  switch (kind) {
    case GK_FUSED:
      if (sm > 65536)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm<PREC, NBT, TNB, GK_FUSED>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
      hipLaunchKernelGGL((k_gemm<PREC, NBT, TNB, GK_FUSED>), grid, block, sm, s, a);
      break;
    case GK_FWD:
      if (sm > 65536)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm<PREC, NBT, TNB, GK_FWD>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
      hipLaunchKernelGGL((k_gemm<PREC, NBT, TNB, GK_FWD>), grid, block, sm, s, a);
      break;
    case GK_ADJ:
      if (sm > 65536)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm<PREC, NBT, TNB, GK_ADJ>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
      hipLaunchKernelGGL((k_gemm<PREC, NBT, TNB, GK_ADJ>), grid, block, sm, s, a);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Column groups of one frequency in the tiled kernel.
int tiled_groups(int nb, int nvb) {
  const int tnb = nb <= 16 ? 1 : (nb <= 32 ? 2 : 4);
  return (nvb + tnb - 1) / tnb;
}

template <int PREC>
hipError_t launch_prec(int kind, const GemmArgs& a, hipStream_t s) {
  if constexpr (PREC == MDD_PREC_BF16) {
    if (a.nb <= 16) return launch_cfg<PREC, 1, 1>(kind, a, s);
    if (a.nb <= 32) return launch_cfg<PREC, 2, 2>(kind, a, s);
    return launch_cfg<PREC, 4, 4>(kind, a, s);
  } else {
    if (a.nb > 16 || (kind == GK_FUSED && a.nr <= SPLIT_PIPE_KC))
      return launch_gemm_split(kind, PREC, a, s);  // operands split once, in LDS
    return launch_cfg<PREC, 1, 1>(kind, a, s);
  }
}

}  // namespace

int gemm_loss_parts(int precision, int nb, int nvb) {
  const bool fp32 = precision == MDD_PREC_FP32 || precision == MDD_PREC_FP32_CGEMM;
  return fp32 ? nvb : tiled_groups(nb, nvb);
}

hipError_t launch_gemm(int kind, int precision, const GemmArgs& a, hipStream_t s) {
  if (a.nb <= 0 || a.nb > NB_LIMIT) return hipErrorInvalidValue;
  switch (precision) {
    case MDD_PREC_FP32:
    case MDD_PREC_FP32_CGEMM: return launch_gemm_rows(kind, precision, a, s);
    case MDD_PREC_BF16X3: return launch_prec<MDD_PREC_BF16X3>(kind, a, s);
    case MDD_PREC_FP16X3: return launch_prec<MDD_PREC_FP16X3>(kind, a, s);
    case MDD_PREC_BF16: return launch_prec<MDD_PREC_BF16>(kind, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mdd
