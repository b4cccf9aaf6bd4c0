// Float32 per-frequency products with one wavefront per 16-column block (every kind,
// every batch size):
//
//   Res_k = D_{b,k} R_k - U_{b,k}      ([nb x nr] [nr x nvs])
//   G_k   = D_{b,k}^H Res_k            ([nr x nb] [nb x nvs]), written over R_k
//
// A workgroup is up to NW wavefronts on neighbouring 16-column blocks of one frequency,
// which share the rows of D_{b,k} in LDS.  Everything else belongs to one wavefront: it
// streams its block of R_k from HBM straight into MFMA operand registers, one receiver
// chunk ahead of the products, keeps the residual block [16 NBT batch rows x 16 columns]
// in the accumulators, and uses those as the right operand of the adjoint product.  No
// value changes lanes in between: the forward product leaves batch row 4 q + e of a tile
// in lane quarter q, element e, and the adjoint's k-step e takes exactly row 4 q + e from
// lane quarter q (the order of the batch rows in that sum is free, so the left operand is
// read from LDS in the same order).  The residual needs neither LDS nor a barrier.
//
// What bounds it: the float32 matrix unit at 33 and more batch rows, the traffic of R_k and
// G_k and the latency of their first and last accesses below.  Measured (fused kind,
// float32, HIP events; before: tiled, persistent and loader / compute wavefront kernels):
//   nr = nvs   nb   nf    before     now
//      1600    64  200   4394 us  3673 us   143 TFLOP/s of the method's 8 flops per complex
//                                           multiply-add; matrix unit 68 % busy
//       400    48  200    396 us   233 us
//       301    64  257    301 us   220-238 us
//       301    32  257    260 us   127-135 us (forward and adjoint kinds 135 + 123 -> 67 + 68)
//       201    32  257    132 us    74-76 us
//       201    16  257     54 us    45 us   172 MB of R_k and G_k: 3.8 TB/s
// Without the compensated sums the first takes 3513 us, without the staging of D 3319 us
// (timing only): both are vector work, which the float32 matrix unit does not overlap with.
#include <type_traits>

#include "device_common.h"
#include "mdd_internal.h"

namespace mdd {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Left operand of one lane, z = x + i y, prepared once when D is staged, because a vector
// addition between two products holds up the float32 matrix unit for about six cycles
// whatever the occupancy (in a loop of 16x16x4 products alone 155 TFLOP/s; with four
// additions per three products 125).
//   MDD_PREC_FP32: three real products per complex one, (x, x + y, y - x)
//   MDD_PREC_FP32_CGEMM: the four of a plain complex product, (x, y, -y)
struct alignas(16) Left {
  float x, y, z;
};
template <int PREC>
__device__ __forceinline__ Left left_of(float2 v) {
  if constexpr (PREC == MDD_PREC_FP32) return {v.x, v.x + v.y, v.y - v.x};
  else return {v.x, v.y, -v.y};
}

// Accumulators of one complex 16 x 16 tile.  FP32: with A = a + ib, B = c + id,
//   t1 += a (c + d),  t2 += (a + b) d,  t3 += (b - a) c;   Re = t1 - t2, Im = t1 + t3
// and for conj(A):  t1 += a (c + d),  t2 += (b - a) d,  t3 += (a + b) c;
//   Re = t1 + t2, Im = t1 - t3.
// CGEMM: t2 and t3 are Re and Im themselves, t1 is unused.
struct Tile {
  floatx4 t1, t2, t3;
};
template <int PREC>
__device__ __forceinline__ void mac(Left a, float2 b, float bsum, Tile& t, bool fresh = false) {
  if constexpr (PREC == MDD_PREC_FP32) {
    t.t1 = mfma4(a.x, bsum, fresh ? floatx4{0.f, 0.f, 0.f, 0.f} : t.t1);
    t.t2 = mfma4(a.y, b.y, t.t2);
    t.t3 = mfma4(a.z, b.x, t.t3);
  } else {
    t.t2 = mfma4(a.x, b.x, t.t2);
    t.t3 = mfma4(a.x, b.y, t.t3);
    t.t2 = mfma4(a.z, b.y, t.t2);
    t.t3 = mfma4(a.y, b.x, t.t3);
  }
}
template <int PREC>
__device__ __forceinline__ void mac_conj(Left a, float2 b, float bsum, Tile& t) {
  if constexpr (PREC == MDD_PREC_FP32) {
    t.t1 = mfma4(a.x, bsum, t.t1);
    t.t2 = mfma4(a.z, b.y, t.t2);
    t.t3 = mfma4(a.y, b.x, t.t3);
  } else {
    t.t2 = mfma4(a.x, b.x, t.t2);
    t.t3 = mfma4(a.x, b.y, t.t3);
    t.t2 = mfma4(a.y, b.y, t.t2);
    t.t3 = mfma4(a.z, b.x, t.t3);
  }
}

// Adds a group's sum to the running total with the rounding error of that addition kept
// (Kahan's compensated sum): the error goes in front of the next group's products, as
// the value their accumulators start from.  Each group of 64 receivers (32 at up to 16 batch
// rows) starts near zero, so the products' rounding grows with the group and not with nr.
template <int PREC>
__device__ __forceinline__ void fold(Tile& t, floatx4& re, floatx4& im) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float xr = PREC == MDD_PREC_FP32 ? t.t1[i] - t.t2[i] : t.t2[i];
    const float xi = PREC == MDD_PREC_FP32 ? t.t1[i] + t.t3[i] : t.t3[i];
    const float sr = re[i] + xr, si = im[i] + xi;
    if constexpr (PREC == MDD_PREC_FP32) {
      t.t2[i] = (sr - re[i]) - xr;                // subtracted
      t.t3[i] = xi - (si - im[i]);
    } else {
      // Beside an infinite sum the error is inf - inf: the median of a NaN and two bounds is the
      // lower one, which changes no infinity.  A finite sum's error is below 2^104.
      t.t2[i] = __builtin_amdgcn_fmed3f(xr - (sr - re[i]), -0x1p104f, 0x1p104f);
      t.t3[i] = __builtin_amdgcn_fmed3f(xi - (si - im[i]), -0x1p104f, 0x1p104f);
    }
    re[i] = sr;
    im[i] = si;
  }
}

template <int NBT>
struct RowsCfg {
  static constexpr bool WIDE = NBT >= 2;          // left operands prepared in LDS (16 bytes each)
  static constexpr int KC = 32;                   // receivers per chunk
  static constexpr int SUM = NBT == 1 ? 1 : 64 / KC;  // chunks per compensated addition
  static constexpr int KS = KC / 4;               // k-steps per chunk
  static constexpr int MB = 16 * NBT;
  static constexpr int NBUF = 2;                // chunks of R_k in registers (a multiple of SUM)
  static_assert(NBUF % SUM == 0, "groups");
  // LDS row pitch: 2 mod 4 entries, with rows 4..7 and 8..11 of a tile exchanged (phys).
  // A 16-byte read is served 16 lanes at a time, lanes 0-3, 12-15 and 20-27 first: the
  // forward operand (row lr, receiver lq) then touches 8 even and 8 odd 16-byte banks, and
  // the adjoint's (row 4 lq + e, receiver lr) 16 different ones, rows 4 apart being 8 apart
  // in LDS.
  static constexpr int DP = KC + 2;
  static constexpr int SLOT = MB * DP;            // entries per chunk
  static constexpr int ESZ = WIDE ? 16 : 8;
  static __device__ __forceinline__ int phys(int i) {
    return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1);
  }
};

// Wavefronts per SIMD that the registers are cut for.  At up to 16 rows five where D is resident
// (the three-product fused form spills one register so: 230 to 260 receivers 1 % faster than
// with four, 300 the same) and four where its chunks come in turn (with five 9 registers were
// spilled: 700 receivers, 2600 blocks 134 us with five, 116 with four).
constexpr int waves_per_simd(int nbt, int kind, bool rec, bool res, int np) {
  if (np > 1) return kind == GK_FUSED && !res ? 3 : 4;
  if (nbt > 1) return nbt >= 3 || (rec && kind == GK_FWD) ? 2 : 3;
  if (rec) return res ? 4 : 3;
  return res ? 5 : 4;
}

// ACC: the adjoint product is added to what Gout holds (a sum over batches).
//
// REC: with the reciprocity average C_r (nr = nvs) folded in, forward and adjoint kinds.
//   Forward: the right operand is R_k + R_k^T, its mirrored entries read beside the direct
//   ones; the result is halved, which is exact.
//   Adjoint: (G + G^T)(r, v) = sum_b conj(D[b, r]) V[b, v] + V[b, r] conj(D[b, v]), the same
//   product over twice the rows: D and conj(V) on the left (conj(V) staged beside D), V and
//   conj(D) of this block's columns on the right.
// Bound by traffic: the forward form reads R_k twice (the second time from the caches where
// it can), the adjoint's doubled rows cost matrix work.  At 301 traces and 257 bins, with the
// pass over the spectra that this saves (64 to 88 us; forward + adjoint, us):
//   batch  8: 45 + 70, 49 + 70 -> 64, 53      batch 32: 67 + 80, 68 + 80 -> 87, 118
//   batch 16: 46 + 70, 49 + 70 -> 69, 72      batch 64: 110 + 88 -> 140 (forward)
//
// NP = 4 (up to 16 batch rows, few column blocks): the four wavefronts of a workgroup share one
// block.  Wavefront p takes the receiver chunks p, p + 4, ... of both products, staged by
// itself in LDS slots of its own; in between the four add their sums through LDS, so that each
// holds the residual.
template <int PREC, int NBT, int KIND, bool ACC, bool REC, bool RES, int NW, int NP>
__global__ __launch_bounds__(64 * NW * NP)
__attribute__((amdgpu_waves_per_eu(waves_per_simd(NBT, KIND, REC, RES, NP))))
void k_gemm_rows(GemmArgs a, int nslot) {
  using C = RowsCfg<NBT>;
  using E = std::conditional_t<C::WIDE, Left, float2>;
  constexpr int KC = C::KC, KS = C::KS, MB = C::MB, DP = C::DP, SLOT = C::SLOT;
  constexpr int NBUF = C::NBUF, NTH = 64 * NW;
  constexpr int FPT = MB * (KC / 2) / NTH;        // receiver pairs of a D chunk per thread
  static_assert(FPT * NTH == MB * (KC / 2), "split");
  constexpr bool RFWD = REC && KIND == GK_FWD, RADJ = REC && KIND == GK_ADJ;
  constexpr int HALF = RADJ ? MB / 2 : MB;        // rows of D; the others are conj(V)'s
  static_assert(!REC || (PREC == MDD_PREC_FP32 && KIND != GK_FUSED), "reciprocity");
  static_assert(NP == 1 || (NW == 1 && !REC), "a wavefront without a block would miss a barrier");
  extern __shared__ __align__(16) char s_raw[];

  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = NP == 1 ? wid : 0, part = NP == 1 ? 0 : wid;
  const int tid = threadIdx.x - 64 * part, lane = tid & 63;
  E* const s_d = reinterpret_cast<E*>(s_raw) + part * nslot * SLOT;  // nslot chunks of D [row][receiver]
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
  // this wavefront's chunks c = 0 .. nc - 1 are the receivers' chunks NP c + part
  const int nr = a.nr, nc = (nr + NP * KC - 1) / (NP * KC);
  auto chunk = [&](int c) { return NP * c + part; };

  // R_k rows of a chunk -> registers (the right operand's layout: k-step q, lane quarter
  // lq is receiver rstep(q) + RQ lq of the chunk); rows at or past nr are out of bounds: zeros.
  constexpr int RQ = RFWD ? 2 : 1;
  auto rstep = [](int q) { return q / RQ * 4 * RQ + q % RQ; };
  const long long col = ((long long)blk * a.nf + k) * CB;
  unsigned roff[KS];
#pragma unroll
  for (int q = 0; q < KS; ++q) roff[q] = ((unsigned)(rstep(q) + RQ * lq) * rs32 + lr) * 8u;
  // The spectra of up to KC receivers from r0 on, seen from this block's column: what lies
  // past receiver nr is out of bounds (32 rows of at most 256 blocks x 513 bins fit 32 bits).
  auto rows_at = [&](float2* base, int r0, int rows) {
    const int n = max(min(nr - r0, rows), 0);
    return buffer_at(base + r0 * rowstride + col, n ? (unsigned)n * rs32 * 8u - (unsigned)col * 8u : 0u);
  };
  auto load_r = [&](float2 (&dst)[KS], int c) {
    const auto rb = rows_at(a.F, chunk(c) * KC, KC);
#pragma unroll
    for (int q = 0; q < KS; ++q) dst[q] = buffer_get2(rb, roff[q]);
  };
  // The forward product's order over the chunks.  With reciprocity at up to 16 batch rows it
  // alternates around the workgroup's own columns: a mirrored entry is then a direct one of
  // another workgroup's next or last chunk, and still in L2 (301 traces, 8 rows: 76 -> 67 us;
  // with more rows fewer frequencies are under way at once and the order makes no difference).
  const int c0 = blk0 * CB / KC;
  auto ord = [&](int v) {
    if constexpr (!RFWD || NBT > 1) return v;
    const int c = c0 + ((v & 1) ? (v + 1) / 2 : nc - v / 2);
    return v >= nc ? nc : c >= nc ? c - nc : c;
  };
  // The mirrored entries: column lr of this block as a row, RQ neighbouring receivers of the
  // chunk as columns, zeros past receiver nr (what the padding columns of a block hold is not
  // known to be finite).
  unsigned toff[RFWD ? KS / 2 : 1];
  if constexpr (RFWD) {
#pragma unroll
    for (int q = 0; q < KS / 2; ++q) {
      const int r = rstep(2 * q) + RQ * lq;
      toff[q] = ((unsigned)lr * rs32 + (unsigned)(r / CB * a.nf * CB + r % CB)) * 8u;
    }
  }
  auto load_t = [&](float2 (&dst)[RFWD ? KS : 1], int c) {
    if constexpr (RFWD) {
      const int tb = c * (KC / CB), in_row = (tb * a.nf + k) * CB;
      const int n = tb < a.nvb ? min(nr - blk * CB, CB) : 0;
      const auto tr = buffer_at(a.F + blk * CB * rowstride + in_row,
                                n ? (unsigned)n * rs32 * 8u - (unsigned)in_row * 8u : 0u);
#pragma unroll
      for (int q = 0; q < KS / 2; ++q) {
        const int r = rstep(2 * q) + RQ * lq, left = nr - c * KC;
        const float4 z = buffer_get4(tr, r < left ? toff[q] : PAST_END);
        dst[2 * q] = make_float2(z.x, z.y);
        dst[2 * q + 1] = r + 1 < left ? make_float2(z.z, z.w) : make_float2(0.f, 0.f);
      }
    }
  };
  float2 rbuf[NBUF][KS], tbuf[NBUF][RFWD ? KS : 1];
  if constexpr (KIND != GK_ADJ) {                 // in flight while the batch is looked up
#pragma unroll
    for (int i = 0; i < NBUF - 1; ++i) {
      load_r(rbuf[i], ord(i));
      load_t(tbuf[i], ord(i));
    }
  }

  // Batch rows: lane b of every wavefront holds the source of batch entry b, or -1.
  int src = -1;
  if (lane < a.nb) {
    src = a.idx[lane];
    if (src < 0 || src >= a.ns) src = -1;
  }
  const int drow = src >= 0 ? drow_of(a, lane, src) : -1;

  // The thread's receiver pairs of a chunk of D (or V); rows without a source and receivers past the
  // padded row are out of bounds: zeros.
  const char* dbase = reinterpret_cast<const char*>(a.Df + (long long)k * a.dns * a.nrp);
  const unsigned dbytes = (unsigned)a.dns * (unsigned)a.nrp * 8u;
  static_assert(!RADJ || NTH / (KC / 2) == 16, "of_v");  // a thread's rows are 16 apart,
  auto of_v = [&](int q) { return RADJ && 16 * q + 4 * wave >= HALF; };  // a wavefront's four
  unsigned doff[FPT];
#pragma unroll
  for (int q = 0; q < FPT; ++q) {
    const int i = tid + NTH * q, rr = 2 * (i % (KC / 2));
    const int b = i / (KC / 2) - (of_v(q) ? HALF : 0);
    const int row = __shfl(drow, b, 64);
    if (of_v(q))                                  // batch spectra [b][block of 16][k][16]
      doff[q] = (((unsigned)b * a.nvb + rr / CB) * a.nf + k) * (CB * 8u) + (rr % CB) * 8u;
    else
      doff[q] = ((unsigned)row * (unsigned)a.nrp + rr) * 8u;
    if (row < 0) doff[q] = PAST_END;
  }
  constexpr int DB = RES ? 8 / NP : 1;            // chunks of D requested at once
  float4 dv[DB][FPT];
  auto load_d = [&](int own, float4 (&d)[FPT]) {
    const int c = chunk(own);
    const auto db = buffer_at(dbase + (long long)c * KC * 8, dbytes - (unsigned)(c * KC) * 8u);
    const auto vb = buffer_at(a.Bsp + (long long)c * (KC / CB) * a.nf * CB,
                              RADJ ? (unsigned)(a.nb * a.nvb - c * (KC / CB)) * (unsigned)a.nf * (CB * 8u) : 0u);
    const int left_in_row = a.nrp - c * KC;
#pragma unroll
    for (int q = 0; q < FPT; ++q)
      d[q] = buffer_get4(of_v(q) ? vb : db,
                         2 * ((tid + NTH * q) % (KC / 2)) < left_in_row ? doff[q] : PAST_END);
  };
  auto stage_d = [&](int i, const float4 (&d)[FPT]) {  // the i-th chunk of the LDS slots
    E* slot = s_d + (RES ? i : i % nslot) * SLOT;
#pragma unroll
    for (int q = 0; q < FPT; ++q) {
      const int j = tid + NTH * q, b = j / (KC / 2), rr = 2 * (j % (KC / 2));
      float4 v = d[q];
      // used here and not before: hoisted above the step's products, the sums of left_of
      // would wait there for these loads and, in order, for every store before them
      asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
      if (of_v(q)) v = make_float4(v.x, -v.y, v.z, -v.w);
      E* p = slot + C::phys(b) * DP + rr;
      if constexpr (C::WIDE) {
        p[0] = left_of<PREC>(make_float2(v.x, v.y));
        p[1] = left_of<PREC>(make_float2(v.z, v.w));
      } else {
        *reinterpret_cast<float4*>(p) = v;
      }
    }
  };
  auto left = [&](E z) -> Left {
    if constexpr (C::WIDE) return z;
    else return left_of<PREC>(z);
  };
  // Chunk visited at step v of the launch: 0 .. nc - 1 for the forward product, then back
  // down for the adjoint, which finds the last nslot chunks still in LDS.
  constexpr bool FWD = KIND != GK_ADJ;
  const int v0 = FWD ? 0 : nc, v1 = KIND == GK_FWD ? nc : 2 * nc;
  auto chunk_of = [&](int v) { return v < nc ? ord(v) : max(2 * nc - 1 - v, 0); };
  auto staged_at = [&](int v) {                   // step v needs its chunk brought in
    return v < v1 && (v < nc || !FWD || v >= nc + nslot);
  };
  // End of step v: the next step's chunk goes to LDS, the one after that is requested.
  auto advance = [&](int v) {
    if constexpr (!RES) {
      if (staged_at(v + 1)) stage_d(RFWD ? v + 1 : chunk_of(v + 1), dv[0]);
      load_d(chunk_of(v + 2), dv[0]);
      __syncthreads();
    }
  };

  // Data (or the adjoint's operand) entries of the lane: batch row 16 t + 4 lq + e.
  unsigned okrow = 0;                             // bit 4 t + e: the entry counts
  float2 upre[NBT][4];
  auto load_u = [&]() {
#pragma unroll
    for (int t = 0; t < NBT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = t * 16 + lq * 4 + e, row = i < HALF ? i : i - HALF;
        const int s = __shfl(src, row, 64), rowc = min(row, a.nb - 1);
        if (s >= 0 && blk * CB + lr < a.nvs) okrow |= 1u << (4 * t + e);
        if constexpr (RADJ) {                     // V, or conj(D) of this block's columns
          const int dr = max(__shfl(drow, row, 64), 0);
          const float2* pv = a.Bsp + (((size_t)rowc * a.nvb + blk) * a.nf + k) * CB + lr;
          const float2* pd = a.Df + ((long long)k * a.dns + dr) * a.nrp + blk * CB + lr;
          const float2 z = *(i < HALF ? pv : pd);
          upre[t][e] = make_float2(z.x, i < HALF ? z.y : -z.y);
        }
        else if constexpr (KIND == GK_ADJ)
          upre[t][e] = a.Bsp[(((size_t)rowc * a.nvb + blk) * a.nf + k) * CB + lr];
        else if constexpr (KIND == GK_FUSED)
          upre[t][e] = a.Uf[urow_off(a, k, rowc, max(s, 0)) + blk * CB + lr];
      }
  };
  if constexpr (!RES) load_d(chunk_of(v0), dv[0]);
  if constexpr (NBT < 3 || KIND != GK_FUSED) load_u();
  if constexpr (RES) {
#pragma unroll 1
    for (int c0 = 0; c0 < nc; c0 += DB) {
#pragma unroll
      for (int i = 0; i < DB; ++i) load_d(c0 + i, dv[i]);
#pragma unroll
      for (int i = 0; i < DB; ++i)
        if (c0 + i < nc) stage_d(c0 + i, dv[i]);
    }
  } else {
    stage_d(RFWD ? 0 : chunk_of(v0), dv[0]);
    load_d(chunk_of(v0 + 1), dv[0]);
  }
  __syncthreads();

  if (!active) {                                  // a wavefront without a block stages D only
    if constexpr (!RES) {
#pragma unroll 1
      for (int v = v0; v < v1; ++v)
        if (v < nc || !FWD || staged_at(v + 1) || staged_at(v + 2)) advance(v);
    }
    return;
  }

  floatx4 re[NBT], im[NBT];
  if constexpr (FWD) {
    Tile acc[NBT];
#pragma unroll
    for (int t = 0; t < NBT; ++t) {
      const floatx4 z = {0.f, 0.f, 0.f, 0.f};
      re[t] = im[t] = acc[t].t1 = acc[t].t2 = acc[t].t3 = z;
    }
    const E* dl = s_d + C::phys(lr) * DP + RQ * lq;
    // U: v modulo NBUF, which says whether step v begins or ends a group of SUM chunks
    auto step = [&](int v, auto U, float2 (&cur)[KS], float2 (&nxt)[KS]) {
      load_r(nxt, ord(v + NBUF - 1));
      load_t(tbuf[(U + NBUF - 1) % NBUF], ord(v + NBUF - 1));
      // left operands G k-steps at a time, read from LDS one group ahead of their products
      constexpr int G = NBT >= 3 ? 1 : 2;
      const E* dsl = dl + (RES ? ord(v) : v % nslot) * SLOT;
      E av[2][G][NBT];
      auto read_a = [&](int g) {
#pragma unroll
        for (int q = 0; q < G; ++q)
#pragma unroll
          for (int t = 0; t < NBT; ++t) av[g & 1][q][t] = dsl[t * 16 * DP + rstep(G * g + q)];
      };
      read_a(0);
#pragma unroll
      for (int g = 0; g < KS / G; ++g) {
        if (g + 1 < KS / G) read_a(g + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < G; ++q) {
          float2 bv = cur[G * g + q];
          if constexpr (RFWD) bv = cadd(bv, tbuf[U][G * g + q]);
          const float bsum = bv.x + bv.y;
#pragma unroll
          for (int t = 0; t < NBT; ++t) mac<PREC>(left(av[g & 1][q][t]), bv, bsum, acc[t], U % C::SUM == 0 && g + q == 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if ((U + 1) % C::SUM == 0 || v + 1 == nc) {
#pragma unroll
        for (int t = 0; t < NBT; ++t) fold<PREC>(acc[t], re[t], im[t]);
      }
      advance(v);
    };
    int v = 0;
    while (true) {
      step(v, std::integral_constant<int, 0>{}, rbuf[0], rbuf[NBUF - 1]);
      if (++v == nc) break;
      step(v, std::integral_constant<int, 1>{}, rbuf[1], rbuf[0]);
      if (++v == nc) break;
    }
    if constexpr (KIND == GK_FUSED && NBT >= 3) load_u();
    if constexpr (NP > 1) {  // the parts' sums with what they lack, in order: one rounding in all
      __shared__ double2 s_sum[NP][MB][16];
#pragma unroll
      for (int t = 0; t < NBT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double er = PREC == MDD_PREC_FP32 ? -acc[t].t2[e] : acc[t].t2[e];
          s_sum[part][t * 16 + lq * 4 + e][lr] = make_double2(re[t][e] + er, im[t][e] + (double)acc[t].t3[e]);
        }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NBT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          double2 z = s_sum[0][t * 16 + lq * 4 + e][lr];
#pragma unroll
          for (int p = 1; p < NP; ++p) {
            const double2 y = s_sum[p][t * 16 + lq * 4 + e][lr];
            z.x += y.x;
            z.y += y.y;
          }
          re[t][e] = (float)z.x;
          im[t][e] = (float)z.y;
        }
    } else {
#pragma unroll
      for (int t = 0; t < NBT; ++t) {               // the last compensation
        if constexpr (PREC == MDD_PREC_FP32) re[t] -= acc[t].t2;
        else re[t] += acc[t].t2;
        im[t] += acc[t].t3;
      }
    }
  }

  // residual and float64 loss partial (or predicted data, or the adjoint's operand)
  double lpart = 0.0;
#pragma unroll
  for (int t = 0; t < NBT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = t * 16 + lq * 4 + e;
      float2 z = KIND == GK_ADJ ? upre[t][e] : make_float2(re[t][e], im[t][e]);
      if constexpr (KIND == GK_FUSED) z = csub(z, upre[t][e]);
      if (!((okrow >> (4 * t + e)) & 1)) z = make_float2(0.f, 0.f);
      if constexpr (KIND == GK_FUSED) lpart += (double)z.x * z.x + (double)z.y * z.y;
      if constexpr (KIND == GK_FWD) {
        if constexpr (REC) z = cscale(z, 0.5f);
        if (row < a.nb && part == 0) a.Bsp[(((size_t)row * a.nvb + blk) * a.nf + k) * CB + lr] = z;
      }
      re[t][e] = z.x;
      im[t][e] = z.y;
    }
  if constexpr (KIND == GK_FUSED) {
    lpart = wave_sum(lpart);
    if (lane == 0 && part == 0) a.loss_part[k * a.nvb + blk] = lpart * (k == 0 || 2 * k == a.nt ? 1.0 : 2.0);
  }
  if constexpr (KIND == GK_FWD) return;

  // adjoint: G_k = D_b^H Res, 16 receivers at a time, written over R_k (or into Gout)
  float2* gbase = a.Gout ? a.Gout : a.F;
  unsigned goff[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) goff[e] = ((unsigned)(4 * lq + e) * rs32 + lr) * 8u;
  floatx4 sum[NBT];
#pragma unroll
  for (int t = 0; t < NBT; ++t) sum[t] = re[t] + im[t];
  auto visit = [&](int v, auto partial) {         // the first chunk may end inside
    const int c = chunk_of(v);
    const E* da = s_d + (RES ? c : c % nslot) * SLOT + C::phys(4 * lq) * DP + lr;
    constexpr int NG = (KC / 16) * NBT;           // groups of four k-steps: (tile, row block)
    E av[2][4];                                   // left operands, read one group ahead
    auto read_a = [&](int g) {
#pragma unroll
      for (int e = 0; e < 4; ++e) av[g & 1][e] = da[((g % NBT) * 16 + e) * DP + (g / NBT) * 16];
    };
    read_a(0);
#pragma unroll
    for (int m = 0; m < KC / 16; ++m) {
      const int r0 = chunk(c) * KC + m * 16;
      const auto gb = rows_at(gbase, r0, 16);
      float2 old[4];
      if constexpr (ACC) {
#pragma unroll
        for (int e = 0; e < 4; ++e) old[e] = buffer_get2(gb, goff[e]);
      }
      Tile acc;
      const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
      acc.t1 = acc.t2 = acc.t3 = zero;
      // a tile past nr has no products; its stores are issued all the same (and dropped, out
      // of bounds), so that a wait in the loop knows how many accesses are in flight
      if (!partial || r0 < nr) {
#pragma unroll
        for (int t = 0; t < NBT; ++t) {
          const int g = m * NBT + t;
          if (g + 1 < NG) read_a(g + 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            mac_conj<PREC>(left(av[g & 1][e]), make_float2(re[t][e], im[t][e]), sum[t][e], acc);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      const floatx4 gr = PREC == MDD_PREC_FP32 ? acc.t1 + acc.t2 : acc.t2;
      const floatx4 gi = PREC == MDD_PREC_FP32 ? acc.t1 - acc.t3 : acc.t3;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float2 z = make_float2(gr[e], gi[e]);
        if constexpr (REC) z = cscale(z, 0.5f);
        if constexpr (ACC) z = cadd(z, old[e]);
        buffer_put2(gb, goff[e], z);
      }
    }
    if (!RES && (!FWD || staged_at(v + 1) || staged_at(v + 2))) advance(v);
  };
  visit(nc, std::true_type{});
#pragma unroll 1
  for (int v = nc + 1; v < 2 * nc; ++v) visit(v, std::false_type{});
}

template <int PREC, int NBT, bool RES, int NW, int NP = 1>
hipError_t launch_nw(int kind, const GemmArgs& a, int nslot, hipStream_t s) {
  const size_t sm = (size_t)RowsCfg<NBT>::ESZ * RowsCfg<NBT>::SLOT * nslot * NP;
  constexpr size_t sums = NP > 1 ? sizeof(double2) * NP * RowsCfg<NBT>::MB * 16 : 0;  // the kernel's own LDS
  const int ncg = (a.nvb + NW - 1) / NW;
  const dim3 grid(a.nf * ncg), block(64 * NW * NP);
  auto go = [&](auto kernel) {
    if (sm + sums > 65536)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
    hipLaunchKernelGGL(kernel, grid, block, sm, s, a, nslot);
    return hipGetLastError();
  };
  constexpr bool R3 = PREC == MDD_PREC_FP32 && NP == 1;  // reciprocity: the three-product form only
  switch (kind) {
    case GK_FUSED:
      return a.gacc ? go(k_gemm_rows<PREC, NBT, GK_FUSED, true, false, RES, NW, NP>)
                    : go(k_gemm_rows<PREC, NBT, GK_FUSED, false, false, RES, NW, NP>);
    case GK_FWD:
      if constexpr (R3) {
        if (a.rec) return go(k_gemm_rows<PREC, NBT, GK_FWD, false, true, RES, NW, NP>);
      }
      return go(k_gemm_rows<PREC, NBT, GK_FWD, false, false, RES, NW, NP>);
    case GK_ADJ:
      if constexpr (R3) {
        if (a.rec) return go(k_gemm_rows<PREC, NBT, GK_ADJ, false, true, RES, NW, NP>);
      }
      return go(k_gemm_rows<PREC, NBT, GK_ADJ, false, false, RES, NW, NP>);
    default: return hipErrorInvalidValue;
  }
}

// Up to 16 rows: four wavefronts on one block where a wavefront per block would leave the chip
// idle behind its chain of chunks, up to four workgroups a CU (fused, us; a wavefront per block ->
// four, in brackets the kernel before both):
//   receivers  blocks:  60                 200                771                1285
//      64               8.5 ->  7.8 (10)   8.6 ->  8.0 (8)    12 -> 13 (13)      16 -> 18 (17)
//     200               15 ->  9.1 (15)    17 ->  11 (12)     24 -> 20 (21)      25 -> 26 (26)
//     400               26 ->  15 (19)     29 ->  17 (23)     37 -> 31 (34)      39 -> 43 (53)
//    1000               58 ->  24 (44)     57 ->  24 (50)     78 -> 53 (73)      92 -> 90 (133)
// Few receivers leave wavefronts without a chunk: there only up to a workgroup a CU, and not
// with a single chunk (a step of 32 traces 12.9 -> 13.3 us).
inline bool share_block(const GemmArgs& a) {
  return a.nr > 32 && a.nf * a.nvb <= (a.nr > 128 ? 1024 : 256);
}

// LDS slots: the adjoint finds the last nslot chunks of D in LDS and fetches the others
// again, so more slots save fetches and barriers, but only as long as LDS does not take
// workgroups off a CU that the registers allow (5, 3, 2, 2 for NBT 1, 2, 3, 4).  Up to 320
// receivers at 16 batch rows all of D_b fits so, and is staged before the products begin:
// their loops then have no barrier at all (201 receivers, 16 rows: 50 -> 45 us fused).
template <int PREC, int NBT>
hipError_t launch_nbt(int kind, const GemmArgs& a, hipStream_t s) {
  using C = RowsCfg<NBT>;
  const int nc = (a.nr + C::KC - 1) / C::KC, slot = C::ESZ * C::SLOT;
  if constexpr (NBT == 1) {
    if (!a.rec && share_block(a)) {
      const int np = (nc + 3) / 4;                // chunks per wavefront
      return np <= 3 ? launch_nw<PREC, NBT, true, 1, 4>(kind, a, np, s) : launch_nw<PREC, NBT, false, 1, 4>(kind, a, 2, s);
    }
    if (nc * slot <= 45000) return launch_nw<PREC, NBT, true, 4>(kind, a, nc, s);
  }
  const int most = (NBT == 1 ? 32768 : NBT == 2 ? 52300 : 70000) / slot;
  const int nslot = nc < 2 ? 2 : (nc < most ? nc : most);
  return launch_nw<PREC, NBT, false, 4>(kind, a, nslot, s);
}

// Batch rows are padded to the next multiple of 16 only: the products' matrix work grows
// with it (301 receivers, fused: 48 rows 178 us, 64 rows 238 us).
template <int PREC>
hipError_t launch_prec(int kind, const GemmArgs& a, hipStream_t s) {
  // the small fused product keeps the four real products that mdd.h states for it (42 us
  // with three against 45 us at 201 receivers and 16 rows)
  if (kind == GK_FUSED && a.nb <= 16 && a.nr <= 224)
    return launch_nbt<MDD_PREC_FP32_CGEMM, 1>(kind, a, s);
  const int rows = a.rec && kind == GK_ADJ ? 2 * a.nb : a.nb;
  if (rows <= 16) return launch_nbt<PREC, 1>(kind, a, s);
  if (rows <= 32) return launch_nbt<PREC, 2>(kind, a, s);
  if (rows <= 48) return launch_nbt<PREC, 3>(kind, a, s);
  return launch_nbt<PREC, 4>(kind, a, s);
}

}  // namespace

bool gemm_rec(int kind, int precision, int nb) {
  return precision == MDD_PREC_FP32 && (kind == GK_FWD || (kind == GK_ADJ && nb <= 32));
}

hipError_t launch_gemm(int kind, int precision, const GemmArgs& a, hipStream_t s) {
  if (a.nb <= 0 || a.nb > NB_LIMIT) return hipErrorInvalidValue;
  if (a.rec && (a.nr != a.nvs || !gemm_rec(kind, precision, a.nb))) return hipErrorInvalidValue;
  switch (precision) {
    case MDD_PREC_FP32: return launch_prec<MDD_PREC_FP32>(kind, a, s);
    case MDD_PREC_FP32_CGEMM: return launch_prec<MDD_PREC_FP32_CGEMM>(kind, a, s);
    default: return launch_gemm_split(kind, precision, a, s);
  }
}

}  // namespace mdd
