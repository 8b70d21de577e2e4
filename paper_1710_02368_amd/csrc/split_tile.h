// Float32 products on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16), each
// float32 operand split into three bf16 pieces x = h + m + l.
//
// The split is exact: h = bf16(x), m = bf16(x - h), l = x - h - m hold 8 bits
// each, rounded to nearest, and the subtractions are exact.  Every operand is
// split as 2^16 x: a float32 value is a multiple of 2^-149 and a bf16 one of
// 2^-133, which without the factor would take the low bits of values below
// 2^-110, 16 of the 24 at 2^-126.  (Conversion, dot product and MFMA keep
// subnormal values.)  The sums come out 2^32 too large and are scaled back
// before anything else is done with them; in range the factors change no bit.
// A product a*b is the sum of the six piece products
// ah*bh + (ah*bm + am*bh) + (am*bm + ah*bl + al*bh); the three left out are
// below 2^-26 of it.  ah*bh goes to one accumulator, the five small ones to
// a second, added at the end: one rounding per 16 k in the large sum, where
// the float32 MFMA rounds four times.  Measured against 64 bits (K = 64 to
// 2000; normal, sparse, rectified and positive operands) the relative error
// is 0.33 to 0.50 of the float32 MFMA's (K = 784, sparse inputs x normal
// weights: 7.7e-8 against 2.3e-7).  Six bf16 MFMAs take 6/16 of the float32
// MFMAs' cycles at the nominal rates; with random operands the card sustains
// 1.75 PFLOP/s in bf16 (292 TFLOP/s of split products) against 154 in float32.
//
// The split takes 4.5 vector instructions per element: the factor,
// v_cvt_pk_bf16_f32, which rounds two elements to a packed pair, and
// v_dot2c_f32_bf16, which subtracts one piece of that pair from its element
// (dot with (-1, 0) or (0, -1)).  Masks and subtractions instead of the dot
// products (5.5 per element without the factor) overlap with MFMAs, which
// those do not, and still measured slower (forward product 40 x 128 x 2000 x
// 2000: 271 against 256 us; weight gradient 547 against 518).  The factor
// cost a round of 8 x 784-1000-1000-10, m = 128 1897 against 1849 us when it
// came in, of 20 workers 4098 against 3974, of 10 x 784-512-256-10, m = 64 573
// against 553.
//
// Infinities: inf - inf in the split makes NaN where the float32 product
// would keep an infinity, and results of 2^96 and more (operands of 2^111)
// leave the range that the factors leave, so a tile with a non-finite result
// that no NaN operand explains is computed again with float32 MFMAs
// (direct_tile, unexplained).
#pragma once

#include "device_common.h"

namespace agn {
namespace {

typedef float sp_f32x16 __attribute__((ext_vector_type(16)));
typedef float sp_f32x4 __attribute__((ext_vector_type(4)));
typedef float sp_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 sp_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 sp_bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t sp_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t sp_u32x2 __attribute__((ext_vector_type(2)));

constexpr float kSplitScale = 0x1p16f, kSplitUnscale = 0x1p-32f;  // of an operand; of a product of two

// eight float32 values -> the three bf16 pieces of 2^16 times each, 16 bytes each
__device__ __forceinline__ void split8(const float (&x)[8], sp_u32x4& h, sp_u32x4& m, sp_u32x4& l) {
  // (-1, 0) and (0, -1), the first from a register: the compiler would encode
  // it as the inline constant -1.0, which the instruction reads as (0, -1)
  uint32_t u0 = 0x0000BF80u;
  asm("" : "+s"(u0));
  float scale = kSplitScale;  // (from a register too: a literal makes every multiplication eight bytes)
  asm("" : "+s"(scale));
  const sp_bf16x2 n0 = __builtin_bit_cast(sp_bf16x2, u0);
  const sp_bf16x2 n1 = __builtin_bit_cast(sp_bf16x2, 0xBF800000u);
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float x0 = x[2 * p] * scale, x1 = x[2 * p + 1] * scale;
    sp_bf16x2 a, b, c;
    a[0] = (__bf16)x0;
    a[1] = (__bf16)x1;
    const float r0 = __builtin_amdgcn_fdot2_f32_bf16(a, n0, x0, false);
    const float r1 = __builtin_amdgcn_fdot2_f32_bf16(a, n1, x1, false);
    b[0] = (__bf16)r0;
    b[1] = (__bf16)r1;
    const float s0 = __builtin_amdgcn_fdot2_f32_bf16(b, n0, r0, false);
    const float s1 = __builtin_amdgcn_fdot2_f32_bf16(b, n1, r1, false);
    c[0] = (__bf16)s0;
    c[1] = (__bf16)s1;
    h[p] = __builtin_bit_cast(uint32_t, a);
    m[p] = __builtin_bit_cast(uint32_t, b);
    l[p] = __builtin_bit_cast(uint32_t, c);
  }
}

// Shape of a workgroup's tile: WGM x WGN x KW waves; a wave owns WTM x WTN
// outputs (blocks of 32 x 32) over SL slices of 16 k per K step, and the KW
// waves of the same outputs take different slices (their sums are added
// through LDS).
template <int WTM_, int WTN_, int WGM_, int WGN_, int KW_, int SL_>
struct SplitCfg {
  static constexpr int WTM = WTM_, WTN = WTN_, WGM = WGM_, WGN = WGN_, KW = KW_, SL = SL_;
  static constexpr int BM = WTM * WGM, BN = WTN * WGN, BK = 16 * KW * SL, NTH = 64 * WGM * WGN * KW;
  static constexpr int ELD = BN;               // row stride (floats) of the epilogue tile
  static constexpr int EPI = KW * BM * ELD * 4;
  static constexpr int NC = BM * BN / 4 / NTH;  // epilogue chunks of 4 outputs per thread
  static_assert(BM * BN % (4 * NTH) == 0, "whole epilogue chunks per thread");
};

// element (outer o, k) of an operand straight from memory
template <bool KC>
__device__ __forceinline__ float operand_at(const Operand& op, const Gather& g, int64_t w, int64_t t, int64_t o,
                                            int64_t k) {
  int64_t r = KC ? o : k;
  if (op.gather) r = batch_row(w, t, g.mb, g.S, r);
  return reinterpret_cast<const float*>(op.ptr)[w * op.wstride + r * op.ld + (KC ? k : o)];
}

// Where a wave's accumulators lie in the workgroup's tile: block bi covers
// rows 32*bi + i (i = 0..31) of the wave's, or rows MB*i + bi (interleaved);
// columns likewise.
template <class Cfg, bool A_IL, bool B_IL>
struct SplitPlace {
  static constexpr int MB = Cfg::WTM / 32, NB = Cfg::WTN / 32;
  static __device__ __forceinline__ int row(int bi, int i) { return A_IL ? MB * i + bi : 32 * bi + i; }
  static __device__ __forceinline__ int col(int bj, int j) { return B_IL ? NB * j + bj : 32 * bj + j; }
};

// Coordinates of a tile and of a thread in it.
template <class Cfg>
struct SplitCoord {
  int tid, lane, wave, kw, wn, wm, li, lh, worker, m0, n0;
  // this thread's epilogue chunks: 4 outputs at column ec of rows m0 + er0 +
  // i*ERS
  int ecl, ec, er0;
  static constexpr int ERS = Cfg::NTH / (Cfg::BN / 4);

  __device__ __forceinline__ SplitCoord(const GemmArgs& g, int logical) {
    tid = threadIdx.x;
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    kw = wave % Cfg::KW;
    wn = wave / Cfg::KW % Cfg::WGN;
    wm = wave / Cfg::KW / Cfg::WGN;
    li = lane & 31;
    lh = lane >> 5;
    const int tm = (g.M + Cfg::BM - 1) / Cfg::BM, tn = (g.N + Cfg::BN - 1) / Cfg::BN;
    worker = logical / (tm * tn);
    const int rem = logical % (tm * tn);
    // consecutive tiles share an XCD's L2: one worker's few rows of A and a
    // block of its weights, or (batch 1, the evaluation) a block of rows and
    // all of the weights
    const int ti = g.batch == 1 ? rem / tn : rem % tm, tj = g.batch == 1 ? rem % tn : rem / tm;
    m0 = ti * Cfg::BM;
    n0 = tj * Cfg::BN;
    ecl = 4 * (tid % (Cfg::BN / 4));
    ec = n0 + ecl;
    er0 = tid / (Cfg::BN / 4);
  }
};

// Operands of the epilogue, loaded from indices clamped into the matrix (its
// rows are padded to 8; values outside are never stored): the bias, the ReLU
// mask, or the weights (with the snapshot on a round's last step, and Adam's
// moments).  H16: activations and gradients are bf16, and the updated weights'
// bf16 shadow is written beside them.
template <class Cfg, int EPI, bool ADAM, bool H16 = false>
struct SplitEpilogue {
  static constexpr int NC = Cfg::NC;
  static constexpr bool DW = EPI == EPI_DW_UPDATE;
  sp_f32x4 pre[NC], snap[DW ? NC : 1], mo[DW && ADAM ? NC : 1], ve[DW && ADAM ? NC : 1];

  __device__ __forceinline__ void load(const GemmArgs& g, const SplitCoord<Cfg>& c) {
    const int cc = min(c.ec, (g.N - 1) / 4 * 4);
    if (EPI == EPI_DX_MASK || DW) {
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int64_t row = min(c.m0 + c.er0 + i * c.ERS, g.M - 1);
        if (EPI == EPI_DX_MASK) {
          const int64_t e = c.worker * g.mstride + row * g.ldm + cc;
          if (H16) {
            const sp_u32x2 t = *reinterpret_cast<const sp_u32x2*>(reinterpret_cast<const uint16_t*>(g.mask) + e);
            pre[i] = sp_f32x4{__uint_as_float(t[0] << 16), __uint_as_float(t[0] & 0xFFFF0000u),
                              __uint_as_float(t[1] << 16), __uint_as_float(t[1] & 0xFFFF0000u)};
          } else {
            pre[i] = *reinterpret_cast<const sp_f32x4*>(reinterpret_cast<const float*>(g.mask) + e);
          }
        } else {
          const int64_t e = c.worker * g.pstride + row * g.ldw + cc;
          pre[i] = *reinterpret_cast<const sp_f32x4*>(g.w_src + e);
          if (g.last) snap[i] = *reinterpret_cast<const sp_f32x4*>(g.w_snap + e);
          if (ADAM) {
            mo[i] = *reinterpret_cast<const sp_f32x4*>(g.adam.mw + e);
            ve[i] = *reinterpret_cast<const sp_f32x4*>(g.adam.vw + e);
          }
        }
      }
    } else {
      const float* bp = g.bias + c.worker * g.bstride;
#pragma unroll
      for (int e = 0; e < 4; ++e) pre[0][e] = bp[min(c.ec + e, g.N - 1)];
    }
  }

  static __device__ __forceinline__ sp_u32x2 bf16_of(const sp_f32x4& v) {
    return sp_u32x2{(uint32_t)f32_to_bf16_rne(v[0]) | ((uint32_t)f32_to_bf16_rne(v[1]) << 16),
                    (uint32_t)f32_to_bf16_rne(v[2]) | ((uint32_t)f32_to_bf16_rne(v[3]) << 16)};
  }

  // v: this thread's chunks of the product; gb: the bias gradient of row tid
  // (first column tile of a weight gradient)
  __device__ __forceinline__ void store(const GemmArgs& g, const SplitCoord<Cfg>& c, const sp_f32x4 (&v)[NC], float gb) {
    if (!DW) {
      if (c.ec < g.ldo) {  // (columns past N are stored as zeros: the row padding stays zero)
        const int64_t e0 = c.worker * g.ostride + c.ec;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int64_t row = c.m0 + c.er0 + i * c.ERS;
          if (row >= g.M) continue;
          sp_f32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float x = v[i][e];
            if (EPI == EPI_DX_MASK) {
              x = pre[i][e] > 0.f ? x : 0.f;
            } else {
              x += pre[0][e];
              if (EPI == EPI_FWD_RELU) x = x > 0.f ? x : 0.f;
            }
            o[e] = c.ec + e < g.N ? x : 0.f;
          }
          if (H16 && EPI != EPI_FWD_LINEAR)
            *reinterpret_cast<sp_u32x2*>(reinterpret_cast<uint16_t*>(g.out) + e0 + row * g.ldo) = bf16_of(o);
          else
            *reinterpret_cast<sp_f32x4*>(reinterpret_cast<float*>(g.out) + e0 + row * g.ldo) = o;
        }
      }
      return;
    }
    const AdamCoef ac = ADAM ? adam_coef(g.g, g.adam) : AdamCoef{1.f, 1.f};
    const int64_t wo = c.worker * g.pstride;
    if (c.ec < g.N) {
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int64_t row = c.m0 + c.er0 + i * c.ERS;
        if (row >= g.M) continue;
        const int64_t e0 = wo + row * g.ldw + c.ec;
        sp_f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float step = v[i][e];
          if (ADAM) {
            float mm = mo[i][e], vv = ve[i][e];
            step = adam_moments(step, mm, vv, g.adam, ac);
            mo[i][e] = mm;
            ve[i][e] = vv;
          }
          o[e] = pre[i][e] - g.eta * step;
          if (g.last) o[e] = (o[e] - snap[i][e]) / g.lam;
        }
        if (c.ec + 4 <= g.N) {
          *reinterpret_cast<sp_f32x4*>(g.w_dst + e0) = o;
          if (H16 && !g.last) *reinterpret_cast<sp_u32x2*>(g.w_dst16 + e0) = bf16_of(o);
          if (ADAM) {
            *reinterpret_cast<sp_f32x4*>(g.adam.mw + e0) = mo[i];
            *reinterpret_cast<sp_f32x4*>(g.adam.vw + e0) = ve[i];
          }
        } else {
          for (int e = 0; e < 4 && c.ec + e < g.N; ++e) {
            g.w_dst[e0 + e] = o[e];
            if (H16 && !g.last) g.w_dst16[e0 + e] = f32_to_bf16_rne(o[e]);
            if (ADAM) g.adam.mw[e0 + e] = mo[i][e], g.adam.vw[e0 + e] = ve[i][e];
          }
        }
      }
    }
    if (c.n0 == 0 && c.tid < Cfg::BM && c.m0 + c.tid < g.M) {
      const int64_t e = wo + c.m0 + c.tid;
      const float step = ADAM ? adam_dir(gb, g.adam.mb, g.adam.vb, e, g.adam, ac) : gb;
      const float nb = g.b_src[e] - g.eta * step;
      g.b_dst[e] = g.last ? (nb - g.b_snap[e]) / g.lam : nb;
    }
  }
};

// The waves' accumulators to LDS and each thread's chunks back in row order,
// the KW partial sums added in wave order.  lds is free when this is called
// (a barrier lies before); the sums in it stay until the next barrier.
template <class Cfg, class Place>
__device__ __forceinline__ void split_gather(const SplitCoord<Cfg>& c, float* et,
                                             const sp_f32x16 (&acc)[Cfg::WTM / 32][Cfg::WTN / 32],
                                             sp_f32x4 (&v)[Cfg::NC]) {
  constexpr int MB = Cfg::WTM / 32, NB = Cfg::WTN / 32, NC = Cfg::NC, KW = Cfg::KW, BM = Cfg::BM, ELD = Cfg::ELD;
  float* dst = et + (c.kw * BM + c.wm * Cfg::WTM) * ELD + c.wn * Cfg::WTN;
#pragma unroll
  for (int bi = 0; bi < MB; ++bi)
#pragma unroll
    for (int bj = 0; bj < NB; ++bj)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        dst[Place::row(bi, 8 * (r >> 2) + 4 * c.lh + (r & 3)) * ELD + Place::col(bj, c.li)] = acc[bi][bj][r];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const float* src = et + (c.er0 + i * c.ERS) * ELD + c.ecl;
    v[i] = *reinterpret_cast<const sp_f32x4*>(src);
#pragma unroll
    for (int w = 1; w < KW; ++w) v[i] += *reinterpret_cast<const sp_f32x4*>(src + w * BM * ELD);
  }
}

// Whether a result of the tile is not finite although no NaN was found in its
// row of A or its column of B: such a tile has to be computed in float32.  A
// result with a NaN operand is NaN either way, so that the rounds of a model
// that has diverged to NaN run at their ordinary speed; NaNs are looked for
// at kNanProbes k of every row and column (the update of a layer spreads one
// over a whole row of its weights; a NaN that is not found costs the tile its
// second pass, nothing else).  8 x 784-1000-1000-10, m = 128, us per round
// that is waited for: finite 1960; all weights NaN 2050; one weight in 5488 NaN
// 2357 (with every such tile computed again by loads straight from memory:
// 4676 in both).
// lds is free when this returns.
constexpr int kNanProbes = 16;

template <class Cfg, bool A_KC, bool B_KC>
__device__ __forceinline__ bool unexplained(const GemmArgs& g, const SplitCoord<Cfg>& c, float* et,
                                            const sp_f32x4 (&v)[Cfg::NC]) {
  float chk = 0.f;
#pragma unroll
  for (int i = 0; i < Cfg::NC; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) chk += v[i][e] * 0.f;
  if (__builtin_expect(!__syncthreads_or(chk != 0.f), 1)) return false;
  static_assert(Cfg::BM + Cfg::BN <= Cfg::NTH, "a row or a column per thread");
  if (c.tid < Cfg::BM + Cfg::BN) {
    const bool row = c.tid < Cfg::BM;
    const int64_t t = g.a.gather || g.b.gather ? gather_step(g.g) : 0;
    const int o = row ? min(c.m0 + c.tid, g.M - 1) : min(c.n0 + c.tid - Cfg::BM, g.N - 1);
    float sum = 0.f;
    for (int p = 0; p < kNanProbes; ++p) {
      const int64_t k = (int64_t)g.K * p / kNanProbes;
      const float x = row ? operand_at<A_KC>(g.a, g.g, c.worker, t, o, k) : operand_at<B_KC>(g.b, g.g, c.worker, t, o, k);
      sum += x != x ? 1.f : 0.f;
    }
    et[c.tid] = sum;
  }
  __syncthreads();
  bool open = false;
#pragma unroll
  for (int i = 0; i < Cfg::NC; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      open = open || (v[i][e] * 0.f != 0.f && et[c.er0 + i * c.ERS] == 0.f && et[Cfg::BM + c.ecl + e] == 0.f);
  return __syncthreads_or(open);
}

// the six piece products of one slice of 16 k (see the top of this file)
template <int MB, int NB>
__device__ __forceinline__ void split_mfma(const sp_bf16x8 (&a)[3][MB], const sp_bf16x8 (&b)[3][NB],
                                           sp_f32x16 (&acc)[MB][NB], sp_f32x16 (&low)[MB][NB]) {
  constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
  for (int p = 0; p < 6; ++p)
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int bj = 0; bj < NB; ++bj) {
        sp_f32x16& d = p == 0 ? acc[bi][bj] : low[bi][bj];
        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[p]][bi], b[PB[p]][bj], d, 0, 0, 0);
      }
}

}  // namespace
}  // namespace agn
