// Batched bf16 products in small tiles with direct global->LDS loads: the
// products whose 128 x 128 tiles (gemm_bf16_dl.hip) would leave most of the
// card idle, and those whose K those tiles do not take (a forward K that is no
// multiple of 8).
//
// What bounds them is latency: few tiles, each a chain of K steps.  So a tile
// is 64 x 64 (four waves of 32 x 32; 32 x 32 tiles of one wave are slower or
// even at every count of tiles: backward launch 4 x 512 x 512 x 256 8.2 against
// 7.4 us, forward 24 x 128 x 512 x 256 8.1 against 7.8), K goes in steps of 64
// with loads three steps ahead, and a wave runs its own K slices in order, one
// v_mfma_f32_32x32x16_bf16 each -- the sums, and so the results, are those
// of the 128 x 128 tiles bit for bit (the bias gradient's, which only the
// order of its float32 sum changes, aside).  6 workers of 123-517-259-37,
// m = 77, against the register-staged kernels that took these products before
// (128 x 128 tiles, each step's loads waited for): forward 6.7 against 14.3 us
// on average, backward 7.3 and 7.9 against 26.7, first layer 6.6 against 30.2.
#include "split_dl.h"

namespace agn {
namespace {

typedef short bs_i16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bs_bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bs_i16x4 lds_bs_i16x4;

using Quad = SplitCfg<32, 32, 2, 2, 1, 4>;  // 64 x 64, four waves
constexpr int NS16 = 4;                    // LDS stages

// Loads and fragments of one operand, OUT outer indices x BK k of bf16 per
// step.  Rows are 16-byte aligned and zero between their end and the next
// multiple of 8 elements (K-contiguous: those meet zeros of the other operand
// too).  LDS: 16-byte chunks, a load instruction fills 64 of them; K-contiguous
// rows of 8 chunks, chunk (r, q) at 8r + (q ^ key(r)); K-strided rows as stored.
template <class Cfg, int OUT, bool KC>
struct Operand16 {
  static constexpr int BK = Cfg::BK, NW = Cfg::NTH / 64;
  static constexpr int BYTES = OUT * BK * 2, LPS = BYTES / 1024 / NW;
  static constexpr int QR = KC ? BK / 8 : OUT / 8;  // chunks per LDS row
  static_assert(BYTES % (1024 * NW) == 0 && LPS >= 1, "whole load instructions per wave");
  static_assert(!KC || QR == 8, "k chunks per row");

  const char* base;
  const char* zero;
  uint32_t off[LPS];
  int64_t ldb;
  int K, o0, on, wave, lane;
  bool gather, narrow;
  int64_t at, S;

  static __device__ __forceinline__ int key(int r) { return (r & 7) ^ ((r >> 3) & 1); }
  __device__ __forceinline__ void place(int i, int& r, int& first) const {
    const int ch = 64 * (wave + NW * i) + lane;
    r = ch / QR;
    first = 8 * (KC ? (ch % QR) ^ key(r) : ch % QR);
  }
  __device__ __forceinline__ int64_t batch_pos(int64_t j) const {
    const int64_t r = at + j;
    return r < S ? r : r - S < S ? r - S : r % S;
  }

  __device__ __forceinline__ void init(const Operand& op, const Gather& g, int worker, int o0_, int on_, int kk, int wave_,
                                       int lane_, const float* zero_page) {
    K = kk;
    o0 = o0_;
    on = on_;
    wave = wave_;
    lane = lane_;
    zero = reinterpret_cast<const char*>(zero_page);
    ldb = op.ld * 2;
    gather = op.gather;
    narrow = true;
    at = 0;
    S = 1;
    const char* p = reinterpret_cast<const char*>(op.ptr);
    if (gather) {
      S = g.S;
      at = (gather_step(g) * g.mb) % S;
      narrow = S * ldb < (int64_t)1 << 32 && (KC || g.mb <= S);
      p += worker * S * ldb;
    } else {
      p += worker * op.wstride * 2 + (KC ? o0 * ldb : 0);
    }
    base = uniform_ptr(p);
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
      int r, first;
      place(i, r, first);
      if (KC) {
        const int64_t o = min(o0 + r, on - 1);
        off[i] = (uint32_t)((gather ? batch_pos(o) : o - o0) * ldb) + 2 * first;
      } else {
        off[i] = (gather ? 0 : (uint32_t)(r * ldb)) + 2 * min(o0 + first, (on - 1) / 8 * 8);
      }
    }
  }

  __device__ __forceinline__ void fire(int k0, uint32_t lds) const {
    if (k0 + BK <= K && narrow) {
      if (!KC && gather) {
        const uint32_t at0 = (uint32_t)at + k0, n = (uint32_t)S, ld = (uint32_t)ldb;
#pragma unroll
        for (int i = 0; i < LPS; ++i) {
          int r, first;
          place(i, r, first);
          uint32_t pos = at0 + r;
          pos -= pos >= n ? n : 0;
          fire_at(base, pos * ld + off[i], lds + 1024 * (wave + NW * i));
        }
      } else {
        const char* b = base + (KC ? (int64_t)k0 * 2 : k0 * ldb);
#pragma unroll
        for (int i = 0; i < LPS; ++i) fire_at(b, off[i], lds + 1024 * (wave + NW * i));
      }
      return;
    }
    // the step that crosses K, offsets beyond 32 bits: every address from its indices
#pragma unroll 1
    for (int i = 0; i < LPS; ++i) {
      int r, first;
      place(i, r, first);
      const int k = k0 + (KC ? first : r), o = KC ? min(o0 + r, on - 1) : min(o0 + first, (on - 1) / 8 * 8);
      const int64_t row = KC ? (gather ? batch_pos(o) : o - o0) : (gather ? batch_pos(k) : k);
      const char* p = base + row * ldb + 2 * (int64_t)(KC ? k : o);
      if (k >= K) p = zero;
      agn::fire(p, lds + 1024 * (wave + NW * i));
    }
  }

  // the MFMA operand of slice s for the 32 outer indices from w0: 8 k per lane
  __device__ __forceinline__ sp_bf16x8 read(const char* st, int w0, int s) const {
    const int li = lane & 31, lh = lane >> 5;
    if constexpr (KC) {
      const int r = w0 + li;
      return *reinterpret_cast<const sp_bf16x8*>(st + (r * QR + ((2 * s + lh) ^ key(r))) * 16);
    } else {
      // transposing reads: within 16 lanes, lane i receives element e from
      // mem[A(4e + i/4) + i%4], A(j) the address lane j supplies
      const int row = 16 * s + 8 * lh + (li % 16) / 4, col = w0 + 16 * (li / 16) + 4 * (li % 4);
      bs_bf16x4 h[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bs_i16x4 v =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_bs_i16x4*)(st + ((row + 4 * c) * OUT + col) * 2));
        h[c] = __builtin_bit_cast(bs_bf16x4, v);
      }
      return __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7);
    }
  }
};

template <class Cfg>
constexpr int small16_lds() {
  constexpr int st = NS16 * (Cfg::BM + Cfg::BN) * Cfg::BK * 2;
  return st > Cfg::EPI ? st : Cfg::EPI;
}

template <class Cfg, bool A_KC, bool B_KC, int EPI, bool ADAM>
__device__ __forceinline__ void small16_tile(const GemmArgs& g, const int logical, char* lds) {
  constexpr bool DW = EPI == EPI_DW_UPDATE;
  using OpA = Operand16<Cfg, Cfg::BM, A_KC>;
  using OpB = Operand16<Cfg, Cfg::BN, B_KC>;
  constexpr int STAGE = OpA::BYTES + OpB::BYTES, LPS = OpA::LPS + OpB::LPS;
  const SplitCoord<Cfg> c(g, logical);
  OpA la;
  OpB lb;
  la.init(g.a, g.g, c.worker, c.m0, g.M, g.K, c.wave, c.lane, g.zero);
  lb.init(g.b, g.g, c.worker, c.n0, g.N, g.K, c.wave, c.lane, g.zero);
  const uint32_t lds0 = lds_off(lds);
  const int nk = (g.K + Cfg::BK - 1) / Cfg::BK;
  const auto fire_step = [&](int t, int stage) {
    la.fire(t * Cfg::BK, lds0 + stage * STAGE);
    lb.fire(t * Cfg::BK, lds0 + stage * STAGE + OpA::BYTES);
  };
#pragma unroll
  for (int t = 0; t < NS16 - 1; ++t)
    if (t < nk) fire_step(t, t);
  sp_f32x16 acc[1][1];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
  const bool do_bias = DW && c.n0 == 0;
  float bsum = 0.f;
  SplitEpilogue<Cfg, EPI, ADAM, true> epi;
  int st = 0, nxt = NS16 - 1;
  for (int t = 0; t < nk; ++t) {
    // this wave's loads of step t have landed (those of the two steps after
    // it may be in flight; near the end of K fewer are, and all are waited
    // for), then every wave's; every wave is done with the stage that the
    // next loads overwrite
    if (t + NS16 - 2 < nk)
      wait_vm<(NS16 - 2) * LPS>();
    else
      wait_vm<0>();
    wait_lgkm0();
    barrier();
    if (t + NS16 - 1 < nk) fire_step(t + NS16 - 1, nxt);
    if (t + 1 == nk) epi.load(g, c);  // (behind the last wait, which does not count them)
    const char* s0 = lds + st * STAGE;
#pragma unroll
    for (int s = 0; s < Cfg::SL; ++s) {
      const sp_bf16x8 a = la.read(s0, c.wm * 32, s), b = lb.read(s0 + OpA::BYTES, c.wn * 32, s);
      if (DW && do_bias) {
#pragma unroll
        for (int e = 0; e < 8; ++e) bsum += (float)a[e];
      }
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[0][0], 0, 0, 0);
    }
    st = st + 1 == NS16 ? 0 : st + 1;
    nxt = nxt + 1 == NS16 ? 0 : nxt + 1;
  }
  wait_lgkm0();
  barrier();
  float* et = reinterpret_cast<float*>(lds);
  float gb = 0.f;
  if constexpr (DW) {
    if (do_bias) {  // the two lane groups' sums over their k, in lane order
      if (c.wn == 0) et[c.lh * Cfg::BM + c.wm * 32 + c.li] = bsum;
      __syncthreads();
      if (c.tid < Cfg::BM) gb = et[c.tid] + et[Cfg::BM + c.tid];
      __syncthreads();
    }
  }
  sp_f32x4 v[Cfg::NC];
  split_gather<Cfg, SplitPlace<Cfg, false, false>>(c, et, acc, v);
  epi.store(g, c, v, gb);
}

template <class Cfg>
__host__ __device__ inline int tiles_of(const GemmArgs& g) {
  return ((g.M + Cfg::BM - 1) / Cfg::BM) * ((g.N + Cfg::BN - 1) / Cfg::BN) * g.batch;
}

template <class Cfg, bool A_KC, bool B_KC, int EPI, bool ADAM>
__global__ __launch_bounds__(Cfg::NTH) void gemm_bf16_small_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) char lds[small16_lds<Cfg>()];
  small16_tile<Cfg, A_KC, B_KC, EPI, ADAM>(g, xcd_remap(blockIdx.x, tiles_of<Cfg>(g)), lds);
}

// input-gradient tiles, then weight-gradient tiles, of one layer in one launch
template <class Cfg, bool ADAM>
__global__ __launch_bounds__(Cfg::NTH) void gemm_bf16_small_bwd_kernel(GemmArgs dx, GemmArgs dw, int n1, int n1pad) {
  __shared__ __attribute__((aligned(16))) char lds[small16_lds<Cfg>()];
  const int pid = blockIdx.x;
  if (pid < n1pad) {
    if (pid < n1) small16_tile<Cfg, true, false, EPI_DX_MASK, false>(dx, xcd_remap(pid, n1), lds);
  } else {
    small16_tile<Cfg, false, false, EPI_DW_UPDATE, ADAM>(dw, xcd_remap(pid - n1pad, tiles_of<Cfg>(dw)), lds);
  }
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

bool operand_aligned(const Operand& op) {
  return op.vec && aligned16(op.ptr) && op.ld % 8 == 0 && op.wstride % 8 == 0;
}

template <bool A_KC, bool B_KC, int EPI, bool ADAM>
hipError_t go(const GemmArgs& g, hipStream_t s) {
  AGN_LAUNCH((gemm_bf16_small_kernel<Quad, A_KC, B_KC, EPI, ADAM>), dim3(tiles_of<Quad>(g)), dim3(Quad::NTH), 0, s, g);
  return hipGetLastError();
}

}  // namespace

bool gemm_bf16_small_ok(const GemmArgs& g) {
  if (!g.zero || !operand_aligned(g.a) || !operand_aligned(g.b)) return false;
  if (g.epi == EPI_DW_UPDATE)
    return aligned16(g.w_src) && aligned16(g.w_dst) && aligned16(g.w_snap) && ((uintptr_t)g.w_dst16 & 7) == 0 &&
           g.ldw % 8 == 0 && g.pstride % 4 == 0;
  const bool f32 = g.epi == EPI_FWD_LINEAR;
  bool ok = ((uintptr_t)g.out & (f32 ? 15 : 7)) == 0 && g.ldo % 8 == 0 && g.ostride % 4 == 0;
  if (g.epi == EPI_DX_MASK) ok = ok && ((uintptr_t)g.mask & 7) == 0 && g.ldm % 8 == 0 && g.mstride % 4 == 0;
  return ok;
}

hipError_t launch_gemm_bf16_small(int a_kc, int b_kc, const GemmArgs& g, hipStream_t s) {
  if (a_kc && b_kc && g.epi == EPI_FWD_RELU) return go<true, true, EPI_FWD_RELU, false>(g, s);
  if (a_kc && b_kc && g.epi == EPI_FWD_LINEAR) return go<true, true, EPI_FWD_LINEAR, false>(g, s);
  if (!a_kc && !b_kc && g.epi == EPI_DW_UPDATE)
    return g.adam.on ? go<false, false, EPI_DW_UPDATE, true>(g, s) : go<false, false, EPI_DW_UPDATE, false>(g, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_bf16_small_bwd(const GemmArgs& dx, const GemmArgs& dw, hipStream_t s) {
  const int n1 = tiles_of<Quad>(dx), n1pad = (n1 + kNumXcd - 1) / kNumXcd * kNumXcd;
  const dim3 grid(n1pad + tiles_of<Quad>(dw));
  if (dw.adam.on)
    AGN_LAUNCH((gemm_bf16_small_bwd_kernel<Quad, true>), grid, dim3(Quad::NTH), 0, s, dx, dw, n1, n1pad);
  else
    AGN_LAUNCH((gemm_bf16_small_bwd_kernel<Quad, false>), grid, dim3(Quad::NTH), 0, s, dx, dw, n1, n1pad);
  return hipGetLastError();
}

}  // namespace agn
