// Tiles of the split float32 products (split_tile.h) with direct
// global->LDS loads (global_load_lds_dwordx4): raw float32 operand tiles
// travel into LDS ahead of their use, and every wave splits the fragments it
// reads (a 64 x 64 tile's waves take different slices of k, so nothing is
// split twice in it).
//
// LDS layout of an operand tile (16-byte chunks; a load instruction fills 64
// consecutive chunks, lane l chunk l, so the layout is chosen by which global
// chunk each lane loads):
//   K-contiguous (rows = outer index, QR = BK/4 chunks of 4 k per row): chunk
//     (r, q) at r*QR + (q ^ key(r)): 16 consecutive rows read at one q fall
//     in 16 distinct bank groups modulo 256 bytes;
//   K-strided (rows = k, OUT/4 chunks per row): as stored.  A lane reads, at
//     each of its 8 k, the adjacent columns of its wave's blocks (block b of
//     NB covers columns NB*j + b), a wave's 32 lanes 128 or 256 contiguous bytes.
#pragma once

#include <type_traits>

#include "direct_load.h"
#include "split_tile.h"

namespace agn {
namespace {

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// one 64-lane direct load: lane l's 16 bytes from base + off (bytes) to LDS
// byte offset lds + 16*l (base and lds wave-uniform)
__device__ __forceinline__ void fire_at(const void* base, uint32_t off, uint32_t lds) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m0), "v"(off), "s"(base)
               : "memory", "m0");
}

template <class T>
__device__ __forceinline__ const T* uniform_ptr(const T* p) {
  const uint64_t u = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return reinterpret_cast<const T*>((uintptr_t)(((uint64_t)hi << 32) | lo));
}

// one 64-lane direct load of single floats: lane l's 4 bytes to LDS byte
// offset lds + 4*l
__device__ __forceinline__ void fire_word(const void* src, uint32_t lds) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(m0), "v"(src) : "memory", "m0");
}
#pragma clang diagnostic pop

// Loads and fragments of one operand: OUT outer indices, BK k per step.
// Outer indices past the edge repeat the last row (or column chunk); k past K
// reads the zero page.  W = 4: 16 bytes per lane (16-byte rows; between a
// K-contiguous row's last k and the next multiple of 4 lie zeros); W = 1:
// single floats, for a data set whose rows are not aligned.
template <class Cfg, int OUT, int WT, bool KC, int W>
struct DirectOperand {
  static constexpr int BK = Cfg::BK, NW = Cfg::NTH / 64;
  static constexpr int BYTES = OUT * BK * 4;
  static constexpr int LPS = BYTES / (256 * W) / NW;   // load instructions per wave and step
  static constexpr int QR = KC ? BK / 4 : OUT / 4;     // chunks per LDS row
  static constexpr int NBL = WT / 32;                  // blocks of a wave
  static_assert(BYTES % (256 * W * NW) == 0 && LPS >= 1, "whole load instructions per wave");
  static_assert(!KC || QR == 4 || QR == 8 || QR == 16 || QR == 32, "k chunks per row");

  const char* base;      // uniform: the tile's first row of the worker's matrix, or the worker's shard
  const char* zero;
  uint32_t off[LPS];     // byte offset of this lane's words in a step that starts at k = 0 (gathered K-strided rows: of the column)
  int64_t ldb;           // bytes per matrix row
  int K, o0, on, wave, lane;
  bool gather, narrow;   // narrow: a shard lies within 32-bit offsets (and, where rows are picked per step, a batch wraps at most once)
  int64_t at, S;         // gathered: first row of the batch in the shard, shard size
  uint32_t frag[KC ? Cfg::SL : 1];  // LDS byte offsets of this lane's fragments

  static __device__ __forceinline__ int key(int r) {
    return QR == 4 ? ((r >> 1) ^ (r >> 3)) & 3 : QR == 8 ? (r & 7) ^ ((r >> 3) & 1) : (r & 15);
  }
  // LDS row and the first (KC: k, else: column) index of this lane's words in load instruction i
  __device__ __forceinline__ void place(int i, int& r, int& first) const {
    const int word = W * (64 * (wave + NW * i) + lane), ch = word / 4;
    r = ch / QR;
    if (64 * W <= 4 * QR) r = __builtin_amdgcn_readfirstlane(r);  // (one row per instruction)
    first = 4 * (KC ? (ch % QR) ^ key(r) : ch % QR) + word % 4;
  }
  __device__ __forceinline__ int64_t batch_pos(int64_t j) const {  // row of the shard that holds mini-batch row j
    const int64_t r = at + j;
    return r < S ? r : r - S < S ? r - S : r % S;
  }
  __device__ __forceinline__ int column(int first) const {  // clamped column of a K-strided operand
    return W == 4 ? min(o0 + first, (on - 1) / 4 * 4) : min(o0 + first, on - 1);
  }

  __device__ __forceinline__ void init(const Operand& op, const Gather& g, int worker, int o0_, int on_, int kk, int wave_,
                                       int lane_, int w0, int kw, const float* zero_page) {
    K = kk;
    o0 = o0_;
    on = on_;
    wave = wave_;
    lane = lane_;
    zero = reinterpret_cast<const char*>(zero_page);
    ldb = op.ld * 4;
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
      p += worker * op.wstride * 4 + (KC ? o0 * ldb : 0);
    }
    base = uniform_ptr(p);
    if (W == 4) {
#pragma unroll
      for (int i = 0; i < LPS; ++i) {
        int r, first;
        place(i, r, first);
        if (KC) {
          const int64_t o = min(o0 + r, on - 1);
          off[i] = (uint32_t)((gather ? batch_pos(o) : o - o0) * ldb) + 4 * first;
        } else {
          off[i] = (gather ? 0 : (uint32_t)(r * ldb)) + 4 * column(first);
        }
      }
    }
    const int li = lane & 31, lh = lane >> 5;
    if (KC) {
      const int r = w0 + li;
#pragma unroll
      for (int s = 0; s < (KC ? Cfg::SL : 1); ++s) frag[s] = (r * QR + ((4 * (kw * Cfg::SL + s) + 2 * lh) ^ key(r))) * 16;
    } else {
      frag[0] = ((16 * kw * Cfg::SL + 8 * lh) * OUT + w0 + NBL * li) * 4;
    }
  }

  // the loads of the step that starts at k0, into the stage at LDS offset lds
  __device__ __forceinline__ void fire(int k0, uint32_t lds) const {
    if (W == 4 && k0 + BK <= K && narrow) {
      if (!KC && gather) {  // rows picked by the mini-batch index
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
        const char* b = base + (KC ? (int64_t)k0 * 4 : k0 * ldb);
#pragma unroll
        for (int i = 0; i < LPS; ++i) fire_at(b, off[i], lds + 1024 * (wave + NW * i));
      }
      return;
    }
    // the step that crosses K, single floats, offsets beyond 32 bits: every
    // address from its indices (a rolled loop, so that none is kept in registers)
#pragma unroll 1
    for (int i = 0; i < LPS; ++i) {
      int r, first;
      place(i, r, first);
      const int k = k0 + (KC ? first : r), o = KC ? min(o0 + r, on - 1) : column(first);
      const int64_t row = KC ? (gather ? batch_pos(o) : o - o0) : (gather ? batch_pos(k) : k);
      const char* p = base + row * ldb + 4 * (int64_t)(KC ? k : o);
      if (k >= K) p = zero;
      if (W == 4)
        agn::fire(p, lds + 1024 * (wave + NW * i));
      else
        fire_word(p, lds + 256 * (wave + NW * i));
    }
  }

  // this lane's 8 k of its wave's slice s, for each of the wave's blocks
  __device__ __forceinline__ void read(const char* st, int s, float (&x)[NBL][8]) const {
    if constexpr (KC) {
#pragma unroll
      for (int b = 0; b < NBL; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const sp_f32x4 t = *reinterpret_cast<const sp_f32x4*>(st + ((frag[KC ? s : 0] ^ (16 * h)) + b * 32 * QR * 16));
#pragma unroll
          for (int e = 0; e < 4; ++e) x[b][4 * h + e] = t[e];
        }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (NBL == 2) {
          const sp_f32x2 t = *reinterpret_cast<const sp_f32x2*>(st + frag[0] + (16 * s + e) * OUT * 4);
          x[0][e] = t[0];
          x[1][e] = t[1];
        } else {
          x[0][e] = *reinterpret_cast<const float*>(st + frag[0] + (16 * s + e) * OUT * 4);
        }
      }
    }
  }
};

// LDS of a tile with NS stages
template <class Cfg, int NS>
constexpr int direct_lds_bytes() {
  constexpr int stages = NS * (Cfg::BM + Cfg::BN) * Cfg::BK * 4;
  return stages > Cfg::EPI ? stages : Cfg::EPI;
}

template <int N>
__device__ __forceinline__ void split_frag(const float (&x)[N][8], sp_bf16x8 (&f)[3][N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    sp_u32x4 h, m, l;
    split8(x[i], h, m, l);
    f[0][i] = __builtin_bit_cast(sp_bf16x8, h);
    f[1][i] = __builtin_bit_cast(sp_bf16x8, m);
    f[2][i] = __builtin_bit_cast(sp_bf16x8, l);
  }
}

// One workgroup tile of one batched product.  The operands are loaded NS - 1
// steps ahead, the epilogue's behind the last step's arrival, so that no step
// waits for them.
template <class Cfg, int NS, bool A_KC, bool B_KC, int EPI, bool ADAM, int AW = 4, int BW = 4>
__device__ __forceinline__ void direct_tile(const GemmArgs& g, const int logical, char* lds) {
  static_assert(NS >= 2, "stages");
  constexpr int BK = Cfg::BK, MB = Cfg::WTM / 32, NB = Cfg::WTN / 32;
  constexpr bool DW = EPI == EPI_DW_UPDATE;
  using OpA = DirectOperand<Cfg, Cfg::BM, Cfg::WTM, A_KC, AW>;
  using OpB = DirectOperand<Cfg, Cfg::BN, Cfg::WTN, B_KC, BW>;
  const SplitCoord<Cfg> c(g, logical);
  OpA la;
  OpB lb;
  la.init(g.a, g.g, c.worker, c.m0, g.M, g.K, c.wave, c.lane, c.wm * Cfg::WTM, c.kw, g.zero);
  lb.init(g.b, g.g, c.worker, c.n0, g.N, g.K, c.wave, c.lane, c.wn * Cfg::WTN, c.kw, g.zero);
  const uint32_t lds0 = lds_off(lds);
  constexpr int B0 = NS * OpA::BYTES;  // operand B's stages follow operand A's
  const int nk = (g.K + BK - 1) / BK;
  const auto fire_step = [&](int t, int stage) {
    la.fire(t * BK, lds0 + stage * OpA::BYTES);
    lb.fire(t * BK, lds0 + B0 + stage * OpB::BYTES);
  };
  SplitEpilogue<Cfg, EPI, ADAM> epi;

  // bias gradient (first column tile of a weight gradient): sums of dZ over
  // this lane's k
  const bool do_bias = DW && c.n0 == 0;
  float bsum[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) bsum[b] = 0.f;

  // The products of all K steps, from split operands or (F32: the second pass
  // of a tile) from the float32 values.
  sp_f32x16 acc[MB][NB];
  const auto sweep = [&](auto f32) {
    constexpr bool F32 = decltype(f32)::value;
#pragma unroll
    for (int t = 0; t < NS - 1; ++t)
      if (t < nk) fire_step(t, t);
    sp_f32x16 low[MB][NB];
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int bj = 0; bj < NB; ++bj)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[bi][bj][r] = low[bi][bj][r] = 0.f;
    int st = 0, nxt = NS - 1;  // stages of the next step to read and to load

    // Step t has landed: this wave's loads of it (those of the NS - 2 steps
    // after it may be in flight; at the end of K fewer are, and all are waited
    // for), then every wave's; and every wave is done reading the stage the
    // next loads overwrite.
    const auto arrive = [&](int t) {
      constexpr int YOUNGER = (NS - 2) * (OpA::LPS + OpB::LPS);
      if (YOUNGER < 64 && t + NS - 2 < nk)
        wait_vm<YOUNGER < 64 ? YOUNGER : 0>();
      else
        wait_vm<0>();
      wait_lgkm0();
      barrier();
      if (t + NS - 1 < nk) fire_step(t + NS - 1, nxt);
      nxt = nxt + 1 == NS ? 0 : nxt + 1;
      // the epilogue's operands come in behind the last step (the waits above
      // do not count them)
      if (!F32 && t + 1 == nk) epi.load(g, c);
    };
    for (int t = 0; t < nk; ++t) {
      arrive(t);
      const char *sta = lds + st * OpA::BYTES, *stb = lds + B0 + st * OpB::BYTES;
#pragma unroll
      for (int s = 0; s < Cfg::SL; ++s) {
        float xa[MB][8], xb[NB][8];
        la.read(sta, s, xa);
        lb.read(stb, s, xb);
        if constexpr (F32) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int bi = 0; bi < MB; ++bi)
#pragma unroll
              for (int bj = 0; bj < NB; ++bj)
                acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[bi][e], xb[bj][e], acc[bi][bj], 0, 0, 0);
        } else {
          sp_bf16x8 a[3][MB], b[3][NB];
          split_frag<MB>(xa, a);
          split_frag<NB>(xb, b);
          if (DW && do_bias) {
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
              for (int e = 0; e < 8; ++e) bsum[i] += xa[i][e];
          }
          split_mfma<MB, NB>(a, b, acc, low);
        }
      }
      st = st + 1 == NS ? 0 : st + 1;
    }
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int bj = 0; bj < NB; ++bj)
        if (!F32) acc[bi][bj] += low[bi][bj];
    wait_lgkm0();
    barrier();
  };
  sweep(std::false_type{});

  float* et = reinterpret_cast<float*>(lds);
  using Place = SplitPlace<Cfg, !A_KC, !B_KC>;
  float gb = 0.f;
  if constexpr (DW) {
    if (do_bias) {  // the lanes' sums over their k, added in k order
#pragma unroll
      for (int i = 0; i < MB; ++i)
        if (c.wn == 0) et[(2 * c.kw + c.lh) * Cfg::BM + c.wm * Cfg::WTM + Place::row(i, c.li)] = bsum[i];
      __syncthreads();
      if (c.tid < Cfg::BM)
        for (int q = 0; q < 2 * Cfg::KW; ++q) gb += et[q * Cfg::BM + c.tid];
      __syncthreads();
    }
  }
  sp_f32x4 v[Cfg::NC];
  split_gather<Cfg, Place>(c, et, acc, v);
#pragma unroll
  for (int i = 0; i < Cfg::NC; ++i) v[i] *= kSplitUnscale;
  if (__builtin_expect(unexplained<Cfg, A_KC, B_KC>(g, c, et, v), 0)) {
    sweep(std::true_type{});
    split_gather<Cfg, Place>(c, et, acc, v);
  }
  epi.store(g, c, v, gb);
}

}  // namespace
}  // namespace agn
