// Float32 products of the local SGD step as split bf16 products (split_tile.h
// for the arithmetic, split_dl.h for the tiles): the forward products, the
// backward launch of a layer (input gradient, and weight gradient fused with
// the update of W and b), and the first layer's weight gradient.
//
//   forward          H_{l+1} = relu(H_l W_l^T + b_l)    A = H_l   (K-contiguous)
//                                                       B = W_l   (K-contiguous)
//   input gradient   dZ_l = (dZ_{l+1} W_l) * [H_l > 0]  A = dZ    (K-contiguous)
//                                                       B = W_l   (K-strided)
//   weight gradient  dW_l = dZ_{l+1}^T H_l              A = dZ    (K-strided)
//                                                       B = H_l   (K-strided)
// For the first layer the rows of H_0 are the data-set rows that the
// mini-batch index picks (no copy of the batch is made).
//
// What bounds these launches: at 1000 x 1000 x 128 and eight workers one tile
// or two per compute unit, so a tile's own chain (load latency, 16 K steps of
// split, MFMAs and a barrier, the gather of the waves' sums); at forty workers
// of 2000 the matrix pipe (MFMAs and the split's dot products) at 160 TFLOP/s.
// Kernel times against the float32-MFMA kernels these replaced (us, both on
// one card in turn):
//   forward 8 x 128 x 1000 x 1000 / 784     21.7 (average of both) against 20.5
//   forward 20 x 128 x 1000 x 1000 / 784    45.5 against 50.7
//   forward 40 x 128 x 2000 x 2000          267 against 322
//   backward 8 / 20 x 1000 x 1000 x 128     43.6 against 49.8, 101.9 against 125.5
//   first layer 8 / 20 x 1000 x 784 x 128   26.8 against 30.6, 59.8 against 66.1
//   10 x 784-512-256, m = 64                forward 10.6 against 15.0 (average), backward 11.2
//     against 18.0, first layer 16.0 (with the output layer's update) against 20.0 + 7.7
//   5 x 123-517-259, m = 50                 forward (with the logits) 7.8 against 15.2, backward
//     (average of two) 7.4 against 13.5
// Two kinds of launches are slower than the float32-MFMA kernels were, where
// the split's vector work is not hidden: forward products of about 256 64 x 64
// tiles (5 %, above), and backward launches of 256-wide layers at m = 256
// (8 x 512 x 256 x 256 18.9 against 18.4).
#include "head_dw_unit.h"
#include "split_dl.h"

namespace agn {
namespace {

template <class Cfg>
__host__ __device__ inline int tiles_of(const GemmArgs& g) {
  return ((g.M + Cfg::BM - 1) / Cfg::BM) * ((g.N + Cfg::BN - 1) / Cfg::BN) * g.batch;
}

// Tile shapes (see fwd, launch_gemm_f32_bwd and dw for where each is used)
using Wide = SplitCfg<64, 64, 2, 1, 2, 1>;   // 128 x 64, two slices per step: a whole mini-batch per weight tile
using Mid = SplitCfg<64, 64, 1, 1, 4, 1>;    // 64 x 64, four slices
struct Deep : Mid {};                        // ... with three LDS stages: a tile per compute unit
using Flat = SplitCfg<32, 64, 1, 1, 4, 1>;   // 32 x 64, four slices
using Small = SplitCfg<32, 32, 1, 1, 4, 1>;  // 32 x 32, four slices: many tiles of a small product
using MidW = SplitCfg<32, 32, 2, 2, 1, 2>;   // 64 x 64 as four waves of 32 x 32: weight gradients

// LDS stages
template <class Cfg>
constexpr int kStages = 2;
template <>
constexpr int kStages<Wide> = 3;
template <>
constexpr int kStages<Small> = 3;
template <>
constexpr int kStages<Deep> = 3;
template <>
constexpr int kStages<MidW> = 3;

template <class Cfg>
constexpr int lds_of() { return direct_lds_bytes<Cfg, kStages<Cfg>>(); }

template <class Cfg, int EPI, int AW>
__global__ __launch_bounds__(Cfg::NTH, 2) void split_fwd_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) char lds[lds_of<Cfg>()];
  direct_tile<Cfg, kStages<Cfg>, true, true, EPI, false, AW, 4>(
      g, xcd_remap(blockIdx.x, tiles_of<Cfg>(g)), lds);
}

// The backward products of one layer in one launch: the input-gradient tiles
// (long K) first, then the weight-gradient tiles.  Both read dZ_{l+1}; the
// first reads W_l from the step's source parameters, the second writes the
// destination parameters, so they are independent.  Each range is laid out
// over the XCDs on its own (the first is padded to a multiple of 8
// workgroups, the pad workgroups exit at once).
template <class CX, class CW, bool ADAM>
__global__ __launch_bounds__(CX::NTH, 2) void split_bwd_kernel(GemmArgs dx, GemmArgs dw, int n1, int n1pad) {
  static_assert(CX::NTH == CW::NTH, "one workgroup size");
  constexpr int LDS = lds_of<CX>() > lds_of<CW>() ? lds_of<CX>() : lds_of<CW>();
  __shared__ __attribute__((aligned(16))) char lds[LDS];
  const int pid = blockIdx.x;
  if (pid < n1pad) {
    if (pid < n1)
      direct_tile<CX, kStages<CX>, true, false, EPI_DX_MASK, false>(dx, xcd_remap(pid, n1), lds);
  } else {
    direct_tile<CW, kStages<CW>, false, false, EPI_DW_UPDATE, ADAM>(
        dw, xcd_remap(pid - n1pad, tiles_of<CW>(dw)), lds);
  }
}

// A layer's weight gradient by itself (the first layer); with HCM > 0 (the
// class bound of the fused output layer) the first `units` workgroups run the
// output layer's weight-gradient units, which neither read nor write what the
// tiles do.
template <class Cfg, int BW, bool ADAM, int HCM>
__global__ __launch_bounds__(Cfg::NTH, 2) void split_dw_kernel(GemmArgs dw, HeadDwArgs h, int units, int upad) {
  constexpr int HB = HCM > 0 ? hdw_smem_floats<HCM ? HCM : 1>() * 4 : 0;
  constexpr int LDS = lds_of<Cfg>() > HB ? lds_of<Cfg>() : HB;
  __shared__ __attribute__((aligned(16))) char lds[LDS];
  const int pid = blockIdx.x;
  if (HCM > 0 && pid < upad) {
    static_assert(HCM == 0 || Cfg::NTH == 64 * HDW_WAVES, "one unit per workgroup");
    if constexpr (HCM > 0)
      if (pid < units) head_dw_unit<HCM>(h, pid, reinterpret_cast<float*>(lds));
    return;
  }
  direct_tile<Cfg, kStages<Cfg>, false, false, EPI_DW_UPDATE, ADAM, 4, BW>(
      dw, xcd_remap(pid - upad, tiles_of<Cfg>(dw)), lds);
}

int pad8(int n) { return (n + kNumXcd - 1) / kNumXcd * kNumXcd; }

template <class Cfg, int EPI>
hipError_t go_fwd(const GemmArgs& g, hipStream_t s) {
  if (g.a.vec)
    AGN_LAUNCH((split_fwd_kernel<Cfg, EPI, 4>), dim3(tiles_of<Cfg>(g)), dim3(Cfg::NTH), 0, s, g);
  else
    AGN_LAUNCH((split_fwd_kernel<Cfg, EPI, 1>), dim3(tiles_of<Cfg>(g)), dim3(Cfg::NTH), 0, s, g);
  return hipGetLastError();
}

// Forward tile shapes by the product's number of 64 x 64 tiles (us, measured):
//                              tiles   Small   Flat   Deep    Mid
//   10 x 64 x 512 x 784           80    14.2                 19.9
//   4 x 128 x 1000 x 1000        128    17.6   18.7
//   6 x 128 x 1000 x 1000        192    24.1   24.7          26.4
//   8 x 128 x 1000 x 784         256    25.7   22.8          22.6
//   8 x 128 x 1000 x (784, 1000) 256           22.2   21.7        (average of both)
//   12 x 128 x 1000 x 784        384    35.0   29.1          32.0
//   20 x 128 x 1000 x 784        640    54.3   43.7          46.6
//   24 x 128 x 1000 x 784        768           50.0          47.9
//   28 x 128 x 1000 x 784        896           56.4          56.1
// (Deep's 96 KB of LDS leave one workgroup per compute unit, so it ends at a
// tile per unit.)  Data rows that are loaded in single floats need the more
// waves of Flat: 6 x 128 x 1000 x 785, 192 tiles, Small 37.4, Flat 35.2; 8 x,
// 256, Small 53.9, Flat 35.8, Deep 52.3.
constexpr int kFlatTiles = 200, kFlatTilesWords = 128, kDeepTiles = 256, kMidTiles = 700;
// ... and from this many 128 x 64 tiles on, a tile holds a worker's whole
// mini-batch and reads each weight once (Wide against Mid: 40 x 128 x 2000 x
// 784, 1280 tiles, 119 us both, and 255 against 267 at 2000 x 2000; 32 x 128 x
// 2000 x 784, 1024, 99 both; below, Wide wins or loses with how its tiles fill
// the card: 960 96 against 106, 640 77 against 73, 320 48 against 45)
constexpr int kWideTiles = 1024;

template <int EPI>
hipError_t fwd(const GemmArgs& g, hipStream_t s) {
  // (batch 1: the evaluation, whose rows come in chunks of any size; Wide
  // adds a row's products in another order than the rest)
  if (g.batch > 1 && g.M > 64 && tiles_of<Wide>(g) >= kWideTiles) return go_fwd<Wide, EPI>(g, s);
  const int t = tiles_of<Mid>(g);
  if (t >= kMidTiles) return go_fwd<Mid, EPI>(g, s);
  if (t < (g.a.vec ? kFlatTiles : kFlatTilesWords)) return go_fwd<Small, EPI>(g, s);
  return t <= kDeepTiles && g.a.vec ? go_fwd<Deep, EPI>(g, s) : go_fwd<Flat, EPI>(g, s);
}

template <class CX, class CW>
hipError_t go_bwd(const GemmArgs& dx, const GemmArgs& dw, hipStream_t s) {
  const int n1 = tiles_of<CX>(dx), n1pad = pad8(n1);
  const dim3 grid(n1pad + tiles_of<CW>(dw));
  if (dw.adam.on)
    AGN_LAUNCH((split_bwd_kernel<CX, CW, true>), grid, dim3(CX::NTH), 0, s, dx, dw, n1, n1pad);
  else
    AGN_LAUNCH((split_bwd_kernel<CX, CW, false>), grid, dim3(CX::NTH), 0, s, dx, dw, n1, n1pad);
  return hipGetLastError();
}

template <class Cfg, int BW, int HCM>
hipError_t go_dw(const GemmArgs& g, const HeadDwArgs& h, hipStream_t s) {
  const int units = HCM > 0 ? hdw_units(h) : 0, upad = pad8(units);
  const dim3 grid(upad + tiles_of<Cfg>(g));
  if (g.adam.on)
    AGN_LAUNCH((split_dw_kernel<Cfg, BW, true, HCM>), grid, dim3(Cfg::NTH), 0, s, g, h, units, upad);
  else
    AGN_LAUNCH((split_dw_kernel<Cfg, BW, false, HCM>), grid, dim3(Cfg::NTH), 0, s, g, h, units, upad);
  return hipGetLastError();
}

// Weight gradients of at least this many 64 x 64 tiles go in 64 x 64, fewer in
// 32 x 32 (us, 64 x 64 against 32 x 32): 20 x 128 x 256 x 64, 160 tiles, 8.6
// and 8.0; 6 x 128 x 1000 x 128, 192, 11.0 both; 8 x, 256, 11.2 and 12.1; 12 x,
// 384, 14.0 and 15.5.  Backward launches, 12 x 256 x 256 x 128, 192: 12.6 and
// 12.4; 16 x, 256: 12.9 and 14.0; 24 x 256 x 256 x 256, 384: 27.2 and 28.1.
// MidW's third LDS stage: 20 x 1000 x 784 x 128 59.8 against 60.6, backward
// launch 16 x 256 x 256 x 256 19.2 against 21.4.
constexpr int kMidWTiles = 220;
// The input gradient beside them: 32 x 64 tiles from this many 64 x 64 tiles
// on, 32 x 32 below (us of the launch, 32 x 64 against 32 x 32): 8 x 512 x 512 x
// 64, 64 tiles, 13.7 and 12.9; 12 x, 96, 17.1 and 17.9; 14 x, 112, 18.9 and 19.9;
// 8 x 512 x 512 x 128, 128, 17.4 and 19.8.
constexpr int kFlatDxTiles = 100;

template <int HCM>
hipError_t dw(const GemmArgs& g, const HeadDwArgs& h, hipStream_t s) {
  const bool mid = tiles_of<MidW>(g) >= kMidWTiles;
  if (g.b.vec) return mid ? go_dw<MidW, 4, HCM>(g, h, s) : go_dw<Small, 4, HCM>(g, h, s);
  return mid ? go_dw<MidW, 1, HCM>(g, h, s) : go_dw<Small, 1, HCM>(g, h, s);
}

}  // namespace

hipError_t launch_gemm_f32(int a_kc, int b_kc, const GemmArgs& g, hipStream_t s) {
  if (a_kc && b_kc && g.epi == EPI_FWD_RELU) return fwd<EPI_FWD_RELU>(g, s);
  if (a_kc && b_kc && g.epi == EPI_FWD_LINEAR) return fwd<EPI_FWD_LINEAR>(g, s);
  if (!a_kc && !b_kc && g.epi == EPI_DW_UPDATE) return dw<0>(g, HeadDwArgs{}, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_f32_bwd(const GemmArgs& dx, const GemmArgs& dw, hipStream_t s) {
  if (dx.epi != EPI_DX_MASK || dw.epi != EPI_DW_UPDATE) return hipErrorInvalidValue;
  if (gemm_f32_strip_ok(dx, dw)) return launch_gemm_f32_strip_bwd(dx, dw, s);
  if (tiles_of<MidW>(dw) < kMidWTiles) return go_bwd<Small, Small>(dx, dw, s);
  return tiles_of<Mid>(dx) >= kFlatDxTiles ? go_bwd<Flat, MidW>(dx, dw, s) : go_bwd<Small, MidW>(dx, dw, s);
}

bool gemm_f32_dw_head_ok(const HeadDwArgs& h) { return h.C >= 1 && h.C <= 10 && h.n >= 1 && h.d >= 1; }

hipError_t launch_gemm_f32_dw_head(const GemmArgs& g, const HeadDwArgs& h, hipStream_t s) {
  if (!gemm_f32_dw_head_ok(h)) return hipErrorInvalidValue;
  return dw<10>(g, h, s);
}

}  // namespace agn
