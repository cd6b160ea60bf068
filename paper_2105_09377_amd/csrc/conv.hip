// Host side of the direct 2D convolution of Fig. 2a: weight packing, kernel selection, and the
// combine step of split channel sums.
//
//   out[n,o,x,y] = sum_{c,dx,dy} act[n,c,Sh*x+dx-Ph,Sw*y+dy-Pw] * w[o,c,dx,dy]
//
// Kernels, in the order they are tried:
//   * conv_tile_kernel    (conv_tile_kernel.h)  3x3, 5x5 and (no padding) 1x1 windows of strides 1
//                                            and 2, any channel count: small
//                                            independent workgroups, weights from L2 into registers;
//                                            in the workgroup shape that a cost model picks, unless it
//                                            expects the next ones to be faster;
//   * conv_smallc_kernel  (conv_smallc.hip)  fewer input channels than one 32-byte chunk, fewer than half
//                                            a chunk first of all;
//   * conv_direct4_kernel (conv4_kernel.h)   eight waves, producers and consumers; may split the
//                                            channel sum among workgroups;
//   * conv_direct3_kernel (conv_kernels.h)   four waves doing everything, same LDS layout;
//   * conv_direct_kernel  (conv_kernels.h)   the simple general kernel.
// All of them put output channels on MFMA rows and flattened output positions (n, x, y) on MFMA
// columns (lanes), which makes the (N,O,H',W') store of the listing coalesced, read weights from
// the packed copy [o][tap][channel] and form windows out of an LDS patch [row][pixel][channel].
#include "conv_kernels.h"
#include "conv_scan.h"

#include <stdint.h>

#include <array>
#include <mutex>

namespace gs {

// wr[o][tap][c] = w[o][c][tap] for c < C, zero for C <= c < Cpad.  With `wb` also the blocked
// copy (see conv_blocked_weight_offset): element e of 16-byte piece i of block (ob, chunk, tap) is
// w[ob * 32 + i / 2][chunk * CCH + h * G + e][tap] (zero past C), G = elements in 16 bytes, CCH = 2 G,
// h = (i % 2) ^ (((r >> 2) ^ (r >> 3)) & 1) with r = i / 2 -- the swizzle the consumers'
// fragment reads undo; rows past O are zero.  A thread gathers one 16-byte piece, its G elements T_ apart,
// and writes it to both copies (packing and convolving 512 x 7x7 -> 512, 3x3: 18.3 us, 24.9 with an element per
// thread and copy).
template <typename T>
__global__ void __launch_bounds__(256)
conv_repack_kernel(const T* __restrict__ w, T* __restrict__ wr, T* __restrict__ wb, uint64_t* mark, int O, int C, int T_,
                   int Cpad) {
  if (mark && blockIdx.x == 0 && threadIdx.x == 0) *mark = wb ? kBlockedMark : 0;
  constexpr int G = 16 / int(sizeof(T));
  typedef T piece_t __attribute__((ext_vector_type(G)));
  const int nchunk = Cpad / (2 * G);
  const int64_t pieces = (wb ? round_up(O, 32) : int64_t(O)) * T_ * (Cpad / G);
  for (int64_t f = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; f < pieces; f += int64_t(gridDim.x) * blockDim.x) {
    int64_t o;
    int tap, c0;
    if (wb) {
      const int i = int(f % 64), r = i >> 1, h = (i & 1) ^ (((r >> 2) ^ (r >> 3)) & 1);
      const int64_t blk = f / 64, bt = blk / T_;
      tap = int(blk - bt * T_);
      o = bt / nchunk * 32 + r;
      c0 = (int(bt % nchunk) * 2 + h) * G;
    } else {
      const int64_t ot = f / (Cpad / G);
      c0 = int(f - ot * (Cpad / G)) * G;
      o = ot / T_;
      tap = int(ot - o * T_);
    }
    const T* src = w + (o < O ? o : 0) * C * T_ + tap;
    piece_t v;
#pragma unroll
    for (int e = 0; e < G; ++e) v[e] = o < O && c0 + e < C ? src[int64_t(c0 + e) * T_] : T(0);
    if (wb) *reinterpret_cast<piece_t*>(wb + f * G) = v;
    if (o < O) *reinterpret_cast<piece_t*>(wr + (o * T_ + tap) * Cpad + c0) = v;
  }
}

static int conv_cpad(int in_dtype, int C) {
  const int per_step = in_dtype == GS_I8 ? 32 : 16;   // channels in 32 bytes
  return int(round_up(C, per_step));
}

size_t conv_smallc_weight_offset(int in_dtype, int O, int C, int Kh, int Kw) {
  return size_t(round_up(int64_t(O) * Kh * Kw * conv_cpad(in_dtype, C) * int64_t(dtype_size(in_dtype)), 256));
}

// The two copies in front of the blocked one.
static size_t conv_weight_front_bytes(int in_dtype, int O, int C, int Kh, int Kw) {
  const size_t tap_major = size_t(O) * Kh * Kw * conv_cpad(in_dtype, C) * dtype_size(in_dtype);
  const size_t natural = conv_smallc_weight_bytes(in_dtype, O, C, Kh, Kw);
  return natural ? conv_smallc_weight_offset(in_dtype, O, C, Kh, Kw) + natural : tap_major;
}

size_t conv_blocked_weight_bytes(int in_dtype, int O, int C, int Kh, int Kw) {
  // (channel counts that are no whole chunks: only conv_tile_kernel takes them)
  if (C != conv_cpad(in_dtype, C) && (C * int64_t(dtype_size(in_dtype)) < 16 || Kh != Kw || (Kh != 1 && Kh != 3 && Kh != 5))) return 0;
  return size_t(round_up(O, 32)) * Kh * Kw * conv_cpad(in_dtype, C) * dtype_size(in_dtype);
}

static bool conv_blocked_optional(int in_dtype, int C) { return C != conv_cpad(in_dtype, C); }

size_t conv_blocked_weight_offset(int in_dtype, int O, int C, int Kh, int Kw) {
  return size_t(round_up(int64_t(conv_weight_front_bytes(in_dtype, O, C, Kh, Kw)), 256)) + (conv_blocked_optional(in_dtype, C) ? 256 : 0);
}

uint64_t* conv_blocked_mark(const void* packed, int in_dtype, int O, int C, int Kh, int Kw) {
  if (!conv_blocked_optional(in_dtype, C) || !conv_blocked_weight_bytes(in_dtype, O, C, Kh, Kw)) return nullptr;
  return reinterpret_cast<uint64_t*>(static_cast<uint8_t*>(const_cast<void*>(packed)) + conv_blocked_weight_offset(in_dtype, O, C, Kh, Kw) - 256);
}

size_t conv_weight_workspace(int in_dtype, int O, int C, int Kh, int Kw, bool least) {
  const size_t blocked = least && conv_blocked_optional(in_dtype, C) ? 0 : conv_blocked_weight_bytes(in_dtype, O, C, Kh, Kw);
  return blocked ? conv_blocked_weight_offset(in_dtype, O, C, Kh, Kw) + blocked
                 : conv_weight_front_bytes(in_dtype, O, C, Kh, Kw);
}

hipError_t launch_conv_repack(const void* w, void* wr, int in_dtype, int O, int C, int Kh, int Kw,
                              bool blocked, hipStream_t s) {
  const int Cpad = conv_cpad(in_dtype, C);
  if (int64_t(O) * Kh * Kw * Cpad == 0) return hipSuccess;
  if (conv_is_smallc(in_dtype, C)) return launch_conv_smallc_pack(w, wr, in_dtype, O, C, Kh, Kw, blocked, s);
  const int64_t b = ceil_div(round_up(O, 32) * Kh * Kw * Cpad * int64_t(dtype_size(in_dtype)) / 16, 256);
  const dim3 grid(unsigned(b < 65536 ? b : 65536));
  uint8_t* wb = blocked && conv_blocked_weight_bytes(in_dtype, O, C, Kh, Kw)
                    ? static_cast<uint8_t*>(wr) + conv_blocked_weight_offset(in_dtype, O, C, Kh, Kw)
                    : nullptr;
  uint64_t* const mark = conv_blocked_mark(wr, in_dtype, O, C, Kh, Kw);
  if (in_dtype == GS_I8)
    hipLaunchKernelGGL((conv_repack_kernel<uint8_t>), grid, dim3(256), 0, s,
                       static_cast<const uint8_t*>(w), static_cast<uint8_t*>(wr), wb, mark, O, C, Kh * Kw, Cpad);
  else
    hipLaunchKernelGGL((conv_repack_kernel<uint16_t>), grid, dim3(256), 0, s,
                       static_cast<const uint16_t*>(w), static_cast<uint16_t*>(wr),
                       reinterpret_cast<uint16_t*>(wb), mark, O, C, Kh * Kw, Cpad);
  return hipGetLastError();
}

// Host: most patch rows any tile of TP positions needs, or -1 if a tile spans too many images.
// A scan costs some 15 ns per tile that it looks at: 0.8 us for 64 images of 56x56 in tiles of 256, 46 for 111x113,
// whose tiles do not repeat within them.  Each thread keeps the last ones (256, by a hash of the shape), which
// kernels planned anew on every call look up.
int conv_max_rows(const ConvArgs& a, int64_t M, int HWo, int TP) {
  struct Entry {
    std::array<int64_t, 6> key;
    int rows;
    bool set = false;
  };
  static thread_local Entry kept[256];
  const std::array<int64_t, 6> key = {M, HWo, a.Wo, a.Sh, a.Kh, TP};
  uint64_t h = 14695981039346656037u;
  for (int64_t v : key) h = (h ^ uint64_t(v)) * 1099511628211u;
  Entry& e = kept[(h >> 32) & 255];
  if (!e.set || e.key != key) {
    e.rows = scan_patch_rows(M, HWo, a.Wo, a.Sh, a.Kh, TP, kMaxSeg);
    e.key = key;
    e.set = true;
  }
  return e.rows;
}

int conv_num_cus() {
  static int cus = 0;
  if (!cus) {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
      cus = prop.multiProcessorCount;
    if (cus <= 0) cus = 256;
  }
  return cus;
}

template <typename TR, int TO, int TP, int WO, int WP, int CB>
static hipError_t launch_conv_cfg(const ConvArgs& a, const ConvGeom& g, size_t lds_bytes,
                                  hipStream_t s) {
  auto kern = conv_direct_kernel<TR, TO, TP, WO, WP, CB>;
  static std::once_flag once;
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [&]() {
    attr_status = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(kLdsLimit));
  });
  if (attr_status != hipSuccess) return attr_status;
  const int64_t tiles = ceil_div(g.M, TP) * ceil_div(a.O, TO);
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3(unsigned(tiles)), dim3(256), lds_bytes, s, a, g);
  return hipGetLastError();
}

static size_t conv_lds_bytes(int TO, int T, int CB, int rows, int PW) {
  return 256 + size_t(TO) * (T * CB + 16) + size_t(rows) * PW * (CB + 16);
}

template <typename TR, int TO, int TP, int WO, int WP>
static hipError_t launch_conv_tile(const ConvArgs& a, ConvGeom g, hipStream_t s) {
  g.max_rows = conv_max_rows(a, g.M, g.HWo, TP);
  if (g.max_rows < 0) return hipErrorInvalidValue;
  const int cbytes = a.Cpad * TR::kEsz;
  // Largest channel chunk that divides the padded channel count and leaves room for two
  // workgroups per compute unit; failing that, the largest that fits at all.
  const int cands[3] = {128, 64, 32};
  for (int pass = 0; pass < 2; ++pass) {
    const size_t limit = pass == 0 ? kLdsLimit / 2 : kLdsLimit;
    for (int ci = 0; ci < 3; ++ci) {
      const int CB = cands[ci];
      if (cbytes % CB) continue;
      const size_t need = conv_lds_bytes(TO, g.T, CB, g.max_rows, g.PW);
      if (need > limit) continue;
      if (CB == 128) return launch_conv_cfg<TR, TO, TP, WO, WP, 128>(a, g, need, s);
      if (CB == 64) return launch_conv_cfg<TR, TO, TP, WO, WP, 64>(a, g, need, s);
      return launch_conv_cfg<TR, TO, TP, WO, WP, 32>(a, g, need, s);
    }
  }
  return hipErrorInvalidValue;
}

// The few-channel kernel, or launch_conv_tile<64, 64> in its smallest chunk (32 bytes of channels, which every
// padded channel count is a multiple of).  The latter needs at most: 64 consecutive positions touch at most
// ceil(63 / Wo) + 1 output rows of ceil(63 / HWo) + 1 images (64 / HWo where that divides), and n images with R
// output rows between them (R - n) Sh + n Kh patch rows.
bool conv_direct_fits(const ConvArgs& a) {
  const int64_t N = a.N, Wo = a.Wo, HWo = int64_t(a.Ho) * Wo, Kh = a.Kh, Kw = a.Kw;
  if (N * HWo == 0 || a.O == 0) return true;
  if (conv_smallc_fits(a.in_dtype, a.C, a.W, a.Kh, a.Kw, a.Sh, a.Sw, a.Pw, a.Wo)) return true;
  if (Kh > 512 || Kw > 512) return false;
  const int64_t images = 64 % HWo == 0 ? 64 / HWo : ceil_div(63, HWo) + 1, n = images < N ? images : N;
  const int64_t spanned = ceil_div(63, Wo) + 1, R = spanned < N * a.Ho ? spanned : N * a.Ho;
  if (n > kMaxSeg) return false;
  const int64_t one = (R - 1) * a.Sh + Kh, all = (R > n ? R - n : 0) * a.Sh + n * Kh;
  const int64_t PW = round_up(round_up(a.Pw, 2) + int64_t(a.W) + a.Pw, 2);
  return 256 + 64 * (Kh * Kw * 32 + 16) + (one > all ? one : all) * PW * (32 + 16) <= kLdsLimit;
}

// Pipelined kernel instances (conv3_inst.hip), one per element type and tile shape.
hipError_t launch_conv3_bf16_t0(const ConvArgs&, const ConvGeom&, hipStream_t, bool probe);
hipError_t launch_conv3_bf16_t1(const ConvArgs&, const ConvGeom&, hipStream_t, bool probe);
hipError_t launch_conv3_bf16_t2(const ConvArgs&, const ConvGeom&, hipStream_t, bool probe);
hipError_t launch_conv3_i8_t0(const ConvArgs&, const ConvGeom&, hipStream_t, bool probe);
hipError_t launch_conv3_i8_t1(const ConvArgs&, const ConvGeom&, hipStream_t, bool probe);
hipError_t launch_conv3_i8_t2(const ConvArgs&, const ConvGeom&, hipStream_t, bool probe);

// 64 x 256 or 64 x 128 tiles: whichever needs less time by rounds x cost per tile, a wide tile
// costing 1.44 narrow ones (measured: 196 wide tiles of 256 channels at 14x14 take 23.7 us in one
// round, the same layer in 392 narrow tiles 33.0 us in two).  Few tiles therefore go narrow (more
// compute units busy): 256 channels at 14x14, batch 32, 17.9 us in 196 narrow tiles against 23.7
// in 100 wide ones with a two-way split of the channel sum; 512 channels at 7x7, batch 64, with a
// residual, 28 us in 200 narrow tiles against 34 in 104 wide ones split two ways.
static bool conv_prefers_wide_tile(int64_t M, int O) {
  const int64_t cus = 256;
  const int64_t wide = ceil_div(M, 256) * ceil_div(O, 64), narrow = ceil_div(M, 128) * ceil_div(O, 64);
  return double(ceil_div(wide, cus)) * 1.44 < double(ceil_div(narrow, cus));
}

template <typename TR>
static hipError_t launch_conv3(const ConvArgs& a, const ConvGeom& g, hipStream_t s, bool probe = false) {
  constexpr bool i8 = TR::kEsz == 1;
  if (a.C % (16 / TR::kEsz) != 0 || a.C != a.Cpad) return hipErrorInvalidValue;
  // Tile shapes: 64 channels x 256 positions (three weight buffers fit, the best pipeline) while
  // that still gives most compute units a tile; 64 x 128 for small feature maps; 128 x 128 last.
  auto t0 = [&]() { return i8 ? launch_conv3_i8_t0(a, g, s, probe) : launch_conv3_bf16_t0(a, g, s, probe); };
  auto t1 = [&]() { return i8 ? launch_conv3_i8_t1(a, g, s, probe) : launch_conv3_bf16_t1(a, g, s, probe); };
  auto t2 = [&]() { return i8 ? launch_conv3_i8_t2(a, g, s, probe) : launch_conv3_bf16_t2(a, g, s, probe); };
  hipError_t e = hipErrorInvalidValue;
  const bool wide = conv_prefers_wide_tile(g.M, a.O);
  e = wide ? t1() : t2();
  if (e != hipErrorInvalidValue) return e;
  e = wide ? t2() : t1();
  if (e != hipErrorInvalidValue) return e;
  return a.O > 64 ? t0() : e;
}

// Combines the partial sums of a split channel sum: out = cvt(relu(sum_k partial[k] + residual)).
template <typename AccT>
__global__ void __launch_bounds__(256)
conv_splitk_finish_kernel(const AccT* __restrict__ partial, int ksplit, int64_t total,
                          const void* __restrict__ residual, void* __restrict__ out, int out_dtype,
                          int relu) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < total;
       i += int64_t(gridDim.x) * blockDim.x) {
    AccT v = partial[i];
    for (int k = 1; k < ksplit; ++k) v += partial[int64_t(k) * total + i];
    store_result<AccT>(out, residual, out_dtype, i, v, relu);
  }
}

// Same, four results per thread; total and all pointers are multiples of four elements.
template <typename AccT>
__global__ void __launch_bounds__(256)
conv_splitk_finish_vec_kernel(const AccT* __restrict__ partial, int ksplit, int64_t total,
                              const void* __restrict__ residual, void* __restrict__ out, int out_dtype,
                              int relu) {
  typedef AccT acc4_t __attribute__((ext_vector_type(4)));
  const int64_t nvec = total / 4;
  for (int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; q < nvec;
       q += int64_t(gridDim.x) * blockDim.x) {
    acc4_t v = __builtin_nontemporal_load(reinterpret_cast<const acc4_t*>(partial) + q);
    for (int k = 1; k < ksplit; ++k)
      v += __builtin_nontemporal_load(reinterpret_cast<const acc4_t*>(partial + int64_t(k) * total) + q);
    if constexpr (__is_same(AccT, int32_t)) {
      if (residual) v += reinterpret_cast<const acc4_t*>(residual)[q];
      if (relu) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = v[e] > 0 ? v[e] : 0;
      }
      reinterpret_cast<acc4_t*>(out)[q] = v;
    } else if (out_dtype == GS_F32) {
      if (residual) v += reinterpret_cast<const acc4_t*>(residual)[q];
      if (relu) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.0f);
      }
      reinterpret_cast<acc4_t*>(out)[q] = v;
    } else {
      if (residual) {
        const i32x2 r = reinterpret_cast<const i32x2*>(residual)[q];
        v[0] += __uint_as_float(uint32_t(r.x) << 16); v[1] += __uint_as_float(uint32_t(r.x) & 0xffff0000u);
        v[2] += __uint_as_float(uint32_t(r.y) << 16); v[3] += __uint_as_float(uint32_t(r.y) & 0xffff0000u);
      }
      if (relu) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.0f);
      }
      const i32x2 w = {int32_t(pack_bf16x2(v[0], v[1])), int32_t(pack_bf16x2(v[2], v[3]))};
      reinterpret_cast<i32x2*>(out)[q] = w;
    }
  }
}

int conv_pick_ksplit(int in_dtype, int N, int C, int O, int Ho, int Wo) {
  const int64_t M = int64_t(N) * Ho * Wo;
  const int nchunk = conv_cpad(in_dtype, C) / (in_dtype == GS_I8 ? 32 : 16);
  const int64_t tiles = ceil_div(M, conv_prefers_wide_tile(M, O) ? 256 : 128) * ceil_div(O, 64);
  const int cus = 256;
  if (tiles * 4 <= cus && nchunk % 16 == 0) return 4;
  if (tiles * 2 <= cus && nchunk % 8 == 0) return 2;
  return 1;
}

static ConvGeom conv_geom(const ConvArgs& a) {
  ConvGeom g;
  g.T = a.Kh * a.Kw;
  g.XO = int(round_up(a.Pw, 2));
  g.PW = int(round_up(g.XO + a.W + a.Pw, 2));
  g.HWo = a.Ho * a.Wo;
  g.M = int64_t(a.N) * g.HWo;
  g.pair_ok = (a.W % 2 == 0) ? 1 : 0;
  g.max_rows = 0;
  g.tps = 0;
  g.rb_shift = 0;
  g.pos_major = 0;
  g.dHWo = FastDiv::make(uint32_t(g.HWo > 0 ? g.HWo : 1));
  g.dWo = FastDiv::make(uint32_t(a.Wo > 0 ? a.Wo : 1));
  return g;
}

// conv_tile_kernel instances (conv_tile_inst.hip), one per element type and workgroup shape.
using TileLaunch = hipError_t (*)(const ConvArgs&, const TilePlan&, hipStream_t);
#define GS_TILE_DECL(k, i)                                                                 \
  hipError_t launch_conv_tile_bf16_k##k##s##i(const ConvArgs&, const TilePlan&, hipStream_t); \
  hipError_t launch_conv_tile_i8_k##k##s##i(const ConvArgs&, const TilePlan&, hipStream_t);
#define GS_TILE_DECLS(k)                                                                        \
  GS_TILE_DECL(k, 0) GS_TILE_DECL(k, 1) GS_TILE_DECL(k, 2) GS_TILE_DECL(k, 3) GS_TILE_DECL(k, 4) \
  GS_TILE_DECL(k, 1odd) GS_TILE_DECL(k, 2odd) GS_TILE_DECL(k, 3odd) GS_TILE_DECL(k, 4odd)
GS_TILE_DECLS(1) GS_TILE_DECLS(3) GS_TILE_DECLS(5)
#undef GS_TILE_DECLS
#undef GS_TILE_DECL

template <typename TR>
static hipError_t launch_tiles(const ConvArgs& a, const TilePlan& plan, hipStream_t s) {
#define GS_TILE_ROW(t, k)                                                                              \
  {launch_conv_tile_##t##_k##k##s0, launch_conv_tile_##t##_k##k##s1, launch_conv_tile_##t##_k##k##s2, \
   launch_conv_tile_##t##_k##k##s3, launch_conv_tile_##t##_k##k##s4}
  static constexpr TileLaunch bf16[3][kNumTileShapes] = {GS_TILE_ROW(bf16, 1), GS_TILE_ROW(bf16, 3), GS_TILE_ROW(bf16, 5)};
  static constexpr TileLaunch i8[3][kNumTileShapes] = {GS_TILE_ROW(i8, 1), GS_TILE_ROW(i8, 3), GS_TILE_ROW(i8, 5)};
#undef GS_TILE_ROW
#define GS_TILE_ROW(t, k)                                                                                       \
  {nullptr, launch_conv_tile_##t##_k##k##s1odd, launch_conv_tile_##t##_k##k##s2odd, launch_conv_tile_##t##_k##k##s3odd, \
   launch_conv_tile_##t##_k##k##s4odd}
  static constexpr TileLaunch bf16_odd[3][kNumTileShapes] = {GS_TILE_ROW(bf16, 1), GS_TILE_ROW(bf16, 3), GS_TILE_ROW(bf16, 5)};
  static constexpr TileLaunch i8_odd[3][kNumTileShapes] = {GS_TILE_ROW(i8, 1), GS_TILE_ROW(i8, 3), GS_TILE_ROW(i8, 5)};
#undef GS_TILE_ROW
  if (plan.odd) return (TR::kEsz == 1 ? i8_odd : bf16_odd)[a.Kh / 2][plan.shape](a, plan, s);
  return (TR::kEsz == 1 ? i8 : bf16)[a.Kh / 2][plan.shape](a, plan, s);
}

// Time of a layer in each workgroup shape, in microseconds, fitted by window size to measured times of
// 240 (1x1), 620 (3x3) and 200 (5x5) layers of 1 to 128 images, 16 to 512 channels on either side,
// planes of 7x7 to 112x112, strides 1 and 2, both element types (mean error 13 %).  On 500, 400 and 150
// other layers of these ranges, weights packed: the way it picks is 2 to 4 % slower than the fastest one on
// average (at worst 1.4 times for 3x3, 2.1 for 5x5), and 1.5, 2.8 and 4.3 times faster than the kernels
// without this one; 15 of the 1050 layers are slower than in those by more than 3 %, 2 by more than 10.  A workgroup alone takes wg + store + cnt * alone; a compute unit that
// is given one after the other takes 0.6 store + cnt * busy for each.  `store` grows by `cut` for
// planes that are no multiple of a 16-byte store's positions, the chunks by `item` for each patch
// item of a thread beyond the first and by `strided` for stride 2.  `at_once`: workgroups that fit a
// compute unit together.
struct TileCost {
  float base, wg, alone, busy, store, cut, item, at_once, strided;
};
constexpr TileCost kTileCost[3][kNumTileShapes] = {   // shapes as in kTileShapes
    {{1.00f, 4.40f, 0.59f, 3.79f, 1.00f, 1.00f, 0.57f, 2, 0.57f},
     {1.01f, 2.92f, 0.26f, 0.55f, 1.00f, 0.99f, 4.87f, 3, 0.0f},
     {1.00f, 2.66f, 0.44f, 0.62f, 1.00f, 0.99f, 4.15f, 3, 0.0f},
     {1.38f, 0.47f, 0.93f, 0.39f, 1.12f, 0.55f, 1.01f, 3, 0.21f},
     {1.77f, 1.54f, 0.65f, 0.53f, 0.37f, 0.78f, 0.99f, 4, 0.30f}},
    {{0.22f, 5.32f, 0.854f, 1.488f, 1.02f, 1.02f, 0.0f, 2, 0.32f},
     {0.98f, 3.08f, 0.622f, 0.750f, 1.02f, 0.66f, 0.88f, 3, 0.32f},
     {2.35f, 1.32f, 0.637f, 0.706f, 1.02f, 0.68f, 1.58f, 3, 0.23f},
     {1.73f, 2.19f, 0.919f, 1.230f, 0.07f, 5.87f, 0.90f, 3, 0.0f},
     {0.91f, 2.83f, 0.714f, 0.865f, 0.02f, 0.20f, 1.36f, 4, 0.0f}},
    {{0, 0, 0, 0, 0, 0, 0, 1, 0},                     // not taken (tile_geometry)
     {0.99f, 3.53f, 1.15f, 2.35f, 1.00f, 1.06f, 1.30f, 3, 0.01f},
     {1.07f, 3.38f, 1.15f, 2.06f, 0.97f, 0.97f, 0.79f, 3, 0.0f},
     {1.05f, 0.89f, 2.37f, 1.72f, 1.00f, 1.01f, 0.69f, 3, 0.0f},
     {1.02f, 2.72f, 1.18f, 1.35f, 0.03f, 17.0f, 0.99f, 4, 0.18f}},
};

// The same where channels do not fill the last chunk: what a chunk costs in the place of one, with `item` more for each patch item of a
// thread beyond the first; `start` us for each of those, and `groups` us in the shapes that split the channel sum, in front
// of a workgroup's first chunk.  Fitted to 1118 layers of 3x3 and 5x5 windows and 334 of 1x1 in every shape that takes
// them (mean error 13 and 16 %, 32 and 37 with each chunk a tenth dearer and nothing else); the shape it picks is 1.1 and 1.4 %
// slower than the fastest on average, 7.6 and 8.7 before (47 images of 26 bytes 15x26 -> 16, 5x5: four items 15.8 us, one 6.6).
struct TileOdd {
  float chunk, item, start, groups;
};
constexpr TileOdd kTileOdd[2] = {{1.09f, 0, 1.11f, 0.72f}, {0.91f, 0.29f, 0.94f, 0.64f}};     // 1x1, others

// Positions per tile of at most `tp`: fewest rounds over the compute units, then whole output rows
// (a patch row fewer), then the widest.  Multiples of eight, so that stores are whole.
static int tile_positions(int64_t M, int n_ot, int Wo, int tp) {
  int64_t best = INT64_MAX;
  int tps = tp;
  for (int t = tp; t >= tp / 2; t -= 8) {
    const int64_t c = ceil_div(ceil_div(M, t) * n_ot, conv_num_cus()) * 8 - (t % Wo == 0 ? 1 : 0);
    if (c < best) best = c, tps = t;
  }
  return tps;
}

// The layer in workgroup shape `shape` and tiles of `tps` positions, `whole`: whole output rows; false where it does
// not fit (LDS, patch items per thread).
static bool tile_geometry(const ConvArgs& a, const ConvGeom& g0, int shape, int tps, bool whole, TilePlan* p, float* cost) {
  const TileShape sh = kTileShapes[shape];
  const int to = 32 * sh.wo, S = a.Sh, threads = 64 * sh.wo * sh.wp;
  const bool point = a.Kh == 1;        // patch rows are output rows, several chunks at a time
  const int cm = point ? kTileChunks : 1;
  p->shape = shape;
  p->g = g0;
  ConvGeom& g = p->g;
  p->il = 1;                           // a group of il interleaved blocks: il positions lie in one output row
  if (sh.ks == 1 && sh.nj >= 4 && S == 1 && a.Wo % 4 == 0) p->il = 4;
  else if (sh.ks == 1 && sh.nj >= 2 && a.Wo % 2 == 0) p->il = 2;
  const int n_ot = int(ceil_div(a.O, to));
  g.tps = tps;
  ConvArgs r = a;
  if (point) r.Sh = 1;
  const int max_rows = conv_max_rows(r, g.M, g.HWo, g.tps);
  if (max_rows < 0) return false;
  const int64_t segs = (g.tps + g.HWo - 2) / g.HWo + 1;
  const int64_t items = point ? 2 * cm * max_rows * ceil_div(a.W, kTileItem)
                              : 2 * (ceil_div(int64_t(max_rows) * a.W, kTileItem) + segs);
  if (a.Kh == 5 && sh.nj > 2) return false;              // a ring of 25 taps leaves no registers for it
  p->maxi = items <= threads ? 1 : items <= 2 * threads ? 2 : 4;
  if (items > 4 * threads || (sh.nj > 2 && p->maxi > 2)) return false;
  const int nchunk = int(ceil_div(a.Cpad * int64_t(dtype_size(a.in_dtype)), 32 * cm)), cnt = int(ceil_div(nchunk, sh.ks));
  p->odd = a.C * int(dtype_size(a.in_dtype)) % (32 * cm) != 0;
  if (p->odd && shape == 0) return false;                // not built
  p->one = sh.ks > 1 && cnt == 1 && !p->odd;
  const int PH = p->il * S;
  const int lastcol = a.W + a.Pw - 1 > (a.Wo - 1) * S + a.Kw - 1 ? a.W + a.Pw - 1 : (a.Wo - 1) * S + a.Kw - 1;
  const int64_t php = (lastcol / PH + 1) * 16, bufb = 2 * cm * max_rows * PH * php;
  const int64_t patches = sh.ks * (p->one ? 1 : 3) * bufb;
  const int64_t results = (sh.ks > 1 ? int64_t(sh.ks) * sh.wo * sh.wp * sh.nj * 4096 : 0) +
                          int64_t(sh.wo) * sh.wp * 32 * (32 * (sh.nj < 4 ? sh.nj : 4) * 4 + 16);
  const int64_t lds = patches > results ? patches : results;
  const int64_t tiles_m = ceil_div(g.M, g.tps), tiles = tiles_m * n_ot;
  if (lds > kLdsLimit || tiles > 0x7fffffff) return false;
  g.php = int(php);
  g.rowp = PH * g.php;
  g.halfb = max_rows * g.rowp;
  g.bufb = int(bufb);
  p->lds_bytes = int(lds);
  p->tiles = int(tiles);
  // Tile order: the one of the producer / consumer kernel (conv3_inst.hip).
  const double in_b = double(a.N) * a.C * a.H * a.W * dtype_size(a.in_dtype);
  const double w_b = double(a.O) * a.C * a.Kh * a.Kw * dtype_size(a.in_dtype);
  const double ch_first = in_b * n_ot + w_b * (n_ot < 8 ? 8.0 / n_ot : 1.0);
  const double pos_first = in_b + w_b * 8.0 * (w_b > 3.0e6 ? double(ceil_div(tiles_m, 8)) : 1.0);
  g.pos_major = (n_ot > 1 && pos_first < ch_first) ? 1 : 0;
  g.dTiles = FastDiv::make(uint32_t(g.pos_major ? n_ot : tiles_m));
  g.dW = FastDiv::make(uint32_t(a.W));
  g.dXG = FastDiv::make(uint32_t(ceil_div(a.W, kTileItem)));
  const TileCost& c = kTileCost[a.Kh / 2][shape];
  const int group = a.in_dtype == GS_I8 || a.out_dtype == GS_F32 ? 4 : 8;     // positions of a 16-byte store
  const int64_t rows = ceil_div(g.tps, a.Wo);
  const float per_thread = point ? float(2 * cm * (whole ? rows : rows + 1) * ceil_div(a.W, kTileItem)) / threads
                                 : float((rows * S + a.Kh) * a.W) / (2 * threads);
  // Channels that do not fill the last chunk: items beyond the first cost more, in every chunk and before the first one, and
  // channel-sum groups, whose chunks are seldom one for each, start later (TileOdd).
  const TileOdd& od = kTileOdd[point ? 0 : 1];
  const float more = p->odd ? float(p->maxi - 1) : 0.0f;
  const float chunk = (p->odd ? od.chunk + od.item * more : 1.0f) + (S == 2 ? c.strided : 0.0f) + c.item * (per_thread > 1 ? per_thread - 1 : 0.0f);
  const float store = c.store * (g.HWo % group ? 1 + c.cut : 1.0f);
  const float start = p->odd ? od.start * more + (sh.ks > 1 ? od.groups : 0.0f) : 0.0f;
  const float alone = c.wg + start + store + c.alone * cnt * chunk, busy = c.busy * cnt * chunk + 0.6f * store + start;
  const float by_rounds = alone * ceil_div(tiles, int64_t(256 * c.at_once));
  const float by_work = alone + busy * float(ceil_div(tiles, 256) - 1);
  *cost = c.base + (by_rounds > by_work ? by_rounds : by_work);
  return true;
}

// Ways to cut a layer: every workgroup shape with the positions of tile_positions, then, for 1x1 windows, with
// whole output rows.  Those stage the whole rows that a tile touches and nothing around them, so that a tile
// that ends with a row stages no pixel in vain: 40 images of 94x94 x 128 bytes -> 16 in tiles of 120 positions 77 us,
// of 94 26 (31 in the producer / consumer kernel).  Over 211 layers of more than 8 us the cheaper cut is 1.33 times
// faster than the first kind alone, 6 layers lose 3 to 15 %.
constexpr int kTileWays = 2 * kNumTileShapes;
static bool tile_way(const ConvArgs& a, const ConvGeom& g, int way, TilePlan* p, float* cost) {
  const int shape = way % kNumTileShapes;
  const TileShape sh = kTileShapes[shape];
  const int tp = 32 * sh.nj * sh.wp, tps = tile_positions(g.M, int(ceil_div(a.O, 32 * sh.wo)), a.Wo, tp);
  if (way == shape) return tile_geometry(a, g, shape, tps, false, p, cost);
  const int whole = tp / a.Wo * a.Wo;
  return a.Kh == 1 && whole > 0 && whole != tps && tile_geometry(a, g, shape, whole, true, p, cost);
}

// The same for the producer / consumer kernel (290 layers, mean error 14 %).
static float pipelined_cost(const ConvArgs& a, const ConvGeom& g) {
  const bool wide = conv_prefers_wide_tile(g.M, a.O);
  const float narrow = wide ? 1.0f : 0.507f;
  const int64_t tiles = ceil_div(g.M, wide ? 256 : 128) * ceil_div(a.O, 64) * a.ksplit;
  const int chunks = a.Cpad * int(dtype_size(a.in_dtype)) / 32 / a.ksplit;
  return 4.36f + float(ceil_div(tiles, 256)) * narrow *
                     (2.61f * (g.HWo % 4 ? 2.25f : 1.0f) + 1.17f * chunks * (a.Sh == 2 ? 1.63f : 1.0f)) +
         (a.ksplit > 1 ? 3.59f : 0.0f);
}

// A 1x1 window's matrix gathered and multiplied by the dense kernels (fitted to 246 layers; mean error 28 % over 500
// others).  What counts is that it is the faster way for large ones: 128 images of 28x28 x 512 -> 512 142 us
// against 165.  Few channels and many results are where it errs most: 12 images of 103x72 x 64 -> 473 go to the
// tiles, 61 us against 35.  In MB and MFLOP.
static float gathered_cost(const ConvArgs& a, const ConvGeom& g) {
  const float esz = float(dtype_size(a.in_dtype)), m = float(g.M) * 1e-6f;
  return 7.7f + 0.27f * esz * a.C * (m + float(a.N) * a.H * a.W * 1e-6f) + 0.00072f * esz * a.C * a.O * m +
         0.44f * float(dtype_size(a.out_dtype)) * a.O * m * (a.residual ? 2 : 1);
}

// Does conv_tile_kernel take the layer, in a workgroup shape that fits?
template <typename TR>
static bool tile_takes(const ConvArgs& a, bool natural) {
  const bool window = a.Kh == a.Kw && (a.Kh == 3 || a.Kh == 5 || (a.Kh == 1 && a.Ph + a.Pw == 0));
  // Weights as they come are read in 16-byte pieces; channels that do not fill the last chunk: 32-bit offsets of planes.
  const bool whole = a.C * TR::kEsz % (a.Kh == 1 ? 32 * kTileChunks : 32) == 0;
  if (!whole && ((natural && a.C * TR::kEsz % 16 != 0) || int64_t(a.H) * a.W * TR::kEsz >= (1 << 24))) return false;
  return (a.wblk || (natural && a.Kh == 1)) && window && a.Sh == a.Sw && a.Sh <= 2 && a.W >= kTileItem &&
         round_up(a.O, 32) * a.Kh * a.Kw * a.Cpad * TR::kEsz < (int64_t(1) << 32);
}

// How the layer runs on conv_tile_kernel, or shape -1.  A plan depends on the shape alone; each
// thread keeps the last ones it made (64, by a hash of the shape), since making one takes a scan of the tiles
// (conv_max_rows) in up to five workgroup shapes: 5 us for 56x56, up to 0.5 ms for large planes of odd sizes (1x1: twice that).
template <typename TR>
static const TilePlan& plan_tiles(const ConvArgs& a, const ConvGeom& g, bool natural = false) {
  struct Entry {
    std::array<int, 18> key;
    TilePlan plan;
    bool set = false;
  };
  static thread_local Entry kept[64];
  const std::array<int, 18> key = {a.in_dtype, a.out_dtype, a.N, a.C, a.H, a.W, a.O, a.Kh, a.Kw, a.Sh, a.Sw, a.Ph, a.Pw, a.ksplit,
                                   a.Cpad, a.wblk != nullptr, natural, a.residual != nullptr};
  uint32_t h = 2166136261u;
  for (int v : key) h = (h ^ uint32_t(v)) * 16777619u;
  Entry& e = kept[(h >> 16) & 63];
  if (e.set && e.key == key) return e.plan;
  TilePlan best;
  best.shape = -1;
  if (tile_takes<TR>(a, natural)) {
    float least = 0;
    for (int i = 0; i < kTileWays; ++i) {
      TilePlan p;
      float cost;
      if (tile_way(a, g, i, &p, &cost) && (best.shape < 0 || cost < least)) {
        best = p;
        least = cost;
      }
    }
    // The estimates err by 14 % (the gathered matrix's by 28): a tenth in favour of the older way keeps it where
    // it is the faster one.
    if (best.shape >= 0 && (natural ? 0.9f * gathered_cost(a, g) < least
                                    : a.Kh == 3 && launch_conv3<TR>(a, g, nullptr, true) == hipSuccess &&
                                          0.9f * pipelined_cost(a, g) < least))
      best.shape = -1;
  }
  e.key = key;
  e.plan = best;
  e.set = true;
  return e.plan;
}

template <typename TR>
static hipError_t launch_conv_t(const ConvArgs& a_in, hipStream_t s) {
  ConvArgs a = a_in;
  if (a.ksplit < 2 || !a.partial) {
    a.ksplit = 1;
    a.partial = nullptr;
  }
  const ConvGeom g = conv_geom(a);
  if (g.M == 0 || a.O == 0) return hipSuccess;
  // Fewer channels than a chunk: half of one at least on conv_tile_kernel, but 1x1 windows and few results, and all
  // others, as im2col rows formed in LDS.  350 layers of 8 to 15 channels (16 to 31 in bytes), us, in LDS rows / in tiles:
  // 1.5 times faster on average (64 images of 15, 26x14 -> 384, 3x3 stride 2 88 / 6.5; 34 of 29 in bytes, 18x46 -> 400
  // 108 / 20; 2 of 8, 26x20 -> 96 5.7 / 5.6), four below 0.9 (14 of 8, 9x7 -> 2, 5x5, 6.3 / 8.2); 1x1: 10 of 25 in
  // bytes, 73x26 -> 208 53 / 11, but 10 of 9, 12x53 -> 16 5.4 / 6.9.
  const bool rows_first = a.wnat && a.Kh == 1 && a.O <= 64;
  const TilePlan& plan = plan_tiles<TR>(a, g);
  if (plan.shape >= 0 && !rows_first) return launch_tiles<TR>(a, plan, s);
  if (a.wnat) {
    ConvArgs b = a;
    b.wr = a.wnat;
    const hipError_t es = launch_conv_smallc(b, nullptr, s);
    if (es != hipErrorInvalidValue) return es;
  }
  if (plan.shape >= 0) return launch_tiles<TR>(a, plan, s);
  hipError_t e = launch_conv3<TR>(a, g, s);
  if (a.ksplit > 1) {
    if (e == hipSuccess) {
      using AccT = typename TR::acc_t;
      const int64_t total = g.M * a.O;
      const size_t osz = dtype_size(a.out_dtype);
      const bool vec = total % 4 == 0 && reinterpret_cast<uintptr_t>(a.partial) % 16 == 0 &&
                       reinterpret_cast<uintptr_t>(a.out) % (4 * osz) == 0 &&
                       reinterpret_cast<uintptr_t>(a.residual) % (4 * osz) == 0;
      const int64_t b = ceil_div(vec ? total / 4 : total, 256);
      const dim3 grid(unsigned(b < 4096 ? b : 4096));
      if (vec)
        hipLaunchKernelGGL((conv_splitk_finish_vec_kernel<AccT>), grid, dim3(256), 0, s,
                           static_cast<const AccT*>(a.partial), a.ksplit, total, a.residual, a.out,
                           a.out_dtype, a.relu);
      else
        hipLaunchKernelGGL((conv_splitk_finish_kernel<AccT>), grid, dim3(256), 0, s,
                           static_cast<const AccT*>(a.partial), a.ksplit, total, a.residual, a.out,
                           a.out_dtype, a.relu);
      return hipGetLastError();
    }
    if (e != hipErrorInvalidValue) return e;
    a.ksplit = 1;                      // no splitting kernel takes this shape: plain path
    a.partial = nullptr;
    e = launch_conv3<TR>(a, g, s);
  }
  if (e != hipErrorInvalidValue) return e;
  if (a.O > 64) {
    e = launch_conv_tile<TR, 128, 128, 2, 2>(a, g, s);
    if (e != hipErrorInvalidValue) return e;
  }
  e = launch_conv_tile<TR, 64, 128, 1, 4>(a, g, s);
  if (e != hipErrorInvalidValue) return e;
  return launch_conv_tile<TR, 64, 64, 2, 2>(a, g, s);
}

// 1x1 windows without padding on weights in the listing's order (a.wr = ((O),(C))): one launch, no
// packing.  hipErrorInvalidValue where conv_tile_kernel does not take the layer.
template <typename TR>
static hipError_t launch_conv_point_t(const ConvArgs& a_in, hipStream_t s) {
  ConvArgs a = a_in;
  a.Cpad = conv_cpad(a.in_dtype, a.C);
  a.ksplit = 1;
  a.wblk = nullptr;
  const ConvGeom g = conv_geom(a);
  if (g.M == 0 || a.O == 0) return hipSuccess;
  if (a.Kh != 1 || a.Kw != 1) return hipErrorInvalidValue;
  const TilePlan& plan = plan_tiles<TR>(a, g, true);
  return plan.shape >= 0 ? launch_tiles<TR>(a, plan, s) : hipErrorInvalidValue;
}
hipError_t launch_conv_point(const ConvArgs& a, hipStream_t s) {
  return a.in_dtype == GS_I8 ? launch_conv_point_t<I8Traits>(a, s) : launch_conv_point_t<Bf16Traits>(a, s);
}

template <typename TR>
static hipError_t conv_tile_forced_t(const ConvArgs& a_in, int way, bool launch, int* out, hipStream_t s) {
  ConvArgs a = a_in;
  a.ksplit = 1;
  const bool natural = !a.wblk;
  const ConvGeom g = conv_geom(a);
  if (g.M == 0 || a.O == 0 || way >= kTileWays || !tile_takes<TR>(a, natural)) return hipErrorInvalidValue;
  TilePlan p;
  float cost;
  if (way < 0) p = plan_tiles<TR>(a, g, natural);
  else if (!tile_way(a, g, way, &p, &cost)) return hipErrorInvalidValue;
  if (p.shape < 0) return hipErrorInvalidValue;
  out[0] = p.shape; out[1] = p.il; out[2] = p.maxi; out[3] = p.one; out[4] = p.g.tps;
  return launch ? launch_tiles<TR>(a, p, s) : hipSuccess;
}
hipError_t conv_tile_forced(const ConvArgs& a, int way, bool launch, int* out, hipStream_t s) {
  return a.in_dtype == GS_I8 ? conv_tile_forced_t<I8Traits>(a, way, launch, out, s)
                             : conv_tile_forced_t<Bf16Traits>(a, way, launch, out, s);
}

// A residual block's shortcut: its pixels are the centre taps of 3x3 windows padded by one, and both strides are two.
bool conv_projection_fits(const ConvArgs& a) {
  return a.in_dtype == GS_BF16 && a.Kh == 3 && a.Kw == 3 && a.Sh == 2 && a.Sw == 2 && a.Ph == 1 && a.Pw == 1 && a.wblk && a.wproj && a.C == a.Cpad;
}
// Taken wherever the layer alone has a plan, and with that plan: 89 random layers of 16 to 480 channels, 7x7 to 112x112, were 1.11
// to 1.95 times faster than in two launches (6 images of 448 channels 28x58 -> 19 36.5 / 32.8 us, 4 of 224 90x64 -> 112 20.1 /
// 15.3, 1 of 48 28x28 -> 65 10.9 / 6.7), none slower.
hipError_t launch_conv_with_projection(const ConvArgs& a_in, hipStream_t s) {
  ConvArgs a = a_in;
  if (!conv_projection_fits(a)) return hipErrorInvalidValue;
  a.ksplit = 1;
  a.partial = nullptr;
  const ConvGeom g = conv_geom(a);
  if (g.M == 0 || a.O == 0) return hipErrorInvalidValue;
  const TilePlan& plan = plan_tiles<Bf16Traits>(a, g);
  return plan.shape >= 0 ? launch_tiles<Bf16Traits>(a, plan, s) : hipErrorInvalidValue;
}

bool conv_pipelined_takes(const ConvArgs& a_in) {
  ConvArgs a = a_in;
  a.Cpad = conv_cpad(a.in_dtype, a.C);
  if (conv_is_smallc(a.in_dtype, a.C) || !conv_blocked_weight_bytes(a.in_dtype, a.O, a.C, a.Kh, a.Kw)) return false;
  a.wblk = &a;      // asked for, never read
  const ConvGeom g = conv_geom(a);
  if (g.M == 0 || a.O == 0) return false;
  auto takes = [&](int ksplit) {
    a.ksplit = ksplit;
    return (a.in_dtype == GS_I8 ? launch_conv3<I8Traits>(a, g, nullptr, true) : launch_conv3<Bf16Traits>(a, g, nullptr, true)) == hipSuccess;
  };
  const int ksplit = conv_pick_ksplit(a.in_dtype, a.N, a.C, a.O, a.Ho, a.Wo);
  return takes(ksplit) || (ksplit > 1 && takes(1));
}

bool conv_tiles_take(const ConvArgs& a_in) {
  ConvArgs a = a_in;
  a.Cpad = conv_cpad(a.in_dtype, a.C);
  a.ksplit = 1;
  if (conv_is_smallc(a.in_dtype, a.C) || !conv_blocked_weight_bytes(a.in_dtype, a.O, a.C, a.Kh, a.Kw)) return false;
  a.wblk = &a;      // asked for, never read
  const ConvGeom g = conv_geom(a);
  if (g.M == 0 || a.O == 0) return false;
  return (a.in_dtype == GS_I8 ? plan_tiles<I8Traits>(a, g) : plan_tiles<Bf16Traits>(a, g)).shape >= 0;
}

hipError_t launch_conv(const ConvArgs& a, hipStream_t s) {
  return a.in_dtype == GS_I8 ? launch_conv_t<I8Traits>(a, s) : launch_conv_t<Bf16Traits>(a, s);
}

}  // namespace gs
