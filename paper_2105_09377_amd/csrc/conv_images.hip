// Convolution of small images with weights as they come, in one launch and without a workspace: the windows of
// the im2col matrix (Fig. 5) are gathered from whole images in LDS straight into the registers of the MFMAs.
//
// A workgroup has four waves and one tile of 32 output channels x 32 positions.  It copies the images that its
// positions lie in to LDS (consecutive memory, 16-byte loads), and beside them its channels' weights as rows
// that end in zeros at a whole MFMA step.  The waves share the steps of the contraction; a lane's 16 bytes of
// a step are the elements k .. of one position's window, looked up one by one: a table holds for every k = (c,
// dx, dy) the offset c H W + dx W + dy and (dx, dy), by which cells outside the image become zero.  The partial tiles
// meet in LDS and are added pairwise.
//
// What bounds it: the launch, and two latencies (arguments, then images and weights).  Calls of this size are
// paid by the launch -- some 3 us of host time each -- so that gathering the matrix, padding the weights and
// multiplying in launches of their own costs two to three times as much.  40 random calls of up to 4 images of up
// to 16 channels and 32x32, up to 48 results, GPU time alone: the im2col form 1.52 times faster on average (1.14 at least; 2
// images of 1 channel 19x20 -> 30, 1x1: 9.7 -> 4.6 us; 1 of 7 channels 15x9
// -> 8, 3x3 int8 at stride 2: 6.2 -> 4.1), the direct form, against conv_smallc_kernel and against packing first, 1.30 (one
// 1x1 call of 40 7 % slower).  80 others of up to 16 images, 40
// channels and 200 results: none slower.
#include "smallc_copies.h"

#include <mutex>

namespace gs {

constexpr int kImagesThreads = 256, kImagesLds = 158 * 1024;    // of a workgroup that has a compute unit for itself
constexpr int kImagesRS = 160;          // row stride of a partial tile: both half-waves on other banks
constexpr int kImagesExtent = 192;      // rows and columns of an image, at most

struct ImagesArgs {
  ConvArgs c;                           // c.wr: the listing's ((O),(C,Kh,Kw))
  SmallCCopies copies;                  // written by the workgroups behind the tiles
  unsigned tiles;
  int M, K, ppr, wpb;                   // positions, contraction length, 16-byte pieces and LDS bytes of a weight row
  uint32_t lds_w, lds_tab, lds_part;    // LDS: images and a cell of zeros | weights | table | partial tiles
  FastDiv dHWo, dWo, dT, dKw, dtp, dppr;
};

template <typename TR, bool COPIES>
__global__ void __launch_bounds__(kImagesThreads) conv_images_kernel(ImagesArgs p) {
  constexpr int ESZ = TR::kEsz, G = 16 / ESZ, NT = kImagesThreads, NW = NT / 64;
  using T = typename std::conditional<ESZ == 1, uint8_t, uint16_t>::type;
  using acc_t = typename TR::acc_t;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const ConvArgs& a = p.c;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if constexpr (COPIES) {
    if (blockIdx.x >= p.tiles) {
      write_copies(static_cast<const T*>(a.wr), p.copies, (blockIdx.x - p.tiles) * unsigned(NT) + unsigned(tid),
                   (gridDim.x - p.tiles) * unsigned(NT));
      return;
    }
  }
  uint32_t ot, pt;
  p.dtp.divmod(blockIdx.x, &ot, &pt);
  const int o0 = int(ot) * 32, m0 = int(pt) * 32, mend = m0 + 32 < p.M ? m0 + 32 : p.M;
  const int n_first = int(p.dHWo.div(uint32_t(m0))), n_last = int(p.dHWo.div(uint32_t(mend - 1)));
  const int HW = a.H * a.W, CHW = a.C * HW;               // (CHW fits 16 bits: host check)
  const int img_bytes = (n_last - n_first + 1) * CHW * ESZ, Kb = p.K * ESZ;
  const uint8_t* const img = static_cast<const uint8_t*>(a.act) + int64_t(n_first) * CHW * ESZ;
  const uint8_t* const w = static_cast<const uint8_t*>(a.wr);
  const int n_img = (img_bytes + 15) / 16, n_w = 32 * p.ppr;

  // Images and weights, up to eight and four pieces of each thread requested at once.  The last piece of the images and of
  // a row lies 16 bytes in front of the end; what is shorter than a piece comes element by element.
  auto short_piece = [](const uint8_t* at, int bytes) {
    i32x4 v = {0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < 16; ++b) v[b >> 2] |= int32_t((b < bytes ? uint32_t(at[b < bytes ? b : 0]) : 0u) << (8 * (b & 3)));
    return v;
  };
  auto image_piece = [&](int f) {
    if (img_bytes >= 16) return i32x4(*reinterpret_cast<const i32x4_any*>(img + (f * 16 < img_bytes - 16 ? f * 16 : img_bytes - 16)));
    return short_piece(img, img_bytes);
  };
  auto weight_piece = [&](int f) {
    uint32_t r, c;
    p.dppr.divmod(uint32_t(f), &r, &c);
    const uint8_t* const row = w + int64_t(o0 + int(r) < a.O ? o0 + int(r) : a.O - 1) * Kb;   // (rows past O are never stored)
    if (Kb >= 16) {
      const int at = int(c) * 16 < Kb - 16 ? int(c) * 16 : Kb - 16;
      return row_piece_fix(*reinterpret_cast<const i32x4_any*>(row + at), int(c) * 16 - at);
    }
    return c == 0 ? short_piece(row, Kb) : i32x4{0, 0, 0, 0};
  };
  uint32_t* const tab = reinterpret_cast<uint32_t*>(lds + p.lds_tab);
  {
    constexpr int NI = 8, NWP = 4;
    i32x4 iv[NI], wv[NWP];
    for (int base = 0; base < n_img || base / 2 < n_w; base += NI * NT) {     // uniform
      const int b_img = base, b_w = base / 2;
      static_assert(NI == 2 * NWP, "both advance together");
#pragma unroll
      for (int u = 0; u < NWP; ++u)
        if (b_w + u * NT + tid < n_w) wv[u] = weight_piece(b_w + u * NT + tid);
#pragma unroll
      for (int u = 0; u < NI; ++u)
        if (b_img + u * NT + tid < n_img) iv[u] = image_piece(b_img + u * NT + tid);
      if (base == 0) {                                     // while they are on their way: the table and the zeros
        const int steps_k = p.ppr * G;
        for (int k = tid; k < steps_k; k += NT) {
          uint32_t c, t, dx, dy;
          p.dT.divmod(uint32_t(k), &c, &t);
          p.dKw.divmod(t, &dx, &dy);
          // (past K: a row that no image has)
          tab[k] = k < p.K ? (c * uint32_t(HW) + dx * uint32_t(a.W) + dy) | dx << 16 | dy << 24 : 255u << 16;
        }
        if (tid < 4) reinterpret_cast<uint32_t*>(lds + p.lds_w - 16)[tid] = 0;
      }
#pragma unroll
      for (int u = 0; u < NWP; ++u) {
        const int f = b_w + u * NT + tid;
        if (f < n_w) {
          uint32_t r, c;
          p.dppr.divmod(uint32_t(f), &r, &c);
          *reinterpret_cast<i32x4*>(lds + p.lds_w + r * p.wpb + c * 16) = wv[u];
        }
      }
#pragma unroll
      for (int u = 0; u < NI; ++u) {
        const int f = b_img + u * NT + tid;
        if (f < n_img) *reinterpret_cast<i32x4_any*>(lds + (f * 16 < img_bytes - 16 || img_bytes < 16 ? f * 16 : img_bytes - 16)) = iv[u];
      }
    }
  }

  // This lane's position: window origin, and the LDS index of its first element (may lie in front of the image).
  int m = m0 + (lane & 31);
  m = m < mend ? m : mend - 1;                             // its results are dropped
  uint32_t n, pos, ho, wo;
  p.dHWo.divmod(uint32_t(m), &n, &pos);
  p.dWo.divmod(pos, &ho, &wo);
  const int ih0 = int(ho) * a.Sh - a.Ph, iw0 = int(wo) * a.Sw - a.Pw;
  const int at0 = (int(n) - n_first) * CHW + ih0 * a.W + iw0;
  const int zero_at = int(p.lds_w - 16) / ESZ;
  const T* const cells = reinterpret_cast<const T*>(lds);
  const uint8_t* const wrow = lds + p.lds_w + (lane & 31) * p.wpb + (lane >> 5) * 16;

  typename TR::accv_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0;
  lds_barrier();
  for (int st = wave; st < p.ppr / 2; st += NW) {          // uniform
    const i32x4 wf = *reinterpret_cast<const i32x4*>(wrow + st * 32);
    const uint32_t* const te = tab + st * (2 * G) + (lane >> 5) * G;
    uint32_t e[G];
#pragma unroll
    for (int q = 0; q < G / 4; ++q) {
      const i32x4 t4 = *reinterpret_cast<const i32x4*>(te + 4 * q);
#pragma unroll
      for (int i = 0; i < 4; ++i) e[4 * q + i] = uint32_t(t4[i]);
    }
    uint32_t x[G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const bool in = uint32_t(ih0 + int((e[i] >> 16) & 255u)) < uint32_t(a.H) && uint32_t(iw0 + int(e[i] >> 24)) < uint32_t(a.W);
      x[i] = cells[in ? at0 + int(e[i] & 0xffffu) : zero_at];
    }
    i32x4 yf;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      if constexpr (ESZ == 2) yf[d] = int32_t(x[2 * d] | x[2 * d + 1] << 16);
      else yf[d] = int32_t(x[4 * d] | x[4 * d + 1] << 8 | x[4 * d + 2] << 16 | x[4 * d + 3] << 24);
    }
    acc = TR::mfma(wf, yf, acc);
  }
  typedef acc_t acc4_t __attribute__((ext_vector_type(4)));
  uint8_t* const part = lds + p.lds_part;
#pragma unroll
  for (int v = 0; v < 16; ++v)
    *reinterpret_cast<acc_t*>(part + wave * (32 * kImagesRS) + (8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * kImagesRS + (lane & 31) * 4) = acc[v];
  lds_barrier();
  const int row = tid >> 3, o = o0 + row;                  // four neighbouring positions of a channel
  acc4_t t[NW];
#pragma unroll
  for (int q = 0; q < NW; ++q) t[q] = *reinterpret_cast<const acc4_t*>(part + q * (32 * kImagesRS) + row * kImagesRS + (tid & 7) * 16);
#pragma unroll
  for (int step = 1; step < NW; step *= 2)                 // pairwise: fewer roundings than a chain
#pragma unroll
    for (int q = 0; q < NW; q += 2 * step) t[q] += t[q + step];
  if (o >= a.O) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int mm = m0 + (tid & 7) * 4 + i;
    if (mm >= mend) break;
    uint32_t img_n, at;
    p.dHWo.divmod(uint32_t(mm), &img_n, &at);
    store_result<acc_t>(a.out, a.residual, a.out_dtype, (int64_t(img_n) * a.O + o) * int64_t(p.dHWo.d) + at, t[0][i], a.relu);
  }
}

template <typename TR>
static hipError_t launch_images_t(const ConvArgs& a, void* packed, hipStream_t s) {
  constexpr int ESZ = TR::kEsz;
  const int64_t HWo = int64_t(a.Ho) * a.Wo, M = a.N * HWo, CHW = int64_t(a.C) * a.H * a.W, K = int64_t(a.C) * a.Kh * a.Kw;
  if (M == 0 || a.O == 0) return hipErrorInvalidValue;
  if (CHW > 65535 || int64_t(a.C - 1) * a.H * a.W + int64_t(a.Kh - 1) * a.W + a.Kw > 65536 || a.H > kImagesExtent || a.W > kImagesExtent || a.Kh > 32 || a.Kw > 32 || a.Ph > 32 || a.Pw > 32 ||
      M >= (int64_t(1) << 30) || K * ESZ > 1024)
    return hipErrorInvalidValue;
  const int64_t touched = 32 % HWo == 0 ? 32 / HWo : 30 / HWo + 2, images = touched < a.N ? touched : a.N;
  ImagesArgs p;
  p.c = a;
  p.M = int(M);
  p.K = int(K);
  p.ppr = int(round_up(K * ESZ, 32) / 16);
  p.wpb = p.ppr * 16 + 16;
  p.lds_w = uint32_t(round_up(images * CHW * ESZ, 16) + 16);
  p.lds_tab = p.lds_w + 32 * uint32_t(p.wpb);
  p.lds_part = p.lds_tab + uint32_t(p.ppr) * (16 / ESZ) * 4;
  const int64_t lds_bytes = int64_t(p.lds_part) + (kImagesThreads / 64) * 32 * kImagesRS;
  const int64_t tiles_p = ceil_div(M, 32), tiles = tiles_p * ceil_div(a.O, 32);
  // Every tile copies its images again: one round of tiles, where two workgroups share a compute unit or one has it.
  if (images * CHW * ESZ > kImagesLds || lds_bytes > kImagesLds || tiles > (lds_bytes <= 80 * 1024 ? 512 : 256)) return hipErrorInvalidValue;
  p.tiles = unsigned(tiles);
  p.dHWo = FastDiv::make(uint32_t(HWo));
  p.dWo = FastDiv::make(uint32_t(a.Wo));
  p.dT = FastDiv::make(uint32_t(a.Kh * a.Kw));
  p.dKw = FastDiv::make(uint32_t(a.Kw));
  p.dtp = FastDiv::make(uint32_t(tiles_p));
  p.dppr = FastDiv::make(uint32_t(p.ppr));
  int64_t grid = tiles;
  if (packed) {
    int64_t elements;
    p.copies = smallc_copies(packed, a.wblk != nullptr, a.in_dtype, a.O, a.C, a.Kh, a.Kw, &elements);
    if (elements >= (int64_t(1) << 30)) return hipErrorInvalidValue;   // (32-bit indices)
    const int64_t wanted = ceil_div(elements * ESZ / 16, kImagesThreads);
    grid += wanted < 512 ? wanted : 512;
  }
  const auto kern = packed ? conv_images_kernel<TR, true> : conv_images_kernel<TR, false>;
  static std::once_flag once[2];
  static hipError_t attr_status[2];        // (hipSuccess is zero)
  std::call_once(once[packed != nullptr], [&]() {
    attr_status[packed != nullptr] = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kImagesLds);
  });
  if (attr_status[packed != nullptr] != hipSuccess) return attr_status[packed != nullptr];
  hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(kImagesThreads), size_t(lds_bytes), s, p);
  return hipGetLastError();
}

hipError_t launch_conv_images(const ConvArgs& a, void* packed, hipStream_t s) {
  return a.in_dtype == GS_I8 ? launch_images_t<I8Traits>(a, packed, s) : launch_images_t<Bf16Traits>(a, packed, s);
}

}  // namespace gs
