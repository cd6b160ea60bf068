// Depth-wise windows: every channel convolved with its own single-channel filter.
//
// In the paper's operators (Table 1, Table 2) this is the concat, along the channel dimension, of
// the 2D-convolution program of Fig. 2a applied to channel c of the activations and filter c of
// the weights (slice ... 1 c c+1 / slice ... 0 c c+1): C independent one-channel convolutions.
// No contraction over channels is left: 2*Kh*Kw operations per 2-byte input element.  The kernels are built
// like the pooling kernel: every input byte leaves HBM once, however much the windows overlap.
// depthwise_kernel multiplies and adds in scalar registers, depthwise_tile_kernel makes a contraction over
// columns of it, with a banded matrix of the taps.
//
// A task is a contiguous run of the input: G whole planes (small images) or a band of rows of one
// plane (large images).  Its workgroup copies the run into LDS with aligned 16-byte reads -- a plain
// linear copy that does not care how long a row is or where a plane starts -- and every thread
// then produces strips of 8 neighbouring outputs of one output row from LDS.  Cells outside the
// image are never read as data: rows outside are skipped, columns outside are replaced by zero in
// the (few) strips that touch the left or right border.  The 16-byte loads of the next task are in
// flight while the current one is computed.
#include "common.h"

#include <string.h>

namespace gs {

namespace {

constexpr int kVX = 8;             // outputs per strip
constexpr int kMaxVec = 8;         // 16-byte loads per thread and task
constexpr int kDwTileLds = 40 * 1024;   // of a workgroup of depthwise_tile_kernel
constexpr int kGuard = 64;         // bytes of LDS in front of the copy (reads of columns < 0 land here)

struct DwArgs {
  const void* in;
  const void* w;
  void* out;
  int out_dtype, relu;
  int C, H, W, Ho, Wo, Kh, Kw, Sh, Sw, Ph, Pw;
  int G;            // planes per task (1 when a plane is cut into bands)
  int HB, bands;    // output rows per band, bands per plane
  int XS;           // strips per output row
  int KKP;          // filter taps padded to a multiple of 4
  int64_t planes, groups, tasks, total;   // N*C, ceil(planes / G), groups * bands, elements of the input
  int vec_in, vec_out, pair_out;
  uint32_t lds_w;   // byte offset of the filters in LDS
  FastDiv dXS, dHo, dKK;
  int step_r, step_xs;   // 256 items further: step_r rows of strips and step_xs strips
};

template <typename T> struct DwElem;
template <> struct DwElem<uint16_t> {
  using acc = float;
  __device__ static inline float cvt(uint16_t v) { return bf16_bits_to_float(v); }
};
template <> struct DwElem<int8_t> {
  using acc = int32_t;
  __device__ static inline int32_t cvt(int8_t v) { return v; }
};

struct DwTask {
  int64_t plane0;
  int gcount, ho0, nho, R;   // planes, first output row, output rows, rows of strips
  int ih1;           // end of the input rows copied
  int64_t ebase;     // first element (16-byte aligned) of the copy
  int nvec;          // 16-byte vectors in the copy
  int shift;         // LDS element index of (g, ih, iw) is (g*H + ih)*W + iw - shift
};

template <int VY>
__device__ __forceinline__ DwTask dw_task(const DwArgs& a, int64_t task, int epv) {
  DwTask t;
  const int64_t grp = task / a.bands;
  const int band = int(task - grp * a.bands);
  t.plane0 = grp * a.G;
  const int64_t left = a.planes - t.plane0;
  t.gcount = left < a.G ? int(left) : a.G;
  t.ho0 = band * a.HB;
  t.nho = a.Ho - t.ho0 < a.HB ? a.Ho - t.ho0 : a.HB;
  t.R = t.gcount * ((t.nho + VY - 1) / VY);
  int ih0 = t.ho0 * a.Sh - a.Ph;
  ih0 = ih0 < 0 ? 0 : ih0;
  int ih1 = (t.ho0 + t.nho - 1) * a.Sh - a.Ph + a.Kh;
  ih1 = ih1 > a.H ? a.H : ih1;
  ih1 = ih1 < ih0 ? ih0 : ih1;
  t.ih1 = ih1;
  const int64_t e0 = (t.plane0 * a.H + ih0) * a.W;
  const int64_t e1 = ((t.plane0 + t.gcount - 1) * a.H + ih1) * a.W;
  t.ebase = e0 / epv * epv;
  t.nvec = int((e1 + epv - 1) / epv - e0 / epv);
  t.shift = int(t.ebase - t.plane0 * a.H * a.W);
  return t;
}

// Streaming where neighbouring lines are written together; strips of several rows leave a line's halves to
// different instructions, which the cache joins.
template <int VY, typename V>
__device__ __forceinline__ void dw_store(V v, V* p) {
  if constexpr (VY > 1) *p = v;
  else __builtin_nontemporal_store(v, p);
}

// KH, KW, SW > 0: window and horizontal stride fixed at compile time; 0: run-time loops.
// VY > 1 (vertical stride 1): a thread produces strips of VY output rows, one below the other, from
// VY + KH - 1 input rows, each read, converted and cut at the border once.  The kernel is bound by the
// instructions it issues, and with one row per strip two thirds of a 3x3 window's conversions repeat
// what the rows above and below do.
// EDGE: stride 1, "same" padding, rows of a multiple of eight: a strip's own eight columns are one
// aligned vector of LDS and always inside the image, only its KW - 1 neighbours can be outside.
template <typename T, int KH, int KW, int SW, int VY, bool EDGE>
__global__ void __launch_bounds__(256, VY > 1 ? 3 : 1)
depthwise_kernel(DwArgs a) {
  using A = typename DwElem<T>::acc;
  constexpr int ESZ = int(sizeof(T));
  constexpr int EPV = 16 / ESZ;
  constexpr bool FIXED = KH > 0;
  typedef T vec_t __attribute__((ext_vector_type(EPV)));
  extern __shared__ __attribute__((aligned(16))) uint8_t dw_lds[];
  T* const stage = reinterpret_cast<T*>(dw_lds + kGuard);
  A* const wl = reinterpret_cast<A*>(dw_lds + a.lds_w);
  const T* const in = static_cast<const T*>(a.in);
  const int tid = threadIdx.x;
  const int kh = FIXED ? KH : a.Kh, kw = FIXED ? KW : a.Kw, sw = FIXED ? SW : a.Sw;
  const int kk = kh * kw;

  vec_t val[kMaxVec];
  auto issue_loads = [&](const DwTask& t) {
#pragma unroll
    for (int u = 0; u < kMaxVec; ++u) {
      const int v = u * 256 + tid;
      const int64_t e = t.ebase + int64_t(v) * EPV;
#pragma unroll
      for (int i = 0; i < EPV; ++i) val[u][i] = 0;
      if (v < t.nvec) {
        if (a.vec_in && e + EPV <= a.total) {
          val[u] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(in + e));   // read once
        } else {
#pragma unroll
          for (int i = 0; i < EPV; ++i)
            if (e + i < a.total) val[u][i] = in[e + i];
        }
      }
    }
  };

  int64_t task = blockIdx.x;
  if (task >= a.tasks) return;
  DwTask cur = dw_task<VY>(a, task, EPV);
  issue_loads(cur);
  for (; task < a.tasks; task += gridDim.x) {
    __syncthreads();                                   // the previous task has been computed
#pragma unroll
    for (int u = 0; u < kMaxVec; ++u) {
      const int v = u * 256 + tid;
      if (v < cur.nvec) *reinterpret_cast<vec_t*>(stage + v * EPV) = val[u];
    }
    for (int id = tid; id < cur.gcount * kk; id += 256) {   // the filters of this task's planes
      uint32_t g, i;
      a.dKK.divmod(uint32_t(id), &g, &i);
      const int c = int((cur.plane0 + g) % a.C);
      wl[int(g) * a.KKP + int(i)] = DwElem<T>::cvt(static_cast<const T*>(a.w)[int64_t(c) * kk + int(i)]);
    }
    __syncthreads();
    const DwTask t = cur;
    if (task + gridDim.x < a.tasks) {
      cur = dw_task<VY>(a, task + gridDim.x, EPV);
      issue_loads(cur);
    }

    // Strips are numbered along the rows: neighbouring lanes read neighbouring 16 bytes of LDS
    // and write neighbouring 16 bytes of the result.
    const int items = a.XS * t.R;
    // (row of strips, strip) of this thread's item: divided once, then stepped by 256 items.
    uint32_t r, xs;
    a.dXS.divmod(uint32_t(tid), &r, &xs);
    const int64_t obase = t.plane0 * a.Ho * a.Wo;       // results of the task's first plane
    for (int id = tid; id < items; id += 256, r += a.step_r, xs += a.step_xs) {
      if (int(xs) >= a.XS) {
        xs -= a.XS;
        ++r;
      }
      uint32_t g = 0, yl = r;
      if (a.G > 1) a.dHo.divmod(r, &g, &yl);           // G > 1: whole planes
      const int y = t.ho0 + int(yl) * VY;
      const int x0 = int(xs) * kVX;
      const int iw0 = x0 * sw - a.Pw;                   // column of the first element of the span
      const A* wg = wl + __mul24(int(g), a.KKP);
      A accs[VY][kVX];
#pragma unroll
      for (int vy = 0; vy < VY; ++vy)
#pragma unroll
        for (int v = 0; v < kVX; ++v) accs[vy][v] = 0;
      if constexpr (FIXED) {
        constexpr int SPAN = (kVX - 1) * SW + KW;
        constexpr int KKP = (KH * KW + 3) / 4 * 4;
        A wr[KKP];
#pragma unroll
        for (int q = 0; q < KKP / 4; ++q) {
          typedef A a4 __attribute__((ext_vector_type(4)));
          const a4 w4 = *reinterpret_cast<const a4*>(wg + 4 * q);
#pragma unroll
          for (int i = 0; i < 4; ++i) wr[4 * q + i] = w4[i];
        }
        // All LDS reads of the strip first (rows outside the image read nothing and count as
        // zeros), then straight-line arithmetic: the reads of the KH rows overlap.
        const int ih_first = __mul24(y, a.Sh) - a.Ph;
        // 24-bit multiplies: LDS indices are far below 2^23
        const T* row0 = stage + (__mul24(__mul24(int(g), a.H) + ih_first, a.W) + iw0 - t.shift);
        constexpr int RIN = VY - 1 + KH;                // input rows of the strip
        T raw[RIN][SPAN];
#pragma unroll
        for (int ky = 0; ky < RIN; ++ky) {
#pragma unroll
          for (int j = 0; j < SPAN; ++j) raw[ky][j] = 0;
          // rows past the copy belong to output rows past the task's, which are not written
          if (ih_first + ky >= 0 && ih_first + ky < t.ih1) {
            const T* row = row0 + ky * a.W;
            if constexpr (EDGE) {
              typedef T own_t __attribute__((ext_vector_type(kVX)));
              constexpr int P = KW / 2;
              const own_t own = *reinterpret_cast<const own_t*>(row + P);
#pragma unroll
              for (int j = 0; j < P; ++j) {
                raw[ky][j] = row[j];
                raw[ky][P + kVX + j] = row[P + kVX + j];
              }
#pragma unroll
              for (int j = 0; j < kVX; ++j) raw[ky][P + j] = own[j];
            } else {
#pragma unroll
              for (int j = 0; j < SPAN; ++j) raw[ky][j] = row[j];
            }
          }
        }
        // Element j of a span sits in column iw0 + j: columns left of the image (only the first
        // KW - 1 elements can be) and right of it hold a neighbouring row's data and count as zero.
        const int lo_bad = -iw0, hi_ok = a.W - iw0;
#pragma unroll
        for (int r_in = 0; r_in < RIN; ++r_in) {
          A e[SPAN];
#pragma unroll
          for (int j = 0; j < SPAN; ++j) {
            e[j] = DwElem<T>::cvt(raw[r_in][j]);
            if (EDGE ? j < KW / 2 : j < KW - 1) e[j] = j >= lo_bad ? e[j] : A(0);
            if (!EDGE || j >= KW / 2 + kVX) e[j] = j < hi_ok ? e[j] : A(0);
          }
#pragma unroll
          for (int vy = 0; vy < VY; ++vy) {
            const int ky = r_in - vy;
            if (ky < 0 || ky >= KH) continue;
#pragma unroll
            for (int v = 0; v < kVX; ++v)
#pragma unroll
              for (int kx = 0; kx < KW; ++kx) accs[vy][v] += e[v * SW + kx] * wr[ky * KW + kx];
          }
        }
      } else {
        for (int ky = 0; ky < kh; ++ky) {
          const int ih = y * a.Sh - a.Ph + ky;
          if (ih < 0 || ih >= a.H) continue;
          const T* row = stage + ((int(g) * a.H + ih) * a.W - t.shift);
          for (int kx = 0; kx < kw; ++kx) {
            const A wv = wg[ky * kw + kx];
#pragma unroll
            for (int v = 0; v < kVX; ++v) {
              const int iw = iw0 + v * sw + kx;
              if (iw >= 0 && iw < a.W && x0 + v < a.Wo) accs[0][v] += DwElem<T>::cvt(row[iw]) * wv;
            }
          }
        }
      }
#pragma unroll
      for (int vy = 0; vy < VY; ++vy) {
        if (vy > 0 && y + vy >= t.ho0 + t.nho) break;
        A* const acc = accs[vy];
        if (a.relu) {
#pragma unroll
          for (int v = 0; v < kVX; ++v) acc[v] = acc[v] > A(0) ? acc[v] : A(0);
        }
        // within a task the results are fewer than 2^23 rows of fewer than 2^23 values
        const int64_t o = obase + (int64_t(__mul24(__mul24(int(g), a.Ho) + y + vy, a.Wo)) + x0);
        if (a.vec_out && x0 + kVX <= a.Wo) {
          if (a.out_dtype == GS_BF16) {
            if constexpr (__is_same(A, float)) {
              typedef uint32_t u4 __attribute__((ext_vector_type(4)));
              u4 p;
#pragma unroll
              for (int q = 0; q < 4; ++q) p[q] = pack_bf16x2(acc[2 * q], acc[2 * q + 1]);
              dw_store<VY>(p, reinterpret_cast<u4*>(static_cast<uint16_t*>(a.out) + o));
            }
          } else {                                        // 32-bit results: two 16-byte stores
            typedef A a4 __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              const a4 p = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
              dw_store<VY>(p, reinterpret_cast<a4*>(static_cast<A*>(a.out) + o) + q);
            }
          }
        } else if (__is_same(A, float) && a.out_dtype == GS_BF16 && a.pair_out) {
          // rows of an even number of results: pairs never straddle the end of a row
          if constexpr (__is_same(A, float)) {
#pragma unroll
            for (int q = 0; q < kVX / 2; ++q)
              if (x0 + 2 * q < a.Wo)
                reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(a.out) + o)[q] = pack_bf16x2(acc[2 * q], acc[2 * q + 1]);
          }
        } else {
#pragma unroll
          for (int v = 0; v < kVX; ++v) {
            if (x0 + v < a.Wo) {
              if constexpr (__is_same(A, float)) {
                if (a.out_dtype == GS_BF16) static_cast<uint16_t*>(a.out)[o + v] = float_to_bf16_bits(acc[v]);
                else static_cast<float*>(a.out)[o + v] = acc[v];
              } else {
                static_cast<int32_t*>(a.out)[o + v] = acc[v];
              }
            }
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Unit strides on the matrix units.  A tile is 16 x 16 results of one plane: for every filter row, a banded matrix of
// the filter's taps (16 result columns x the 64 bytes of input columns around them) times the input rows in LDS
// (those columns x 16 result rows), as one 16x16 MFMA.  Both operands are 16 bytes per lane: the input as it lies in a
// padded row of LDS, the band from a row of zeros with the taps in its middle, read once per plane.  With columns on
// the MFMA rows a lane holds four neighbouring results of a row.
//
// A band's zeros meet input values too, so an infinity or NaN in the 64 bytes reaches results that it is no
// part of, as NaN.  A tile with a result that is not finite is worked out again with zeros in the place of such values, and
// tap by tap where a window holds one: a result never depends on what its window does not hold.
//
// What bounds it: a wave waits for its stores before it writes the next plane into LDS (loads and stores share a
// counter), and each pair of tiles is a chain of LDS reads, products and stores.  It needs 106 to 123 registers, of 128 for four
// workgroups on a compute unit; with the places of the pieces in two registers each it spilled 8 to 26 and kept that
// counter busy with scratch (5x5 to f32, 351 planes of 89x45 in 7 images, 23.6 -> 21.9).  The kernels of scalar
// multiply-adds are bound by their instructions, 300 per eight results against some 60 per 512 here.  Errors
// of f32 results against 64 bits are 0.90 to 0.95 of theirs.  See launch_depthwise_t for times.
// ---------------------------------------------------------------------------------------------
struct DwTileArgs {
  const void* in;
  const void* w;
  void* out;
  int relu, C, H, W, Ho, Wo, P;       // P: padding on every side
  int G;                              // planes per task
  int cpr;                            // 16-byte pieces of a row
  int pitch, plane_lds, lds_w;        // LDS: bytes of a row, of a plane; where the taps are
  int64_t planes, tasks;
  int dx, dy, second;                 // from a pair's first tile to its second: columns, rows, bytes of LDS
  FastDiv dcpr, dH, dT, dTX;          // pieces per row, rows, pairs of tiles per plane and in a row of them
  int pieces;                         // of a plane
};

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// K: window; OUT: GS_BF16, GS_F32 or GS_I32.
template <typename T, int K, int OUT>
__global__ void __launch_bounds__(256, 4) depthwise_tile_kernel(DwTileArgs a) {
  constexpr int ESZ = int(sizeof(T)), E = 16 / ESZ;     // elements of a piece; zeros in front of a row too
  constexpr bool INT = __is_same(T, int8_t);
  using A = typename DwElem<T>::acc;
  typedef A acc4_t __attribute__((ext_vector_type(4)));
  constexpr int kBand = 96 * ESZ;                       // a row of taps: zeros around them on both sides
  extern __shared__ __attribute__((aligned(16))) uint8_t dw_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const T* const in = static_cast<const T*>(a.in);
  const int64_t plane_in = int64_t(a.H) * a.W;

  // Pieces of a task: row by row, the last of a row moved down to its start (zeros behind the row's end).
  // Where they come from and go to is the same for every task, 16 bits each (a task's pieces are 32 KB): bytes from its first
  // plane's start; above them the LDS offset, and in its low bit whether the row ends there.
  i32x4 val[kMaxVec];
  uint32_t way[kMaxVec];
  static_assert(kMaxVec * 256 * 16 <= 0x10000 && kDwTileLds <= 0x10000, "16 bits");
  auto way_of = [&](int u) {              // (taken apart where it is used: two registers per piece are not kept)
    uint32_t v = way[u];
    asm volatile("" : "+v"(v));
    return v;
  };
#pragma unroll
  for (int u = 0; u < kMaxVec; ++u) {
    uint32_t row, c, g, y;                              // (planes lie one behind the other)
    a.dcpr.divmod(uint32_t(u * 256 + tid), &row, &c);
    a.dH.divmod(row, &g, &y);
    const int col = int(c) * E < a.W - E ? int(c) * E : a.W - E;
    const uint32_t dst = (g * uint32_t(a.plane_lds) + (y + uint32_t(a.P)) * uint32_t(a.pitch) + (c + 1) * 16) | (int(c) + 1 == a.cpr ? 1u : 0u);
    way[u] = (((row * uint32_t(a.W) + uint32_t(col)) * ESZ) & 0xffffu) | dst << 16;
  }
  const int over = (a.cpr * E - a.W) * ESZ;             // bytes by which a row's last piece is moved down
  auto gcount_of = [&](int64_t task) { return int(a.planes - task * a.G < a.G ? a.planes - task * a.G : a.G); };
  auto issue_loads = [&](int64_t task) {
    const int n = gcount_of(task) * a.pieces;
    const uint8_t* const base = reinterpret_cast<const uint8_t*>(in + task * a.G * plane_in);
#pragma unroll
    for (int u = 0; u < kMaxVec; ++u)
      if (u * 256 + tid < n) val[u] = __builtin_nontemporal_load(reinterpret_cast<const i32x4_any*>(base + (way_of(u) & 0xffffu)));
  };
  int64_t task = blockIdx.x;
  if (task >= a.tasks) return;
  issue_loads(task);
  // Cells around the planes stay zero for good.
  for (int off = tid * 16; off < a.lds_w + a.G * K * kBand; off += 256 * 16) *reinterpret_cast<i32x4*>(dw_lds + off) = i32x4{0, 0, 0, 0};

  const int n16 = lane & 15, grp = lane >> 4;
  for (; task < a.tasks; task += gridDim.x) {
    const int gcount = gcount_of(task);
    __syncthreads();                                    // the previous task has been computed
#pragma unroll
    for (int u = 0; u < kMaxVec; ++u) {
      if (u * 256 + tid < gcount * a.pieces) {
        const uint32_t at = way_of(u) >> 16;
        if (over) val[u] = row_piece_fix(val[u], at & 1 ? over : 0);      // uniform
        *reinterpret_cast<i32x4*>(dw_lds + (at & ~1u)) = val[u];
      }
    }
    for (int id = tid; id < gcount * K * K; id += 256) {
      const int g = id / (K * K), i = id - g * (K * K), c = int((task * a.G + g) % a.C);
      reinterpret_cast<T*>(dw_lds + a.lds_w + (g * K + i / K) * kBand)[32 + i % K] =
          static_cast<const T*>(a.w)[int64_t(c) * (K * K) + i];
    }
    __syncthreads();
    const int64_t plane0 = task * a.G;
    if (task + gridDim.x < a.tasks) issue_loads(task + gridDim.x);

    // Two tiles side by side (one above the other in planes of one column of tiles) at a time; a run of them for each
    // wave.
    const int pairs = gcount * int(a.dT.d);
    int t = wave * pairs / 4;
    const int t_end = (wave + 1) * pairs / 4;
    int have = -1;
    i32x4 band[K];
    for (; t < t_end; ++t) {                            // uniform
      uint32_t g, r, ty, tx;
      a.dT.divmod(uint32_t(t), &g, &r);
      a.dTX.divmod(r, &ty, &tx);
      if (int(g) != have) {
        have = int(g);
        // band[m][k] = tap k - E - m + P: element j of this lane is k = grp E + j of row m = n16
#pragma unroll
        for (int dy = 0; dy < K; ++dy) {
          const T* const from = reinterpret_cast<const T*>(dw_lds + a.lds_w + (have * K + dy) * kBand) + 32 + grp * E - E - n16 + a.P;
          band[dy] = *reinterpret_cast<const i32x4_any*>(from);
        }
      }
      const int x0 = int(tx) * (16 + a.dx), y0 = int(ty) * (16 + a.dy);
      const uint8_t* const rows = dw_lds + have * a.plane_lds + (y0 + n16) * a.pitch + x0 * ESZ + grp * 16;
      i32x4 x[2][K];
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int dy = 0; dy < K; ++dy) x[q][dy] = *reinterpret_cast<const i32x4*>(rows + q * a.second + dy * a.pitch);
      acc4_t acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
      for (int dy = 0; dy < K; ++dy)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if constexpr (INT) acc[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(band[dy], x[q][dy], acc[q], 0, 0, 0);
          else acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, band[dy]), __builtin_bit_cast(bf16x8, x[q][dy]), acc[q], 0, 0, 0);
        }
      // This lane's results: of tile q row y0 + q dy + n16, columns x0 + q dx + 4 grp ..
      if constexpr (!INT) {
        float zero[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) zero[q] = (acc[q][0] * 0.0f + acc[q][1] * 0.0f) + (acc[q][2] * 0.0f + acc[q][3] * 0.0f);
        const float z = zero[0] + zero[1];              // NaN if any of them is not finite
        if (__any(z != z)) {
          // The products again with zeros in the place of what is not finite ..
#pragma unroll
          for (int q = 0; q < 2; ++q) acc[q] = acc4_t{0, 0, 0, 0};
#pragma unroll 1
          for (int dy = 0; dy < K; ++dy) {
            const T* const from = reinterpret_cast<const T*>(dw_lds + a.lds_w + (have * K + dy) * kBand) + 32 + grp * E - E - n16 + a.P;
            const i32x4 taps = *reinterpret_cast<const i32x4_any*>(from);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              i32x4 v = *reinterpret_cast<const i32x4*>(rows + q * a.second + dy * a.pitch);
#pragma unroll
              for (int d = 0; d < 4; ++d) {
                const uint32_t u = uint32_t(v[d]);
                const uint32_t lo = (u & 0x7f80u) == 0x7f80u ? 0 : 0xffffu, hi = (u & 0x7f800000u) == 0x7f800000u ? 0 : 0xffff0000u;
                v[d] = int32_t(u & (lo | hi));
              }
              acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, taps), __builtin_bit_cast(bf16x8, v), acc[q], 0, 0, 0);
            }
          }
          // .. and tap by tap the results whose windows hold it.
#pragma unroll 1
          for (int i = 0; i < 8; ++i) {
            const int q = i >> 2;
            const T* const cells = reinterpret_cast<const T*>(dw_lds + have * a.plane_lds + (y0 + q * a.dy + n16) * a.pitch) + E + x0 + q * a.dx + 4 * grp + (i & 3) - a.P;
            const T* const taps = reinterpret_cast<const T*>(dw_lds + a.lds_w + have * K * kBand) + 32;
            float sum = 0.0f;
            bool held = false;
#pragma unroll 1
            for (int dy = 0; dy < K; ++dy)
#pragma unroll 1
              for (int dx = 0; dx < K; ++dx) {
                const T cell = cells[dy * (a.pitch / ESZ) + dx];
                held = held || (cell & 0x7f80) == 0x7f80;
                sum += DwElem<T>::cvt(cell) * DwElem<T>::cvt(taps[dy * (kBand / ESZ) + dx]);
              }
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (e == i && held) acc[e >> 2][e & 3] = sum;
          }
        }
      }
      if (a.relu) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[q][i] = acc[q][i] > A(0) ? acc[q][i] : A(0);
      }
      const int64_t oplane = (plane0 + have) * a.Ho;
      if constexpr (OUT == GS_BF16) {
        // The tiles' halves change places between neighbouring groups of lanes: then a lane holds eight neighbouring
        // columns of one tile, lanes of even groups of the first.
        uint32_t lo[2], hi[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          lo[q] = pack_bf16x2(acc[q][0], acc[q][1]);
          hi[q] = pack_bf16x2(acc[q][2], acc[q][3]);
        }
        const auto l = __builtin_amdgcn_permlane16_swap(lo[0], lo[1], false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi[0], hi[1], false, false);
        const i32x4 v = {int32_t(l[0]), int32_t(h[0]), int32_t(l[1]), int32_t(h[1])};
        const int q = grp & 1, y = y0 + q * a.dy + n16, xs = x0 + q * a.dx + 8 * (grp >> 1);
        if (y < a.Ho && xs < a.Wo) {
          uint16_t* const dst = static_cast<uint16_t*>(a.out) + (oplane + y) * a.Wo + xs;
          if (xs + 8 <= a.Wo) {
            typedef int32_t i32x4_half __attribute__((ext_vector_type(4), aligned(2)));
            *reinterpret_cast<i32x4_half*>(dst) = v;
          } else {
#pragma unroll
            for (int i = 0; i < 7; ++i)
              if (xs + i < a.Wo) dst[i] = uint16_t(uint32_t(v[i >> 1]) >> (16 * (i & 1)));
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int y = y0 + q * a.dy + n16, xs = x0 + q * a.dx + 4 * grp;
          if (y < a.Ho && xs < a.Wo) {
            typedef int32_t i32x4_word __attribute__((ext_vector_type(4), aligned(4)));
            A* const dst = static_cast<A*>(a.out) + (oplane + y) * a.Wo + xs;
            if (xs + 4 <= a.Wo) {
              *reinterpret_cast<i32x4_word*>(dst) = __builtin_bit_cast(i32x4, acc[q]);
            } else {
#pragma unroll
              for (int i = 0; i < 3; ++i)
                if (xs + i < a.Wo) dst[i] = acc[q][i];
            }
          }
        }
      }
    }
  }
}

int dw_num_cus() {
  static int n = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      cus = 256;
    return cus;
  }();
  return n;
}

// What the EDGE kernels take.
bool dw_edge(const DepthwiseArgs& d) {
  return d.Sw == 1 && d.W % kVX == 0 && d.Wo == d.W && d.Pw == d.Kw / 2;
}

template <typename T, int VY>
hipError_t launch_depthwise_rows(const DepthwiseArgs& d, hipStream_t s) {
  constexpr int ESZ = int(sizeof(T));
  constexpr int EPV = 16 / ESZ;
  constexpr int kResident = VY > 1 ? 3 : 4;   // workgroups per compute unit that the registers allow
  using A = typename DwElem<T>::acc;
  DwArgs a;
  memset(&a, 0, sizeof(a));
  a.in = d.in; a.w = d.w; a.out = d.out; a.out_dtype = d.out_dtype; a.relu = d.relu;
  a.C = d.C; a.H = d.H; a.W = d.W; a.Ho = d.Ho; a.Wo = d.Wo; a.Kh = d.Kh; a.Kw = d.Kw;
  a.Sh = d.Sh; a.Sw = d.Sw; a.Ph = d.Ph; a.Pw = d.Pw;
  a.planes = int64_t(d.N) * d.C;
  a.total = a.planes * d.H * d.W;
  if (a.planes == 0 || d.Ho <= 0 || d.Wo <= 0) return hipSuccess;
  if (a.total >= (int64_t(1) << 40)) return hipErrorInvalidValue;
  // positions inside a plane (of the input and of the result) are 32-bit in the kernel
  if ((int64_t(d.H) + 64) * (int64_t(d.W) + 64) >= (int64_t(1) << 31)) return hipErrorInvalidValue;
  // The copy of a task: at most kMaxVec * 256 vectors, two of them spent on the ragged ends.
  const int64_t cap = int64_t(kMaxVec * 256 - 2) * EPV;           // elements
  const int64_t plane = int64_t(d.H) * d.W;
  if (plane <= cap) {
    // Planes per task: the strips of a task are worked off 256 at a time, and the chip holds
    // `slots` tasks at once; take the G with the fewest (rounds + one round of fixed cost) x passes.
    int gmax = int(cap / plane);
    gmax = gmax > 64 ? 64 : gmax;
    const int64_t slots = int64_t(dw_num_cus()) * kResident;
    const int64_t strips = ceil_div(d.Wo, kVX) * ceil_div(d.Ho, VY);
    int64_t best = -1;
    a.G = 1;
    for (int g = 1; g <= gmax; ++g) {
      const int64_t cost = ceil_div(ceil_div(a.planes, g), slots) * (ceil_div(strips * g, 256) + 1);
      if (best < 0 || cost <= best) {
        best = cost;
        a.G = g;
      }
    }
    a.HB = d.Ho;
    a.bands = 1;
  } else {
    a.G = 1;
    const int64_t rows = cap / d.W;                                 // input rows that fit
    if (rows < d.Kh) return hipErrorInvalidValue;
    int64_t hb = (rows - d.Kh) / d.Sh + 1;
    hb = hb > d.Ho ? d.Ho : hb;
    a.bands = int(ceil_div(d.Ho, hb));
    a.HB = int(ceil_div(d.Ho, a.bands));
  }
  a.groups = ceil_div(a.planes, a.G);
  a.tasks = a.groups * a.bands;
  a.XS = int(ceil_div(d.Wo, kVX));
  a.KKP = int(round_up(int64_t(d.Kh) * d.Kw, 4));
  a.dXS = FastDiv::make(uint32_t(a.XS));
  a.step_r = 256 / a.XS;
  a.step_xs = 256 % a.XS;
  a.dHo = FastDiv::make(uint32_t(ceil_div(d.Ho, VY)));
  a.dKK = FastDiv::make(uint32_t(d.Kh * d.Kw));
  a.vec_in = reinterpret_cast<uintptr_t>(d.in) % 16 == 0;
  a.vec_out = d.Wo % kVX == 0 && reinterpret_cast<uintptr_t>(d.out) % 16 == 0;
  a.pair_out = d.Wo % 2 == 0 && reinterpret_cast<uintptr_t>(d.out) % 4 == 0;
  // LDS: guard, the copy, room for the last strip's reads past the end of a row, the filters.
  const int64_t span_max = int64_t(kVX) * d.Sw + d.Kw;
  const int64_t copy_bytes = int64_t(kMaxVec) * 256 * 16;
  a.lds_w = uint32_t(round_up(kGuard + copy_bytes + span_max * ESZ, 16));
  const size_t lds = a.lds_w + size_t(a.G) * a.KKP * sizeof(A);
  if (d.Pw * ESZ > kGuard || lds > 64 * 1024) return hipErrorInvalidValue;
  int per_cu = int((160 * 1024) / (lds + 512));
  per_cu = per_cu < 1 ? 1 : per_cu > kResident ? kResident : per_cu;
  int64_t grid = int64_t(dw_num_cus()) * per_cu;
  if (grid > a.tasks) grid = a.tasks;
  grid = ceil_div(a.tasks, ceil_div(a.tasks, grid));     // the same number of tasks for everyone
  const dim3 g{unsigned(grid)}, b{256};
  if constexpr (VY == 4) {
    hipLaunchKernelGGL((depthwise_kernel<T, 3, 3, 1, 4, true>), g, b, lds, s, a);
  } else if constexpr (VY == 2) {
    if (dw_edge(d)) hipLaunchKernelGGL((depthwise_kernel<T, 5, 5, 1, 2, true>), g, b, lds, s, a);
    else hipLaunchKernelGGL((depthwise_kernel<T, 5, 5, 1, 2, false>), g, b, lds, s, a);
  } else if (d.Kh == 3 && d.Kw == 3 && d.Sw == 1) {
    hipLaunchKernelGGL((depthwise_kernel<T, 3, 3, 1, 1, false>), g, b, lds, s, a);
  } else if (d.Kh == 3 && d.Kw == 3 && d.Sw == 2) {
    hipLaunchKernelGGL((depthwise_kernel<T, 3, 3, 2, 1, false>), g, b, lds, s, a);
  } else if (d.Kh == 5 && d.Kw == 5 && d.Sw == 1) {
    hipLaunchKernelGGL((depthwise_kernel<T, 5, 5, 1, 1, false>), g, b, lds, s, a);
  } else if (d.Kh == 5 && d.Kw == 5 && d.Sw == 2) {    // (31 x 372 planes of 21x22 int8 34.0 us in the kernel of any window, 11.7)
    hipLaunchKernelGGL((depthwise_kernel<T, 5, 5, 2, 1, false>), g, b, lds, s, a);
  } else {
    hipLaunchKernelGGL((depthwise_kernel<T, 0, 0, 0, 1, false>), g, b, lds, s, a);
  }
  return hipGetLastError();
}

// hipErrorInvalidValue where the kernel does not take the call.
template <typename T>
hipError_t launch_depthwise_tiles(const DepthwiseArgs& d, hipStream_t s) {
  constexpr int ESZ = int(sizeof(T)), E = 16 / ESZ;
  const int K = d.Kh;
  if (d.Sh != 1 || d.Sw != 1 || K != d.Kw || (K != 3 && K != 5) || d.Ph != d.Pw || d.Ph > K / 2 || d.W < E) return hipErrorInvalidValue;
  DwTileArgs a;
  memset(&a, 0, sizeof(a));
  a.in = d.in; a.w = d.w; a.out = d.out; a.relu = d.relu;
  a.C = d.C; a.H = d.H; a.W = d.W; a.Ho = d.Ho; a.Wo = d.Wo; a.P = d.Ph;
  a.planes = int64_t(d.N) * d.C;
  if (a.planes == 0 || d.Ho <= 0 || d.Wo <= 0) return hipSuccess;
  if (a.planes * d.H * d.W >= (int64_t(1) << 40) || int64_t(d.H) * d.W >= (1 << 20)) return hipErrorInvalidValue;
  a.cpr = int(ceil_div(d.W, E));
  a.pieces = d.H * a.cpr;
  const bool beside = d.Wo > 16;                         // pairs of tiles
  const int TX = int(ceil_div(d.Wo, beside ? 32 : 16)), TY = int(ceil_div(d.Ho, beside ? 16 : 32));
  a.dx = beside ? 16 : 0;
  a.dy = 16 - a.dx;
  // A tile reads the 64 bytes from a piece in front of its first column on, in 16 + K - 1 rows; a row holds the pieces
  // of the data behind one of zeros.  An odd number of pieces: the 16 rows of a read on 16 bank groups.
  int64_t pitch = 16 * (1 + a.cpr);
  const int64_t reach = (int64_t(TX) * (16 + a.dx) - 16) * ESZ + 64;
  if (pitch < reach) pitch = reach;
  if (pitch / 16 % 2 == 0) pitch += 16;
  int64_t rows = int64_t(TY) * (16 + a.dy) + K - 1;
  if (rows < d.H + 2 * d.Ph) rows = d.H + 2 * d.Ph;
  a.pitch = int(pitch);
  a.plane_lds = int(rows * pitch);
  a.second = beside ? 16 * ESZ : 16 * a.pitch;
  const int taps = K * 96 * ESZ;
  if (a.pieces > kMaxVec * 256 || a.plane_lds + taps > kDwTileLds) return hipErrorInvalidValue;
  // As many planes as a task's loads and a quarter of the LDS hold, but four tasks for every compute unit.
  int64_t G = kMaxVec * 256 / a.pieces, fit = kDwTileLds / (a.plane_lds + taps), fill = a.planes / (4 * dw_num_cus());
  G = G < fit ? G : fit;
  G = G < fill ? G : fill;
  a.G = int(G < 1 ? 1 : G);
  a.tasks = ceil_div(a.planes, a.G);
  a.lds_w = a.G * a.plane_lds;
  a.dcpr = FastDiv::make(uint32_t(a.cpr));
  a.dH = FastDiv::make(uint32_t(d.H));
  a.dT = FastDiv::make(uint32_t(TX * TY));
  a.dTX = FastDiv::make(uint32_t(TX));
  const size_t lds = size_t(a.lds_w) + size_t(a.G) * taps;
  int64_t grid = int64_t(dw_num_cus()) * 4;
  if (grid > a.tasks) grid = a.tasks;
  grid = ceil_div(a.tasks, ceil_div(a.tasks, grid));     // the same number of tasks for everyone
  const dim3 g{unsigned(grid)}, b{256};
  if constexpr (__is_same(T, int8_t)) {
    if (K == 3) hipLaunchKernelGGL((depthwise_tile_kernel<T, 3, GS_I32>), g, b, lds, s, a);
    else hipLaunchKernelGGL((depthwise_tile_kernel<T, 5, GS_I32>), g, b, lds, s, a);
  } else if (d.out_dtype == GS_BF16) {
    if (K == 3) hipLaunchKernelGGL((depthwise_tile_kernel<T, 3, GS_BF16>), g, b, lds, s, a);
    else hipLaunchKernelGGL((depthwise_tile_kernel<T, 5, GS_BF16>), g, b, lds, s, a);
  } else {
    if (K == 3) hipLaunchKernelGGL((depthwise_tile_kernel<T, 3, GS_F32>), g, b, lds, s, a);
    else hipLaunchKernelGGL((depthwise_tile_kernel<T, 5, GS_F32>), g, b, lds, s, a);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_depthwise_t(const DepthwiseArgs& d, hipStream_t s) {
  // Unit strides on the matrix units where the 16x32 or 32x16 results of a step are mostly results, there are enough of them, and,
  // for 3x3, columns are unaligned (us, strips / tiles):
  //   5x5: 32 images of 128 planes of 112x112 101 / 63, 11 of 330 51x101 64 / 36, 3 of 314 100x17 14.4 / 8.9, 10 of 65 49x19 to
  //   f32 9.4 / 6.9; but 18 of 361 planes of 8x49 14.2 / 16.2, 16 of 511 27x20 to bfloat16 18.4 / 19.7;
  //   3x3: 17 of 313 80x99 85 / 61, 14 of 276 28x68 int8 25 / 16, 32 of 256 28x28 16.5 / 13.9; but 32 of 128 112x112 (aligned) 52.3 /
  //   57.3 (to f32 72 / 82), 32 of 512 14x14 9.7 / 16.0, 2 of 361 51x19 to f32 6.3 / 6.3.
  const int64_t step = d.Wo > 16 ? round_up(d.Wo, 32) * round_up(d.Ho, 16) : round_up(d.Wo, 16) * round_up(d.Ho, 32);
  const int64_t plane = int64_t(d.Ho) * d.Wo, results = int64_t(d.N) * d.C * plane;
  if (d.Kh == 5 ? plane * 100 >= step * (d.out_dtype == GS_BF16 ? 54 : 45) && results >= (__is_same(T, int8_t) ? 2000000 : 300000) : plane * 100 >= step * 70 && results >= 900000 && !dw_edge(d)) {
    const hipError_t e = launch_depthwise_tiles<T>(d, s);
    if (e != hipErrorInvalidValue) return e;
  }
  // Several rows per strip (four for 3x3; two for 5x5, whose twenty-five filter taps leave registers for no
  // more) where every compute unit still has 256 strips, few of the rows are past the end, and it was the
  // faster way over 32 images (us, one row per strip against several):
  //   3x3 bfloat16 to bfloat16, aligned columns: 128 planes of 112x112 67.1 / 52.4, 56x56 20.9 / 17.6; but not
  //   with unaligned columns (512 of 14x14 9.8 / 11.7, 128 of 57x61 to f32 44.1 / 48.9) or int8 (56x56 21.0 / 22.0),
  //   nor to f32 with aligned ones, where it depends on the size (128 of 112x112 70.4 / 64.6, 56x56 19.0 / 20.5,
  //   48x64 18.1 / 18.8);
  //   5x5 to bfloat16: 128 of 112x112 139.5 / 97.4, 57x61 53.1 / 47.0, 256 of 14x14 11.1 / 9.2; to 32 bits only
  //   with aligned columns (int8, 56x56 36.1 / 34.0, 55x55 44.8 / 47.6).
  if (d.Sw == 1 && d.Sh == 1 && d.Ho >= 6) {
    const bool edge = dw_edge(d), narrow = d.out_dtype == GS_BF16;
    const int64_t row_strips = int64_t(d.N) * d.C * ceil_div(d.Wo, kVX), fill = int64_t(dw_num_cus()) * 256;
    if constexpr (__is_same(T, uint16_t))
      if (d.Kh == 3 && d.Kw == 3 && edge && narrow && row_strips * ceil_div(d.Ho, 4) >= fill)
        return launch_depthwise_rows<T, 4>(d, s);
    if (d.Kh == 5 && d.Kw == 5 && (edge || narrow) && row_strips * ceil_div(d.Ho, 2) >= fill)
      return launch_depthwise_rows<T, 2>(d, s);
  }
  return launch_depthwise_rows<T, 1>(d, s);
}

}  // namespace

hipError_t launch_depthwise(const DepthwiseArgs& d, hipStream_t s) {
  for (int v : {d.H, d.W, d.Ho, d.Wo})
    if (v > (1 << 20)) return hipErrorInvalidValue;
  for (int v : {d.Kh, d.Kw, d.Sh, d.Sw, d.Ph, d.Pw})
    if (v < 0 || v > 64) return hipErrorInvalidValue;
  if (d.Kh < 1 || d.Kw < 1 || d.Sh < 1 || d.Sw < 1) return hipErrorInvalidValue;
  // Padding is smaller than the window: no window lies wholly outside the image, and the reads of
  // the last strip of a row stay within the LDS reserved behind the copy.
  if (d.Ph >= d.Kh || d.Pw >= d.Kw) return hipErrorInvalidValue;
  return d.in_dtype == GS_I8 ? launch_depthwise_t<int8_t>(d, s) : launch_depthwise_t<uint16_t>(d, s);
}

}  // namespace gs
