// Direct 2D convolution (Fig. 2a) for inputs with fewer channels than one 32-byte channel chunk
// (the 3-channel stem of a CNN).  With so few channels the contraction length K = C*Kh*Kw is
// short, so the whole im2col row of a position fits in LDS: a workgroup forms the rows of the
// im2col matrix of Fig. 5 for 128 positions *in LDS* -- never in memory -- and multiplies them
// with the weight matrix ((O),(K)), which already is K-contiguous in the listing's (C,Kh,Kw)
// order.
//
// A task is up to 128 consecutive positions of one output row (n, x).  Persistent workgroups
// (8 waves) stage the C*Kh input rows of a task in LDS (16-byte loads issued one task ahead into
// registers, padding cells zero), gather the task's [position][k] tile through a table
// k -> LDS offset, run the MFMAs (wave w: positions 32 (w % 4) .. + 31 against channels 32 (w / 4) .. + 31), and
// write the results through a per-wave LDS staging area as 8- or 16-byte stores with residual add
// and ReLU fused.  The weight tile of 64 output channels is loaded once per workgroup.
//
// Row-window form (DR).  When a window row is at most 16 bytes (Kw <= 8 bf16 / 16 int8) and
// consecutive windows start a whole number of dwords apart (Sw * element size a multiple of 4),
// the contraction index is laid out as (c, dx, dy padded to 16 bytes): the 16 bytes an MFMA lane
// needs for position y and row (c, dx) are then the 16 bytes of the staged input row starting at
// column y*Sw - Pw, so the B fragments are read straight from the staged rows with the columns
// past Kw masked to zero, and no [position][k] tile is formed at all.  The first data column of a
// staged row is Pw, which puts every window on a dword boundary (16-byte LDS reads off a dword
// boundary are several times slower); the staged data may then sit off a dword boundary and is
// written with stores aligned to the element only, which the hardware's unaligned mode allows
// and which are few.  The weights get a second copy in that order, zero in the padding.  Where that
// fills the chip, conv_rows_kernel makes tasks of two output rows.
#include "smallc_copies.h"

#include <limits.h>

#include <mutex>

namespace gs {

struct SmallCArgs {
  ConvArgs c;
  SmallCCopies copies;   // written on the side where a.wr is the listing's tensor itself
  unsigned groups;  // workgroups that share the tasks; those behind them, if any, write the copies
  int K, Kp;        // contraction length and its padding to whole 32-byte MFMA steps (elements)
  int pitch, XO;    // LDS input-row pitch (elements) and first data column
  int wpb;          // LDS bytes per weight / tile row: Kp * esz + 16
  int tile_bytes;   // LDS bytes of the [128][wpb] tile region (at least the four staging areas)
  int xtiles;       // 128-position tasks per output row
  int otiles;       // 64-channel tiles
  int64_t tasks;    // N * Ho * xtiles * otiles
  int vec_ok;       // input rows are whole 16-byte vectors
  uint32_t dr_mask[4];   // row-window form: keeps the first Kw elements of a 16-byte window
  FastDiv dvpr, dW, dhalo, dKh, dT, dKw, dchunk;
  FastDiv dkh2, dxt, dpairs;   // conv_rows_kernel: Kh + Sh, position tiles, pairs of output rows
};

constexpr int kSmallCBatch = 4;   // 16-byte vectors a thread stages per task
constexpr int kSmallCThreads = 512;

// RAW: a.wr is the listing's ((O),(C,Kh,Kw)) tensor itself, not one of the packed copies, which the kernel writes on
// the side (a kernel of its own: with a run-time branch the other one took up to 0.3 us longer).
template <typename TR, bool DR, bool RAW>
__global__ void __launch_bounds__(kSmallCThreads) conv_smallc_kernel(SmallCArgs p) {
  constexpr int NT = kSmallCThreads;
  using T = typename std::conditional<TR::kEsz == 1, uint8_t, uint16_t>::type;
  constexpr int ESZ = TR::kEsz;
  constexpr int EPV = 16 / ESZ;
  constexpr int RS = 32 * 4 + 16;          // epilogue staging row stride in bytes
  typedef T outv_t __attribute__((ext_vector_type(EPV)));
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const ConvArgs& a = p.c;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nrows = a.C * a.Kh;
  const int row_bytes = p.pitch * ESZ;
  // LDS: weights [64][wpb] | tile [128][wpb] (reused as 4 staging areas) | input rows (+ zero row) | table
  uint8_t* wl = lds;
  uint8_t* tl = wl + 64 * p.wpb;
  T* stage = reinterpret_cast<T*>(tl + p.tile_bytes);
  const int zero_row = nrows * p.pitch;
  uint32_t* tab = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(stage) +
                                              round_up(int64_t(nrows + 1) * row_bytes, 16));
  const T* in = static_cast<const T*>(a.act);
  const int vpr = a.W * ESZ / 16;
  const int halo = p.pitch - a.W;
  const bool vec_ok = p.vec_ok != 0;

  // Workgroup b runs on XCD b % 8.  Within each round of `groups` tasks an XCD takes a contiguous
  // run of them, so that the input rows shared by neighbouring output rows meet in one L2.
  const unsigned groups = RAW ? p.groups : gridDim.x;
  int64_t task = blockIdx.x;
  if (groups % 8 == 0) task = int64_t(blockIdx.x % 8) * (groups / 8) + blockIdx.x / 8;
  const bool aside = RAW && blockIdx.x >= groups;
  if (!aside && task >= p.tasks) return;
  // task -> (o tile, n, x, position tile): the channel tile changes slowest so that a workgroup
  // almost never reloads its weights
  const int64_t per_o = p.tasks / p.otiles;
  auto decode = [&](int64_t t, int* ot, int* n, int* ho, int* xt) {
    *ot = int(t / per_o);
    int64_t r = t - int64_t(*ot) * per_o;
    *xt = int(r % p.xtiles);
    r /= p.xtiles;
    *ho = int(r % a.Ho);
    *n = int(r / a.Ho);
  };

  // -- written once: padding cells, zero row, table k -> LDS byte offset of (c, dx, dy) at column 0
  for (int id = tid; id < nrows * halo; id += NT) {
    uint32_t r, h;
    p.dhalo.divmod(uint32_t(id), &r, &h);
    stage[int(r) * p.pitch + (int(h) < p.XO ? int(h) : a.W + int(h))] = T(0);
  }
  for (int id = tid; id < p.pitch; id += NT) stage[zero_row + id] = T(0);
  for (int k = tid; !DR && k < p.Kp; k += NT) {
    int off = zero_row;
    if (k < p.K) {
      uint32_t c, t, dx, dy;
      p.dT.divmod(uint32_t(k), &c, &t);
      p.dKw.divmod(t, &dx, &dy);
      off = (int(c) * a.Kh + int(dx)) * p.pitch + p.XO - a.Pw + int(dy);
    }
    tab[k] = uint32_t(off * ESZ);
  }

  i32x4 val[kSmallCBatch];
  auto issue_loads = [&](int64_t t) {
    int ot, n, ho, xt;
    decode(t, &ot, &n, &ho, &xt);
    const int nvec = nrows * vpr;
#pragma unroll
    for (int u = 0; u < kSmallCBatch; ++u) {
      val[u] = i32x4{0, 0, 0, 0};
      if (u * NT < nvec) {                             // uniform: skip batches past the last vector
        const int id = u * NT + tid;
        uint32_t r, v, c, dx;
        p.dvpr.divmod(uint32_t(id), &r, &v);
        p.dKh.divmod(r, &c, &dx);
        const int ih = ho * a.Sh + int(dx) - a.Ph;
        if (id < nvec && ih >= 0 && ih < a.H)
          val[u] = *reinterpret_cast<const i32x4*>(in + ((int64_t(n) * a.C + int(c)) * a.H + ih) * a.W + int(v) * EPV);
      }
    }
  };
  if (vec_ok && !aside) issue_loads(task);
  if constexpr (RAW) {
    if (aside || gridDim.x == groups)                  // (the latter while the loads are on their way)
      write_copies(static_cast<const T*>(a.wr), p.copies, (blockIdx.x - (aside ? groups : 0)) * unsigned(NT) + unsigned(tid),
                   (aside ? gridDim.x - groups : groups) * unsigned(NT));
    if (aside) return;
  }

  int cur_ot = -1;
  for (; task < p.tasks; task += groups) {
    int ot, n, ho, xt;
    decode(task, &ot, &n, &ho, &xt);
    const int y0 = xt * 128;
    const int npos = a.Wo - y0 < 128 ? a.Wo - y0 : 128;
    __syncthreads();                                   // the previous task is out of LDS
    if (ot != cur_ot) {                                // weight tile: rows past O and columns past K are zero
      cur_ot = ot;
      const T* wsrc = static_cast<const T*>(a.wr);     // ((O rounded up to 64),(Kp)), zero padded
      if constexpr (RAW) {                             // eight threads to a row, element by element
        const int r = tid >> 3, o = ot * 64 + r;
        const T* row = wsrc + int64_t(o < a.O ? o : 0) * p.K;
        for (int k = tid & 7; k < p.Kp; k += 8) {
          // row-window form: element dy of row k / EPV; otherwise the listing's order
          const int at = DR ? k / EPV * a.Kw + k % EPV : k;
          const bool in = o < a.O && (DR ? k / EPV < nrows && k % EPV < a.Kw : k < p.K);
          *reinterpret_cast<T*>(wl + r * p.wpb + k * ESZ) = in ? row[at] : T(0);
        }
      } else {
        for (int id = tid; id < 64 * (p.Kp / EPV); id += NT) {
          const int r = id / (p.Kp / EPV), v = id - r * (p.Kp / EPV);
          *reinterpret_cast<i32x4*>(wl + r * p.wpb + v * 16) =
              *reinterpret_cast<const i32x4*>(wsrc + (int64_t(ot) * 64 + r) * p.Kp + v * EPV);
        }
      }
    }
    // -- stage the input rows (c, dx): image row ho*Sh + dx - Ph of channel c
    if (vec_ok) {
      const int nvec = nrows * vpr;
#pragma unroll
      for (int u = 0; u < kSmallCBatch; ++u) {
        const int id = u * NT + tid;
        if (u * NT < nvec && id < nvec) {
          uint32_t r, v;
          p.dvpr.divmod(uint32_t(id), &r, &v);
          typedef int32_t word_t __attribute__((aligned(1)));   // aligned to the element only
          word_t* d = reinterpret_cast<word_t*>(reinterpret_cast<uint8_t*>(stage) +
                                                (int(r) * p.pitch + p.XO) * ESZ + int(v) * 16);
          d[0] = val[u][0];
          d[1] = val[u][1];
          d[2] = val[u][2];
          d[3] = val[u][3];
        }
      }
    } else {
      for (int id = tid; id < nrows * a.W; id += NT) {
        uint32_t r, x, c, dx;
        p.dW.divmod(uint32_t(id), &r, &x);
        p.dKh.divmod(r, &c, &dx);
        const int ih = ho * a.Sh + int(dx) - a.Ph;
        stage[int(r) * p.pitch + p.XO + int(x)] =
            (ih >= 0 && ih < a.H) ? in[((int64_t(n) * a.C + int(c)) * a.H + ih) * a.W + int(x)] : T(0);
      }
    }
    __syncthreads();
    if (vec_ok && task + groups < p.tasks) issue_loads(task + groups);
    // -- gather the [position][k] tile: item = (position, 16-byte chunk of k)
    if constexpr (!DR) {
      const int nchunk = p.Kp / EPV;
      const int items = npos * nchunk;
      for (int id = tid; id < items; id += NT) {
        uint32_t pos, j;
        p.dchunk.divmod(uint32_t(id), &pos, &j);
        const uint32_t shift = uint32_t((y0 + int(pos)) * a.Sw * ESZ);
        typedef uint32_t tabv_t __attribute__((ext_vector_type(EPV)));
        const tabv_t offs = *reinterpret_cast<const tabv_t*>(tab + int(j) * EPV);
        outv_t v;
#pragma unroll
        for (int i = 0; i < EPV; ++i)
          v[i] = *reinterpret_cast<const T*>(reinterpret_cast<const uint8_t*>(stage) + offs[i] + shift);
        *reinterpret_cast<outv_t*>(tl + int(pos) * p.wpb + int(j) * 16) = v;
      }
      __syncthreads();
    }
    // -- multiply: wave w owns positions 32 (w % 4) .. + 31 and channels 32 (w / 4) .. + 31
    const int pb_ = wave & 3, ob_ = wave >> 2;
    typename TR::accv_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0;
    if (pb_ * 32 < npos) {
      const uint8_t* ap = wl + (ob_ * 32 + (lane & 31)) * p.wpb + (lane >> 5) * 16;
      const int ksteps = p.Kp * ESZ / 32;
      if constexpr (DR) {
        // K step ks holds input rows 2 ks and 2 ks + 1 (the row after the last is the zero row);
        // lanes past the last position read the last position's windows and are not stored.
        typedef i32x4 win_t __attribute__((aligned(4)));   // windows start on dword boundaries
        const int pos = pb_ * 32 + (lane & 31);
        const uint8_t* bp = reinterpret_cast<const uint8_t*>(stage) +
                            (p.XO - a.Pw + (y0 + (pos < npos ? pos : npos - 1)) * a.Sw) * ESZ +
                            (lane >> 5) * row_bytes;
        const i32x4 keep = {int(p.dr_mask[0]), int(p.dr_mask[1]), int(p.dr_mask[2]), int(p.dr_mask[3])};
        for (int ks = 0; ks < ksteps; ++ks) {
          const i32x4 b = *reinterpret_cast<const win_t*>(bp + ks * 2 * row_bytes) & keep;
          const i32x4 a0 = *reinterpret_cast<const i32x4*>(ap + ks * 32);
          acc = TR::mfma(a0, b, acc);
        }
      } else {
        const uint8_t* bp = tl + (pb_ * 32 + (lane & 31)) * p.wpb + (lane >> 5) * 16;
        for (int ks = 0; ks < ksteps; ++ks) {
          const i32x4 b = *reinterpret_cast<const i32x4*>(bp + ks * 32);
          const i32x4 a0 = *reinterpret_cast<const i32x4*>(ap + ks * 32);
          acc = TR::mfma(a0, b, acc);
        }
      }
    }
    if constexpr (!DR) __syncthreads();                // the tile is free: it becomes the staging areas
    // -- epilogue: out[((n*O + o)*Ho + ho)*Wo + y]
    if (pb_ * 32 < npos) {
      uint8_t* st = tl + wave * (32 * RS);
      const int64_t row0 = ((int64_t(n) * a.O) * a.Ho + ho) * a.Wo + y0 + pb_ * 32;   // o = 0
      const int64_t ostride = int64_t(a.Ho) * a.Wo;
      const bool vec_out = a.Wo % 4 == 0;
      {
        const int m = ob_;
        if (vec_out) {
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int r = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            *reinterpret_cast<typename TR::acc_t*>(st + r * RS + (lane & 31) * 4) = acc[v];
          }
          const int gq = lane & 7, rsub = lane >> 3;   // 8 groups of 4 positions, 8 rows per step
#pragma unroll
          for (int it = 0; it < 4; ++it) {
            const int r = it * 8 + rsub;
            const int o = ot * 64 + m * 32 + r;
            const i32x4 raw = *reinterpret_cast<const i32x4*>(st + r * RS + gq * 16);
            if (o < a.O && pb_ * 32 + gq * 4 < npos) {
              const int64_t addr = row0 + int64_t(o) * ostride + gq * 4;
              if constexpr (__is_same(typename TR::acc_t, int32_t)) {
                i32x4 r4 = raw;
                if (a.residual) r4 += *reinterpret_cast<const i32x4*>(static_cast<const int32_t*>(a.residual) + addr);
                if (a.relu) {
#pragma unroll
                  for (int e = 0; e < 4; ++e) r4[e] = r4[e] > 0 ? r4[e] : 0;
                }
                *reinterpret_cast<i32x4*>(static_cast<int32_t*>(a.out) + addr) = r4;
              } else {
                float f[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] = __int_as_float(raw[e]);
                if (a.out_dtype == GS_F32) {
                  if (a.residual) {
                    const i32x4 q = *reinterpret_cast<const i32x4*>(static_cast<const float*>(a.residual) + addr);
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] += __int_as_float(q[e]);
                  }
                  i32x4 w4;
#pragma unroll
                  for (int e = 0; e < 4; ++e) w4[e] = __float_as_int(a.relu ? fmaxf(f[e], 0.0f) : f[e]);
                  *reinterpret_cast<i32x4*>(static_cast<float*>(a.out) + addr) = w4;
                } else {
                  if (a.residual) {
                    const uint2 q = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(a.residual) + addr);
                    f[0] += __uint_as_float(q.x << 16); f[1] += __uint_as_float(q.x & 0xffff0000u);
                    f[2] += __uint_as_float(q.y << 16); f[3] += __uint_as_float(q.y & 0xffff0000u);
                  }
#pragma unroll
                  for (int e = 0; e < 4; ++e) f[e] = a.relu ? fmaxf(f[e], 0.0f) : f[e];
                  uint2 w2;
                  w2.x = pack_bf16x2(f[0], f[1]);
                  w2.y = pack_bf16x2(f[2], f[3]);
                  *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + addr) = w2;
                }
              }
            }
          }
        } else {
          const int pos = pb_ * 32 + (lane & 31);
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int o = ot * 64 + m * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            if (pos < npos && o < a.O)
              store_result<typename TR::acc_t>(a.out, a.residual, a.out_dtype,
                                               row0 + int64_t(o) * ostride + (lane & 31), acc[v], a.relu);
          }
        }
      }
    }
  }
}

// Row-window form for many rows: a task is two output rows (n, x), (n, x + 1) of up to 128 positions,
// whose input rows are staged once (C (Kh + Sh) instead of 2 C Kh).  Wave w multiplies 32 positions of row w / 4
// with all 64 channels of the tile, so that every window is read once, positions on the MFMA rows:
// a lane then holds four consecutive positions of a channel, which reach the staging rows as 16-byte
// LDS stores and memory as 16 bytes per lane.  Two workgroups per compute unit take turns between
// LDS, matrix unit and memory.
template <typename TR, bool RAW>
__global__ void __launch_bounds__(kSmallCThreads, 4) conv_rows_kernel(SmallCArgs p) {
  constexpr int NT = kSmallCThreads;
  using T = typename std::conditional<TR::kEsz == 1, uint8_t, uint16_t>::type;
  constexpr int ESZ = TR::kEsz, EPV = 16 / ESZ;
  constexpr bool INT = __is_same(typename TR::acc_t, int32_t);
  constexpr int RS = 32 * 4 + 16;          // row stride of the results' staging
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const ConvArgs& a = p.c;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kh2 = a.Kh + a.Sh, nrows = a.C * kh2;     // staged rows: row c * kh2 + i is image row x * Sh - Ph + i of channel c
  const int row_bytes = p.pitch * ESZ;
  // LDS: weights [64][wpb] | results' staging, one area per wave | input rows and a zero row
  uint8_t* const wl = lds;
  uint8_t* const st = lds + 64 * p.wpb + wave * (32 * RS);
  T* const stage = reinterpret_cast<T*>(lds + 64 * p.wpb + p.tile_bytes);
  const T* in = static_cast<const T*>(a.act);
  const int vpr = a.W * ESZ / 16, nvec = nrows * vpr;
  const int halo = p.pitch - a.W;

  // Within each round of `groups` tasks an XCD takes a contiguous run of them (see conv_smallc_kernel).
  const unsigned groups = RAW ? p.groups : gridDim.x;
  int64_t task = blockIdx.x;
  if (groups % 8 == 0) task = int64_t(blockIdx.x % 8) * (groups / 8) + blockIdx.x / 8;
  const bool aside = RAW && blockIdx.x >= groups;
  if (!aside && task >= p.tasks) return;
  const int64_t per_o = p.tasks / p.otiles;
  const int pairs = (a.Ho + 1) / 2;
  auto decode = [&](int64_t t, int* ot, int* n, int* ho, int* xt) {
    *ot = int(t / per_o);
    const uint32_t r = uint32_t(t - int64_t(*ot) * per_o), q = p.dxt.div(r);     // (tasks per channel tile fit 31 bits: host check)
    *xt = int(r - q * uint32_t(p.xtiles));
    *n = int(p.dpairs.div(q));
    *ho = 2 * int(q - uint32_t(*n) * uint32_t(pairs));
  };
  // what is written once: padding cells and the zero row
  for (int id = tid; id < nrows * halo; id += NT) {
    uint32_t r, h;
    p.dhalo.divmod(uint32_t(id), &r, &h);
    stage[int(r) * p.pitch + (int(h) < p.XO ? int(h) : a.W + int(h))] = T(0);
  }
  for (int id = tid; id < p.pitch; id += NT) stage[nrows * p.pitch + id] = T(0);

  i32x4 val[kSmallCBatch];
  auto issue_loads = [&](int64_t t) {
    int ot, n, ho, xt;
    decode(t, &ot, &n, &ho, &xt);
#pragma unroll
    for (int u = 0; u < kSmallCBatch; ++u) {
      val[u] = i32x4{0, 0, 0, 0};
      if (u * NT < nvec) {                               // uniform: skip batches past the last vector
        const int id = u * NT + tid;
        uint32_t r, v, c, i;
        p.dvpr.divmod(uint32_t(id), &r, &v);
        p.dkh2.divmod(r, &c, &i);
        const int ih = ho * a.Sh + int(i) - a.Ph;
        if (id < nvec && ih >= 0 && ih < a.H)
          val[u] = *reinterpret_cast<const i32x4*>(in + ((int64_t(n) * a.C + int(c)) * a.H + ih) * a.W + int(v) * EPV);
      }
    }
  };
  if (p.vec_ok && !aside) issue_loads(task);
  if constexpr (RAW) {
    if (aside || gridDim.x == groups)                    // (the latter while the loads are on their way)
      write_copies(static_cast<const T*>(a.wr), p.copies, (blockIdx.x - (aside ? groups : 0)) * unsigned(NT) + unsigned(tid),
                   (aside ? gridDim.x - groups : groups) * unsigned(NT));
    if (aside) return;
  }

  const int pb = wave & 3, rr = wave >> 2;               // position block, row of the task
  const int half = lane >> 5;
  const i32x4 keep = {int(p.dr_mask[0]), int(p.dr_mask[1]), int(p.dr_mask[2]), int(p.dr_mask[3])};
  const int ksteps = p.Kp * ESZ / 32;
  int cur_ot = -1;
  for (; task < p.tasks; task += groups) {
    int ot, n, ho, xt;
    decode(task, &ot, &n, &ho, &xt);
    const int y0 = xt * 128;
    const int npos = a.Wo - y0 < 128 ? a.Wo - y0 : 128;
    lds_barrier();                                       // the previous task's rows have been read
    if (ot != cur_ot) {                                  // weights: rows past O and columns past the window are zero
      cur_ot = ot;
      const T* wsrc = static_cast<const T*>(a.wr);       // ((O rounded up to 64),(Kp)), zero padded; raw: ((O),(C,Kh,Kw))
      if constexpr (RAW) {                               // eight threads to a row, element by element
        const int r = tid >> 3, o = ot * 64 + r;
        const T* row = wsrc + int64_t(o < a.O ? o : 0) * p.K;
        for (int k = tid & 7; k < p.Kp; k += 8) {
          const bool ok = o < a.O && k / EPV < a.C * a.Kh && k % EPV < a.Kw;
          *reinterpret_cast<T*>(wl + r * p.wpb + k * ESZ) = ok ? row[k / EPV * a.Kw + k % EPV] : T(0);
        }
      } else {
        for (int id = tid; id < 64 * (p.Kp / EPV); id += NT) {
          const int r = id / (p.Kp / EPV), v = id - r * (p.Kp / EPV);
          *reinterpret_cast<i32x4*>(wl + r * p.wpb + v * 16) =
              *reinterpret_cast<const i32x4*>(wsrc + (int64_t(ot) * 64 + r) * p.Kp + v * EPV);
        }
      }
    }
    if (p.vec_ok) {
#pragma unroll
      for (int u = 0; u < kSmallCBatch; ++u) {
        const int id = u * NT + tid;
        if (u * NT < nvec && id < nvec) {
          uint32_t r, v;
          p.dvpr.divmod(uint32_t(id), &r, &v);
          typedef int32_t word_t __attribute__((aligned(1)));   // aligned to the element only
          word_t* d = reinterpret_cast<word_t*>(reinterpret_cast<uint8_t*>(stage) + (int(r) * p.pitch + p.XO) * ESZ + int(v) * 16);
          d[0] = val[u][0];
          d[1] = val[u][1];
          d[2] = val[u][2];
          d[3] = val[u][3];
        }
      }
    } else {
      for (int id = tid; id < nrows * a.W; id += NT) {
        uint32_t r, x, c, i;
        p.dW.divmod(uint32_t(id), &r, &x);
        p.dkh2.divmod(r, &c, &i);
        const int ih = ho * a.Sh + int(i) - a.Ph;
        stage[int(r) * p.pitch + p.XO + int(x)] =
            (ih >= 0 && ih < a.H) ? in[((int64_t(n) * a.C + int(c)) * a.H + ih) * a.W + int(x)] : T(0);
      }
    }
    lds_barrier();
    if (p.vec_ok && task + groups < p.tasks) issue_loads(task + groups);
    if (pb * 32 >= npos || ho + rr >= a.Ho) continue;    // uniform; the barriers are at the loop's head
    // -- multiply: K step ks holds window rows 2 ks and 2 ks + 1 (c, dx); lanes past the last position
    // read the last position's windows and are not stored
    typename TR::accv_t acc[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0;
    {
      typedef i32x4 win_t __attribute__((aligned(4)));   // windows start on dword boundaries
      const int pos = pb * 32 + (lane & 31);
      const uint8_t* const b0 = reinterpret_cast<const uint8_t*>(stage) +
                                (p.XO - a.Pw + (y0 + (pos < npos ? pos : npos - 1)) * a.Sw) * ESZ;
      const uint8_t* ap = wl + (lane & 31) * p.wpb + half * 16;
      // window row r, its row dx in the channel (a single one: never past it), its LDS offset
      int r = half, dx = a.Kh == 1 ? INT_MIN / 2 : half;
      int at = (rr * a.Sh + (a.Kh == 1 ? half * kh2 : half)) * row_bytes;
      const int step = a.Kh == 1 ? 2 * kh2 * row_bytes : 2 * row_bytes, skip = (kh2 - a.Kh) * row_bytes;
      const int last = a.C * a.Kh, zero = nrows * row_bytes;
      auto window = [&]() { return *reinterpret_cast<const win_t*>(b0 + (r < last ? at : zero)); };
      // the next step's fragments are requested in front of the MFMAs
      i32x4 b = window(), w0 = *reinterpret_cast<const i32x4*>(ap), w1 = *reinterpret_cast<const i32x4*>(ap + 32 * p.wpb);
      for (int ks = 1; ks < ksteps; ++ks) {
        r += 2;
        dx += 2;
        const bool wrap = dx >= a.Kh;                    // into the next channel
        at += wrap ? step + skip : step;
        dx -= wrap ? a.Kh : 0;
        ap += 32;
        const i32x4 bn = window(), w0n = *reinterpret_cast<const i32x4*>(ap);
        const i32x4 w1n = *reinterpret_cast<const i32x4*>(ap + 32 * p.wpb);
        acc[0] = TR::mfma(b & keep, w0, acc[0]);
        acc[1] = TR::mfma(b & keep, w1, acc[1]);
        b = bn;
        w0 = w0n;
        w1 = w1n;
      }
      acc[0] = TR::mfma(b & keep, w0, acc[0]);
      acc[1] = TR::mfma(b & keep, w1, acc[1]);
    }
    // -- write-back: out[((n*O + o)*Ho + ho + rr)*Wo + y], 32 channels at a time
    const int m0 = y0 + pb * 32, mlim = y0 + npos;
    const int64_t ostride = int64_t(a.Ho) * a.Wo;
    const int64_t row0 = (int64_t(n) * a.O * a.Ho + ho + rr) * a.Wo;                    // o = 0, y = 0
    const int esz_out = INT || a.out_dtype == GS_F32 ? 4 : 2;
    typedef int32_t i32x4_bytes __attribute__((ext_vector_type(4), aligned(1)));   // 16 bytes at any address
    static_for<2>([&](auto m_) {
      constexpr int m = decltype(m_)::value;
      static_for<4>([&](auto q_) {
        constexpr int q = decltype(q_)::value;
        const auto t = __builtin_shufflevector(acc[m], acc[m], 4 * q, 4 * q + 1, 4 * q + 2, 4 * q + 3);
        *reinterpret_cast<i32x4*>(st + (lane & 31) * RS + (8 * q + 4 * half) * 4) = __builtin_bit_cast(i32x4, t);
      });
      const int o0 = ot * 64 + m * 32;
      // 16 bytes per lane, aligned to the element only; the group that the row's end cuts value by value
      auto cut_group = [&](int r, int y, int count) {
        for (int e = 0; e < count; ++e)
          store_result<typename TR::acc_t>(a.out, a.residual, a.out_dtype, row0 + int64_t(o0 + r) * ostride + y + e,
                                           *reinterpret_cast<const typename TR::acc_t*>(st + r * RS + (y - m0 + e) * 4), a.relu);
      };
      if (esz_out == 2) {
        const int g = lane & 3, rsub = lane >> 2, y = m0 + g * 8;
#pragma unroll
        for (int it = 0; it < 2; ++it) {
          const int r = it * 16 + rsub;
          const i32x4 lo = *reinterpret_cast<const i32x4*>(st + r * RS + g * 32);
          const i32x4 hi = *reinterpret_cast<const i32x4*>(st + r * RS + g * 32 + 16);
          if (y >= mlim || o0 + r >= a.O) continue;
          if (y + 8 > mlim) {
            cut_group(r, y, mlim - y);
            continue;
          }
          const int64_t at = row0 + int64_t(o0 + r) * ostride + y;
          float f[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) f[e] = __int_as_float(e < 4 ? lo[e & 3] : hi[e & 3]);
          if (a.residual) {
            const i32x4 q = *reinterpret_cast<const i32x4_bytes*>(static_cast<const uint16_t*>(a.residual) + at);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              f[2 * e] += __uint_as_float(uint32_t(q[e]) << 16);
              f[2 * e + 1] += __uint_as_float(uint32_t(q[e]) & 0xffff0000u);
            }
          }
          i32x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            w[e] = int32_t(a.relu ? pack_bf16x2(fmaxf(f[2 * e], 0.0f), fmaxf(f[2 * e + 1], 0.0f)) : pack_bf16x2(f[2 * e], f[2 * e + 1]));
          *reinterpret_cast<i32x4_bytes*>(static_cast<uint16_t*>(a.out) + at) = w;
        }
      } else {
        const int g = lane & 7, rsub = lane >> 3, y = m0 + g * 4;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int r = it * 8 + rsub;
          i32x4 w = *reinterpret_cast<const i32x4*>(st + r * RS + g * 16);
          if (y >= mlim || o0 + r >= a.O) continue;
          if (y + 4 > mlim) {
            cut_group(r, y, mlim - y);
            continue;
          }
          const int64_t at = row0 + int64_t(o0 + r) * ostride + y;
          if (a.residual) {
            const i32x4 q = *reinterpret_cast<const i32x4_bytes*>(static_cast<const int32_t*>(a.residual) + at);
#pragma unroll
            for (int e = 0; e < 4; ++e)
              w[e] = INT ? w[e] + q[e] : __float_as_int(__int_as_float(w[e]) + __int_as_float(q[e]));
          }
          if (a.relu) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              w[e] = INT ? (w[e] > 0 ? w[e] : 0) : __float_as_int(fmaxf(__int_as_float(w[e]), 0.0f));
          }
          *reinterpret_cast<i32x4_bytes*>(static_cast<int32_t*>(a.out) + at) = w;
        }
      }
    });
  }
}

template <typename T>
__global__ void __launch_bounds__(256) conv_smallc_pack_kernel(const T* __restrict__ w, SmallCCopies c) {
  write_copies(w, c, int64_t(blockIdx.x) * blockDim.x + threadIdx.x, int64_t(gridDim.x) * blockDim.x);
}

static int smallc_kp(int in_dtype, int C, int Kh, int Kw) {
  const int per = in_dtype == GS_I8 ? 32 : 16;
  return int(round_up(int64_t(C) * Kh * Kw, per));
}

bool conv_is_smallc(int in_dtype, int C) { return C * int(dtype_size(in_dtype)) < 32 && C > 0; }

// The row-window copy exists when a window row fits 16 bytes (whether it is used depends on the
// stride, which the packing call does not know).
static bool smallc_has_rows_copy(int in_dtype, int Kw) { return Kw * int(dtype_size(in_dtype)) <= 16; }
static size_t smallc_natural_bytes(int in_dtype, int O, int C, int Kh, int Kw) {
  return size_t(round_up(O, 64)) * smallc_kp(in_dtype, C, Kh, Kw) * dtype_size(in_dtype);
}
static size_t smallc_rows_offset(int in_dtype, int O, int C, int Kh, int Kw) {
  return size_t(round_up(int64_t(smallc_natural_bytes(in_dtype, O, C, Kh, Kw)), 256));
}

size_t conv_smallc_weight_bytes(int in_dtype, int O, int C, int Kh, int Kw) {
  if (!conv_is_smallc(in_dtype, C)) return 0;
  if (!smallc_has_rows_copy(in_dtype, Kw)) return smallc_natural_bytes(in_dtype, O, C, Kh, Kw);
  return smallc_rows_offset(in_dtype, O, C, Kh, Kw) + size_t(round_up(O, 64)) * round_up(C * Kh, 2) * 16;
}

SmallCCopies smallc_copies(void* packed, bool blocked, int in_dtype, int O, int C, int Kh, int Kw, int64_t* elements) {
  SmallCCopies c;
  uint8_t* const natural = static_cast<uint8_t*>(packed) + conv_smallc_weight_offset(in_dtype, O, C, Kh, Kw);
  c.taps = packed;
  c.natural = natural;
  c.blocked = blocked && conv_blocked_weight_bytes(in_dtype, O, C, Kh, Kw)
                  ? static_cast<uint8_t*>(packed) + conv_blocked_weight_offset(in_dtype, O, C, Kh, Kw) : nullptr;
  c.mark = conv_blocked_mark(packed, in_dtype, O, C, Kh, Kw);
  c.rows = smallc_has_rows_copy(in_dtype, Kw) ? natural + smallc_rows_offset(in_dtype, O, C, Kh, Kw) : nullptr;
  c.O = O; c.O64 = int(round_up(O, 64)); c.C = C; c.Kh = Kh; c.Kw = Kw;
  c.Cpad = in_dtype == GS_I8 ? 32 : 16;                // one chunk: fewer channels than that
  c.Kp = smallc_kp(in_dtype, C, Kh, Kw);
  c.rows2 = int(round_up(C * Kh, 2));
  const int64_t taps = int64_t(O) * Kh * Kw * c.Cpad, rows = int64_t(c.O64) * c.rows2 * 16 / int64_t(dtype_size(in_dtype));
  const int64_t blocks = c.blocked ? int64_t(conv_blocked_weight_bytes(in_dtype, O, C, Kh, Kw) / dtype_size(in_dtype)) : 0;
  *elements = taps + int64_t(c.O64) * c.Kp + (c.rows ? rows : 0) + blocks;
  return c;
}

hipError_t launch_conv_smallc_pack(const void* w, void* packed, int in_dtype, int O, int C, int Kh, int Kw,
                                   bool blocked, hipStream_t s) {
  int64_t elements;
  const SmallCCopies c = smallc_copies(packed, blocked, in_dtype, O, C, Kh, Kw, &elements);
  if (elements == 0) return hipSuccess;
  const int64_t b = ceil_div(elements * int64_t(dtype_size(in_dtype)) / 16, 256);   // (every copy is whole pieces)
  const dim3 grid(unsigned(b < 4096 ? b : 4096));
  if (in_dtype == GS_I8)
    hipLaunchKernelGGL((conv_smallc_pack_kernel<uint8_t>), grid, dim3(256), 0, s, static_cast<const uint8_t*>(w), c);
  else
    hipLaunchKernelGGL((conv_smallc_pack_kernel<uint16_t>), grid, dim3(256), 0, s, static_cast<const uint16_t*>(w), c);
  return hipGetLastError();
}

static int smallc_num_cus() {
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

// LDS of a workgroup: weights, staged input rows, and tiles or staging of the results.
struct SmallCLayout {
  bool dr;                       // row-window form
  int R;                         // its output rows per task
  int Kp, wpb, XO, pitch;        // see SmallCArgs
  int64_t tile_bytes, stage_bytes, lds_bytes;
  bool fits;
};
static SmallCLayout smallc_layout(int in_dtype, int C, int W, int Kh, int Kw, int Sh, int Sw, int Pw, int Wo, int rows = 1) {
  const int esz = int(dtype_size(in_dtype)), epd = 4 / esz;
  SmallCLayout l;
  // Row-window form: windows a whole number of dwords apart, a window row within 16 bytes.
  l.dr = smallc_has_rows_copy(in_dtype, Kw) && (Sw * esz) % 4 == 0;
  l.Kp = l.dr ? int(round_up(C * Kh, 2)) * (16 / esz) : smallc_kp(in_dtype, C, Kh, Kw);
  l.wpb = l.Kp * esz + 16;
  // First data column of a staged row.  Row-window form: exactly Pw, so that window y starts
  // y*Sw elements into the row, on a dword boundary (the staged data itself may then sit off one).
  l.XO = l.dr ? Pw : int(round_up(Pw, epd));
  const int64_t reach = int64_t(l.XO) - Pw + int64_t(Wo - 1) * Sw + Kw;
  const int64_t width = reach > l.XO + W ? reach : l.XO + W;
  l.pitch = int(round_up(width, epd));
  if ((l.pitch / epd) % 2 == 0) l.pitch += epd;        // an odd number of dwords spreads the gather over banks
  constexpr int kStaging = (kSmallCThreads / 64) * 32 * (32 * 4 + 16);   // one staging area per wave
  l.tile_bytes = (!l.dr && 128 * int64_t(l.wpb) > kStaging) ? 128 * int64_t(l.wpb) : kStaging;
  l.R = l.dr ? rows : 1;
  const int64_t staged = (int64_t(C) * (Kh + (l.R - 1) * Sh) + 1) * l.pitch * esz;
  l.stage_bytes = round_up(staged, 16);
  l.lds_bytes = 64 * int64_t(l.wpb) + l.tile_bytes + l.stage_bytes + (l.R > 1 ? 0 : int64_t(l.Kp) * 4);
  l.fits = l.lds_bytes <= 96 * 1024 && staged <= (1 << 20);
  return l;
}

bool conv_smallc_fits(int in_dtype, int C, int W, int Kh, int Kw, int Sh, int Sw, int Pw, int Wo) {
  return conv_is_smallc(in_dtype, C) && smallc_layout(in_dtype, C, W, Kh, Kw, Sh, Sw, Pw, Wo).fits;
}

// `a.wr` must point at the natural-order weight copy, or, with `packed`, at the weights themselves: a call that
// brings its weights then needs no packing launch in front, and its kernel writes the copies to `packed` on
// the side.  Returns hipErrorInvalidValue when the shape does not fit (LDS), or where packing first is the
// faster way, so that the caller can fall back.
template <typename TR>
static hipError_t launch_smallc_t(const ConvArgs& a, void* packed, hipStream_t s) {
  const bool raw = packed != nullptr;
  constexpr int ESZ = TR::kEsz;
  constexpr int EPV = 16 / ESZ, EPD = 4 / ESZ;
  SmallCLayout l = smallc_layout(a.in_dtype, a.C, a.W, a.Kh, a.Kw, a.Sh, a.Sw, a.Pw, a.Wo);
  if (!l.fits) return hipErrorInvalidValue;
  // Pairs of rows where they fill the chip: a task of two costs 1.6 of one (64 x 3 x 224x224 -> 64, 7x7 at
  // stride 2, on 512 workgroups: 3584 pairs 62 us, 7168 rows 75; one image 7.5 and 6.5, 16 of 150x150 25.1
  // and 23.8).
  if (l.dr) {
    const int64_t slots = 2 * smallc_num_cus(), per_row = int64_t(a.N) * ceil_div(a.Wo, 128) * ceil_div(a.O, 64);
    const SmallCLayout two = smallc_layout(a.in_dtype, a.C, a.W, a.Kh, a.Kw, a.Sh, a.Sw, a.Pw, a.Wo, 2);
    const bool whole = (a.W * ESZ) % 16 != 0 || int64_t(a.C) * (a.Kh + a.Sh) * (a.W * ESZ / 16) <= kSmallCThreads * kSmallCBatch;
    if (two.fits && whole && 1.6 * double(ceil_div(per_row * ((a.Ho + 1) / 2), slots)) < double(ceil_div(per_row * a.Ho, slots))) l = two;
  }
  const bool dr = l.dr;
  const int64_t lds_bytes = l.lds_bytes;
  SmallCArgs p;
  p.c = a;
  p.K = a.C * a.Kh * a.Kw;
  p.Kp = l.Kp;
  p.wpb = l.wpb;
  p.XO = l.XO;
  p.pitch = l.pitch;
  p.tile_bytes = int(l.tile_bytes);
  int64_t elements = 0;
  if (raw) {
    p.copies = smallc_copies(packed, a.wblk != nullptr, a.in_dtype, a.O, a.C, a.Kh, a.Kw, &elements);
    if (elements >= (int64_t(1) << 30)) return hipErrorInvalidValue;   // (32-bit indices, a step of at most 2^30 threads)
  }
  if (dr && !raw)
    p.c.wr = static_cast<const uint8_t*>(a.wr) + smallc_rows_offset(a.in_dtype, a.O, a.C, a.Kh, a.Kw);
  if (dr) {
    for (int d = 0; d < 4; ++d) {
      uint32_t m = 0;
      for (int e = 0; e < EPD; ++e)
        if (d * EPD + e < a.Kw) m |= (ESZ == 2 ? 0xffffu : 0xffu) << (e * ESZ * 8);
      p.dr_mask[d] = m;
    }
  }
  p.vec_ok = ((a.W * ESZ) % 16 == 0 && reinterpret_cast<uintptr_t>(a.act) % 16 == 0 &&
              int64_t(a.C) * (a.Kh + (l.R - 1) * a.Sh) * (a.W * ESZ / 16) <= kSmallCThreads * kSmallCBatch) ? 1 : 0;
  p.xtiles = int(ceil_div(a.Wo, 128));
  p.otiles = int(ceil_div(a.O, 64));
  const int per_image = int(ceil_div(a.Ho, l.R));      // (tensors have fewer than 2^31 elements: so do tasks per channel tile)
  p.tasks = int64_t(a.N) * per_image * p.xtiles * p.otiles;
  p.dkh2 = FastDiv::make(uint32_t(a.Kh + (l.R - 1) * a.Sh));
  p.dxt = FastDiv::make(uint32_t(p.xtiles > 0 ? p.xtiles : 1));
  p.dpairs = FastDiv::make(uint32_t(per_image > 0 ? per_image : 1));
  if (p.tasks == 0) return hipSuccess;
  if (p.tasks > (int64_t(1) << 40)) return hipErrorInvalidValue;
  p.dvpr = FastDiv::make(uint32_t(a.W * ESZ / 16 > 0 ? a.W * ESZ / 16 : 1));
  p.dW = FastDiv::make(uint32_t(a.W));
  p.dhalo = FastDiv::make(uint32_t(p.pitch - a.W > 0 ? p.pitch - a.W : 1));
  p.dKh = FastDiv::make(uint32_t(a.Kh));
  p.dT = FastDiv::make(uint32_t(a.Kh * a.Kw));
  p.dKw = FastDiv::make(uint32_t(a.Kw));
  p.dchunk = FastDiv::make(uint32_t(p.Kp / EPV));
  constexpr decltype(&conv_rows_kernel<TR, false>) kernels[6] = {
      conv_smallc_kernel<TR, false, false>, conv_smallc_kernel<TR, true, false>, conv_rows_kernel<TR, false>,
      conv_smallc_kernel<TR, false, true>, conv_smallc_kernel<TR, true, true>, conv_rows_kernel<TR, true>};
  const int which = (l.R > 1 ? 2 : dr) + 3 * raw;
  const auto kern = kernels[which];
  static std::once_flag once[6];
  static hipError_t attr_status[6];        // (hipSuccess is zero)
  std::call_once(once[which], [&]() {
    attr_status[which] = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
  });
  if (attr_status[which] != hipSuccess) return attr_status[which];
  int per_cu = int((160 * 1024) / (lds_bytes + 512));
  per_cu = per_cu < 1 ? 1 : per_cu > 4 ? 4 : per_cu;
  int64_t grid = int64_t(smallc_num_cus()) * per_cu;
  if (grid > p.tasks) grid = p.tasks;
  const int64_t per_group = ceil_div(p.tasks, grid);   // tasks of a workgroup
  grid = ceil_div(p.tasks, per_group);
  // Weights as they come save the packing launch (1.9 us), but a workgroup reads them element by element, some 13 ns
  // for each of K at every change of its channel tile, the first time beside its input loads.  Measured over 85
  // layers, packed first / as they are: 24 images of 6 x 49x71 -> 205, 7x7 (K = 294, four channel tiles, three
  // tasks) 42.8 / 58.7 us, 2 of 8 x 78x152 -> 441, 5x5 45.8 / 53.1, 2 of 15 x 64x113 -> 13, 5x5 (K = 375) 14.7 /
  // 15.9; 15 of 2 x 26x27 -> 264, 3x3 (K = 18, five tiles) 24.9 / 23.5, 64 of 3 x 224x224 -> 64, 7x7 stride 2
  // (K = 147) 66 / 64, 3 x 8x8 -> 4, 3x3 7.2 / 5.4.
  const int64_t tiles_each = p.otiles < per_group ? p.otiles : per_group;
  if (raw && (2 * tiles_each - 1) * p.K > 256) return hipErrorInvalidValue;
  // The copies go to workgroups of their own while there is room for them: 3 x 8x8 -> 4, 3x3 5.4 us, some
  // 0.2 more where the others write them, 5.0 without copies.
  p.groups = unsigned(grid);
  const int64_t room = int64_t(smallc_num_cus()) * per_cu - grid, wanted = ceil_div(elements / EPV, kSmallCThreads);
  grid += wanted < room ? wanted : room;
  hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(kSmallCThreads), size_t(lds_bytes), s, p);
  return hipGetLastError();
}

hipError_t launch_conv_smallc(const ConvArgs& a, void* packed, hipStream_t s) {
  if (!conv_is_smallc(a.in_dtype, a.C)) return hipErrorInvalidValue;
  return a.in_dtype == GS_I8 ? launch_smallc_t<I8Traits>(a, packed, s) : launch_smallc_t<Bf16Traits>(a, packed, s);
}

}  // namespace gs
