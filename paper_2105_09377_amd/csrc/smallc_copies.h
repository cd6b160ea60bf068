// The packed copies of the weights of few-channel convolutions, written by whichever kernel has a call's weights in hand.
#pragma once
#include "common.h"

#include <type_traits>

namespace gs {

// The packed copies of few-channel weights ((O),(C,Kh,Kw)) (glenside_conv2d_pack_weights).
struct SmallCCopies {
  void* taps;        // ((O),(Kh,Kw,Cpad)), zeros for channels past C; null: no copies are made
  void* natural;     // ((O rounded up to 64),(Kp)), zeros in the padding
  void* rows;        // row-window copy ((O rounded up to 64),(C*Kh rounded up to 2, 16 bytes)): element dy of row
                     // r = c*Kh + dx is w[o][c][dx][dy], zeros for dy >= Kw and in the padding row; or null
  void* blocked;     // the copy in 1 KB blocks (see conv_blocked_weight_offset), one chunk of channels; or null
  uint64_t* mark;    // whether it is there (see there); or null
  int O, O64, C, Kh, Kw, Cpad, Kp, rows2;
};

// `packed`: the copies one after the other, as the packing call leaves them.  *elements: of all of them.
SmallCCopies smallc_copies(void* packed, bool blocked, int in_dtype, int O, int C, int Kh, int Kw, int64_t* elements);

// Thread `first` of `step` writes its share of the 16-byte pieces, all copies in one loop: a thread has one
// latency to wait for where there are threads enough (3 x 8x8 -> 4, 3x3 in bytes, the whole call, all workgroups
// writing: 5.0 us without copies, 5.8 with this, 6.5 with one loop after the other).  I: an index type that holds all copies' element counts plus step.
template <typename T, typename I>
__device__ __forceinline__ void write_copies(const T* __restrict__ w, const SmallCCopies& c, I first, I step) {
  constexpr int G = 16 / int(sizeof(T));
  typedef T piece_t __attribute__((ext_vector_type(G)));
  if (c.mark && first == 0) *c.mark = c.blocked ? kBlockedMark : 0;
  const I O = I(c.O), C = I(c.C), taps = I(c.Kh) * I(c.Kw), K = C * taps, nrows = C * I(c.Kh), rows2 = I(c.rows2);
  const I per_tap = I(c.Cpad / G), per_row = I(c.Kp / G);
  const I n_taps = O * taps * per_tap, n_natural = I(c.O64) * per_row, n_rows = c.rows ? I(c.O64) * rows2 : 0;
  const I n_blocked = c.blocked ? I((c.O + 31) / 32) * taps * 64 : 0;
  for (I f = first; f < n_taps + n_natural + n_rows + n_blocked; f += step) {
    // elements src, src + by, ... of the weights, `count` of them (none where it is not positive), then zeros
    I src, by = 1;
    int count;
    piece_t* dst;
    if (f < n_taps) {
      const I ot = f / per_tap, ch = (f - ot * per_tap) * G, o = ot / taps;
      src = (o * C + ch) * taps + (ot - o * taps);
      by = taps;
      count = int(C) - int(ch);
      dst = static_cast<piece_t*>(c.taps) + f;
    } else if (f < n_taps + n_natural) {
      const I at = f - n_taps, o = at / per_row, k = (at - o * per_row) * G;
      src = o * K + k;
      count = o < O ? int(K) - int(k) : 0;
      dst = static_cast<piece_t*>(c.natural) + at;
    } else if (f >= n_taps + n_natural + n_rows) {         // (the order within a block: conv_repack_kernel)
      const I at = f - n_taps - n_natural - n_rows, block = at / 64, i = at - block * 64, r = i >> 1, ob = block / taps;
      const I o = ob * 32 + r, ch = ((i & 1) ^ (((r >> 2) ^ (r >> 3)) & 1)) * G;
      src = o < O ? (o * C + ch) * taps + (block - ob * taps) : 0;
      by = taps;
      count = o < O ? int(C) - int(ch) : 0;
      dst = static_cast<piece_t*>(c.blocked) + at;
    } else {
      const I at = f - n_taps - n_natural, o = at / rows2, r = at - o * rows2;
      src = (o * nrows + r) * I(c.Kw);
      count = o < O && r < nrows ? c.Kw : 0;
      dst = static_cast<piece_t*>(c.rows) + at;
    }
    piece_t v;
#pragma unroll
    for (int e = 0; e < G; ++e) {
      const T x = w[e < count ? src + I(e) * by : 0];    // (loads without a branch: all are on their way at once)
      v[e] = e < count ? x : T(0);
    }
    *dst = v;
  }
}

}  // namespace gs
