// `compute dotProd (cartProd a0 a1)` as an MFMA contraction:  C[i][j] = sum_k X[i][k] * Y[j][k].
//
// Both operands are K-contiguous (each access index of a0 / a1 owns one contiguous compute
// element), which is exactly the operand order the MFMA wants, so tiles are copied global -> LDS
// with 16-byte loads and no transposition.  A workgroup of 4 to 16 waves owns a BM x BN output tile
// (the concat-on-access-dimensions blocking of Sec. 5.4); the K loop walks 128-byte slabs (the
// pair/reduceSum blocking on the compute dimension) through two to four LDS buffers, the next slabs'
// global loads in flight while the current one feeds the MFMAs; fragment reads run one K step
// ahead of the MFMAs and the per-slab barrier sits under the slab's last MFMAs.  The kernels are
// written in bytes: a slab row is 128 bytes = 64 bf16 or 128 int8, one MFMA eats 32 bytes of K
// per row.
//
// Three kernels:
//   gemm_nt_dma_kernel     : aligned operands, K a whole number of 32-byte MFMA steps (the last
//                            slab may be short).  Slabs go global -> LDS
//                            directly (global_load_lds, 16 bytes per lane, no register staging);
//                            because such a load writes 64 x 16 contiguous bytes, rows cannot be
//                            padded, so bank conflicts are avoided by an XOR swizzle of the
//                            16-byte columns instead.
//   gemm_nt_any_kernel     : ragged K, unaligned rows: 16-byte loads at any address, register-staged; rows
//                            of fewer than 16 bytes as one piece.
//   gemm_nt_ksplit_kernel  : few result tiles, any alignment, rows of at least 16 bytes: the K slabs of a
//                            small tile are dealt to the waves of its workgroup.
//
// Result element (i, j) is stored at (j / jp) * (I * jp) + i * jp + (j % jp): jp = J gives the
// plain row-major ((I, J), ()) result; jp = H'*W' with j = flattened (n, h', w') and i = o gives
// the (N, O, H', W') layout of the convolution listings, i.e. the reshape/squeeze/transpose tail
// of Fig. 5 folded into the store.  Columns j sit on the lanes, so stores are coalesced along j.
//
// Workgroups are renumbered so that each of the 8 XCDs (which have private L2 caches and receive
// consecutive workgroup ids round-robin) works on a compact block of the tile grid.
#include "common.h"

#include <stdlib.h>

#include <mutex>

namespace gs {

constexpr int kSlabBytes = 128;             // K bytes per slab row
constexpr int kRowBytes = kSlabBytes + 16;  // LDS row stride: odd multiple of 16 B, conflict-free b128
constexpr int kXcds = 8;

// Every argument is requested at once: one latency instead of one per use.
__device__ __forceinline__ void request_args(const GemmArgs& a) {
  asm volatile("" ::"s"(a.x), "s"(a.y), "s"(a.out), "s"(a.residual), "s"(a.I), "s"(a.J), "s"(a.K), "s"(a.ldx), "s"(a.ldy), "s"(a.jp),
               "s"(a.bm), "s"(a.bn), "s"(a.relu), "s"(a.vj), "s"(a.out_dtype));
}

// Map the hardware workgroup id to a tile so that an XCD's workgroups cover a compact region:
// XCD x gets the contiguous range of "logical" ids [x*n/8, (x+1)*n/8), and logical ids walk the
// grid in column bands of `band` tile rows.
__device__ inline void tile_of_block(uint32_t bid, uint32_t nblocks, int64_t tiles_i, int64_t tiles_j,
                                     int64_t* ti, int64_t* tj) {
  const uint32_t per = nblocks / kXcds, rem = nblocks % kXcds;   // (fewer than 2^31 tiles: host check)
  const uint32_t x = bid % kXcds, l = bid / kXcds;
  // XCDs 0..rem-1 own (per + 1) ids.
  const uint32_t logical = x * per + (x < rem ? x : rem) + l;
  constexpr uint32_t band = 8;
  const uint64_t band_size = band * uint64_t(tiles_j);           // (more than 32 bits: one band)
  const uint32_t b = band_size > logical ? 0 : logical / uint32_t(band_size);
  const uint32_t r = logical - b * uint32_t(band_size);
  const uint32_t rows_here = (b * band + band <= uint32_t(tiles_i)) ? band : uint32_t(tiles_i) - b * band;
  const uint32_t q = r / rows_here;
  *ti = b * band + (r - q * rows_here);
  *tj = q;
}

// Offset of column j in a row of the result (see the top).  64-bit divisions are routines of more than a
// hundred instructions: plain rows need none, other results seldom more than 32 bits.
__device__ __forceinline__ int64_t column_offset(const GemmArgs& a, int64_t j) {
  if (a.jp >= a.J) return j;
  if (a.J <= 0x7fffffff) {
    const uint32_t q = uint32_t(j) / uint32_t(a.jp);
    return int64_t(q) * (a.I * a.jp) + (uint32_t(j) - q * uint32_t(a.jp));
  }
  return (j / a.jp) * (a.I * a.jp) + (j % a.jp);
}

// The rows [i0, ilim) and columns [j0, jlim) a tile may touch.  Unblocked: tile (ti, tj) starts at
// (ti * BM, tj * BN) and ends with the matrix.  Blocked: tiles are counted block by block
// (ceil(bm / BM) tile rows per block row) and end with their block; a tile past the end of a
// smaller last block is empty.
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(v)));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(v) >> 32));
  return int64_t((uint64_t(hi) << 32) | lo);
}
struct TileBox {
  int64_t i0, j0, ilim, jlim;
};
__host__ __device__ inline int64_t tile_count(int64_t extent, int64_t block, int tile) {
  return block > 0 ? ceil_div(extent, block) * ceil_div(block, tile) : ceil_div(extent, tile);
}
__device__ inline void tile_span(int64_t t, int64_t extent, int64_t block, int tile, int64_t* lo, int64_t* lim) {
  if (block <= 0) {
    *lo = t * tile;
    *lim = extent;
    return;
  }
  const int64_t per = ceil_div(block, tile), b = t / per;
  *lo = b * block + (t - b * per) * tile;
  const int64_t end = (b + 1) * block;
  *lim = end < extent ? end : extent;
}
template <int BM, int BN>
__device__ inline TileBox tile_box(const GemmArgs& a, int64_t ti, int64_t tj) {
  TileBox b;
  tile_span(ti, a.I, a.bm, BM, &b.i0, &b.ilim);
  tile_span(tj, a.J, a.bn, BN, &b.j0, &b.jlim);
  return b;
}

// Result write-back of one wave: acc[m][n] holds the 32x32 blocks of rows iw .. and columns jw ..
// (a lane holds column lane % 32, rows 8*(v/4) + 4*(lane/32) + v%4 of a block).
//
// Vector form (a.vj = 8 or 4 consecutive columns j are contiguous and aligned in the result): the
// wave stages one 32-row block of its results in `stage` (32 rows of WN * 4 + 16 bytes of LDS that
// nobody else touches) as 32-bit values and writes it back a.vj columns per lane, so a store
// instruction carries 16 (or 8) bytes per lane instead of one element.
//
// Row form (a.vj = 2: a plain row-major result of any row length and alignment): the same with
// eight columns per lane wherever they lie; the group that the end of the result cuts is written
// value by value.  Stores aligned to the element only are cheap here (rows of 1531 bfloat16: 12.7 us
// for the product against 15.6 with groups moved to aligned addresses and 17.8 value by value).
template <typename TR, int MI, int NJ>
__device__ __forceinline__ void write_tile(const GemmArgs& a, const TileBox& box, typename TR::accv_t (&acc)[MI][NJ],
                                           int64_t iw, int64_t jw, uint8_t* stage, int lane) {
  constexpr int WN = NJ * 32;
  // Results larger than the last-level cache are streamed past L2.
  const bool stream_out = a.I * a.J * 4 > (int64_t(128) << 20);

  if (a.vj >= 2) {
    constexpr int RS = WN * 4 + 16;                 // staging row stride in bytes
    const bool has_res = a.residual != nullptr;
    auto write_back = [&](auto vj_, auto kind_, auto ragged_) {
      constexpr bool RAGGED = decltype(ragged_)::value;
      using v4 = std::conditional_t<RAGGED, i32x4_any, i32x4>;
      constexpr int VJ = decltype(vj_)::value;       // columns per lane
      constexpr int kind = decltype(kind_)::value;   // 0: int32, 1: f32, 2: bf16
      constexpr int NV = VJ / 4;                     // 16-byte pieces of 32-bit values per lane
      constexpr int LPR = WN / VJ, RPP = 64 / LPR, NP = 32 / RPP;   // lanes per row, rows per pass, passes
      const int cq = lane % LPR, rsub = lane / LPR;
      const int64_t jg = jw + cq * VJ;
      const bool j_ok = jg < box.jlim;
      const int64_t jq = j_ok ? jg : 0;
      const int64_t jbase = column_offset(a, jq);
      static_for<MI>([&](auto m_) {
        constexpr int m = decltype(m_)::value;
        static_for<NJ>([&](auto n_) {
          constexpr int n = decltype(n_)::value;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int r = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            *reinterpret_cast<typename TR::acc_t*>(stage + r * RS + (n * 32 + (lane & 31)) * 4) = acc[m][n][v];
          }
        });
        i32x4 raw[NP][NV];
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int q = 0; q < NV; ++q)
            raw[p][q] = *reinterpret_cast<const i32x4*>(stage + (p * RPP + rsub) * RS + cq * VJ * 4 + q * 16);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          const int64_t i = iw + m * 32 + p * RPP + rsub;
          const bool ok = j_ok && i < box.ilim;
          const int64_t addr = ok ? jbase + i * a.jp : 0;
          if (RAGGED && jg + VJ > box.jlim) {
            if (ok)
#pragma unroll
              for (int e = 0; e < VJ; ++e)
                if (jg + e < box.jlim)
                  store_result<typename TR::acc_t>(a.out, a.residual, a.out_dtype, addr + e,
                                                   __builtin_bit_cast(typename TR::acc_t, int32_t(raw[p][e >> 2][e & 3])), a.relu);
            continue;
          }
          if constexpr (kind == 2) {
            float f[VJ];
#pragma unroll
            for (int e = 0; e < VJ; ++e) f[e] = __int_as_float(raw[p][e >> 2][e & 3]);
            if (has_res) {
              uint32_t rq[VJ / 2];
              if constexpr (VJ == 8) {
                const i32x4 t = *reinterpret_cast<const v4*>(static_cast<const uint16_t*>(a.residual) + addr);
                rq[0] = t[0]; rq[1] = t[1]; rq[2] = t[2]; rq[3] = t[3];
              } else {
                const i32x2 t = *reinterpret_cast<const i32x2*>(static_cast<const uint16_t*>(a.residual) + addr);
                rq[0] = t[0]; rq[1] = t[1];
              }
#pragma unroll
              for (int e = 0; e < VJ / 2; ++e) {
                f[2 * e] += __uint_as_float(rq[e] << 16);
                f[2 * e + 1] += __uint_as_float(rq[e] & 0xffff0000u);
              }
            }
            uint32_t w[VJ / 2];
#pragma unroll
            for (int e = 0; e < VJ / 2; ++e) {
              const float lo = a.relu ? fmaxf(f[2 * e], 0.0f) : f[2 * e];
              const float hi = a.relu ? fmaxf(f[2 * e + 1], 0.0f) : f[2 * e + 1];
              w[e] = pack_bf16x2(lo, hi);
            }
            if (ok) {
              uint16_t* dst = static_cast<uint16_t*>(a.out) + addr;
              if constexpr (VJ == 8) {
                const v4 w4 = {int(w[0]), int(w[1]), int(w[2]), int(w[3])};
                if (stream_out) __builtin_nontemporal_store(w4, reinterpret_cast<v4*>(dst));
                else *reinterpret_cast<v4*>(dst) = w4;
              } else {
                const i32x2 w2 = {int(w[0]), int(w[1])};
                if (stream_out) __builtin_nontemporal_store(w2, reinterpret_cast<i32x2*>(dst));
                else *reinterpret_cast<i32x2*>(dst) = w2;
              }
            }
          } else {
#pragma unroll
            for (int q = 0; q < NV; ++q) {
              v4 r4 = raw[p][q];
              if (has_res) {
                const v4 t = *reinterpret_cast<const v4*>(static_cast<const int32_t*>(a.residual) + addr + q * 4);
                if constexpr (kind == 0) {
                  r4 += t;
                } else {
#pragma unroll
                  for (int e = 0; e < 4; ++e) r4[e] = __float_as_int(__int_as_float(r4[e]) + __int_as_float(t[e]));
                }
              }
              if (a.relu) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  if constexpr (kind == 0) r4[e] = r4[e] > 0 ? r4[e] : 0;
                  else r4[e] = __float_as_int(fmaxf(__int_as_float(r4[e]), 0.0f));
                }
              }
              if (ok) {
                v4* dst = reinterpret_cast<v4*>(static_cast<int32_t*>(a.out) + addr + q * 4);
                if (stream_out) __builtin_nontemporal_store(r4, dst);
                else *dst = r4;
              }
            }
          }
        }
      });
    };
    using c8 = std::integral_constant<int, 8>;
    using c4 = std::integral_constant<int, 4>;
    auto by_width = [&](auto kind_) {
      if (a.vj == 8) write_back(c8{}, kind_, std::false_type{});
      else if (a.vj == 4) write_back(c4{}, kind_, std::false_type{});
      else write_back(c8{}, kind_, std::true_type{});
    };
    if constexpr (__is_same(typename TR::acc_t, int32_t)) by_width(std::integral_constant<int, 0>{});
    else if (a.out_dtype == GS_BF16) by_width(std::integral_constant<int, 2>{});
    else by_width(std::integral_constant<int, 1>{});
    return;
  }
  static_for<NJ>([&](auto n_) {
    constexpr int n = decltype(n_)::value;
    const int64_t j = jw + n * 32 + (lane & 31);
    const bool j_ok = j < box.jlim;
    const int64_t jbase = column_offset(a, j);
    static_for<MI>([&](auto m_) {
      constexpr int m = decltype(m_)::value;
      const int64_t ibase = iw + m * 32 + 4 * (lane >> 5);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t i = ibase + 8 * (v >> 2) + (v & 3);
        if (j_ok && i < box.ilim)
          store_result<typename TR::acc_t>(a.out, a.residual, a.out_dtype, jbase + i * a.jp,
                                           acc[m][n][v], a.relu, stream_out);
      }
    });
  });
}

// ---------------------------------------------------------------------------------------------
// Rows at any byte address: 16-byte pieces are loaded where they lie and pass through registers, so that LDS rows can be aligned and padded.
// ---------------------------------------------------------------------------------------------
// A row of Kb < 16 bytes as one piece: every byte requested at once, the ones past the end replaced by zero.
__device__ __forceinline__ i32x4 short_row(const uint8_t* row, int64_t Kb) {
  if (Kb <= 0) return i32x4{0, 0, 0, 0};
  uint32_t byte[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) byte[t] = row[t < Kb ? t : 0];
  uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
  for (int t = 0; t < 16; ++t) w[t >> 2] |= (t < Kb ? byte[t] : 0u) << (8 * (t & 3));
  return i32x4{int32_t(w[0]), int32_t(w[1]), int32_t(w[2]), int32_t(w[3])};
}

// Any alignment, any K of at least 16 bytes.  Slabs of 128 bytes of K go global -> registers -> LDS;
// two slabs are in flight in registers while one is multiplied and the next sits in the other LDS
// buffer.  Bound by LDS traffic (a slab of a 128x128 tile is written once, 436 cycles at 75 bytes per
// cycle, and read as 98 to 128 KB of fragments, 610 to 800 at 160, against 256-512 of MFMAs) and by what rows
// off the 16-byte boundary cost the loads (2047 x 1531 x 1001 e4m3 13.5 us, x 1008 10.5).  2047 x 1531 x 1001:
// e4m3 70.6 -> 12.6 us, int8 74.7 -> 15.1, bf16 155.8 -> 16.5 (first: 16-byte pieces gathered byte by byte).
// SHORT: rows of fewer than 16 bytes (empty ones included): one piece per row, one MFMA step, and the
// result is what takes the time.
template <typename TR, int BM, int BN, int WGM, int WGN, bool SHORT>
__global__ void __launch_bounds__(WGM * WGN * 64) gemm_nt_any_kernel(GemmArgs a) {
  request_args(a);
  constexpr int NT = WGM * WGN * 64, D = 2;
  constexpr int WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NJ = WN / 32;
  constexpr int XCH = BM * 8 / NT, YCH = BN * 8 / NT;   // 16-byte pieces per thread per slab
  static_assert(BM * 8 % NT == 0 && BN * 8 % NT == 0, "whole pieces");
  constexpr int kXBytes = BM * kRowBytes, kYBytes = BN * kRowBytes, kBuf = kXBytes + kYBytes;
  static_assert(WGM * WGN * 32 * (WN * 4 + 16) <= 2 * kBuf, "write-back staging must fit in the slab buffers");
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  int64_t ti, tj;
  tile_of_block(blockIdx.x, gridDim.x, tile_count(a.I, a.bm, BM), tile_count(a.J, a.bn, BN), &ti, &tj);
  const TileBox box = tile_box<BM, BN>(a, ti, tj);
  const int64_t i0 = box.i0, j0 = box.j0;
  if (i0 >= box.ilim || j0 >= box.jlim) return;          // past the end of a smaller last block
  const int64_t Kb = a.K * TR::kEsz;
  const int nslab = int(ceil_div(Kb, kSlabBytes));
  const int kc = (tid & 7) * 16;                         // NT % 8 == 0: the same column for every piece
  // rows past the end of an operand are clamped: their products are never stored
  const uint8_t *xp[XCH], *yp[YCH];
#pragma unroll
  for (int r = 0; r < XCH; ++r) {
    const int64_t i = i0 + ((tid + NT * r) >> 3);
    xp[r] = static_cast<const uint8_t*>(a.x) + (i < box.ilim ? i : box.ilim - 1) * a.ldx * TR::kEsz;
  }
#pragma unroll
  for (int r = 0; r < YCH; ++r) {
    const int64_t j = j0 + ((tid + NT * r) >> 3);
    yp[r] = static_cast<const uint8_t*>(a.y) + (j < box.jlim ? j : box.jlim - 1) * a.ldy * TR::kEsz;
  }

  typename TR::accv_t acc[MI][NJ];
  static_for<MI>([&](auto m_) {
    static_for<NJ>([&](auto n_) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[decltype(m_)::value][decltype(n_)::value][v] = 0;
    });
  });

  constexpr int KST = TR::kStep, P = KST / 32;           // bytes of K per MFMA step; 16-byte pieces per lane
  if constexpr (SHORT) {
    for (int r = tid; r < BM + BN; r += NT) {
      const int64_t i = r < BM ? i0 + r : j0 + r - BM, lim = r < BM ? box.ilim : box.jlim;
      const uint8_t* row = static_cast<const uint8_t*>(r < BM ? a.x : a.y) +
                           (i < lim ? i : lim - 1) * (r < BM ? a.ldx : a.ldy) * TR::kEsz;
      i32x4* dst = reinterpret_cast<i32x4*>(lds + r * kRowBytes);
      dst[0] = short_row(row, Kb);
#pragma unroll
      for (int f = 1; f < KST / 16; ++f) dst[f] = i32x4{0, 0, 0, 0};
    }
  }
  i32x4 piece[D][XCH + YCH];
  auto load = [&](int slab, auto slot_) {
    constexpr int slot = decltype(slot_)::value;
    const int64_t kb = int64_t(slab < nslab ? slab : nslab - 1) * kSlabBytes + kc;
    const int64_t at = kb < Kb - 16 ? kb : Kb - 16;
#pragma unroll
    for (int r = 0; r < XCH; ++r) piece[slot][r] = *reinterpret_cast<const i32x4_any*>(xp[r] + at);
#pragma unroll
    for (int r = 0; r < YCH; ++r) piece[slot][XCH + r] = *reinterpret_cast<const i32x4_any*>(yp[r] + at);
  };
  uint8_t* const mine = lds + (tid >> 3) * kRowBytes + kc;
  auto store = [&](int slab, auto slot_, int buf) {
    constexpr int slot = decltype(slot_)::value;
    if (slab == nslab - 1) {                             // uniform: the end of the rows
      const int64_t over = int64_t(slab) * kSlabBytes + kc - (Kb - 16);
#pragma unroll
      for (int r = 0; r < XCH + YCH; ++r) piece[slot][r] = row_piece_fix(piece[slot][r], over);
    }
    uint8_t* dst = mine + buf * kBuf;
#pragma unroll
    for (int r = 0; r < XCH; ++r) *reinterpret_cast<i32x4*>(dst + r * (NT / 8) * kRowBytes) = piece[slot][r];
#pragma unroll
    for (int r = 0; r < YCH; ++r)
      *reinterpret_cast<i32x4*>(dst + kXBytes + r * (NT / 8) * kRowBytes) = piece[slot][XCH + r];
  };
  const uint8_t* const frag = lds + (lane & 31) * kRowBytes + (lane >> 5) * (KST / 2);
  auto multiply = [&](int buf) {
    const uint8_t* xs = frag + buf * kBuf + wm * WM * kRowBytes;
    const uint8_t* ys = frag + buf * kBuf + kXBytes + wn * WN * kRowBytes;
#pragma unroll
    for (int ks = 0; ks < (SHORT ? 1 : kSlabBytes / KST); ++ks) {
      i32x4 xf[MI * P], yf[NJ * P];
#pragma unroll
      for (int m = 0; m < MI; ++m)
#pragma unroll
        for (int f = 0; f < P; ++f)
          xf[m * P + f] = *reinterpret_cast<const i32x4*>(xs + m * 32 * kRowBytes + ks * KST + f * 16);
#pragma unroll
      for (int n = 0; n < NJ; ++n)
#pragma unroll
        for (int f = 0; f < P; ++f)
          yf[n * P + f] = *reinterpret_cast<const i32x4*>(ys + n * 32 * kRowBytes + ks * KST + f * 16);
#pragma unroll
      for (int m = 0; m < MI; ++m)
#pragma unroll
        for (int n = 0; n < NJ; ++n) acc[m][n] = mfma_pieces<TR>(&xf[m * P], &yf[n * P], acc[m][n]);
    }
  };

  if constexpr (SHORT) {
    lds_barrier();
    multiply(0);
    lds_barrier();
  } else {
    static_for<D>([&](auto d_) { load(decltype(d_)::value, d_); });
    store(0, std::integral_constant<int, 0>{}, 0);
    load(D, std::integral_constant<int, 0>{});
    lds_barrier();
    for (int s0 = 0; s0 < nslab; s0 += D) {
      static_for<D>([&](auto i_) {
        constexpr int i = decltype(i_)::value;
        using Next = std::integral_constant<int, (i + 1) % D>;
        const int s = s0 + i;
        if (s < nslab) {                                   // uniform
          if (s + 1 < nslab) {
            store(s + 1, Next{}, (i + 1) & 1);
            load(s + 1 + D, Next{});
          }
          multiply(i & 1);
          lds_barrier();
        }
      });
    }
  }
  write_tile<TR, MI, NJ>(a, box, acc, i0 + wm * WM, j0 + wn * WN, lds + wave * (32 * (WN * 4 + 16)), lane);
}

// ---------------------------------------------------------------------------------------------
// Few tiles: 32x32 result tiles whose K slabs are dealt to the NW waves of a workgroup.  A wave
// moves and multiplies its own slabs in LDS of its own, two at a time, without any barrier; the
// NW partial tiles are added pairwise at the end.  Bound by one memory latency, the launch and
// the final exchange: with up to 2 NW slabs all of K is requested at once.  kDirect: aligned rows of whole MFMA steps,
// transferred global -> LDS; kStaged: any alignment, rows of at least 16 bytes, through registers.
// ---------------------------------------------------------------------------------------------
enum KsplitLoad { kDirect, kStaged };   // see gemm_nt_ksplit_kernel
template <typename TR, int NW, KsplitLoad LOAD>
__global__ void __launch_bounds__(NW * 64) gemm_nt_ksplit_kernel(GemmArgs a) {
  request_args(a);
  constexpr int KST = TR::kStep, P = KST / 32, KS = kSlabBytes / KST;
  constexpr int kOp = 32 * kSlabBytes;                   // bytes of one operand's slab
  constexpr int kWaveBytes = 4 * kOp;                         // two slabs of both operands
  constexpr int RS = 160;                                // row stride of a partial tile: both half-waves on other banks
  static_assert(32 * RS <= kWaveBytes, "a partial tile takes the place of its wave's slabs");
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t tiles_j = tile_count(a.J, a.bn, 32);
  const uint32_t row = blockIdx.x / uint32_t(tiles_j);    // (tiles_j is the grid at most)
  const TileBox box = tile_box<32, 32>(a, row, blockIdx.x - row * uint32_t(tiles_j));
  const int64_t i0 = uniform64(box.i0), j0 = uniform64(box.j0);
  if (i0 >= box.ilim || j0 >= box.jlim) return;          // past the end of a smaller last block
  const int64_t Kb = a.K * TR::kEsz, ldxb = a.ldx * TR::kEsz, ldyb = a.ldy * TR::kEsz;
  const int nslab = int(ceil_div(Kb, kSlabBytes));
  const int cnt = nslab > wave ? (nslab - wave + NW - 1) / NW : 0;   // slabs wave, wave + NW, ...

  // Piece q of a slab: row q * 8 + lane / 8; LDS rows of 128 bytes, 16-byte column c of row r at
  // column c ^ ((r / 2) % 8) (conflict-free fragment reads).
  const int col = lane & 7;
  const uint8_t *xp[4], *yp[4];
  int swz[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = q * 8 + (lane >> 3);
    swz[q] = ((r / 2) & 7) ^ col;
    const int64_t i = i0 + r < box.ilim ? i0 + r : box.ilim - 1, j = j0 + r < box.jlim ? j0 + r : box.jlim - 1;
    xp[q] = static_cast<const uint8_t*>(a.x) + i * ldxb;
    yp[q] = static_cast<const uint8_t*>(a.y) + j * ldyb;
  }
  uint8_t* const mine = lds + wave * kWaveBytes;
  const uint32_t mine_addr = lds_addr_of(lds) + wave * kWaveBytes;

  i32x4 piece[2][8];
  auto issue = [&](int t, auto slot_) {                  // slab number t of this wave
    constexpr int slot = decltype(slot_)::value;
    const int64_t k0 = int64_t(wave + t * NW) * kSlabBytes;
    if constexpr (LOAD == kDirect) {
      // a transfer lands at lane * 16: the lane fetches the column that belongs there; columns past
      // the end of a row are not multiplied and re-read column 0
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t at = k0 + (k0 + swz[q] * 16 < Kb ? swz[q] * 16 : 0);
        lds_dma16(xp[q] + at, mine_addr + slot * 2 * kOp + q * 1024);
        lds_dma16(yp[q] + at, mine_addr + slot * 2 * kOp + kOp + q * 1024);
      }
    } else {
      const int64_t kb = k0 + col * 16;
      const int64_t at = kb < Kb - 16 ? kb : Kb - 16;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        piece[slot][q] = *reinterpret_cast<const i32x4_any*>(xp[q] + at);
        piece[slot][4 + q] = *reinterpret_cast<const i32x4_any*>(yp[q] + at);
      }
    }
  };

  typename TR::accv_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0;
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  if (cnt > 0) issue(0, S0{});
  if (cnt > 1) issue(1, S1{});
  asm volatile("" ::"s"(a.relu), "s"(a.vj), "s"(a.jp), "s"(a.residual), "s"(a.out), "s"(a.out_dtype));
  for (int t0 = 0; t0 < cnt; t0 += 2) {
    static_for<2>([&](auto i_) {
      constexpr int i = decltype(i_)::value;
      const int t = t0 + i;
      if (t < cnt) {                                     // uniform
        const int slab = wave + t * NW;
        if constexpr (LOAD == kDirect) {
          if (t + 1 < cnt) wait_vmem<8>();               // the next slab's transfers stay in flight
          else wait_vmem<0>();
        } else {
          if (slab == nslab - 1) {
            const int64_t over = int64_t(slab) * kSlabBytes + col * 16 - (Kb - 16);
#pragma unroll
            for (int q = 0; q < 8; ++q) piece[i][q] = row_piece_fix(piece[i][q], over);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            uint8_t* dst = mine + i * 2 * kOp + (q * 8 + (lane >> 3)) * kSlabBytes + swz[q] * 16;
            *reinterpret_cast<i32x4*>(dst) = piece[i][q];
            *reinterpret_cast<i32x4*>(dst + kOp) = piece[i][4 + q];
          }
        }
        // K steps of this slab: the transferred form multiplies whole steps only, the staged form is zero past K
        const int64_t left = Kb - int64_t(slab) * kSlabBytes;
        const int steps = left >= kSlabBytes ? KS : int((left + KST - 1) / KST);
        const uint8_t* xs = mine + i * 2 * kOp + (lane & 31) * kSlabBytes;
        i32x4 xf[KS * P], yf[KS * P];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int f = 0; f < P; ++f) {
            const int at = ((P * (2 * ks + (lane >> 5)) + f) ^ (((lane & 31) / 2) & 7)) << 4;
            xf[ks * P + f] = *reinterpret_cast<const i32x4*>(xs + at);
            yf[ks * P + f] = *reinterpret_cast<const i32x4*>(xs + kOp + at);
          }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          if (ks < steps) acc = mfma_pieces<TR>(&xf[ks * P], &yf[ks * P], acc);
        if (t + 2 < cnt) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // all fragments of this buffer have been read
          issue(t + 2, i_);
        }
      }
    });
  }
  // Partial tiles, each in its wave's own LDS; 256 threads add four neighbouring columns each.
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  typedef typename TR::acc_t acc4_t __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int v = 0; v < 16; ++v)
    *reinterpret_cast<typename TR::acc_t*>(mine + (8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * RS + (lane & 31) * 4) = acc[v];
  __syncthreads();
  if (tid >= 256) return;
  const uint8_t* part = lds + (tid >> 3) * RS + (tid & 7) * 16;
  acc4_t t[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) t[w] = *reinterpret_cast<const acc4_t*>(part + w * kWaveBytes);
#pragma unroll
  for (int step = 1; step < NW; step *= 2)               // pairwise: fewer roundings than a chain
#pragma unroll
    for (int w = 0; w < NW; w += 2 * step) t[w] += t[w + step];
  acc4_t sum = t[0];
  const int64_t i = i0 + (tid >> 3), j = j0 + (tid & 7) * 4;
  if (i >= box.ilim || j >= box.jlim) return;
  if (a.vj >= 4) {
    const int64_t addr = column_offset(a, j) + i * a.jp;
    if constexpr (__is_same(typename TR::acc_t, float)) {
      if (a.out_dtype == GS_BF16) {
        if (a.residual) {
          const uint2 t = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(a.residual) + addr);
          sum += acc4_t{__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xffff0000u), __uint_as_float(t.y << 16),
                        __uint_as_float(t.y & 0xffff0000u)};
        }
        if (a.relu)
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[e] = fmaxf(sum[e], 0.0f);
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + addr) = uint2{pack_bf16x2(sum[0], sum[1]), pack_bf16x2(sum[2], sum[3])};
        return;
      }
    }
    if (a.residual) sum += *reinterpret_cast<const acc4_t*>(static_cast<const typename TR::acc_t*>(a.residual) + addr);
    if (a.relu)
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[e] = sum[e] > 0 ? sum[e] : 0;
    *reinterpret_cast<acc4_t*>(static_cast<typename TR::acc_t*>(a.out) + addr) = sum;
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (j + e < box.jlim)
      store_result<typename TR::acc_t>(a.out, a.residual, a.out_dtype, column_offset(a, j + e) + i * a.jp,
                                       sum[e], a.relu);
}

// ---------------------------------------------------------------------------------------------
// Direct-to-LDS kernel.  LDS slab layout: row r at r*128 bytes, 16-byte column c of that row at
// position c ^ ((r / 2) % 8).  One transfer instruction fills 8 rows: lane i lands at
// (row i/8, position i%8) and therefore fetches global column (i%8) ^ swizzle(row).
// ---------------------------------------------------------------------------------------------

template <typename TR, int BM, int BN, int WGM, int WGN, int SB, int NS>
__global__ void __launch_bounds__(WGM * WGN * 64) gemm_nt_dma_kernel(GemmArgs a) {
  request_args(a);
  constexpr int NW = WGM * WGN;                   // waves per workgroup
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  static_assert(SB == 64 || SB == 128, "K bytes per slab row");
  static_assert(NS >= 2, "slab buffers");
  constexpr int WM = BM / WGM, WN = BN / WGN;     // wave tile
  constexpr int MI = WM / 32, NJ = WN / 32;       // 32x32 MFMA blocks per wave
  constexpr int C = SB / 16;                      // 16-byte columns per slab row
  constexpr int RPB = 256 / SB;                   // slab rows per 256 bytes (one pass over the 64 banks)
  constexpr int RPI = 1024 / SB;                  // slab rows filled by one transfer instruction
  constexpr int XQ = BM / RPI / NW, YQ = BN / RPI / NW, Q = XQ + YQ;   // transfer instructions per wave and slab
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile rows must split over the waves");
  constexpr int kXBytes = BM * SB, kYBytes = BN * SB;
  constexpr int KST = TR::kStep;                  // bytes of K per row and MFMA
  constexpr int P = KST / 32;                     // 16-byte pieces a lane holds per operand block
  constexpr int KS = SB / KST;                    // MFMA K steps per slab

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int64_t tiles_i = tile_count(a.I, a.bm, BM), tiles_j = tile_count(a.J, a.bn, BN);
  int64_t ti, tj;
  tile_of_block(blockIdx.x, gridDim.x, tiles_i, tiles_j, &ti, &tj);
  const TileBox box = tile_box<BM, BN>(a, ti, tj);
  // the tile origin is the same for every lane: say so, the transfers take their base in scalar registers
  const int64_t i0 = uniform64(box.i0), j0 = uniform64(box.j0);
  if (i0 >= box.ilim || j0 >= box.jlim) return;          // past the end of a smaller last block

  const uint8_t* X = static_cast<const uint8_t*>(a.x);
  const uint8_t* Y = static_cast<const uint8_t*>(a.y);
  const int64_t ldxb = a.ldx * TR::kEsz, ldyb = a.ldy * TR::kEsz;
  // K is a whole number of MFMA steps; the last slab may hold fewer than KS of them.
  const int64_t Kb = a.K * TR::kEsz;
  const int nslab = int(ceil_div(Kb, SB));
  const int tail_steps = int((Kb - int64_t(nslab - 1) * SB) / KST);   // 1..KS steps in the last slab

  // LDS slab layout: row r at r * SB bytes, its 16-byte column c at position c ^ swizzle(r) with
  // swizzle(r) = (r / RPB) % C.  The LDS has 64 four-byte banks and serves a 16-byte read 16 lanes
  // at a time; the 16 consecutive rows those lanes read in one K step then fall on 16 different
  // 16-byte bank groups.  A transfer instruction fills RPI consecutive rows: lane i lands at
  // (row i / C, position i % C) and therefore fetches global column (i % C) ^ swizzle(row).
  // Rows past the end of an operand are clamped: their products land in accumulators that are
  // never stored.
  const int lrow = lane / C;
  const int lcol = ((lane % C) ^ (((wave * RPI + lrow) / RPB) % C)) * 16;
  static_assert((NW * RPI / RPB) % C == 0, "the swizzle of a transfer's rows must not depend on q");
  // Sources are a wave-uniform 64-bit base (the tile's first row, advanced by the slab in scalar
  // registers) plus a 32-bit byte offset per lane and instruction (the host keeps 256 rows of
  // either operand below 4 GB).
  const uint8_t* const xbase = X + i0 * ldxb;
  const uint8_t* const ybase = Y + j0 * ldyb;
  uint32_t xoff[XQ], yoff[YQ];
#pragma unroll
  for (int q = 0; q < XQ; ++q) {
    int64_t row = (wave + q * NW) * RPI + lrow;
    row = i0 + row < box.ilim ? row : box.ilim - 1 - i0;
    xoff[q] = uint32_t(row * ldxb + lcol);
  }
#pragma unroll
  for (int q = 0; q < YQ; ++q) {
    int64_t row = (wave + q * NW) * RPI + lrow;
    row = j0 + row < box.jlim ? row : box.jlim - 1 - j0;
    yoff[q] = uint32_t(row * ldyb + lcol);
  }
  // In a short last slab the 16-byte columns past K are not multiplied; their lanes re-read
  // column 0 of the slab instead of running past the end of the row (and of the matrix).
  const uint32_t tail_fix = (lcol >= tail_steps * KST) ? uint32_t(lcol) : 0u;
  // LDS: [X buffers 0 .. NS-1 | Y buffers 0 .. NS-1].
  constexpr int kYBase = NS * kXBytes;
  static_assert((MI - 1) * 32 * SB < 65536 && (NJ - 1) * 32 * SB < 65536, "blocks by immediate offset");
  const uint32_t lds0 = lds_addr_of(lds);
  // Transfer instruction idx (0 .. Q - 1) of slab `slab` into buffer `buf`.
  auto issue_one = [&](int slab, int buf, auto idx_) {
    constexpr int idx = decltype(idx_)::value;
    const int64_t k0 = int64_t(slab) * SB;
    const uint32_t fix = slab == nslab - 1 ? tail_fix : 0u;
    if constexpr (idx < XQ)
      lds_dma16_off(xbase + k0, xoff[idx] - fix, lds0 + buf * kXBytes + (wave + idx * NW) * 1024);
    else
      lds_dma16_off(ybase + k0, yoff[idx - XQ] - fix,
                    lds0 + kYBase + buf * kYBytes + (wave + (idx - XQ) * NW) * 1024);
  };

  typename TR::accv_t acc[MI][NJ];
  static_for<MI>([&](auto m_) {
    static_for<NJ>([&](auto n_) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[decltype(m_)::value][decltype(n_)::value][v] = 0;
    });
  });

  // Fragment addresses in the buffer being multiplied: row (lane % 32) of a 32-row block, 16-byte
  // columns P*(2*ks + lane/32) + f for the pieces f < P, swizzled; one address register per
  // operand, K step and piece, moved to the next buffer once per slab; the 32-row blocks of a wave
  // by immediate offset.
  const uint8_t* xa[KS * P];
  const uint8_t* ya[KS * P];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int f = 0; f < P; ++f) {
      const int koff = ((P * (2 * ks + (lane >> 5)) + f) ^ (((lane & 31) / RPB) % C)) << 4;
      xa[ks * P + f] = lds + (wm * WM + (lane & 31)) * SB + koff;
      ya[ks * P + f] = lds + kYBase + (wn * WN + (lane & 31)) * SB + koff;
    }
  // The K loop is software-pipelined by hand.  Slabs s+1 .. s+NS-1 are in flight (or landed)
  // while slab s is multiplied.  The fragments of K step k + 1 are requested before the MFMAs of
  // step k are issued (two register sets; scheduling barriers keep the compiler from undoing that
  // order, its own wait-count insertion does the rest), and the workgroup barrier of a slab sits
  // in front of the MFMAs of its LAST step, so those MFMAs cover the barrier and the latency of
  // the next slab's first fragments.  At that barrier every wave has (a) received all of its
  // fragments of the current slab (lgkmcnt 0), so its buffer may be overwritten by slab s+NS, and
  // (b) waited for its own direct-to-LDS transfers of slab s+1 (vmcnt: the counter belongs to the
  // issuing wave and transfers complete in order), so after the barrier all of that slab is in LDS.
  // The fragment reads are ordinary loads, not asm: a register written by an asm read would be
  // "defined" for the compiler at once, and copies it makes of such a register (across the loop's
  // back edge, under register pressure) would run before the data has arrived.  The loop bodies
  // are free of branches (steady state and drain are separate loops) so that the accumulators
  // stay in place.
  i32x4 fr[2][(MI + NJ) * P];
  auto request = [&](auto ks_, auto slot_) {
    constexpr int ks = decltype(ks_)::value, slot = decltype(slot_)::value;
#pragma unroll
    for (int m = 0; m < MI; ++m)
#pragma unroll
      for (int f = 0; f < P; ++f)
        fr[slot][m * P + f] = *reinterpret_cast<const i32x4*>(xa[ks * P + f] + m * 32 * SB);
#pragma unroll
    for (int n = 0; n < NJ; ++n)
#pragma unroll
      for (int f = 0; f < P; ++f)
        fr[slot][(MI + n) * P + f] = *reinterpret_cast<const i32x4*>(ya[ks * P + f] + n * 32 * SB);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](auto slot_) {
    constexpr int slot = decltype(slot_)::value;
#pragma unroll
    for (int m = 0; m < MI; ++m)
#pragma unroll
      for (int n = 0; n < NJ; ++n)
        acc[m][n] = mfma_pieces<TR>(&fr[slot][m * P], &fr[slot][(MI + n) * P], acc[m][n]);
    __builtin_amdgcn_sched_barrier(0);
  };
  using I0 = std::integral_constant<int, 0>;
  static_assert(KS % 2 == 0, "register sets alternate per K step and restart with every slab");
  int s = 0, buf = 0;               // slab being multiplied and its buffer (s % NS)
  // One full slab (another slab follows it).  ISSUE: slab s + NS exists and is requested.
  auto full_slab = [&](auto issue_) {
    constexpr bool ISSUE = decltype(issue_)::value;
    static_for<KS>([&](auto ks_) {
      constexpr int ks = decltype(ks_)::value;
      constexpr int slot = ks & 1;
      if constexpr (ks + 1 < KS) {
        request(std::integral_constant<int, ks + 1>{}, std::integral_constant<int, slot ^ 1>{});
        multiply(std::integral_constant<int, slot>{});
      } else {
        // slabs s+1 .. min(s+NS-1, last) are outstanding; s+1 must have landed
        if constexpr (ISSUE) wait_vmem<(NS - 2) * Q>();
        else wait_vmem<0>();
        lds_barrier_tracked();         // lgkmcnt(0), then the workgroup barrier
        const int done_buf = buf;
        const bool wrap = buf + 1 == NS;
        buf = wrap ? 0 : buf + 1;
        const int dx = wrap ? -(NS - 1) * kXBytes : kXBytes, dy = wrap ? -(NS - 1) * kYBytes : kYBytes;
#pragma unroll
        for (int k = 0; k < KS * P; ++k) {
          xa[k] += dx;
          ya[k] += dy;
        }
        request(I0{}, std::integral_constant<int, slot ^ 1>{});
        // the transfers of slab s + NS, into the buffer just drained, go between this step's MFMAs
        static_for<(MI * NJ > (ISSUE ? Q : 0) ? MI * NJ : Q)>([&](auto i_) {
          constexpr int i = decltype(i_)::value;
          if constexpr (i < MI * NJ) {
            constexpr int m = i / NJ, n = i % NJ;
            acc[m][n] = mfma_pieces<TR>(&fr[slot][m * P], &fr[slot][(MI + n) * P], acc[m][n]);
          }
          if constexpr (ISSUE && i < Q) issue_one(s + NS, done_buf, i_);
          __builtin_amdgcn_sched_barrier(0);
        });
        ++s;
      }
    });
  };

  static_for<NS>([&](auto b_) {
    if (decltype(b_)::value < nslab)
      static_for<Q>([&](auto idx_) { issue_one(decltype(b_)::value, decltype(b_)::value, idx_); });
  });
  // Arguments that only the epilogue reads are fetched here: a scalar load left pending across
  // the K loop would make every wait for LDS fragments a wait for everything (scalar loads return
  // out of order on the same counter).
  asm volatile("" ::"s"(a.relu), "s"(a.vj), "s"(a.jp), "s"(a.residual), "s"(a.out), "s"(a.out_dtype));
  if (nslab >= NS) wait_vmem<(NS - 1) * Q>();
  else wait_vmem<0>();
  lds_barrier_tracked();
  request(I0{}, I0{});
  while (s + NS < nslab) full_slab(std::true_type{});     // steady state
  while (s + 1 < nslab) full_slab(std::false_type{});     // drain: nothing left to request
  static_for<KS>([&](auto ks_) {    // last slab: 1..KS steps; its first fragments are on their way
    constexpr int ks = decltype(ks_)::value;
    constexpr int slot = ks & 1;
    if (ks < tail_steps) {                         // uniform
      if constexpr (ks + 1 < KS) {
        if (ks + 1 < tail_steps)
          request(std::integral_constant<int, ks + 1>{}, std::integral_constant<int, slot ^ 1>{});
      }
      multiply(std::integral_constant<int, slot>{});
    }
  });
  __syncthreads();   // every wave is done with the slabs: their memory becomes epilogue staging

  write_tile<TR, MI, NJ>(a, box, acc, i0 + wm * WM, j0 + wn * WN, lds + wave * (32 * (WN * 4 + 16)), lane);
}

// Launch with `lds_bytes` of dynamic LDS, one workgroup per tile.
template <auto KERN>
static hipError_t launch_tiles(const GemmArgs& a, int bm, int bn, int threads, int lds_bytes, hipStream_t s) {
  static std::once_flag once;
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [&]() {
    attr_status = hipFuncSetAttribute(reinterpret_cast<const void*>(KERN), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
  });
  if (attr_status != hipSuccess) return attr_status;
  const int64_t tiles = tile_count(a.I, a.bm, bm) * tile_count(a.J, a.bn, bn);
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(KERN, dim3(unsigned(tiles)), dim3(threads), lds_bytes, s, a);
  return hipGetLastError();
}
template <typename TR, int BM, int BN, int WGM, int WGN, int SB, int NS>
static hipError_t launch_dma(const GemmArgs& a, hipStream_t s) {
  constexpr int slab_bytes = NS * (BM + BN) * SB, staging = WGM * WGN * 32 * (BN / WGN * 4 + 16);
  constexpr int lds_bytes = slab_bytes > staging ? slab_bytes : staging;     // (the staging of the results takes the slabs' place)
  static_assert(lds_bytes <= 160 * 1024, "LDS of a compute unit");
  return launch_tiles<gemm_nt_dma_kernel<TR, BM, BN, WGM, WGN, SB, NS>>(a, BM, BN, WGM * WGN * 64, lds_bytes, s);
}
template <typename TR, int BM, int BN, int WGM, int WGN, bool SHORT>
static hipError_t launch_any(const GemmArgs& a, hipStream_t s) {
  return launch_tiles<gemm_nt_any_kernel<TR, BM, BN, WGM, WGN, SHORT>>(a, BM, BN, WGM * WGN * 64, 2 * (BM + BN) * kRowBytes, s);
}
template <typename TR, int NW, KsplitLoad LOAD>
static hipError_t launch_ksplit(const GemmArgs& a, hipStream_t s) {
  return launch_tiles<gemm_nt_ksplit_kernel<TR, NW, LOAD>>(a, 32, 32, NW * 64, NW * 4 * 32 * kSlabBytes, s);
}

// Few tiles: what a workgroup of the 64x64 kernels waits for is one slab after the other, so up to
// 512 tiles of 32x32 the K slabs are dealt to waves instead (256 x 512 x 784 bf16: 4.2 us against
// 6.4 in 32 tiles of 64x64; 512 x 1024 x 1024: 6.0 against 7.4; with twice the tiles 10.6 against
// 7.4).  That holds at any K up to 256 tiles.  Between 257 and 512, where K is long, it holds while the tiles
// of a row are a multiple of the 8 XCDs, whose L2 then keeps its columns (512 x 1024 x 8192: 24.5 against
// 32.2), and not otherwise (384 x 1300 x 8192: 50.2 against 32.4; 1024 x 288 x 8192: 37.4 against 31.9), where
// it is still faster than 64x64 tiles with two slab buffers were (64.1 and 63.4).
// Eight waves need the LDS of a compute unit for themselves and pay from the ninth slab on
// (300 x 300 x 8192 int8: 9.2 against 9.6 us; 512 tiles of eight slabs: 8.5 against 6.3).
template <typename TR>
static bool few_tiles(const GemmArgs& a, bool* eight) {
  const int64_t t32 = tile_count(a.I, a.bm, 32) * tile_count(a.J, a.bn, 32);
  *eight = t32 <= 256 && a.K * TR::kEsz > 8 * kSlabBytes;
  return t32 <= 512;
}

// Tile choice of the direct-to-LDS kernel (times in us, bf16 unless said otherwise).
template <typename TR>
static hipError_t launch_dma_tiles(const GemmArgs& a, hipStream_t s) {
  const int64_t t64 = tile_count(a.I, a.bm, 64) * tile_count(a.J, a.bn, 64);
  const int64_t t128 = tile_count(a.I, a.bm, 128) * tile_count(a.J, a.bn, 128);
  const int64_t t256 = tile_count(a.I, a.bm, 256) * tile_count(a.J, a.bn, 256);
  // extent a tile can fill: the block when the result is cut into blocks
  const int64_t fi = a.bm > 0 && a.bm < a.I ? a.bm : a.I, fj = a.bn > 0 && a.bn < a.J ? a.bn : a.J;
  const int64_t slabs = ceil_div(a.K * TR::kEsz, kSlabBytes);
  // Short K: the write-back of smaller tiles overlaps another tile's products (6271 x 7864 x 64 34.1 in 256x256
  // tiles, 26.5 in 128x128).  Long K: from 180 tiles on the larger ones pay although they do not fill the chip (2272 x 5160 x
  // 1536, 189 tiles, 46.7 in 128x128 tiles, 43.6).  Over 80 products each, all types: 1.14 and 1.15 times faster (int8 1.11 and
  // 1.14), two slower (one slab, e4m3 to bfloat16, 2018 x 8168: 11.0 / 12.1).
  if (((t256 >= 256 && slabs > 4) || (t256 >= 180 && slabs >= 16)) && fi >= 256 && fj >= 256)
    return launch_dma<TR, 256, 256, 2, 4, 128, 2>(a, s);
  // few rows (a convolution's output channels against many positions) or few columns (100352 x 64 x 576
  // takes 32.2 against 36.2 in half-empty 128x128 tiles)
  if (a.I <= 64 && ceil_div(fj, 256) * ceil_div(a.J, fj) >= 192) return launch_dma<TR, 64, 256, 1, 4, 128, 2>(a, s);
  if (a.J <= 64 && ceil_div(fi, 256) * ceil_div(a.I, fi) >= 192) return launch_dma<TR, 256, 64, 4, 1, 128, 2>(a, s);
  bool eight;
  if (few_tiles<TR>(a, &eight))
    return eight ? launch_ksplit<TR, 8, kDirect>(a, s) : launch_ksplit<TR, 4, kDirect>(a, s);
  if (t128 >= 192 && (a.bm <= 0 || fi >= 128) && (a.bn <= 0 || fj >= 128)) {
    // One tile per compute unit: halves of it where K is short, since two workgroups overlap what is not a
    // product (2936 x 1112 x 256 to f32 8.9 in 128x128 tiles, 8.3), else a third slab buffer in the place of the
    // second workgroup (2048^3 20.9 against 23.1 in halves).  Eight waves: with four, what each does between its
    // products lies open (2746 x 1408 x 2112 e4m3 14.1 against 13.5, 3230 x 1704 x 128 8.0 against 7.0, 7413 x 3000 x 256 25.9
    // against 23.4).  80 products for each of these lines, 16 of each pair of types: 1.12 times faster on average at up to 16 slabs
    // (int8 1.05, others 1.07 to 1.22), 1.05 beyond (1.02), 1.06 from two rounds on (1.03; 1.13 where results are bfloat16); two of
    // 240 slower, by 4 % (2390 x 5224 x 192 bf16 to f32 19.6 / 20.3).
    if (t128 <= 256 && slabs <= 16) return launch_dma<TR, 64, 128, 2, 4, 128, 3>(a, s);
    if (t128 <= 256) return launch_dma<TR, 128, 128, 2, 4, 128, 3>(a, s);
    return launch_dma<TR, 128, 128, 2, 4, 128, 2>(a, s);
  }
  // more tiles of 64x64 than one round of the chip, fewer of 64x128, long K: 7519 x 240 x 7232 e4m3 31.7 / 25.1; over 130 products
  // 1.06 times faster, one in ten 4 to 9 % slower, without a pattern in types, tiles or K
  if (t64 > 256 && slabs > 16 && tile_count(a.I, a.bm, 64) * tile_count(a.J, a.bn, 128) <= 256 && (a.bn <= 0 || fj >= 128))
    return launch_dma<TR, 64, 128, 2, 4, 128, 3>(a, s);
  // 1024^3: 10.9 with two slab buffers, 7.9 with three, 7.4 with four; 1024 x 2048 x 1024, two
  // workgroups per compute unit: 11.4, 9.6, 9.9
  if (t64 <= 256) return launch_dma<TR, 64, 64, 2, 2, 128, 4>(a, s);
  return launch_dma<TR, 64, 64, 2, 2, 128, 3>(a, s);
}

template <typename TR>
static hipError_t launch_t(const GemmArgs& a, hipStream_t s) {
  const bool vec = (a.ldx * TR::kEsz) % 16 == 0 && (a.ldy * TR::kEsz) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(a.x) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(a.y) % 16 == 0;
  // whole MFMA steps, and 256 rows of either operand within reach of a 32-bit byte offset
  const bool dma = vec && a.K > 0 && (a.K * TR::kEsz) % TR::kStep == 0 && a.ldx * TR::kEsz < (int64_t(1) << 23) &&
                   a.ldy * TR::kEsz < (int64_t(1) << 23);
  // Columns per lane of the vector write-back: groups of vj columns must not straddle a jp
  // boundary or the end of the result, and must be 16-byte (8-byte for 4 bfloat16) aligned.
  GemmArgs v = a;
  v.vj = 1;
  const size_t osz = dtype_size(a.out_dtype);
  for (int cand = 8; cand >= 4 && v.vj == 1; cand /= 2) {
    const size_t al = cand * osz < 16 ? cand * osz : 16;
    if (a.jp % cand == 0 && a.J % cand == 0 && a.bn % cand == 0 && reinterpret_cast<uintptr_t>(a.out) % al == 0 &&
        reinterpret_cast<uintptr_t>(a.residual) % al == 0)
      v.vj = cand;
  }
  if (v.vj == 1 && a.jp >= a.J) v.vj = 2;    // plain rows
  // Rows of fewer than 16 bytes: one MFMA step per tile, in tiles as large as the others at any size (8192 x
  // 8192 x 7 bf16 to f32 51.8 us, 133 with 64x64 tiles gathered byte by byte, 980 in 32x32 tiles dealt to
  // waves; 64 x 64 x 7 3.2, 7.9 and 5.1).
  const bool is_short = a.K * TR::kEsz < 16;
  if (dma) return launch_dma_tiles<TR>(v, s);
  bool eight;
  if (!is_short && few_tiles<TR>(v, &eight))
    return eight ? launch_ksplit<TR, 8, kStaged>(v, s) : launch_ksplit<TR, 4, kStaged>(v, s);
  // 128x128 tiles need 160 of them to be the faster ones: 2047 x 1531 x 1001 e4m3 (192 tiles) 12.6 us
  // against 16.9 in 64x64 tiles, 1702 x 1221 x 300 (140 tiles) 7.8 against 7.4.  One for each compute unit: 16 waves, whose
  // loads and write-back overlap (13.5 with 8; 3000^3 bf16, 576 tiles, 97.7 against 91.3).  Fewer: 128x64 tiles where those are one
  // round and 64x64 ones more (1103 x 1072 x 1893 e4m3 15.9 in 64x64 tiles, 12.3; 780 x 1730 x 987 bf16 16.1, 13.8; over 130 products 1.1 times faster, three up to 7 % slower).  Results (or
  // blocks) of up to 64 rows or columns would leave half of every tile empty (100000 x 10 x 65 bf16 to
  // bf16: 17.4 against 12.0; 64 x 40000 x 1001 bf16 to f32: 30.4 against 24.0).
  const int64_t t128 = tile_count(a.I, a.bm, 128) * tile_count(a.J, a.bn, 128);
  const int64_t fi = a.bm > 0 && a.bm < a.I ? a.bm : a.I, fj = a.bn > 0 && a.bn < a.J ? a.bn : a.J;
  if (t128 >= 160 && fi > 64 && fj > 64) {
    if (is_short) return launch_any<TR, 128, 128, 2, 4, true>(v, s);
    return t128 <= 256 ? launch_any<TR, 128, 128, 4, 4, false>(v, s) : launch_any<TR, 128, 128, 2, 4, false>(v, s);
  }
  if (!is_short && fi > 64 && tile_count(a.I, a.bm, 64) * tile_count(a.J, a.bn, 64) > 256 &&
      tile_count(a.I, a.bm, 128) * tile_count(a.J, a.bn, 64) <= 256)
    return launch_any<TR, 128, 64, 4, 2, false>(v, s);
  return is_short ? launch_any<TR, 64, 64, 2, 2, true>(v, s) : launch_any<TR, 64, 64, 2, 2, false>(v, s);
}

bool gemm_few_tiles(int64_t I, int64_t J) { return ceil_div(I, 32) * ceil_div(J, 32) <= 512; }

hipError_t launch_gemm(const GemmArgs& a, hipStream_t s) {
  if (a.I == 0 || a.J == 0) return hipSuccess;
  if (ceil_div(a.I, 32) * ceil_div(a.J, 32) > 0x7fffffff) return hipErrorInvalidValue;
  if (a.in_dtype == GS_I8) return launch_t<I8Traits>(a, s);
  if (a.in_dtype == GS_F8) return launch_t<Fp8Traits>(a, s);
  return launch_t<Bf16Traits>(a, s);
}

}  // namespace gs
