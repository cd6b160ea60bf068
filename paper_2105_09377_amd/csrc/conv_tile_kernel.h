// Direct convolution (Fig. 2a) in small independent workgroups, several of which share a compute
// unit, so that one multiplies while another waits for memory or writes its results back.
//
// A workgroup has KS x WO x WP waves.  The KS groups split the channel chunks (Fig. 6's last
// blocking rule inside a workgroup: the partial sums meet in LDS at the end); within a group wave
// (wo, wp) owns 32 output channels x NJ blocks of 32 positions, and the group's waves share one
// patch: the input rows that the tile's positions need, one chunk of 32 bytes of channels at a
// time, in three LDS buffers.  All waves do everything: request the patch of the chunk after next
// (registers), multiply, pack the next chunk's patch into LDS, one barrier per chunk.
//
// Weights never touch the LDS.  A wave needs a 1 KB fragment per tap and chunk, and the blocked
// copy of the weights holds exactly these fragments: they are loaded from L2 into a ring of KH * KW
// register sets, each refilled with the next chunk's tap as soon as its MFMAs have been issued.
//
// Patch layout [half][row][phase][slot] in 16-byte cells (half: which 16 bytes of the 32-byte
// channel chunk).  Column p of a patch row (p = input column + Pw) lies at phase p % PH, slot
// p / PH with PH = IL * S.  The IL blocks of a block group interleave their positions -- lane n of
// block j is position IL * n + j of the group -- so that the cell of (block j, tap column kw) is
// column PH * n' + j * S + kw: lanes read consecutive slots of one phase, at any stride, and equal
// j * S + kw share one read.  IL = 4: 6 reads for 12 MFMAs of a 3x3 kernel row instead of 12, which
// matters because with one read per MFMA the LDS would be as busy as the matrix units.  IL positions
// must lie in one output row (Wo % IL == 0).  Consecutive slots do not meet in the banks; a wave whose
// positions go on in the next patch row does, since a row's pitch does not continue the banks (56
// columns, IL = 4: two of 16 lanes), and so does the write-back of bfloat16, whose lanes read 32 bytes
// apart: 323 conflict cycles per wave on 64 channels at 56x56.
//
// What bounds it: a wave issues in order, so what is not an MFMA has to be issued under one (see the
// loop); a chunk of 36 MFMAs (1152 cycles) takes 1800 cycles with one workgroup per compute unit,
// 2450 before its loads and LDS stores were dealt out between the MFMAs.  On top come 1.9 us from
// the launch to the first MFMA and 2 us of write-back, which only other workgroups can cover.
// Against the kernels that these 3x3 layers took before, in turn on one card, launches among others: 64
// channels at 56x56, batch 32, 17.4 -> 15.1 us (int8 15.3 -> 13.5); one image of 56x56 x 64 6.8 -> 4.7,
// 28x28 x 128 9.1 -> 5.0 to 6.0, 14x14 x 256 10.2 -> 6.0 (two launches before); 8 images of 14x14 x 256
// 13.2 -> 7.7; 16 of 7x7 x 512 18.0 -> 11.5; chunk counts that are no multiple of four (80 channels,
// 30x12 -> 112, 6 images) 29.5 -> 5.5.  Random layers of all sizes: see kTileCost in conv.hip.
#pragma once
#include "conv4_kernel.h"
#include "conv_tile_schedule.h"

namespace gs {

// What chunks multiply that a layer does not have.
static __device__ __attribute__((aligned(16))) const uint8_t kTileZeros[1024] = {};

typedef int32_t i32x4_bytes __attribute__((ext_vector_type(4), aligned(1)));   // 16 bytes at any address

// CM: 32-byte channel chunks that a step of the chunk loop ("chunk" below) holds.  One, except for
// 1x1 windows, whose single tap would leave too little between two barriers: there CM chunks take
// the place of the taps, each with a patch of its own, and a patch row is the input row of an output
// row (no padding; the rows between are not read, but at stride 2 the columns between are staged with
// the others: half of the cells and of the patch buffer are never read).  NAT: weights in the listing's order
// ((O),(C)) instead of the blocked copy.  ODD: the channels do not fill the last chunk.  What a patch item would
// read past them is clamped to the last channel (in bounds) and becomes zero on its way into the LDS, so that an infinity
// never meets the zero weights behind the last channel; 32-byte chunks that a 1x1 window's last step lacks multiply a page
// of zeros.  That is two more instructions per load and one or two per loaded register, so whole chunks keep kernels of
// their own.  Where the blocked copy turns out not to have been written (ConvArgs::wmark), the fragments come from the copy in the listing's order
// that is always there, 32 pieces of 32 bytes each.  50 random layers of 16 to 480 channels, us against the kernels of whole LDS rows that they took before:
// 3.4 times faster on average, at least 1.05 (29 images of 148 channels 18x10 -> 44, 3x3 bf16, 32.1 -> 7.3; 20 of 166 channels
// 75x14 -> 16 int8 at stride 2 37.0 -> 8.1; 7 of 161 channels 67x37 -> 64, 1x1, 32.5 -> 9.2).
//
// PROJ: a 1x1 projection of the same input at the same stride beside a 3x3 convolution padded by one (a residual
// block's shortcut).  Its pixels are the centre tap's: one more weight fragment and NJ more MFMAs a chunk on fragments that
// are in registers anyway, and a second write-back, instead of a launch that stages the input again.  The second accumulators
// take two workgroups of four waves to a compute unit in the place of three, and the instance of four blocks and two items
// spills seven registers.  The ResNet-18-shaped stack with its three projections so, us: one image 145 -> 134, 64 images
// 530 -> 510 (128 to 512 channels at 28x28 to 7x7).
template <typename TR, int KH, int KW, int CM, bool NAT, int S, int IL, int NJ, int WO, int WP, int KS, int MAXI, bool ONE,
          bool ODD, bool PROJ = false>
__global__ void __launch_bounds__(64 * WO * WP * KS, 2) conv_tile_kernel(ConvArgs a, ConvGeom g) {
  static_assert(NJ % IL == 0, "whole groups of interleaved blocks");
  static_assert(CM == 1 || KH * KW == 1, "chunks take the place of taps");
  static_assert(!PROJ || (KH == 3 && KW == 3 && !ODD), "the centre tap's fragments, whole chunks");
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  constexpr int ESZ = TR::kEsz;
  constexpr int G = 16 / ESZ;             // channels per 16-byte cell
  constexpr int CCH = CM * 32 / ESZ;      // channels per chunk
  constexpr int VW = kTileItem, LD = VW * ESZ / 4;        // pixels and dwords of a patch load
  // (ONE: a group has a single chunk and writes no cells in a loop; its schedule is the shortest one)
  using SC = TileSchedule<ESZ, KH, KW, CM, S, IL, NJ, VW, ONE ? 1 : MAXI>;
  constexpr int KR = SC::KR, T = KR * KW, PH = IL * S, GP = SC::GP, NG = SC::NG, NSG = SC::NSG;
  constexpr int STEPS = SC::STEPS, SLOTS = SC::SLOTS, QUOTA = SC::QUOTA;
  constexpr int NBUF = ONE ? 1 : 3;       // patch buffers (ONE: a group has a single chunk)
  constexpr int NW = WO * WP, NT = 64 * NW;
  constexpr bool INT = __is_same(typename TR::acc_t, int32_t);
  using acc_t = typename TR::acc_t;
  typedef int32_t ld2_t __attribute__((ext_vector_type(2), aligned(1)));
  typedef int32_t ld1_t __attribute__((aligned(1)));
  struct Piece { int32_t w[LD]; };        // one load: VW pixels of a channel
  constexpr bool PART = ODD && CM > 1;    // the last step may lack 32-byte chunks

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NW, w = wave % NW, wo = w / WP, wp = w % WP;
  const int gt = tid - kg * NT;           // thread within the group

  // Every argument is requested at once: one latency instead of one per use.
  asm volatile("" ::"s"(a.act), "s"(a.wblk), "s"(a.out), "s"(a.residual), "s"(a.C), "s"(a.H), "s"(a.W), "s"(a.O),
               "s"(a.Ph), "s"(a.Pw), "s"(a.Wo), "s"(a.Cpad), "s"(a.relu), "s"(a.out_dtype), "s"(g.HWo), "s"(g.M), "s"(g.tps),
               "s"(g.pos_major));
  asm volatile("" ::"s"(g.dHWo.mul), "s"(g.dHWo.shift), "s"(g.dHWo.one), "s"(g.dWo.mul), "s"(g.dWo.shift), "s"(g.dWo.one),
               "s"(g.dW.mul), "s"(g.dW.shift), "s"(g.dW.one), "s"(g.dTiles.d), "s"(g.dTiles.mul), "s"(g.dTiles.shift),
               "s"(g.dTiles.one), "s"(g.php), "s"(g.rowp), "s"(g.halfb), "s"(g.bufb));

  uint64_t mark = kBlockedMark;           // (requested here, read where the weights' addresses are made)
  if constexpr (ODD && !NAT)
    if (a.wmark) mark = *a.wmark;

  // Tile: renumbered so that an XCD owns a contiguous range (see conv4_kernel.h).
  int m0, mend, o0;
  {
    const int n_tiles = int(gridDim.x), x = int(blockIdx.x) & 7;
    const int per = n_tiles >> 3, rem = n_tiles & 7;
    const int tile = x * per + (x < rem ? x : rem) + (int(blockIdx.x) >> 3);
    const int q = int(g.dTiles.div(uint32_t(tile))), r = tile - q * int(g.dTiles.d);
    const int mt = g.pos_major ? q : r;
    o0 = (g.pos_major ? r : q) * (32 * WO);
    m0 = mt * g.tps;
    mend = m0 + g.tps < int(g.M) ? m0 + g.tps : int(g.M);
  }
  const TileSegs ts = tile_segs(m0, mend, g);
  // Chunks of a group, and of this one: the last groups have fewer or none where KS does not divide them.
  const int n_blocks = a.Cpad / (32 / ESZ);               // 32-byte chunks
  const int n_chunks = (n_blocks + CM - 1) / CM, most = (n_chunks + KS - 1) / KS, left = n_chunks - kg * most;
  const int cnt = KS == 1 ? most : left < 0 ? 0 : left < most ? left : most;
  const int first = cnt > 0 ? kg * most : 0;              // (a group without chunks loads the first one and leaves it)

  // ---- weights: fragments of (32 channels, chunk, tap), 1 KB each -------------------------------
  // (rows and blocks past O are never stored)
  constexpr int kTap = NAT ? 32 : 1024;   // bytes from a tap to the next
  int tap_step = kTap, chunk_step = T * kTap;             // (constants but where a copy may be missing)
  const uint8_t* wsrc;
  if constexpr (NAT) {
    wsrc = static_cast<const uint8_t*>(a.wr) + int64_t(first) * (T * kTap);
  } else {
    const int n_oblk = (a.O + 31) / 32;
    int ob = o0 / 32 + wo;
    ob = ob < n_oblk ? ob : n_oblk - 1;
    wsrc = static_cast<const uint8_t*>(a.wblk) + (int64_t(ob) * n_blocks + int64_t(first) * CM) * (KH * KW * kTap);
  }
  // lane's 16 bytes of a fragment: row lane % 32, half lane / 32, in the block's order (conv_repack_kernel)
  uint32_t wlane = uint32_t((lane & 31) * 32 + (((lane >> 5) ^ ((((lane & 31) >> 2) ^ ((lane & 31) >> 3)) & 1)) << 4));
  if constexpr (NAT) {
    const int o = o0 + wo * 32 + (lane & 31);
    wlane = uint32_t(o < a.O ? o : a.O - 1) * uint32_t(a.C * ESZ) + uint32_t(lane >> 5) * 16u;   // (fits: host check)
  }
  if constexpr (ODD && !NAT) {
    if (mark != kBlockedMark) {           // uniform
      const int o = o0 + wo * 32 + (lane & 31);
      tap_step = CM > 1 ? 32 : a.Cpad * ESZ;
      chunk_step = 32 * CM;
      wsrc = static_cast<const uint8_t*>(a.wr) + first * chunk_step;
      wlane = uint32_t(o < a.O ? o : a.O - 1) * uint32_t(KH * KW * a.Cpad * ESZ) + uint32_t(lane >> 5) * 16u;
    }
  }
  i32x4 ring[T], proj_tap;
  auto load_tap = [&](int ch, auto tap_) {
    constexpr int tap = decltype(tap_)::value;
    const uint8_t* at = wsrc + int64_t(ch) * chunk_step + tap * tap_step + wlane;
    if constexpr (PART) {                 // (tap: a chunk of the step)
      const int c = (first + ch) * CM + tap;
      if constexpr (NAT) at = (2 * c + (lane >> 5)) * G < a.C ? at : kTileZeros;     // rows are whole 16-byte pieces: host check
      else at = c < n_blocks ? at : kTileZeros + lane * 16;
    }
    ring[tap] = *reinterpret_cast<const i32x4*>(at);
  };

  // (the projection's blocks: one tap)
  const uint8_t* psrc = nullptr;
  if constexpr (PROJ) {
    asm volatile("" ::"s"(a.wproj), "s"(a.out_proj));
    const int n_oblk = (a.O + 31) / 32, ob = o0 / 32 + wo < n_oblk ? o0 / 32 + wo : n_oblk - 1;
    psrc = static_cast<const uint8_t*>(a.wproj) + (int64_t(ob) * n_blocks + first) * 1024 + wlane;
  }
  auto load_proj = [&](int ch) { proj_tap = *reinterpret_cast<const i32x4*>(psrc + int64_t(ch) * 1024); };

  // ---- patch items: VW pixels, consecutive in the rows a segment needs, x one half of a chunk ----
  const int64_t plane = int64_t(a.H) * a.W * ESZ;
  const uint8_t* asrc = static_cast<const uint8_t*>(a.act) + int64_t(first) * CCH * plane;
  // The extents of the first two segments are scalars; a tile that touches more than two images
  // (small planes) walks them.
  // (1x1 windows: in output rows)
  constexpr bool PT = KH * KW == 1;
  constexpr int SR = PT ? 1 : S;
  const int Ph = PT ? 0 : a.Ph, Pw = PT ? 0 : a.Pw;
  int ihlo0, rows0, ihlo1 = 0, rows1 = 0;
  seg_extent(ts, 0, g, SR, Ph, KH, &ihlo0, &rows0);
  if (ts.nseg > 1) seg_extent(ts, 1, g, SR, Ph, KH, &ihlo1, &rows1);
  uint32_t src[MAXI];
  int dst[MAXI][VW], c_of[MAXI];          // c_of (ODD): the item's first channel within a chunk
  bool item_ok[MAXI];
  {
    auto valid = [&](int ihlo, int rows, int* vlo, int* items, int* len) {
      if constexpr (PT) {                   // row by row: the rows between are not wanted
        *vlo = ihlo;
        *len = 0;
        *items = rows * int(g.dXG.d);
        return;
      }
      *vlo = ihlo > 0 ? ihlo : 0;
      const int vhi = ihlo + rows < a.H ? ihlo + rows : a.H;
      *len = vhi > *vlo ? (vhi - *vlo) * a.W : 0;
      *items = (*len + VW - 1) / VW;
    };
    int vlo0, it0, len0, vlo1 = 0, it1 = 0, len1 = 0;
    valid(ihlo0, rows0, &vlo0, &it0, &len0);
    if (ts.nseg > 1) valid(ihlo1, rows1, &vlo1, &it1, &len1);
#pragma unroll
    for (int i = 0; i < MAXI; ++i) {
      int rem = gt + NT * i, seg = 0, base = 0, ihlo = ihlo0, vlo = vlo0, items = it0, len = len0;
      if (ts.nseg == 2) {                   // uniform
        if (rem >= 2 * CM * it0) {
          rem -= 2 * CM * it0;
          seg = 1; base = rows0; ihlo = ihlo1; vlo = vlo1; items = it1; len = len1;
        }
      } else if (ts.nseg > 2) {
        int rows = rows0;
        while (rem >= 2 * CM * items && seg + 1 < ts.nseg) {
          rem -= 2 * CM * items;
          base += rows;
          ++seg;
          seg_extent(ts, seg, g, SR, Ph, KH, &ihlo, &rows);
          valid(ihlo, rows, &vlo, &items, &len);
        }
      }
      item_ok[i] = rem < 2 * CM * items;
      // half: which 16 bytes of the chunk's 32 CM
      int half = rem >= items ? 1 : 0;
      if constexpr (CM > 1) half = int((float(rem) + 0.5f) / float(items));   // (exact: both below 2^16)
      const int k = item_ok[i] ? rem - half * items : 0;
      half = item_ok[i] ? half : 0;
      c_of[i] = half * G;
      int row, col, cell;
      if constexpr (PT) {
        const int r = int(g.dXG.div(uint32_t(k)));
        col = (k - r * int(g.dXG.d)) * VW;
        col = col < a.W - VW ? col : a.W - VW;            // the last item ends with the row
        row = (vlo + r) * S;
        cell = base + r;
      } else {
        int f = k * VW < len - VW ? k * VW : len - VW;    // the last item ends with the range
        f = f > 0 ? f + vlo * a.W : vlo * a.W;
        row = int(g.dW.div(uint32_t(f)));
        col = f - row * a.W;
        cell = base + row - ihlo;
      }
      // byte offsets from the tensor's start fit 32 bits (fewer than 2^31 elements)
      src[i] = item_ok[i] ? uint32_t((ts.n_first + seg) * a.C + half * G) * uint32_t(plane) + uint32_t(row * a.W + col) * uint32_t(ESZ) : 0u;
      cell = half * g.halfb + cell * g.rowp;
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        const uint32_t c = uint32_t(col + Pw);
        dst[i][e] = cell + int(c % PH) * g.php + int(c / PH) * 16;
        if (++col == a.W) {                               // rows are at least VW long: at most one wrap
          col = 0;
          cell += g.rowp;
        }
      }
    }
  }
  Piece preg0[MAXI][G], preg[MAXI][G];
  // ODD: channels that item i has in chunk `ch`, G at most and below one if it has none.
  auto channels = [&](int ch, int i) {
    const int n = a.C - (first + ch) * CCH - c_of[i];
    return n < G ? n : G;
  };
  const int plane32 = ODD ? int(plane) : 0;               // (128 planes fit 31 bits: host check)
  int lim[MAXI];                                          // ODD: byte offset of the last channel that the loads may touch
  auto set_lim = [&](int ch) {
    if constexpr (ODD)
#pragma unroll
      for (int i = 0; i < MAXI; ++i) lim[i] = (channels(ch, i) - 1) * plane32;
  };
  auto load_piece = [&](const uint8_t* b, Piece (&preg)[MAXI][G], auto i_, auto t_) {
    constexpr int i = decltype(i_)::value, t = decltype(t_)::value;
    const uint8_t* at;
    if constexpr (ODD) at = b + (src[i] + uint32_t(t * plane32 < lim[i] ? t * plane32 : lim[i]));
    else at = b + int64_t(t) * plane + src[i];
    if constexpr (LD == 2) {
      const i32x2 v = *reinterpret_cast<const ld2_t*>(at);
      preg[i][t].w[0] = v[0]; preg[i][t].w[1] = v[1];
    } else {
      preg[i][t].w[0] = *reinterpret_cast<const ld1_t*>(at);
    }
  };
  auto load_patch = [&](int ch, Piece (&preg)[MAXI][G]) {
    static_for<MAXI>([&](auto i_) {
      static_for<G>([&](auto t_) { load_piece(asrc + int64_t(ch) * CCH * plane, preg, i_, t_); });
    });
  };
  uint8_t* const patch = lds + kg * NBUF * g.bufb;
  // Pixel p of item i: element t of the cell is channel t of the half; one byte permute per two sources.
  // (ODD: `ch` is the patch's chunk; an item's first cell clears the channels it does not have)
  auto store_cell = [&](uint8_t* pb, Piece (&preg)[MAXI][G], int ch, auto i_, auto p_) {
    constexpr int i = decltype(i_)::value, p = decltype(p_)::value;
    if constexpr (ODD && p == 0) {
      const int n = channels(ch, i);
#pragma unroll
      for (int t = 0; t < G; ++t)
#pragma unroll
        for (int d = 0; d < LD; ++d) preg[i][t].w[d] = t < n ? preg[i][t].w[d] : 0;
    }
    i32x4 cell;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      if constexpr (ESZ == 2) {
        cell[d] = int32_t(__builtin_amdgcn_perm(preg[i][2 * d + 1].w[p / 2], preg[i][2 * d].w[p / 2],
                                                p % 2 ? 0x07060302u : 0x05040100u));
      } else {
        const uint32_t sel = uint32_t((4 + p % 4) << 8 | p % 4);
        const uint32_t lo = __builtin_amdgcn_perm(preg[i][4 * d + 1].w[p / 4], preg[i][4 * d].w[p / 4], sel);
        const uint32_t hi = __builtin_amdgcn_perm(preg[i][4 * d + 3].w[p / 4], preg[i][4 * d + 2].w[p / 4], sel);
        cell[d] = int32_t(__builtin_amdgcn_perm(hi, lo, 0x05040100u));
      }
    }
    asm volatile("" : "+v"(cell));        // outside the branch: only the store is masked
    if (item_ok[i]) *reinterpret_cast<i32x4*>(pb + dst[i][p]) = cell;
  };
  // Vector loads that go with slot `slot` of a chunk (see the loop below): pieces of the patch at
  // `next_patch`, and taps of chunk `ch`.
  auto slot_loads = [&](const uint8_t* next_patch, Piece (&preg)[MAXI][G], int ch, auto slot_) {
    constexpr int slot = decltype(slot_)::value, step = slot / SLOTS, s = slot % SLOTS;
    if constexpr (!ONE)
      static_for<QUOTA>([&](auto k_) {
        constexpr int wk = SC::piece(slot, decltype(k_)::value) - SC::CELLS;
        if constexpr (wk >= 0 && wk < G * MAXI)
          load_piece(next_patch, preg, std::integral_constant<int, wk / G>{}, std::integral_constant<int, wk % G>{});
      });
    constexpr int kw = s / GP - (IL - 1) * S, gi = step % NSG * GP + s % GP;   // the last use of tap kw in its row
    if constexpr (gi == NG - 1 && kw >= 0) load_tap(ch, std::integral_constant<int, step / NSG * KW + kw>{});
    if constexpr (PROJ && gi == NG - 1 && kw == 1 && step / NSG == 1) load_proj(ch);
  };
  // The first loads, in the order in which the loop issues them, so that its waits (loads complete
  // in order) are exact from the first chunk on.
  set_lim(0);
  load_patch(0, preg0);
  __builtin_amdgcn_sched_barrier(0);
  set_lim(cnt > 1 ? 1 : 0);
  static_for<STEPS * SLOTS>([&](auto slot_) {
    slot_loads(asrc + int64_t(cnt > 1 ? 1 : 0) * CCH * plane, preg, 0, slot_);
    __builtin_amdgcn_sched_barrier(0);
  });

  // Padding cells (halo columns, rows outside the image) are written once: the buffers start as zeros.
  {
    const i32x4 z = {0, 0, 0, 0};
    const int bytes = NBUF * g.bufb;
    for (int off = gt * 16; off < bytes; off += NT * 16) *reinterpret_cast<i32x4*>(patch + off) = z;
  }

  // ---- fragment addresses: window origin of the first block's position of each block group -------
  const int wpos = wp * 32 * NJ;          // first position of this wave, relative to m0
  int fb[NG];                             // by block group
#pragma unroll
  for (int gi = 0; gi < NG; ++gi) {
    int m = m0 + wpos + gi * 32 * IL + IL * (lane & 31);
    m = m < mend ? m : mend - IL;         // a valid stand-in; its results are dropped (tiles hold whole groups of IL)
    int img = ts.n_first;
    if (ts.nseg > 1) img = int(g.dHWo.div(uint32_t(m)));
    const int p = m - img * g.HWo;
    const int ho = int(g.dWo.div(uint32_t(p))), wo_ = p - ho * a.Wo;
    const int si = img - ts.n_first;
    int base = si ? rows0 : 0, ihlo = si ? ihlo1 : ihlo0;
    if (ts.nseg > 2) {
      int rows = 0;
      base = 0;
      for (int s_ = 0; s_ <= si; ++s_) {
        base += rows;
        seg_extent(ts, s_, g, SR, Ph, KH, &ihlo, &rows);
      }
    }
    fb[gi] = (lane >> 5) * g.halfb + (base + ho * SR - Ph - ihlo) * g.rowp + (wo_ / IL) * 16;
  }

  typename TR::accv_t acc[NJ], pacc[PROJ ? NJ : 1];
  static_for<NJ>([&](auto j_) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      acc[decltype(j_)::value][v] = 0;
      if constexpr (PROJ) pacc[decltype(j_)::value][v] = 0;
    }
  });

  lds_barrier();                          // zeros are in place
  static_for<MAXI>([&](auto i_) { static_for<VW>([&](auto p_) { store_cell(patch, preg0, 0, i_, p_); }); });
  lds_barrier();

  // ---- chunks --------------------------------------------------------------------------------------
  // A wave issues in order, and a global load holds it for some 40 cycles, so everything else is
  // dealt out between the MFMAs (32 cycles each, two in a row never on the same accumulators): a
  // slot is one fragment, the MFMAs that need it, the request of the fragment that takes its
  // register in the next step, and one piece of other work -- first the cells of the next chunk's
  // patch (LDS), then the loads of the chunk after it, and each tap's refill behind its last use.
  // The chunk's one barrier stands in front of its last step, whose slots request the first
  // fragments of the next chunk.  With three buffers that is enough: a wave writes the buffer that
  // was read two chunks ago, and who has passed the last barrier is done with that one.
  i32x4 fr[SLOTS];
  auto request = [&](const uint8_t* pb, auto step_, auto s_) {
    constexpr int step = decltype(step_)::value, q = decltype(s_)::value / GP, gi = step % NSG * GP + decltype(s_)::value % GP;
    if constexpr (SC::used(decltype(s_)::value))
      fr[decltype(s_)::value] = *reinterpret_cast<const i32x4*>(pb + fb[gi] + step / NSG * (CM > 1 ? 2 * g.halfb : g.rowp) + (q % PH) * g.php + (q / PH) * 16);
  };
  int cur = 0;                                                 // LDS offset of the chunk's buffer
  auto chunk = [&](auto last_, int ch) {
    constexpr bool LAST = decltype(last_)::value;
    const uint8_t* const pb = patch + cur;
    const int nxt = cur + g.bufb < NBUF * g.bufb ? cur + g.bufb : 0;
    uint8_t* const nb = patch + nxt;
    const int ch2 = ch + 2 < cnt ? ch + 2 : ch;                // surplus at the end: no branch
    const uint8_t* const asrc2 = asrc + int64_t(ch2) * CCH * plane;
    if constexpr (!LAST) set_lim(ch2);
    static_for<STEPS>([&](auto step_) {
      constexpr int step = decltype(step_)::value, kh = step / NSG;   // kernel row, or chunk of CM
      static_for<SLOTS>([&](auto s_) {
        constexpr int s = decltype(s_)::value, q = s / GP, gi = step % NSG * GP + s % GP, slot = step * SLOTS + s;
        static_for<IL>([&](auto j_) {
          constexpr int j = IL - 1 - decltype(j_)::value, kw = q - j * S;
          if constexpr (kw >= 0 && kw < KW)
            acc[gi * IL + j] = TR::mfma(fr[s], ring[kh * KW + kw], acc[gi * IL + j]);
          if constexpr (PROJ && kw == 1 && kh == 1) pacc[gi * IL + j] = TR::mfma(fr[s], proj_tap, pacc[gi * IL + j]);
        });
        if constexpr (step + 1 < STEPS) request(pb, std::integral_constant<int, step + 1>{}, s_);
        else if constexpr (!LAST) request(nb, std::integral_constant<int, 0>{}, s_);
        if constexpr (!LAST) {
          static_for<QUOTA>([&](auto k_) {
            constexpr int wk = SC::piece(slot, decltype(k_)::value);
            if constexpr (wk < SC::CELLS)
              store_cell(nb, preg, ch + 1, std::integral_constant<int, wk / VW>{}, std::integral_constant<int, wk % VW>{});
          });
          slot_loads(asrc2, preg, ch + 1, std::integral_constant<int, slot>{});
          // The cells are in LDS when at most the fragments requested behind them are outstanding (the
          // counter ends at 15; a request moved in front of its slot's cells or behind them waits for more).
          if constexpr (slot == SC::BARRIER) {
            constexpr int reads = SC::reads_behind_cells();
            asm volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" ::"n"(reads < 15 ? reads : 15) : "memory");
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    cur = nxt;
  };
  static_for<SLOTS>([&](auto s_) { request(patch, std::integral_constant<int, 0>{}, s_); });
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (!ONE)
    for (int ch = 0; ch + 1 < cnt; ++ch) chunk(std::false_type{}, ch);
  if (KS == 1 || cnt > 0) chunk(std::true_type{}, cnt - 1);
  if constexpr (KS > 1 && !ONE)
    for (int i = cnt > 0 ? cnt : 1; i < most; ++i) lds_barrier();   // the barriers of the chunks that this group does not have
  lds_barrier();                          // every wave is done with the patches

  // ---- write-back: out[(img*O + o)*HWo + p] -----------------------------------------------------
  // SP positions at a time: staged in LDS of the wave's own as [channel][position] rows of 32-bit
  // values (16-byte stores), read back along the rows and written PG positions per lane.
  // (both results one after the other: the staging of one may not meet the reads of the other.  The pointers are values of the
  // closure: read from the arguments, whether there is a residual was asked at every store, 159 waits instead of 100 in 2529
  // instructions instead of 2168; 64 channels at 56x56, batch 32, int8 13.7 -> 12.5 us, bfloat16 15.3 -> 14.8)
  auto write_back = [&](auto& acc, void* out, const void* residual, int relu) {
  constexpr int SP = 32 * (NJ < 4 ? NJ : 4), RS = SP * 4 + 16;
  constexpr int kRed = KS > 1 ? KS * NW * NJ * 4096 : 0;
  uint8_t* const stage = lds + kRed + w * (32 * RS);
  if constexpr (KS > 1) {
    // The groups' partial sums meet in LDS; quads of registers are dealt to the groups' waves, added
    // pairwise (fewer roundings than a chain) and staged.
    static_assert(IL == 1 && SP == 32 * NJ, "a quad is four consecutive positions of the one pass");
    typedef acc_t acc4_t __attribute__((ext_vector_type(4)));
    uint8_t* const red = lds + w * (NJ * 4096) + lane * 16;
    static_for<NJ * 4>([&](auto u_) {
      constexpr int j = decltype(u_)::value / 4, q = decltype(u_)::value % 4;
      const auto v = __builtin_shufflevector(acc[j], acc[j], 4 * q, 4 * q + 1, 4 * q + 2, 4 * q + 3);
      *reinterpret_cast<i32x4*>(red + kg * (NW * NJ * 4096) + (j * 4 + q) * 1024) = __builtin_bit_cast(i32x4, v);
    });
    lds_barrier();
#pragma unroll 1
    for (int u = kg; u < NJ * 4; u += KS) {
      acc4_t t[KS];
#pragma unroll
      for (int k = 0; k < KS; ++k) t[k] = *reinterpret_cast<const acc4_t*>(red + k * (NW * NJ * 4096) + u * 1024);
#pragma unroll
      for (int st = 1; st < KS; st *= 2)
#pragma unroll
        for (int k = 0; k < KS; k += 2 * st) t[k] += t[k + st];
      *reinterpret_cast<i32x4*>(stage + (lane & 31) * RS + (u / 4 * 32 + 8 * (u % 4) + 4 * (lane >> 5)) * 4) =
          __builtin_bit_cast(i32x4, t[0]);
    }
    lds_barrier();
  }
  const int ow = o0 + wo * 32;
  const bool has_res = residual != nullptr;
  // ReLU as one maximum with a run-time operand: zero, or a NaN, which fmaxf ignores.
  const float lo_f = relu ? 0.0f : __builtin_nanf("");
  const int lo_i = relu ? 0 : INT_MIN;
  auto stage_pass = [&](auto ps_) {       // positions ps * SP .. of this wave
    constexpr int ps = decltype(ps_)::value;
    uint8_t* const row = stage + (lane & 31) * RS;
    static_for<SP / 32 / IL>([&](auto gi_) {
      constexpr int gi = decltype(gi_)::value, b = ps * (SP / 32) + gi * IL;
      static_for<16 * IL / 4>([&](auto u_) {              // four consecutive positions: IL blocks x 4 / IL registers
        constexpr int v = decltype(u_)::value * (4 / IL);
        const int n = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        i32x4 t;
        static_for<4>([&](auto e_) {
          constexpr int e = decltype(e_)::value;
          t[e] = __builtin_bit_cast(int32_t, acc_t(acc[b + e % IL][v + e / IL]));
        });
        *reinterpret_cast<i32x4*>(row + (gi * 32 * IL + n * IL) * 4) = t;
      });
    });
  };
  // A group of PG consecutive positions (16 bytes) that lies within one image and the tile goes out
  // with one store per lane, aligned to the element only; the groups that an image's end or the
  // tile's cuts follow value by value, all lanes on one group's 32 x PG values.
  auto write_rows = [&](auto ps_, auto kind_) {
    constexpr int ps = decltype(ps_)::value;
    constexpr int kind = decltype(kind_)::value;           // 0: int32, 1: f32, 2: bf16
    constexpr int PG = kind == 2 ? 8 : 4, LPR = SP / PG, RPI = 64 / LPR, NIT = 32 / RPI;
    const int start = m0 + wpos + ps * SP;                 // first position of the pass
    if (start >= mend) return;
    auto mine = [&](int it) { return KS == 1 || it % KS == kg; };   // steps are dealt to the groups' waves
    const int gq = lane % LPR, rsub = lane / LPR;
    const int m = start + gq * PG;
    const int img = int(g.dHWo.div(uint32_t(m < mend ? m : start))), p = (m < mend ? m : start) - img * g.HWo;
    const bool whole = m + PG <= mend && p + PG <= g.HWo;
    const uint32_t base = whole ? uint32_t(img) * uint32_t(a.O) * uint32_t(g.HWo) + uint32_t(p) : 0u;
    auto addr_of = [&](int it) {
      const int o = ow + it * RPI + rsub;
      return whole && o < a.O ? base + uint32_t(o) * uint32_t(g.HWo) : 0u;
    };
    i32x4 res[NIT];
    if (has_res && int64_t(a.O) * g.M >= PG) {             // (a lane without a group reads the first values)
#pragma unroll
      for (int it = 0; it < NIT; ++it)
        if (mine(it))
          res[it] = *reinterpret_cast<const i32x4_bytes*>(static_cast<const uint8_t*>(residual) +
                                                          int64_t(addr_of(it)) * (kind == 2 ? 2 : 4));
    }
    i32x4 raw[NIT][PG / 4];
#pragma unroll
    for (int it = 0; it < NIT; ++it)
#pragma unroll
      for (int h = 0; h < PG / 4; ++h)
        if (mine(it)) raw[it][h] = *reinterpret_cast<const i32x4*>(stage + (it * RPI + rsub) * RS + (gq * PG + h * 4) * 4);
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      if (!mine(it)) continue;
      const bool ok = whole && ow + it * RPI + rsub < a.O;
      i32x4_bytes* const dst =
          reinterpret_cast<i32x4_bytes*>(static_cast<uint8_t*>(out) + int64_t(addr_of(it)) * (kind == 2 ? 2 : 4));
      i32x4 r;
      if constexpr (kind == 0) {
        r = raw[it][0];
        if (has_res) r += res[it];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = r[e] > lo_i ? r[e] : lo_i;
      } else {
        float f[PG];
#pragma unroll
        for (int e = 0; e < PG; ++e) f[e] = __int_as_float(raw[it][e / 4][e % 4]);
        if (has_res) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if constexpr (kind == 1) {
              f[e] += __int_as_float(res[it][e]);
            } else {
              f[2 * e] += __uint_as_float(uint32_t(res[it][e]) << 16);
              f[2 * e + 1] += __uint_as_float(uint32_t(res[it][e]) & 0xffff0000u);
            }
          }
        }
#pragma unroll
        for (int e = 0; e < PG; ++e) f[e] = fmaxf(f[e], lo_f);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          r[e] = kind == 1 ? __float_as_int(f[e]) : int32_t(pack_bf16x2(f[2 * e % PG], f[(2 * e + 1) % PG]));
      }
      if (ok) *dst = r;
    }
    // cut groups: where an image or the tile ends inside a group
    if (((g.HWo | g.tps) & (PG - 1)) == 0) return;         // uniform
    const int len = mend - start < SP ? mend - start : SP;
    const int img0 = int(g.dHWo.div(uint32_t(start)));
    for (int end = (img0 + 1) * g.HWo - start;; end += g.HWo) {      // uniform
      const int cut = end < len ? end : len;
      if (cut % PG != 0) {
        const int gpos = cut / PG * PG, e = lane % PG, mm = start + gpos + e;
        const int im = int(g.dHWo.div(uint32_t(mm < mend ? mm : start)));
        const uint32_t at = uint32_t(im) * uint32_t(a.O) * uint32_t(g.HWo) + uint32_t(mm - im * g.HWo);
#pragma unroll
        for (int it = 0; it < PG / 2; ++it) {
          const int row = it * (64 / PG) + lane / PG;
          if (mine(it) && mm < mend && ow + row < a.O)
            store_result<acc_t>(out, residual, a.out_dtype, at + uint32_t(ow + row) * uint32_t(g.HWo),
                                *reinterpret_cast<const acc_t*>(stage + row * RS + (gpos + e) * 4), relu);
        }
      }
      if (end >= len) break;
    }
  };
  static_for<32 * NJ / SP>([&](auto ps_) {
    if constexpr (KS == 1) stage_pass(ps_);
    if constexpr (INT) write_rows(ps_, std::integral_constant<int, 0>{});
    else if (a.out_dtype == GS_BF16) write_rows(ps_, std::integral_constant<int, 2>{});
    else write_rows(ps_, std::integral_constant<int, 1>{});
  });
  };
  write_back(acc, a.out, a.residual, a.relu);
  if constexpr (PROJ) {
    lds_barrier();
    write_back(pacc, a.out_proj, nullptr, 0);
  }
}

}  // namespace gs
