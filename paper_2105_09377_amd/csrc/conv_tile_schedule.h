// The order of work within a chunk of conv_tile_kernel, as numbers: plain C++, so that the kernel takes
// its counts from the same place as a replay of the order without a GPU.
//
// A chunk is STEPS * SLOTS slots.  A slot issues, in this order, the MFMAs of its fragment, the request
// (LDS read) of the fragment that takes its register in the next step, and its share of the other work:
// QUOTA pieces from slot 1 on, first the cells of the next chunk's patch (LDS writes), then the loads of
// the patch after it.  The chunk's one barrier stands behind the last slot of step STEPS - 2.
#pragma once

namespace gs {

// What template parameters mean: see conv_tile_kernel.h.  VW: pixels, and so cells, of a patch item.
template <int ESZ, int KH, int KW, int CM, int S, int IL, int NJ, int VW, int MAXI>
struct TileSchedule {
  static constexpr int G = 16 / ESZ;                      // loads of a patch item: channels per 16-byte cell
  static constexpr int KR = KH * CM;                      // kernel rows, or chunks of CM
  static constexpr int NQ = (IL - 1) * S + KW;            // distinct window columns of IL interleaved blocks
  static constexpr int GP = IL == 1 && NJ > 1 ? 2 : 1;    // block groups that take turns within a step
  static constexpr int NG = NJ / IL, NSG = NG / GP, STEPS = KR * NSG, SLOTS = NQ * GP;
  static constexpr int CELLS = VW * MAXI, LOADS = G * MAXI;
  static constexpr int QUOTA = (CELLS + LOADS + STEPS * SLOTS - 2) / (STEPS * SLOTS - 1);
  static constexpr int BARRIER = SLOTS * (STEPS - 1) - 1; // the slot in front of the barrier

  // Does slot s of a step multiply anything?  With 1x1 windows at stride 2 every second window column lies
  // between two blocks' pixels: its fragment is neither requested nor counted.
  static constexpr bool used(int s) {
    const int q = s / GP;
    for (int j = 0; j < IL; ++j)
      if (q - j * S >= 0 && q - j * S < KW) return true;
    return false;
  }
  // Piece k of a slot: a cell if it is below CELLS, otherwise load piece - CELLS (none past LOADS).
  static constexpr int piece(int slot, int k) { return slot > 0 ? (slot - 1) * QUOTA + k : CELLS + LOADS; }
  static constexpr int last_cell_slot() { return (CELLS + QUOTA - 1) / QUOTA; }
  // LDS reads behind the last cell and in front of the barrier.  Within a slot the request comes first, so
  // the last cell's own slot adds none.  LDS operations of a wave complete in order: once no more than
  // these are outstanding, every cell is in LDS.
  static constexpr int reads_behind_cells() {
    int n = 0;
    for (int slot = last_cell_slot() + 1; slot <= BARRIER; ++slot) n += used(slot % SLOTS) ? 1 : 0;
    return n;
  }
  static_assert(CELLS <= QUOTA * BARRIER, "the cells are written before the barrier");
};

}  // namespace gs
