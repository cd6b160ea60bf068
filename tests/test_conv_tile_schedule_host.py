"""conv_tile_kernel without a GPU.  The chunk barrier: the order of every built instance is replayed from the
numbers that the kernel itself is compiled with, and no patch cell may be outstanding behind the barrier's wait.
The planner: every built instance is reached, and no other."""

import os
import random
import subprocess

import pytest

import tile_instances
from paper_2105_09377_amd import binding as gs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

REPLAY = r"""
#include <cstdio>
#include "conv_tile_schedule.h"
using namespace gs;
// One line: the parameters, the wait's count, then the LDS operations up to the barrier: R a read, W a cell.
template <int ESZ, int K, int CM, int S, int IL, int NJ, int MAXI> void replay() {
  using SC = TileSchedule<ESZ, K, K, CM, S, IL, NJ, 4, MAXI>;
  std::printf("%d %d %d %d %d %d %d ", ESZ, K, S, IL, NJ, MAXI, SC::reads_behind_cells());
  for (int slot = 0; slot < SC::STEPS * SC::SLOTS; ++slot) {
    if (SC::used(slot % SC::SLOTS)) std::printf("R");
    for (int k = 0; k < SC::QUOTA; ++k)
      if (SC::piece(slot, k) < SC::CELLS) std::printf("W");
    if (slot == SC::BARRIER) std::printf("|");
  }
  std::printf("\n");
}
template <int ESZ, int K, int CM, int S, int IL, int NJ> void items() {
  replay<ESZ, K, CM, S, IL, NJ, 1>();
  replay<ESZ, K, CM, S, IL, NJ, 2>();
  if constexpr (NJ <= 2) replay<ESZ, K, CM, S, IL, NJ, 4>();
}
template <int ESZ, int K, int CM, int NJ> void strides() {
  items<ESZ, K, CM, 1, 1, NJ>();
  items<ESZ, K, CM, 2, 1, NJ>();
  if constexpr (NJ >= 2) { items<ESZ, K, CM, 1, 2, NJ>(); items<ESZ, K, CM, 2, 2, NJ>(); }
  if constexpr (NJ >= 4) items<ESZ, K, CM, 1, 4, NJ>();
}
template <int ESZ> void all() {
  strides<ESZ, 1, 4, 4>(); strides<ESZ, 1, 4, 2>(); strides<ESZ, 1, 4, 1>();
  strides<ESZ, 3, 1, 4>(); strides<ESZ, 3, 1, 2>(); strides<ESZ, 3, 1, 1>();
  strides<ESZ, 5, 1, 2>(); strides<ESZ, 5, 1, 1>();
}
int main() { all<1>(); all<2>(); }
"""


def test_every_cell_is_written_before_the_chunk_barrier(tmp_path):
    src, exe = tmp_path / "replay.cpp", tmp_path / "replay"
    src.write_text(REPLAY)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2105_09377_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(lines) == 2 * (2 * (5 * 2 + 4 * 3 + 2 * 3) + 4 * 3 + 2 * 3)
    for line in lines:
        esz, k, stride, il, nj, maxi, reads, ops = line.split()
        before, behind = ops.split("|")
        assert before.count("W") == 4 * int(maxi) and "W" not in behind, line
        # A wave's LDS operations complete in order, so a wait for n leaves at most the last n outstanding; the
        # counter holds 15.  Waiting for fewer than are behind the last cell would only cost time.
        assert int(reads) == len(before) - 1 - before.rindex("W"), line
        assert "W" not in before[len(before) - min(int(reads), 15):], line
        # 3x3 and 5x5 windows use every fragment; two blocks of 1x1 windows at stride 2 use two of three
        per_step = (int(il) - 1) * int(stride) + int(k)
        if k != "1" or stride == "1":
            assert ops.count("R") % per_step == 0, line


@pytest.mark.parametrize("dtype", ["bf16", "i8"])
def test_every_instance_has_a_layer(dtype):
    for k, natural in ((1, False), (1, True), (3, False), (5, False)):
        for shape in tile_instances.SHAPES:
            assert set(tile_instances.layers(dtype, k, natural, shape)) == tile_instances.built(dtype, k, shape), (k, natural, shape)


def test_the_planner_picks_built_instances():
    rng, seen = random.Random(8), set()
    for _ in range(1500):
        dtype, k, s = rng.choice(["bf16", "i8"]), rng.choice([1, 3, 5]), rng.choice([1, 2])
        code, unit = (gs.GS_I8, 32) if dtype == "i8" else (gs.GS_BF16, 16)
        c = unit * (4 if k == 1 else 1) * rng.randint(1, 8)
        x = tile_instances.ap((rng.choice([1, 2, 7, 32]), c, rng.randint(k, 112), rng.randint(k, 112)), 1, code)
        w = tile_instances.ap((16 * rng.randint(1, 32), c, k, k), 1, code)
        st, (shape, *instance, _positions) = tile_instances.call(x, w, s, k // 2, None, 0, None, 0x10000, -1, None)
        if st == gs.GS_OK:
            seen.add(shape)
            assert (s, *instance) in tile_instances.built(dtype, k, shape)
    assert seen == set(tile_instances.SHAPES)


@pytest.mark.parametrize("natural", [False, True])
@pytest.mark.parametrize("dtype,n,c,h,w,o,s", [("i8", 40, 128, 94, 94, 16, 1), ("bf16", 94, 64, 56, 98, 27, 1), ("bf16", 41, 64, 96, 104, 336, 2),
                                               ("i8", 48, 128, 79, 79, 50, 1)])
def test_wide_planes_of_1x1_windows_are_cut_at_row_ends(dtype, n, c, h, w, o, s, natural):
    """Whole rows are staged: a tile that ends within one stages up to three times the pixels that it multiplies."""
    code = gs.GS_I8 if dtype == "i8" else gs.GS_BF16
    st, plan = tile_instances.call(tile_instances.ap((n, c, h, w), 1, code), tile_instances.ap((o, c, 1, 1), 1, code), s, 0, None, 0,
                                   None, None if natural else 0x10000, -1, None)
    assert natural or st == gs.GS_OK        # (in the listing's order the gathered matrix may be the faster way)
    assert st != gs.GS_OK or plan[4] % ((w - 1) // s + 1) == 0


@pytest.mark.parametrize("dtype,n,c,h,w,o,k,s,p", [("i8", 47, 26, 15, 26, 16, 5, 1, 0), ("bf16", 6, 8, 75, 27, 3, 3, 2, 1), ("i8", 7, 22, 12, 29, 110, 3, 2, 0),
                                                   ("bf16", 4, 33, 82, 29, 22, 5, 1, 2), ("bf16", 23, 12, 45, 10, 16, 1, 1, 0), ("i8", 4, 18, 8, 45, 16, 3, 1, 0)])
def test_few_items_per_thread_where_channels_do_not_fill_a_chunk(dtype, n, c, h, w, o, k, s, p):
    """Every patch item clears the channels that it does not have: of these layers a thread with one or two is over in 0.4 to 0.7
    of the time of one with four."""
    code = gs.GS_I8 if dtype == "i8" else gs.GS_BF16
    st, plan = tile_instances.call(tile_instances.ap((n, c, h, w), 1, code), tile_instances.ap((o, c, k, k), 1, code), s, p, None, 0,
                                   None, 0x10000, -1, None)
    assert st == gs.GS_OK and plan[2] <= 2
