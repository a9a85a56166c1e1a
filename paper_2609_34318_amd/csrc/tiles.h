// Tile geometry that the host plan and the kernels must agree on (no HIP types here: the
// plan is also built as plain host C++).
#pragma once

namespace hydra {

// Query rows per tile of the key-stationary backward kernel (three 32-row sub-blocks).  The
// plan lays out the stored dS with it: one slot per (key item, query tile), each slot
// holding the 3 x 4 blocks of 32 queries x 32 keys.
constexpr int KV_QTILE_ROWS = 96;
constexpr int DS_BLOCK_BYTES = 32 * 32 * 2;                               // bf16
constexpr int DS_TILE_BYTES = (KV_QTILE_ROWS / 32) * 4 * DS_BLOCK_BYTES;  // 24 KB

// Tile rows of the other side in each kernel's loop.
constexpr int FWD_TILE_ROWS = 64;
constexpr int DQ_TILE_ROWS = 96;

// Launch records: the 16 ints of a work item, then (launch_units in plan.h)
enum Record {
  REC_EDGE = 16,  // document boundary of the first row: its start for query items, its end for key items
  REC_DOC0,       // document indices of the first and the last row
  REC_DOC1,
  REC_SLOT,       // key items: first dS slot
  REC_T0,         // first tile of the walk and the one past the last (-1: all tiles); for dK/dV of its
  REC_T1,         // group * tiles
  REC_PART,       // part of a split item, or -1
  REC_INTS = 24
};

// A work item split over several workgroups: each leaves its accumulators in a part of the
// caller's scratch, as its registers hold them (one 1 KB row of 64 lanes x 16 bytes per four
// registers).  Per wave: 32 rows x 128 (O, with two more rows for the running max and sum, or
// dV) or x 192 columns (dQ, dK) in fp32.
constexpr int PART_WAVE_128 = 32 * 128 * 4;
constexpr int PART_WAVE_192 = 32 * 192 * 4;
constexpr int PART_WAVE_O = PART_WAVE_128 + 512;
constexpr int FWD_PART_BYTES = 8 * PART_WAVE_O;
constexpr int DQ_PART_BYTES = 8 * PART_WAVE_192;
constexpr int KV_PART_BYTES = 4 * (PART_WAVE_128 + PART_WAVE_192);
// Parts of one launch (over all its heads).
constexpr int MAX_PARTS = 256;

}  // namespace hydra
