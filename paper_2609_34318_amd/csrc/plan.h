// Host-side argument checks and work planning for one ring step (no HIP calls).
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

#include "hydra_attn.h"
#include "tiles.h"

namespace hydra {

constexpr int kDqk = 192;
constexpr int kDv = 128;
constexpr int kQTile = 256;    // query rows per query-stationary workgroup (8 waves x 32)
constexpr int kKvTile = 128;   // key rows per key-stationary workgroup (4 waves x 32)
constexpr int kItemInts = 16;  // int32 per work item
constexpr int kUnitInts = REC_INTS;  // int32 per launch record: a work item and what its kernel would else look up

// Checked and normalised view of a hydra_problem_t.
struct Problem {
  int H = 0;
  int Hkv = 0;  // K/V heads (divides H)
  float scale = 0.f;
  std::vector<int32_t> cu;     // n_docs + 1 boundaries
  hydra_chunk_t q{}, kv{};
  int64_t nq = 0, nk = 0;
  int q_s = 0, k_s = 0, v_s = 0;  // token-row strides of q, k, v in elements
};

// Returns HYDRA_OK or an error status; fills `out` on success.
int check_problem(const hydra_problem_t* p, Problem* out);

// Work items (kItemInts each), heaviest first.  which = 0: query-stationary tiles of
// kQTile rows with their visible key ranges; which = 1: key-stationary tiles of kKvTile
// rows with their visible query ranges.
void plan_items(const Problem& pr, int which, std::vector<int32_t>* items);

int64_t visible_pairs(const Problem& pr);

// The kernel a launch list is for: what a tile of its loop costs, and how many it has.
enum class Kernel { kFwd, kDq, kDkdv };

// A launch list: the records of the units, and of the split items the merges.
struct UnitList {
  std::vector<int32_t> units;   // kUnitInts each, heaviest first; empty: no item is split
  std::vector<int32_t> merges;  // kMergeInts each: the item's first row, rows, first part, parts
  int parts = 0;                // parts per head
};
// What a launch holds ahead of the list that is split, in tiles (a workgroup's own cost included).
struct Ahead {
  int64_t groups = 0;  // workgroups
  double sum = 0, longest = 0, shortest = 0;
  bool merges = false;
};
constexpr int kMergeInts = 4;
constexpr int kMaxMerges = MAX_PARTS / 2;  // a split item has at least two parts
// Workgroups of a launch from which on nothing is split: at two per CU (256) and more the
// heavy-first order fills the chip, and no shape measured there gained.
constexpr int64_t kSplitBelow = 512;
// The most bytes of a split list: its merges, and a unit for every part and every whole item.
constexpr size_t kListBytes = (size_t(kMaxMerges) * kMergeInts + size_t(MAX_PARTS + kSplitBelow) * kUnitInts) * sizeof(int32_t);
static_assert(kListBytes % 256 == 0, "lists end on a region boundary");

// Splits the items of a launch over `heads` heads whose workgroups leave the chip idle (`records`
// from launch_units).  A unit is a record with the tiles of its part, or that of the whole item.
// `ahead`: the workgroups that the same launch starts before these.
void split_units(const Problem& pr, Kernel kernel, const std::vector<int32_t>& records, int heads, UnitList* out,
                 const Ahead& ahead = Ahead{});
// The launch of a list (of the whole `records` when it has no units) as what is ahead of another.
Ahead launch_load(const Problem& pr, Kernel kernel, const std::vector<int32_t>& records, int heads, const UnitList& list);

// The launch records (tiles.h) of plan_items' work items, in the same order, as whole items.  A kernel
// that reads one record instead of searching cu_seqlens has one memory round trip before its first
// copy, not several.  kbase: the first dS slot of each key item (ds_tables).
// `kbase` is empty for query items: their records hold nothing of the key side, so that they are
// the same whether or not the key side is planned (plan_image).
void launch_units(const Problem& pr, int which, const std::vector<int32_t>& items,
                  const std::vector<int32_t>& kbase, std::vector<int32_t>* units);

// Byte offsets of the workspace regions, in this order: what the stored-dS backward alone reads
// (krec, qslots), the key items, what the forward reads too (cu, qitems, and at lists the forward's
// split list), the backward's split lists, D and LSE*log2(e).  lists holds the split lists that a plan has, one after
// another (merges, then units); it has the same size for every problem, so that no problem needs
// more workspace than one with more rows.  For the no-allocation call, which stores no dS and splits
// nothing, those regions are empty.
struct WsLayout {
  size_t krec_off, qslots_off, kitems_off, cu_off, qitems_off, lists_off, d_off, lse2_off, total;
  int64_t n_qitems, n_kitems;
};
WsLayout ws_layout(const Problem& pr, bool noalloc = false);

// A split list in the workspace; no units: the whole items are launched.
struct ListSize {
  int units = 0, merges = 0, parts = 0;
  size_t merges_off = 0, units_off = 0;
};

// What an upload writes: `bytes` at workspace offset `off`.
struct PlanImage {
  size_t off = 0;
  std::vector<char> bytes;
  ListSize fwd, dq, kv;
};
// The calls a plan is for; an upload of up to 16 KB costs some 10 us less than a larger one (ragged 8K
// window: 387 against 397 us for forward and backward), so a call writes what it reads and no more.
enum class PlanFor { kForward, kBackward, kStoredDs };
// lists = false: without the split lists, for a call that launches the whole items.  Every byte of an
// image is a function of the problem alone, and every image a range of the largest: an upload for a
// call on the same problem leaves a plan that a recorded graph still reads as it was.
void plan_image(const Problem& pr, const WsLayout& w, PlanFor call, bool lists, PlanImage* out);

// Bytes of scratch that hold the parts of `l` over `heads` heads.
uint64_t parts_bytes(Kernel kernel, const ListSize& l, int heads);
// Scratch with which every launch of a plan that has split lists uses them (the dK/dV parts, then
// the dQ parts, or the forward's).
uint64_t split_scratch_bytes(const Problem& pr);

// What the no-allocation backward's 32 MiB limit is counted on: D, LSE*log2(e), the documents,
// 64 bytes per query tile, 148 per key tile (128 rows; 4 for each 32 of them), each to 256 bytes.
uint64_t noalloc_bytes(const Problem& pr);
constexpr size_t kNoAllocLimitBytes = size_t(32) << 20;
// A query tile's record takes 32 bytes more than are counted, a key tile's fewer, and a query tile of
// 256 rows counts at least 64 + 256 * 8 (each of the four segments may end in a shorter one): what the
// no-allocation workspace of a problem within the limit takes beyond it is at most
constexpr size_t kNoAllocExtraBytes =
    (kNoAllocLimitBytes / (64 + kQTile * 8) + HYDRA_MAX_SEGS + 1) * (kUnitInts * 4 - 64) / 256 * 256 + 256;

// The stored-dS backward applies when every segment of both chunks starts and ends on a
// multiple of 32 positions: the key-stationary tiles then cut the query rows into 32-row
// blocks that coincide with the query-stationary kernel's per-wave blocks.
bool ds_path_applies(const Problem& pr);

// For the stored-dS backward, from the key items in launch order: kbase[i] = first tile
// slot of item i (slots of 24 KB, one per query tile of the item); the items again in
// row order as records of kItemInts ints, krec[j] = {row0, n, n_ranges, first slot, then
// (first row, rows) of each query range}; kmap32[b] = the row-order index of the item
// holding local key rows [32b, 32b + 32).  Returns the slots per query head.  (qslots, in the
// workspace: per query item, in launch order, the kmap32 entry of the first row of each range.)
int64_t ds_tables(const Problem& pr, const std::vector<int32_t>& kitems, std::vector<int32_t>* kbase,
                  std::vector<int32_t>* kmap32, std::vector<int32_t>* krec);

}  // namespace hydra
