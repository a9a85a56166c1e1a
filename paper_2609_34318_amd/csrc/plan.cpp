// Host-side argument checks and work planning for one ring step.
//
// The plan cuts each side of a ring step into tiles that never straddle a segment, so
// the rows of a tile are consecutive global positions.  For a query tile with positions
// [a, b] the visible keys form one contiguous position interval, [doc_start(a), b]: the
// union over its rows p of [doc_start(p), p] has no gaps because document starts only
// grow with p.  Symmetrically, a key tile [a, b] is seen by the query interval
// [a, doc_end(b) - 1].  Intersecting that interval with each segment of the other chunk
// gives at most HYDRA_MAX_SEGS contiguous ranges of local rows; anything outside them is
// masked (Sec. 2.2) and is never visited.  Tiles are ordered heaviest first, the
// kernel-level counterpart of the scheduler placing the longest sequences first
// (Sec. 5.1.1, Alg. 1, phase 2).
#include "plan.h"

#include "tiles.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>

namespace hydra {

namespace {

constexpr int64_t kMaxRows = int64_t(1) << 30;

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

int64_t chunk_rows(const hydra_chunk_t& c) {
  int64_t n = 0;
  for (int s = 0; s < c.n_segs; ++s) n += c.len[s];
  return n;
}

int check_chunk(const hydra_chunk_t& c, int64_t total) {
  if (c.n_segs < 0 || c.n_segs > HYDRA_MAX_SEGS) return HYDRA_ERR_INVALID;
  for (int s = 0; s < c.n_segs; ++s) {
    if (c.start[s] < 0 || c.len[s] < 0) return HYDRA_ERR_INVALID;
    if (int64_t(c.start[s]) + c.len[s] > total) return HYDRA_ERR_INVALID;
  }
  return HYDRA_OK;
}

// Index d with cu[d] <= pos < cu[d+1] (pos inside the packed window).
int doc_index(const std::vector<int32_t>& cu, int64_t pos) {
  auto it = std::upper_bound(cu.begin(), cu.end(), int32_t(pos));
  return int(it - cu.begin()) - 1;
}

struct Tile {
  int32_t row0, pos0, n;
};

void tiles_of(const hydra_chunk_t& c, int rows_per_tile, std::vector<Tile>* out) {
  int32_t row = 0;
  for (int s = 0; s < c.n_segs; ++s) {
    for (int32_t t = 0; t < c.len[s]; t += rows_per_tile)
      out->push_back({row + t, c.start[s] + t, std::min<int32_t>(rows_per_tile, c.len[s] - t)});
    row += c.len[s];
  }
}

int64_t n_tiles(const hydra_chunk_t& c, int rows_per_tile) {
  int64_t n = 0;
  for (int s = 0; s < c.n_segs; ++s) n += (c.len[s] + rows_per_tile - 1) / rows_per_tile;
  return n;
}

// Ranges of local rows of chunk `c` whose positions fall in [lo, hi] (inclusive).
int ranges_in(const hydra_chunk_t& c, int64_t lo, int64_t hi, int32_t* dst) {
  int n = 0;
  int32_t row = 0;
  for (int s = 0; s < c.n_segs; ++s) {
    int64_t a = std::max<int64_t>(lo, c.start[s]);
    int64_t b = std::min<int64_t>(hi, int64_t(c.start[s]) + c.len[s] - 1);
    if (a <= b) {
      dst[3 * n + 0] = row + int32_t(a - c.start[s]);
      dst[3 * n + 1] = int32_t(a);
      dst[3 * n + 2] = int32_t(b - a + 1);
      ++n;
    }
    row += c.len[s];
  }
  return n;
}

// Pairs (p, k) with p in [qa, qb), k in [ka, kb), k <= p.
int64_t causal_pairs(int64_t qa, int64_t qb, int64_t ka, int64_t kb) {
  if (qb <= qa || kb <= ka) return 0;
  int64_t total = 0;
  int64_t a = std::max(qa, ka), b = std::min(qb, kb);
  if (b > a) {
    int64_t hi = b - ka, lo = a - ka;  // sum of x for x in (lo, hi]
    total += hi * (hi + 1) / 2 - lo * (lo + 1) / 2;
  }
  int64_t full = qb - std::max(qa, kb);
  if (full > 0) total += full * (kb - ka);
  return total;
}

}  // namespace

int check_problem(const hydra_problem_t* p, Problem* out) {
  if (!p || !out) return HYDRA_ERR_INVALID;
  if (p->n_heads <= 0 || p->n_heads > 4096) return HYDRA_ERR_INVALID;
  if (p->d_qk <= 0 || p->d_v <= 0) return HYDRA_ERR_INVALID;
  if (p->d_qk != kDqk || p->d_v != kDv) return HYDRA_ERR_UNSUPPORTED;
  if (!std::isfinite(p->softmax_scale)) return HYDRA_ERR_INVALID;
  if (!p->cu_seqlens || p->n_docs < 1) return HYDRA_ERR_INVALID;
  if (p->cu_seqlens[0] != 0) return HYDRA_ERR_INVALID;
  for (int d = 0; d < p->n_docs; ++d)
    if (p->cu_seqlens[d + 1] < p->cu_seqlens[d]) return HYDRA_ERR_INVALID;
  const int64_t total = p->cu_seqlens[p->n_docs];
  int rc = check_chunk(p->q, total);
  if (rc != HYDRA_OK) return rc;
  rc = check_chunk(p->kv, total);
  if (rc != HYDRA_OK) return rc;
  const int64_t nq = chunk_rows(p->q), nk = chunk_rows(p->kv);
  if (nq > kMaxRows || nk > kMaxRows) return HYDRA_ERR_INVALID;
  if (nq * p->n_heads * kDqk >= (int64_t(1) << 40) || nk * p->n_heads * kDqk >= (int64_t(1) << 40))
    return HYDRA_ERR_INVALID;
  const int hkv = p->n_kv_heads == 0 ? p->n_heads : p->n_kv_heads;
  if (hkv < 0 || hkv > p->n_heads || p->n_heads % hkv != 0) return HYDRA_ERR_INVALID;
  if (nk * hkv * kDqk >= (int64_t(1) << 40)) return HYDRA_ERR_INVALID;
  // The attention launches have one 512-lane workgroup per (tile, head), and a dispatch
  // holds fewer than 2^32 lanes.
  int64_t nqt = 0, nkt = 0;
  for (int s = 0; s < p->q.n_segs; ++s) nqt += (p->q.len[s] + kQTile - 1) / kQTile;
  for (int s = 0; s < p->kv.n_segs; ++s) nkt += (p->kv.len[s] + kKvTile - 1) / kKvTile;
  if (nqt * p->n_heads >= (int64_t(1) << 23) || nkt * hkv >= (int64_t(1) << 23)) return HYDRA_ERR_INVALID;
  // token-row strides: 0 = dense; else >= dense, a multiple of 8 (16-byte rows), < 2^22
  auto stride = [](int32_t s, int64_t dense, int* dst) {
    if (s == 0) s = int32_t(dense);
    if (s < dense || s % 8 != 0 || s >= (1 << 22)) return false;
    *dst = s;
    return true;
  };
  if (!stride(p->q_tok_stride, int64_t(p->n_heads) * kDqk, &out->q_s) ||
      !stride(p->k_tok_stride, int64_t(hkv) * kDqk, &out->k_s) ||
      !stride(p->v_tok_stride, int64_t(hkv) * kDv, &out->v_s))
    return HYDRA_ERR_INVALID;
  if (nq * out->q_s >= (int64_t(1) << 40) || nk * out->k_s >= (int64_t(1) << 40)) return HYDRA_ERR_INVALID;
  out->H = p->n_heads;
  out->Hkv = hkv;
  out->scale = p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / std::sqrt(float(kDqk));
  out->cu.assign(p->cu_seqlens, p->cu_seqlens + p->n_docs + 1);
  out->q = p->q;
  out->kv = p->kv;
  out->nq = nq;
  out->nk = nk;
  return HYDRA_OK;
}

void plan_items(const Problem& pr, int which, std::vector<int32_t>* items) {
  const hydra_chunk_t& own = which == 0 ? pr.q : pr.kv;
  const hydra_chunk_t& other = which == 0 ? pr.kv : pr.q;
  std::vector<Tile> tiles;
  tiles_of(own, which == 0 ? kQTile : kKvTile, &tiles);
  const size_t n = tiles.size();
  std::vector<int32_t> raw(n * kItemInts, 0);
  std::vector<int64_t> cost(n, 0);
  for (size_t i = 0; i < n; ++i) {
    const Tile& t = tiles[i];
    int32_t* it = &raw[i * kItemInts];
    it[0] = t.row0;
    it[1] = t.pos0;
    it[2] = t.n;
    const int64_t first = t.pos0, last = int64_t(t.pos0) + t.n - 1;
    int64_t lo, hi;
    if (which == 0) {  // keys seen by queries [first, last]
      lo = pr.cu[doc_index(pr.cu, first)];
      hi = last;
    } else {           // queries that see keys [first, last]
      lo = first;
      hi = int64_t(pr.cu[doc_index(pr.cu, last) + 1]) - 1;
    }
    it[3] = ranges_in(other, lo, hi, it + 4);
    for (int r = 0; r < it[3]; ++r) cost[i] += it[4 + 3 * r + 2];
  }
  std::vector<size_t> order(n);
  std::iota(order.begin(), order.end(), size_t(0));
  std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return cost[a] > cost[b]; });
  items->resize(n * kItemInts);
  for (size_t i = 0; i < n; ++i)
    std::copy(&raw[order[i] * kItemInts], &raw[order[i] * kItemInts] + kItemInts, &(*items)[i * kItemInts]);
}

void launch_units(const Problem& pr, int which, const std::vector<int32_t>& items,
                  const std::vector<int32_t>& kbase, std::vector<int32_t>* units) {
  const size_t n = items.size() / kItemInts;
  units->assign(n * kUnitInts, 0);
  for (size_t i = 0; i < n; ++i) {
    const int32_t* it = &items[i * kItemInts];
    int32_t* u = &(*units)[i * kUnitInts];
    std::copy(it, it + kItemInts, u);
    const int d0 = doc_index(pr.cu, it[1]), d1 = doc_index(pr.cu, int64_t(it[1]) + it[2] - 1);
    u[REC_EDGE] = which == 0 ? pr.cu[d0] : pr.cu[d0 + 1];
    u[REC_DOC0] = d0;
    u[REC_DOC1] = d1;
    u[REC_T1] = u[REC_PART] = -1;
    if (!kbase.empty()) u[REC_SLOT] = kbase[i];
  }
}

namespace {

constexpr int kCus = 256;

// In tiles of the kernel's loop: what a workgroup costs besides its tiles (its own rows in, the
// first copies, its rows out), and what a split is charged for its merge.  Measured, 2.4 GHz: a
// forward tile takes 1.6 to 1.7 us, a dQ tile 3.0 us, a dK/dV tile 2.5 to 2.9 us; a workgroup's own
// cost 4 to 6 us.  A merge takes longer than it is charged, by its parts (least squares over 150
// windows and ring steps, whole and in up to 32 parts an item: forward 4.6 us and 0.047 us a part of
// 132 KB, dK/dV 2.4 us and 0.060 us a part of 160 KB, so up to 17 and 18 us), but charged by the part
// the choices got worse where dQ fills the chip beside dK/dV (1.5K rows of 16 heads on 2: 81 to
// 114 us; recompute backward over the windows 3% slower, the forward and the stored-dS backward 1%
// faster).
struct SplitCost {
  double group, merge;
};
SplitCost split_cost(Kernel k) {
  return k == Kernel::kFwd ? SplitCost{3.0, 4.0} : SplitCost{2.0, 2.5};
}

// Parts are of four tiles and more; items of fewer than eight stay whole.
constexpr int64_t kMinPart = 4;

int tile_rows(Kernel k) { return k == Kernel::kFwd ? FWD_TILE_ROWS : k == Kernel::kDq ? DQ_TILE_ROWS : KV_QTILE_ROWS; }

int64_t record_tiles(const Problem& pr, Kernel kernel, const int32_t* u) {
  const int rows = tile_rows(kernel);
  int64_t t = 0;
  for (int r = 0; r < u[3]; ++r) t += (u[4 + 3 * r + 2] + rows - 1) / rows;
  return kernel == Kernel::kDkdv ? t * (pr.H / pr.Hkv) : t;
}

}  // namespace

Ahead launch_load(const Problem& pr, Kernel kernel, const std::vector<int32_t>& records, int heads, const UnitList& list) {
  Ahead a;
  const std::vector<int32_t>& units = list.units.empty() ? records : list.units;
  const double group = split_cost(kernel).group;
  for (size_t i = 0; i < units.size(); i += kUnitInts) {
    const int32_t* u = &units[i];
    const double t = group + double(u[REC_T1] < 0 ? record_tiles(pr, kernel, u) : u[REC_T1] - u[REC_T0]);
    a.sum += t * heads;
    a.longest = std::max(a.longest, t);
    a.shortest = i == 0 ? t : std::min(a.shortest, t);
  }
  a.groups = int64_t(units.size()) / kUnitInts * heads;
  a.merges = !list.merges.empty();
  return a;
}

void split_units(const Problem& pr, Kernel kernel, const std::vector<int32_t>& records, int heads, UnitList* out,
                 const Ahead& ahead) {
  *out = UnitList{};
  const int64_t n = int64_t(records.size()) / kUnitInts;
  if (n == 0 || heads <= 0 || n * heads >= kSplitBelow) return;
  std::vector<int64_t> tiles(static_cast<size_t>(n));
  int64_t longest = 0;
  for (int64_t i = 0; i < n; ++i) {
    tiles[size_t(i)] = record_tiles(pr, kernel, &records[size_t(i) * kUnitInts]);
    longest = std::max(longest, tiles[size_t(i)]);
  }
  if (longest < 2 * kMinPart) return;
  // The launch's time with items of more than `most` tiles cut into near-equal parts: one round
  // ends with its longest workgroup; several are filled evenly but for about half a workgroup, and
  // take no less than the shortest of the longest workgroups that must share a CU: two of 257, three
  // of 513 (16K ring step of 6 heads: 192 workgroups of 128 and 64 tiles take 246 us, as 288 of 64
  // tiles, which an even share puts at 0.8 times that, 273).
  // Behind a full round of others the first workgroup starts when the shortest of those ends; and
  // where those are merged, a merge is no launch of its own.  (2K rows x 16 heads: dQ alone took
  // 240 parts to fill the chip; behind dK/dV its 128 whole items do.)
  const SplitCost cost = split_cost(kernel);
  auto parts_of = [](int64_t t, int64_t most) { return t > most ? (t + most - 1) / most : int64_t(1); };
  auto time_of = [&](int64_t most, int64_t* parts) {
    int64_t units = 0;
    double sum = 0, top = 0;
    *parts = 0;
    for (int64_t t : tiles) {
      const int64_t k = parts_of(t, most);
      units += k;
      if (k > 1) *parts += k;
      sum += double(t) + double(k) * cost.group;
      top = std::max(top, double((t + k - 1) / k) + cost.group);
    }
    if (ahead.groups + units * heads <= kCus) return std::max(top, ahead.longest);
    const double start = ahead.groups >= kCus ? ahead.shortest : 0;
    double t = std::max({start + top, ahead.longest, (ahead.sum + sum * heads) / kCus + 0.5 * sum / double(units)});
    if (ahead.groups > 0) return t;
    // workgroups by length, in 128 steps
    int64_t count[128] = {}, more = 0;
    for (int64_t x : tiles) {
      const int64_t k = parts_of(x, most);
      count[int(127 * (double(x) / double(k) + cost.group) / top)] += k * heads;
    }
    int b = 127;
    for (int64_t r = 1; r * kCus < units * heads; ++r) {
      while (more + count[b] <= r * kCus) more += count[b--];
      t = std::max(t, double(r + 1) * top * b / 127);
    }
    return t;
  };
  int64_t parts = 0, best_most = longest;
  double best = time_of(longest, &parts);
  for (int d = 2; d <= 32; ++d) {
    const int64_t most = (longest + d - 1) / d;
    if (most < kMinPart) break;
    const double t = time_of(most, &parts) + (ahead.merges ? 0 : cost.merge);
    if (parts * heads > MAX_PARTS) break;
    if (t < best) {
      best = t;
      best_most = most;
    }
  }
  if (best_most == longest) return;
  std::vector<std::pair<int64_t, size_t>> order;  // tiles, unit
  for (int64_t i = 0; i < n; ++i) {
    const int32_t* u = &records[size_t(i) * kUnitInts];
    const int64_t t = tiles[size_t(i)], k = parts_of(t, best_most);
    if (k > 1) {
      const int32_t m[kMergeInts] = {u[0], u[2], int32_t(out->parts), int32_t(k)};
      out->merges.insert(out->merges.end(), m, m + kMergeInts);
    }
    for (int64_t j = 0; j < k; ++j) {
      const size_t at = out->units.size();
      out->units.insert(out->units.end(), u, u + kUnitInts);
      out->units[at + REC_T0] = int32_t(t * j / k);
      out->units[at + REC_T1] = k > 1 ? int32_t(t * (j + 1) / k) : -1;
      out->units[at + REC_PART] = k > 1 ? out->parts++ : -1;
      order.push_back({t * (j + 1) / k - t * j / k, at});
    }
  }
  std::stable_sort(order.begin(), order.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
  std::vector<int32_t> sorted;
  sorted.reserve(out->units.size());
  for (const auto& o : order)
    sorted.insert(sorted.end(), out->units.begin() + int64_t(o.second), out->units.begin() + int64_t(o.second) + kUnitInts);
  out->units.swap(sorted);
}

int64_t visible_pairs(const Problem& pr) {
  int64_t total = 0;
  const int n_docs = int(pr.cu.size()) - 1;
  for (int qs = 0; qs < pr.q.n_segs; ++qs) {
    const int64_t qa = pr.q.start[qs], qb = qa + pr.q.len[qs];
    if (qb <= qa) continue;
    for (int ks = 0; ks < pr.kv.n_segs; ++ks) {
      const int64_t ka = pr.kv.start[ks], kb = ka + pr.kv.len[ks];
      if (kb <= ka) continue;
      // documents overlapping the query segment
      int d0 = doc_index(pr.cu, qa), d1 = doc_index(pr.cu, qb - 1);
      for (int d = std::max(d0, 0); d <= d1 && d < n_docs; ++d) {
        const int64_t da = pr.cu[d], db = pr.cu[d + 1];
        total += causal_pairs(std::max(qa, da), std::min(qb, db), std::max(ka, da), std::min(kb, db));
      }
    }
  }
  return total;
}

bool ds_path_applies(const Problem& pr) {
  if (pr.nq == 0 || pr.nk == 0) return false;
  for (const hydra_chunk_t* c : {&pr.q, &pr.kv})
    for (int s = 0; s < c->n_segs; ++s)
      if (c->start[s] % 32 != 0 || c->len[s] % 32 != 0) return false;
  return true;
}

int64_t ds_tables(const Problem& pr, const std::vector<int32_t>& kitems, std::vector<int32_t>* kbase,
                  std::vector<int32_t>* kmap32, std::vector<int32_t>* krec) {
  const int64_t n = int64_t(kitems.size()) / kItemInts;
  kbase->assign(size_t(n), 0);
  kmap32->assign(size_t((pr.nk + 31) / 32), -1);
  krec->assign(size_t(n) * kItemInts, 0);
  std::vector<int64_t> order(static_cast<size_t>(n));
  std::iota(order.begin(), order.end(), int64_t(0));
  std::sort(order.begin(), order.end(),
            [&](int64_t x, int64_t y) { return kitems[size_t(x) * kItemInts] < kitems[size_t(y) * kItemInts]; });
  int64_t slots = 0;
  for (int64_t i = 0; i < n; ++i) {
    const int32_t* it = &kitems[size_t(i) * kItemInts];
    (*kbase)[size_t(i)] = int32_t(slots);
    for (int r = 0; r < it[3]; ++r) slots += (it[4 + 3 * r + 2] + KV_QTILE_ROWS - 1) / KV_QTILE_ROWS;
  }
  for (int64_t j = 0; j < n; ++j) {
    const int64_t i = order[size_t(j)];
    const int32_t* it = &kitems[size_t(i) * kItemInts];
    int32_t* rec = &(*krec)[size_t(j) * kItemInts];
    rec[0] = it[0];
    rec[1] = it[2];
    rec[2] = it[3];
    rec[3] = (*kbase)[size_t(i)];
    for (int r = 0; r < it[3]; ++r) {
      rec[4 + 2 * r] = it[4 + 3 * r];
      rec[5 + 2 * r] = it[6 + 3 * r];
    }
    for (int32_t b = it[0] / 32; b < (it[0] + it[2] + 31) / 32; ++b) (*kmap32)[size_t(b)] = int32_t(j);
  }
  return slots;
}

uint64_t noalloc_bytes(const Problem& pr) {
  const size_t nq = size_t(n_tiles(pr.q, kQTile)), nk = size_t(n_tiles(pr.kv, kKvTile));
  size_t n = 0;
  for (size_t part : {pr.cu.size() * 4, nq * 64, nk * 64, nk * 4, size_t((pr.nk + 31) / 32) * 4, nk * 64,
                      size_t(pr.H) * size_t(pr.nq) * 4, size_t(pr.H) * size_t(pr.nq) * 4})
    n = align_up(n + part, 256);
  return n;
}

WsLayout ws_layout(const Problem& pr, bool noalloc) {
  WsLayout w{};
  const int64_t nqt = n_tiles(pr.q, kQTile), nkt = n_tiles(pr.kv, kKvTile);
  w.n_qitems = nqt;
  w.n_kitems = nkt;
  size_t off = 0;
  w.krec_off = off;
  if (!noalloc) off = align_up(off + size_t(nkt) * kItemInts * sizeof(int32_t), 256);
  w.qslots_off = off;
  if (!noalloc) off = align_up(off + size_t(nqt) * HYDRA_MAX_SEGS * sizeof(int32_t), 256);
  w.kitems_off = off;
  off = align_up(off + size_t(nkt) * kUnitInts * sizeof(int32_t), 256);
  w.cu_off = off;
  off = align_up(off + pr.cu.size() * sizeof(int32_t), 256);
  w.qitems_off = off;
  off = align_up(off + size_t(nqt) * kUnitInts * sizeof(int32_t), 256);
  w.lists_off = off;
  if (!noalloc) off += 3 * kListBytes;
  w.d_off = off;
  off = align_up(off + size_t(pr.H) * size_t(pr.nq) * sizeof(float), 256);
  w.lse2_off = off;
  off = align_up(off + size_t(pr.H) * size_t(pr.nq) * sizeof(float), 256);
  w.total = off;
  return w;
}

void plan_image(const Problem& pr, const WsLayout& w, PlanFor call, bool lists, PlanImage* out) {
  *out = PlanImage{};
  const bool backward = call != PlanFor::kForward;
  out->off = call == PlanFor::kStoredDs ? w.krec_off : backward ? w.kitems_off : w.cu_off;
  auto put = [&](size_t off, const std::vector<int32_t>& v) {
    const size_t at = off - out->off, end = at + v.size() * sizeof(int32_t);
    if (out->bytes.size() < end) out->bytes.resize(end, 0);
    if (!v.empty()) std::memcpy(out->bytes.data() + at, v.data(), v.size() * sizeof(int32_t));
  };
  std::vector<int32_t> qitems, kitems, qrec, krecs;
  plan_items(pr, 0, &qitems);
  launch_units(pr, 0, qitems, {}, &qrec);
  if (backward) {
    std::vector<int32_t> kbase, kmap32, krec;
    plan_items(pr, 1, &kitems);
    ds_tables(pr, kitems, &kbase, &kmap32, &krec);
    if (call == PlanFor::kStoredDs) {
      std::vector<int32_t> qslots(qitems.size() / kItemInts * HYDRA_MAX_SEGS, 0);
      for (size_t i = 0; i < qitems.size() / kItemInts; ++i) {
        const int32_t* it = &qitems[i * kItemInts];
        for (int r = 0; r < it[3]; ++r) qslots[i * HYDRA_MAX_SEGS + size_t(r)] = kmap32[size_t(it[4 + 3 * r]) / 32];
      }
      put(w.krec_off, krec);
      put(w.qslots_off, qslots);
    }
    launch_units(pr, 1, kitems, kbase, &krecs);
    put(w.kitems_off, krecs);
  }
  put(w.cu_off, pr.cu);
  put(w.qitems_off, qrec);
  if (!lists) return;
  // the split lists last, one after another, so that only what is there is copied
  size_t end = w.lists_off;
  auto put_list = [&](Kernel kernel, const std::vector<int32_t>& records, int heads, Ahead* ahead) {
    UnitList l;
    split_units(pr, kernel, records, heads, &l, ahead ? *ahead : Ahead{});
    if (ahead) *ahead = launch_load(pr, kernel, records, heads, l);
    if (l.units.empty()) return ListSize{};
    ListSize z{int(l.units.size()) / kUnitInts, int(l.merges.size()) / kMergeInts, l.parts, 0, 0};
    auto next = [&](const std::vector<int32_t>& v) {
      const size_t at = end;
      put(at, v);
      end = align_up(at + v.size() * sizeof(int32_t), 256);
      return at;
    };
    z.merges_off = next(l.merges);
    z.units_off = next(l.units);
    return z;
  };
  out->fwd = put_list(Kernel::kFwd, qrec, pr.H, nullptr);
  if (backward) {
    // one split whatever the heads of a pass: dK and dV then sum in the same order on every path
    Ahead ahead;
    out->kv = put_list(Kernel::kDkdv, krecs, pr.Hkv, &ahead);
    out->dq = put_list(Kernel::kDq, qrec, pr.H, &ahead);
  }
}

uint64_t parts_bytes(Kernel kernel, const ListSize& l, int heads) {
  const int bytes = kernel == Kernel::kFwd ? FWD_PART_BYTES : kernel == Kernel::kDq ? DQ_PART_BYTES : KV_PART_BYTES;
  return uint64_t(l.parts) * uint64_t(heads) * uint64_t(bytes);
}

uint64_t split_scratch_bytes(const Problem& pr) {
  if (n_tiles(pr.q, kQTile) * pr.H >= kSplitBelow && n_tiles(pr.kv, kKvTile) * pr.Hkv >= kSplitBelow) return 0;
  PlanImage img;
  plan_image(pr, ws_layout(pr), PlanFor::kBackward, true, &img);
  return std::max(parts_bytes(Kernel::kFwd, img.fwd, pr.H),
                  parts_bytes(Kernel::kDkdv, img.kv, pr.Hkv) + parts_bytes(Kernel::kDq, img.dq, pr.H));
}

}  // namespace hydra
