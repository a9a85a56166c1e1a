// Split launch lists of random problems: each item's tiles are covered once by its units, in
// order; parts are numbered without gaps; the merges name them; the list
// fits its workspace region.  And the plan images: what a forward's upload writes is what the
// complete plan has there.  And the no-allocation call's array, for the largest problems it takes; and a split that would need a second round.  Built with g++ (no GPU code) by tests/test_split_units.py.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <map>
#include <random>
#include <vector>

#include "plan.h"

using namespace hydra;

namespace {
std::mt19937_64 rng(11);
int64_t uni(int64_t lo, int64_t hi) { return std::uniform_int_distribution<int64_t>(lo, hi)(rng); }
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s (trial %d)\n", #x, trial); return 1; } } while (0)
}  // namespace

int main() {
  int split = 0, whole = 0;
  for (int trial = 0; trial < 600; ++trial) {
    const int n_docs = int(uni(1, 6));
    std::vector<int32_t> cu(size_t(n_docs) + 1, 0);
    for (int d = 0; d < n_docs; ++d) cu[size_t(d) + 1] = cu[size_t(d)] + int32_t(uni(0, trial % 3 ? 3000 : 20000));
    hydra_problem_t p{};
    const int grp = int(uni(1, 4));
    p.n_kv_heads = int32_t(uni(1, 6));
    p.n_heads = p.n_kv_heads * grp;
    p.d_qk = 192;
    p.d_v = 128;
    p.cu_seqlens = cu.data();
    p.n_docs = n_docs;
    for (hydra_chunk_t* c : {&p.q, &p.kv}) {
      c->n_segs = int32_t(uni(1, 3));
      for (int s = 0; s < c->n_segs; ++s) {
        const int64_t a = uni(0, cu.back()), b = uni(a, cu.back());
        c->start[s] = int32_t(a);
        c->len[s] = int32_t(b - a);
      }
    }
    Problem pr;
    CHECK(check_problem(&p, &pr) == HYDRA_OK);
    const WsLayout w = ws_layout(pr);
    PlanImage all, bwd, fwd, whole_only;
    plan_image(pr, w, PlanFor::kStoredDs, true, &all);
    plan_image(pr, w, PlanFor::kBackward, true, &bwd);
    plan_image(pr, w, PlanFor::kForward, true, &fwd);
    plan_image(pr, w, PlanFor::kStoredDs, false, &whole_only);
    CHECK(bwd.off >= all.off && bwd.off + bwd.bytes.size() == all.off + all.bytes.size());
    CHECK(std::equal(bwd.bytes.begin(), bwd.bytes.end(), all.bytes.begin() + int64_t(bwd.off - all.off)));
    CHECK(bwd.kv.units_off == all.kv.units_off && bwd.dq.units_off == all.dq.units_off && bwd.fwd.units_off == all.fwd.units_off);
    CHECK(all.off + all.bytes.size() <= w.d_off && fwd.off >= all.off);
    CHECK(fwd.off + fwd.bytes.size() <= all.off + all.bytes.size());
    CHECK(std::equal(fwd.bytes.begin(), fwd.bytes.end(), all.bytes.begin() + int64_t(fwd.off - all.off)));
    CHECK(fwd.fwd.units == all.fwd.units && fwd.fwd.units_off == all.fwd.units_off && fwd.dq.units + fwd.kv.units == 0);
    CHECK(fwd.fwd.merges == all.fwd.merges && fwd.fwd.merges_off == all.fwd.merges_off);
    CHECK(whole_only.off == all.off && whole_only.bytes.size() <= all.bytes.size());
    CHECK(std::equal(whole_only.bytes.begin(), whole_only.bytes.end(), all.bytes.begin()));
    CHECK(whole_only.fwd.units + whole_only.dq.units + whole_only.kv.units == 0);
    CHECK(split_scratch_bytes(pr) == std::max(parts_bytes(Kernel::kFwd, all.fwd, pr.H),
                                              parts_bytes(Kernel::kDkdv, all.kv, pr.Hkv) + parts_bytes(Kernel::kDq, all.dq, pr.H)));
    size_t list_bytes = 0;
    Ahead ahead;  // dQ goes behind dK/dV
    for (Kernel k : {Kernel::kFwd, Kernel::kDkdv, Kernel::kDq}) {
      std::vector<int32_t> items, rec;
      plan_items(pr, k == Kernel::kDkdv ? 1 : 0, &items);
      launch_units(pr, k == Kernel::kDkdv ? 1 : 0, items, {}, &rec);
      const int heads = k == Kernel::kDkdv ? pr.Hkv : pr.H;
      const int64_t rows = k == Kernel::kFwd ? FWD_TILE_ROWS : k == Kernel::kDq ? DQ_TILE_ROWS : KV_QTILE_ROWS;
      UnitList l;
      split_units(pr, k, rec, heads, &l, ahead);
      if (k == Kernel::kDkdv) {
        ahead = launch_load(pr, k, rec, heads, l);
        const size_t groups = (l.units.empty() ? rec : l.units).size() / kUnitInts * size_t(heads);
        CHECK(ahead.groups == int64_t(groups) && ahead.merges == !l.merges.empty());
        CHECK(ahead.shortest <= ahead.longest && ahead.longest * double(groups) >= ahead.sum);
      }
      if (l.units.empty()) {
        CHECK(l.merges.empty() && l.parts == 0);
        ++whole;
        continue;
      }
      ++split;
      CHECK(l.parts * heads <= MAX_PARTS && l.parts >= 2);
      list_bytes += (l.merges.size() * 4 + 255) / 256 * 256 + (l.units.size() * 4 + 255) / 256 * 256;
      CHECK(w.lists_off + list_bytes <= w.d_off);
      CHECK(l.merges.size() <= size_t(kMaxMerges) * kMergeInts);
      const ListSize& z = k == Kernel::kFwd ? all.fwd : k == Kernel::kDq ? all.dq : all.kv;
      CHECK(z.parts == l.parts && size_t(z.units) * kUnitInts == l.units.size());
      // the units of every item, by first row, in the order of their tiles
      std::map<int32_t, std::vector<const int32_t*>> by_row;
      for (size_t i = 0; i < l.units.size(); i += kUnitInts) by_row[l.units[i]].push_back(&l.units[i]);
      std::vector<int> used(size_t(l.parts), 0);
      int64_t longest = 0, last = INT64_MAX;
      for (size_t i = 0; i < l.units.size(); i += kUnitInts) {  // heaviest first
        const int32_t* u = &l.units[i];
        int64_t t = 0;
        for (int r = 0; r < u[3]; ++r) t += (u[4 + 3 * r + 2] + rows - 1) / rows;
        if (k == Kernel::kDkdv) t *= pr.H / pr.Hkv;
        const int64_t n = (u[REC_T1] < 0 ? t : u[REC_T1]) - u[REC_T0];
        CHECK(n <= last);
        last = n;
        longest = std::max(longest, n);
      }
      size_t n_merges = 0;
      for (size_t i = 0; i < rec.size(); i += kUnitInts) {
        const int32_t* it = &rec[i];
        auto& us = by_row[it[0]];
        CHECK(!us.empty());
        for (const int32_t* u : us) CHECK(std::equal(it, it + REC_T0, u));
        std::sort(us.begin(), us.end(), [](const int32_t* a, const int32_t* b) { return a[REC_T0] < b[REC_T0]; });
        if (us.size() == 1) {
          CHECK(us[0][REC_T0] == 0 && us[0][REC_T1] == -1 && us[0][REC_PART] == -1);
          continue;
        }
        int64_t t = 0;
        for (int r = 0; r < it[3]; ++r) t += (it[4 + 3 * r + 2] + rows - 1) / rows;
        if (k == Kernel::kDkdv) t *= pr.H / pr.Hkv;
        int32_t next = 0;
        for (size_t j = 0; j < us.size(); ++j) {
          CHECK(us[j][REC_T0] == next && us[j][REC_T1] > next && us[j][REC_PART] == us[0][REC_PART] + int32_t(j));
          next = us[j][REC_T1];
          ++used[size_t(us[j][REC_PART])];
        }
        CHECK(next == t);
        bool named = false;
        for (size_t g = 0; g < l.merges.size(); g += kMergeInts)
          if (l.merges[g] == it[0])
            named = l.merges[g + 1] == it[2] && l.merges[g + 2] == us[0][REC_PART] && l.merges[g + 3] == int32_t(us.size());
        CHECK(named);
        ++n_merges;
      }
      CHECK(n_merges * kMergeInts == l.merges.size());
      CHECK(std::all_of(used.begin(), used.end(), [](int x) { return x == 1; }));
    }
  }
  // 192 workgroups of 128 and of 64 tiles, which 96 of the longer ones cut in two would make two
  // rounds of the chip: whole
  {
    const int trial = -1;
    int32_t cu[2] = {0, 16384};
    hydra_problem_t p{};
    p.n_heads = 6;
    p.n_kv_heads = 3;
    p.d_qk = 192;
    p.d_v = 128;
    p.cu_seqlens = cu;
    p.n_docs = 1;
    p.q = {2, {4096, 12288}, {4096, 4096}};
    p.kv = {2, {0, 8192}, {4096, 4096}};
    Problem pr;
    CHECK(check_problem(&p, &pr) == HYDRA_OK);
    PlanImage img;
    plan_image(pr, ws_layout(pr), PlanFor::kBackward, true, &img);
    CHECK(img.fwd.units == 0);
  }
  // the no-allocation call's array at its limit: the most rows that are accepted, where the query
  // side, the key side or the documents take it, in one segment or four with short last tiles
  for (int trial = 0; trial < 200; ++trial) {
    std::vector<int32_t> cu(size_t(trial % 20 == 3 ? uni(1, 4000000) : 1) + 1, 0);
    cu.back() = 1 << 30;
    hydra_problem_t p{};
    p.n_heads = trial % 5 ? int32_t(uni(1, 64)) : 1;
    p.d_qk = 192;
    p.d_v = 128;
    p.cu_seqlens = cu.data();
    p.n_docs = int32_t(cu.size()) - 1;
    const bool by_keys = trial % 2;
    hydra_chunk_t &a = by_keys ? p.kv : p.q, &b = by_keys ? p.q : p.kv;
    a.n_segs = b.n_segs = trial % 3 ? 4 : 1;
    for (int s = 0; s < b.n_segs; ++s) b.len[s] = int32_t(uni(0, 300));
    auto bytes = [&](int64_t rows) {
      for (int s = 1; s < a.n_segs; ++s) a.len[s] = trial % 7 ? 1 : 257;
      a.len[0] = int32_t(rows);
      Problem pr;
      return check_problem(&p, &pr) == HYDRA_OK ? noalloc_bytes(pr) : UINT64_MAX;
    };
    int64_t lo = 0, hi = 1 << 29;
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) / 2;
      (bytes(mid) <= kNoAllocLimitBytes ? lo : hi) = mid;
    }
    CHECK(bytes(lo) <= kNoAllocLimitBytes);
    Problem pr;
    CHECK(check_problem(&p, &pr) == HYDRA_OK);
    CHECK(ws_layout(pr, true).total <= kNoAllocLimitBytes + kNoAllocExtraBytes);
    CHECK(lo > 1000);
  }
  std::printf("split %d whole %d\n", split, whole);
  return 0;
}
