// Backward of one ring step, differentiating with the final merged O and LSE of each row:
//   D_i = <dO_i, O_i>,  P = exp(S - LSE),  dV += P^T dO,  dS = P o (dO V^T - D),
//   dK += scale dS^T Q,  dQ += scale dS K.
// Two kernels:
//   bwd_pre        -D = -rowsum(dO o O) and LSE * log2(e)                (HBM-bound)
//   bwd_recompute  dK/dV workgroups, key-stationary: recompute S and dP per query tile,
//                  accumulate dK^T, dV^T; then dQ workgroups, query-stationary: recompute S^T
//                  and dP^T per key tile, accumulate dQ^T
// or, where dS is stored, bwd_pre, bwd_dkdv_ds and bwd_dq_ds (below).
// Splitting dQ from dK/dV recomputes S and dP once more but needs no atomics and is
// deterministic: every output row is owned by exactly one workgroup.  Both kinds
// stream their other-side tiles through swizzled LDS stages filled by direct
// buffer->LDS copies issued ahead of use.
#include "kernels.h"
#include "prof.h"

namespace hydra {

// ------------------------------------------------------------------ D = rowsum(dO * O)
__global__ __launch_bounds__(256) void bwd_pre_kernel(const uint16_t* __restrict__ o,
                                                      const uint16_t* __restrict__ dO,
                                                      const float* __restrict__ lse,
                                                      float* __restrict__ D, float* __restrict__ lse2,
                                                      int nq, int H) {
  const int sub = threadIdx.x & 15;
  const int64_t total = (int64_t)nq * H;
  // (row, head) pairs, 16 lanes each, strided over a capped grid; the 16 lanes of a pair
  // stay together, so the reduction below always has all of them
  for (int64_t rh = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); rh < total; rh += (int64_t)gridDim.x * 16) {
    const u32x4 uo = ldg16(o + rh * DV + sub * 8);
    const u32x4 ud = ldg16(dO + rh * DV + sub * 8);
    float acc = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      acc += __uint_as_float(uo[w] << 16) * __uint_as_float(ud[w] << 16);
      acc += __uint_as_float(uo[w] & 0xffff0000u) * __uint_as_float(ud[w] & 0xffff0000u);
    }
    acc += __shfl_xor(acc, 8, 16);
    acc += __shfl_xor(acc, 4, 16);
    acc += __shfl_xor(acc, 2, 16);
    acc += __shfl_xor(acc, 1, 16);
    if (sub == 0) {
      const int row = (int)(rh / H), head = (int)(rh % H);
      const int64_t li = (int64_t)head * nq + row;
      D[li] = -acc;
      lse2[li] = lse[li] * LOG2E;
    }
  }
}

// ------------------------------------------------------------------ dQ (query-stationary)
constexpr int DQ_BK = DQ_TILE_ROWS;  // keys per tile: 96 measured faster than 64 and 128
constexpr int DQ_KBYTES = DQ_BK * DQK * 2;            // 36 KB
constexpr int DQ_STAGE = DQ_KBYTES + DQ_BK * DV * 2;  // 60 KB
constexpr int DQ_NSTAGE = 2;  // measured faster than three stages
constexpr int DQ_WAVES = 8;                           // 256 query rows per workgroup
constexpr int DQ_COPY_WAVES = 4;                      // the 12 copies per column block split evenly over 4

__device__ __forceinline__ void dq_issue(lds_char* stage, const AttnArgs& a, const Tile k, int kv_head, int wave) {
  if (wave >= DQ_COPY_WAVES) return;  // wave-uniform
  const int koff = dma_lane_off<DQK>(a.k_s, kv_head, wave, lane_now());
  const int voff = dma_lane_off<DV>(a.v_s, kv_head, wave, lane_now());
  dma_tile<DQK, DQ_BK, DQ_COPY_WAVES>(stage, tile_rsrc(a.k, k.row0, k.n, a.k_s), koff, a.k_s, wave);
  dma_tile<DV, DQ_BK, DQ_COPY_WAVES>(stage + DQ_KBYTES, tile_rsrc(a.v, k.row0, k.n, a.v_s), voff, a.v_s, wave);
}

// stage 0 | stage 1; before the loop the waves' Q, then dO rows from the start of stage 1, after it
// their outputs
constexpr int DQ_LDS = DQ_STAGE + DQ_WAVES * own_bytes<DQK>();
static_assert(DQ_LDS >= DQ_NSTAGE * DQ_STAGE && DQ_LDS >= DQ_WAVES * ROWS_OUT_BYTES, "LDS");

__device__ __forceinline__ void bwd_dq_body(const AttnArgs& a, int block, lds_char* smem) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, known to the compiler
  const int m = lane & 31;
  int hl, item;
  xcd_head_item(block, a.q_heads, a.n_items, hl, item);
  const int head = a.q_head0 + hl;
  const Item it(a.items, item);
  const TileRanges kr = tile_ranges(it, DQ_BK);
  const int t0 = it.t0, n_tiles = (it.t1 < 0 ? kr.nt : it.t1) - t0;  // this unit's tiles
  if (n_tiles == 0) return;  // uniform over the workgroup
  const int kv_head = head / a.grp;  // grouped K/V heads: contiguous groups of query heads
  const float sl2 = a.scale * LOG2E;

  // this wave's rows: [q_row0, q_row0 + q_n) at positions from q_pos0 on (q_n = 0: none)
  const int q_n = min(32, max(it.n - 32 * wave, 0));
  const int q_row0 = it.row0 + 32 * wave, q_pos0 = it.pos0 + 32 * wave;
  const int q_last = q_n > 0 ? q_pos0 + q_n - 1 : -1;

  lds_char* own = smem + DQ_STAGE + wave * own_bytes<DQK>();
  own_rows_issue<DQK>(own, a.q, q_row0, q_n, a.q_s, head, lane);
  Tile cur = tile_at(kr, t0, DQ_BK);
  dq_issue(smem, a, cur, kv_head, wave);
  // rows past the end repeat the last one (an empty wave the item's first row)
  const int mc = q_n > 0 ? min(m, q_n - 1) : -32 * wave;
  float lse2 = a.lse2[(int64_t)head * a.nq + q_row0 + mc];
  float neg_D = a.Dvec[(int64_t)head * a.nq + q_row0 + mc];
  const int lo_q = doc_edge<false>(a.cu, it.d0, it.d1, it.edge0, q_pos0 + mc);
  const int lo_first = __builtin_amdgcn_readfirstlane(lo_q);
  const int lo_last = __builtin_amdgcn_readlane(lo_q, 31);
  settle(lse2);
  settle(neg_D);
  bf16x8 qf[DQK / 16], df[DV / 16];
  wait_dma();
  own_rows_read<DQK>(own, lane, qf);
  own_rows_issue<DV>(own, a.dO, q_row0, q_n, a.H * DV, head, lane);
  wait_dma();
  own_rows_read<DV>(own, lane, df);

  f32x16 acc[DQK / 32];
#pragma unroll
  for (int c = 0; c < DQK / 32; ++c) acc[c] = f32x16{};

  OperandOffsets o = operand_offsets(lane);

  for (int t = 0; t < n_tiles; ++t) {
    refresh(o);
    const int kpos = cur.pos0, kn = cur.n;
    lds_char* Ks = smem + (t % DQ_NSTAGE) * DQ_STAGE;
    lds_char* Vs = Ks + DQ_KBYTES;
    wait_dma();  // tile t's copies, the only ones in flight
    if (kn < DQ_BK && wave < DQ_COPY_WAVES) {
      clear_tail<DQK, DQ_BK, DQ_COPY_WAVES>(Ks, kn, wave, lane_now());
      clear_tail<DV, DQ_BK, DQ_COPY_WAVES>(Vs, kn, wave, lane_now());
    }
    barrier_lds();
    if (t + 1 < n_tiles) {
      cur = tile_at(kr, t0 + t + 1, DQ_BK);
      dq_issue(smem + ((t + 1) % DQ_NSTAGE) * DQ_STAGE, a, cur, kv_head, wave);
    }
    // a wave none of whose rows sees the tile leaves the matrix cores to the others
    if (kpos > q_last || kpos + kn <= lo_first) continue;
    const bool full = (kn == DQ_BK) && (lo_last <= kpos) && (kpos + DQ_BK - 1 <= q_pos0);

    static_for<DQ_BK / 32>([&](auto kb_) {
      constexpr int kb = decltype(kb_)::value;
      f32x16 s = f32x16{}, dp = f32x16{};
#pragma unroll
      for (int t2 = 0; t2 < DQK / 16; ++t2) s = mfma(op_b128<DQ_BK>(Ks, o, 32 * kb, t2), qf[t2], s);
#pragma unroll
      for (int t2 = 0; t2 < DV / 16; ++t2) dp = mfma(op_b128<DQ_BK>(Vs, o, 32 * kb, t2), df[t2], dp);

      float ds[16];
      if (full) {
#pragma unroll
        for (int e = 0; e < 16; ++e) ds[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], sl2, -lse2)) * (dp[e] + neg_D);
      } else {
        // key kpos + key(e) is visible iff lo_q <= it <= pos_q and key(e) < kn, i.e. iff
        // 0 <= base + c(e) < lim with base = kpos - lo_q + 32*kb + 8*hh; masked entries get
        // exp2(-inf) = 0.  pos_q is formed here: this kernel has no register to spare for it.
        const int ml = lane_now();
        const int pos_q = (ml & 31) < q_n ? q_pos0 + (ml & 31) : -1;
        const int base = kpos - lo_q + 32 * kb + 8 * (ml >> 5);
        const int lim = max(0, min(pos_q + 1, kpos + kn) - lo_q);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int r = base + 16 * (e >> 3) + (e & 7);
          const bool vis = (unsigned)r < (unsigned)lim;
          ds[e] = __builtin_amdgcn_exp2f(vis ? __builtin_fmaf(s[e], sl2, -lse2) : -INFINITY) * (dp[e] + neg_D);
        }
      }
      const bf16x8 dsf[2] = {to_bf16x8(ds), to_bf16x8(ds + 8)};

      // dQ^T[c][q] += K^T[c][key] dS^T[key][q]; K^T fragments by LDS transpose reads, three
      // column blocks per group; a group's products are issued before the next group loads.
      bf16x8 f[2][3];
      op_tr_x3<DQ_BK, 32 * kb, 0>(Ks, o, f[0]);
      static_for<4>([&](auto g_) {
        constexpr int gq = decltype(g_)::value, half = gq >> 1, c0 = 3 * (gq & 1);
#pragma unroll
        for (int j = 0; j < 3; ++j) acc[c0 + j] = mfma(f[gq & 1][j], dsf[half], acc[c0 + j]);
        if constexpr (gq + 1 < 4)
          op_tr_x3<DQ_BK, 32 * kb + 16 * ((gq + 1) >> 1), 3 * ((gq + 1) & 1)>(Ks, o, f[(gq + 1) & 1]);
        sched_fence();
      });
    });
  }

  if (it.part >= 0) {
    part_store(part_at(a, hl, it.part, DQ_PART_BYTES) + wave * PART_WAVE_192, lane_now(), acc);
    return;
  }
  barrier_lds();  // every wave is past its last tile
  rows_add<DQK / 64>(smem + wave * ROWS_OUT_BYTES, lane_now(), acc, a.scale, a.dq + ((int64_t)q_row0 * a.H + head) * DQK,
                     a.H * DQK, q_n);
}

// ------------------------------------------------------------------ dK, dV (key-stationary)
// Eight waves share 128 keys as four pairs, one pair per SIMD, 32 keys per pair.  The two
// waves of a pair split the work so that each fits in 256 registers (two waves per SIMD,
// whose matrix and vector work then overlap):
//   wave A: S = Q K^T, P = exp(S - LSE) (masked), dV^T += dO^T P
//   wave B: dP - D = dO V^T - D, dS = P o (dP - D), dK^T += Q^T dS
// P crosses from A to B through LDS (rounded to bf16, the value the dV product uses).  Per
// 96-query tile: barrier, start the copy of the next tile (LDS holds two), phase 1 (A: S
// and P, B: dP - D), barrier, phase 2 (A: dV, B: dS and dK).
constexpr int KV_BQ = KV_QTILE_ROWS;                             // query rows per tile
constexpr int KV_NSB = KV_BQ / 32;                               // 32-row sub-blocks per tile
constexpr int KV_VEC = 128;                                      // LDS slots per vector (LSE2, D)
constexpr int KV_QBYTES = KV_BQ * DQK * 2;                       // 36 KB
constexpr int KV_OBYTES = KV_BQ * DV * 2;                        // 24 KB
constexpr int KV_STAGE = KV_QBYTES + KV_OBYTES + 2 * KV_VEC * 4;  // + LSE2 and D
constexpr int KV_NSTAGE = 2;  // measured faster than three stages
constexpr int KV_PBYTES = 4 * KV_NSB * 2048;                     // P: 4 pairs x sub-blocks x 32x32 bf16
constexpr int KV_LDS = KV_NSTAGE * KV_STAGE + KV_PBYTES;
// The copies are issued by the four role-B waves only (role A's first phase is the longer one).

// One tile of a key item's walk: query tile qt of query head `member` of the group.  Each
// member's tiles are walked last first.  Every range of a key item ends where its document or
// segment ends, which is the same row for most items, so the workgroups running together start
// at the same query tiles and stream them through the L2 together (walked first to last, they
// would start at their own key positions, each on its own tiles).
struct KvTile {
  int member, qt;
  Tile q;
};
__device__ __forceinline__ KvTile kv_tile(const TileRanges qr, int member, int qt) {
  return {member, qt, tile_at(qr, qt, KV_BQ)};
}
__device__ __forceinline__ KvTile kv_next(const TileRanges qr, const KvTile& t) {
  return t.qt > 0 ? kv_tile(qr, t.member, t.qt - 1) : kv_tile(qr, t.member + 1, qr.nt - 1);
}

// Starts the copy of tile t into an LDS stage.  wave_b: 0 .. 3, the issuing wave among the
// role-B waves.
__device__ __forceinline__ void kv_issue(lds_char* dst, const AttnArgs& a, const KvTile& t, int qoff, int ooff, int head0,
                                         int wave_b, int lane) {
  const int row0 = t.q.row0, n = t.q.n;
  dma_tile<DQK, KV_BQ, 4>(dst, tile_rsrc(a.q, row0, n, a.q_s), qoff + t.member * (DQK * 2), a.q_s, wave_b);
  dma_tile<DV, KV_BQ, 4>(dst + KV_QBYTES, tile_rsrc(a.dO, row0, n, a.H * DV), ooff + t.member * (DV * 2), a.H * DV,
                         wave_b);
  // LSE2 (waves 0, 2) and D (waves 1, 3) of the tile's rows, 64 per copy; rows past the tile's
  // end are not copied
  static_assert(KV_BQ > 64 && KV_BQ <= 2 * 64 && KV_BQ <= KV_VEC, "two 64-row copies per vector");
  const float* vec = (wave_b & 1) ? a.Dvec : a.lse2;
  const int r0 = 32 * (wave_b & 2);  // 0 or 64
  dma_vec64(dst + KV_QBYTES + KV_OBYTES + (wave_b & 1) * (KV_VEC * 4) + r0 * 4,
            vec + (int64_t)(head0 + t.member) * a.nq + row0 + r0, min(max(n - r0, 0), 64), lane);
}

// clear_tail of the four role-B waves' copies of a short tile (Q, dO and D; a masked row's LSE
// never enters a product).
__device__ __forceinline__ void kv_clear_tail(lds_char* stage, int n, int wave_b, int lane) {
  clear_tail<DQK, KV_BQ, 4>(stage, n, wave_b, lane);
  clear_tail<DV, KV_BQ, 4>(stage + KV_QBYTES, n, wave_b, lane);
  const int r = 32 * (wave_b & 2) + lane;  // waves 1 and 3 copied D, 64 rows each
  if ((wave_b & 1) && r >= n && r < KV_BQ)
    *reinterpret_cast<__attribute__((address_space(3))) float*>(stage + KV_QBYTES + KV_OBYTES + KV_VEC * 4 + 4 * r) = 0.f;
}

// STORE_DS: also store dS (bf16, as the MFMA operand registers hold it) for the query-
// stationary dQ kernel that reads it back instead of recomputing S and dP.
template <bool STORE_DS>
__device__ __forceinline__ void bwd_dkdv_body(const AttnArgs& a, int block, lds_char* smem) {
  lds_char* pbuf = smem + KV_NSTAGE * KV_STAGE;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, known to the compiler
  const int pair = wave & 3, role = wave >> 2;  // role 0: S, P, dV   role 1: dP, dS, dK
  const int m = lane & 31, hh = lane >> 5;
  // one K/V head per workgroup; its dK/dV sum over the group's query heads head0 ..
  int kvl, item_idx;
  xcd_head_item(block, a.kv_heads, a.n_items, kvl, item_idx);
  const int kv_head = a.kv_head0 + kvl;
  const int head0 = kv_head * a.grp;
  const Item it(a.items, item_idx);
  const TileRanges qr = tile_ranges(it, KV_BQ);
  // this unit's (query head, query tile) pairs
  const int t0 = it.t0, n_tiles = (it.t1 < 0 ? qr.nt * a.grp : it.t1) - t0;
  if (n_tiles == 0) return;  // uniform over the workgroup
  const int k_row0 = it.row0, k_pos0 = it.pos0, k_n = it.n;

  const int kj = pair * 32 + m;
  const bool k_valid = kj < k_n;
  const int pos_k = k_valid ? k_pos0 + kj : 0x7fffffff;
  const int hi_k = doc_edge<true>(a.cu, it.d0, it.d1, it.edge0, k_pos0 + min(kj, k_n - 1));
  const int kn_w = min(32, max(0, k_n - pair * 32));  // valid keys of this pair
  const int wk_first = k_pos0 + pair * 32, wk_last = wk_first + kn_w - 1;
  // document ends of the pair's first and last key (lanes past the end repeat the last one)
  const int hi_first = __builtin_amdgcn_readfirstlane(hi_k);
  const int hi_last = __builtin_amdgcn_readlane(hi_k, 31);
  const float sl2 = a.scale * LOG2E;
  const int qoff = dma_lane_off<DQK>(a.q_s, head0, pair, lane);  // role B's copy lanes (wave b = pair)
  const int ooff = dma_lane_off<DV>(a.H * DV, head0, pair, lane);
  const int poff = pair * (KV_NSB * 2048) + lane * 16;  // this lane's P slot: + sb*2048 + half*1024
  const bool active = kn_w > 0;               // uniform over the pair
  // first dS slot of this key item (stored-dS backward only)
  const int ds_slot0 = it.ds_slot, ds_head0 = kvl * a.grp;

  // The two roles run separate copies of the tile loop, with the same copies and the same
  // two barriers per tile: each copy keeps only its own role's operands and accumulators
  // live, which leaves registers for reading LDS operands well ahead of their products.
  auto run = [&](auto role_c) {
    constexpr int ROLE = decltype(role_c)::value;
    // role A keeps K^T fragments (B operand of S) and dV^T; role B V^T fragments (B operand
    // of dP) and dK^T
    constexpr int NF = ROLE == 0 ? DQK / 16 : DV / 16;
    constexpr int NACC = ROLE == 0 ? DV / 32 : DQK / 32;
    const int member0 = t0 / qr.nt;
    KvTile cur = kv_tile(qr, member0, qr.nt - 1 - (t0 - member0 * qr.nt));
    // the pair's K (role A) and V rows (role B) come through LDS, from the start of stage 1 on
    static_assert(KV_STAGE + 4 * (own_bytes<DQK>() + own_bytes<DV>()) <= KV_LDS, "LDS");
    bf16x8 bf[NF];
    if constexpr (ROLE == 0) {
      lds_char* own = smem + KV_STAGE + pair * own_bytes<DQK>();
      own_rows_issue<DQK>(own, a.k, k_row0 + pair * 32, kn_w, a.k_s, kv_head, lane);
      wait_dma();
      own_rows_read<DQK>(own, lane, bf);
    } else {
      lds_char* own = smem + KV_STAGE + 4 * own_bytes<DQK>() + pair * own_bytes<DV>();
      own_rows_issue<DV>(own, a.v, k_row0 + pair * 32, kn_w, a.v_s, kv_head, lane);
      kv_issue(smem, a, cur, qoff, ooff, head0, pair, lane);
      wait_dma();
      own_rows_read<DV>(own, lane, bf);
    }

    f32x16 acc[NACC];
#pragma unroll
    for (int c = 0; c < NACC; ++c) acc[c] = f32x16{};
    OperandOffsets o = operand_offsets(lane);

    for (int t = 0; t < n_tiles; ++t) {
      refresh(o);
      const int qpos = cur.q.pos0, qn = cur.q.n;
      const int64_t ds_off = (int64_t)(ds_head0 + cur.member) * a.ds_head_bytes +
                             (int64_t)(ds_slot0 + cur.qt) * DS_TILE_BYTES;  // this tile's dS slot
      const bool more = t + 1 < n_tiles;
      if (more) cur = kv_next(qr, cur);
      // a pair whose keys no row of the tile sees leaves the matrix cores to the others
      const bool sees = active && qpos + qn > wk_first && qpos < hi_last;
      if constexpr (ROLE == 1) {
        wait_dma();  // tile t's copies, the only ones in flight
        if (qn < KV_BQ) kv_clear_tail(smem + (t % KV_NSTAGE) * KV_STAGE, qn, pair, lane_now());
      }
      barrier_lds();
      if constexpr (ROLE == 1)
        if (more) kv_issue(smem + ((t + 1) % KV_NSTAGE) * KV_STAGE, a, cur, qoff, ooff, head0, pair, lane);
      const lds_char* Qs = smem + (t % KV_NSTAGE) * KV_STAGE;
      const lds_char* Os = lds_opaque(Qs + KV_QBYTES);
      const lds_char* vec_s = lds_opaque(Qs + KV_QBYTES + KV_OBYTES);  // LSE2 then D, KV_VEC slots each

      if constexpr (ROLE == 0) {
        // ---------------- phase 1: S, P = exp(S - LSE) (masked), P to LDS for role B
        bf16x8 pk[KV_BQ / 16];  // P of this tile, bf16: rows 16*g .. 16*g+15 in pk[g]
        if (sees) {
          // S of the 32-row sub-blocks.  Left to itself the compiler issues each read just
          // before its product and waits for it there; instead sub-block 0's reads are all
          // issued first, and each next sub-block's as the current one's products free
          // their registers.
          const RowBases qr_b = row_bases(Qs, o);
          bf16x8 qa[DQK / 16];
#pragma unroll
          for (int t2 = 0; t2 < DQK / 16; ++t2) qa[t2] = op_b128<KV_BQ>(qr_b, 0, t2);
          sched_fence();
          f32x16 sc[KV_NSB];
          static_for<KV_NSB>([&](auto sb_) {
            constexpr int sb = decltype(sb_)::value;
            sc[sb] = f32x16{};
#pragma unroll
            for (int t2 = 0; t2 < DQK / 16; ++t2) {
              sc[sb] = mfma(qa[t2], bf[t2], sc[sb]);
              if constexpr (sb + 1 < KV_NSB) qa[t2] = op_b128<KV_BQ>(qr_b, 32 * (sb + 1), t2);
            }
            sched_fence();
          });
          static_for<KV_BQ / 32>([&](auto sb_) {
            constexpr int sb = decltype(sb_)::value;
            const int qb = qpos + 32 * sb;
            const f32x16& s = sc[sb];
            // this lane's query rows are 32*sb + 8*hh + {0..7, 16..23}
            f32x4 l0, l1, l2, l3;
            lds_x4_f32<128 * sb, 128 * sb + 16, 128 * sb + 64, 128 * sb + 80>(vec_s, 32 * hh, l0, l1, l2, l3);
            const float lse_r[16] = {l0[0], l0[1], l0[2], l0[3], l1[0], l1[1], l1[2], l1[3],
                                     l2[0], l2[1], l2[2], l2[3], l3[0], l3[1], l3[2], l3[3]};
            const bool full = (kn_w == 32) && (qn >= 32 * (sb + 1)) && (wk_last <= qb) && (qb + 31 < hi_first);
            float p[16];
            if (full) {
#pragma unroll
              for (int e = 0; e < 16; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], sl2, -lse_r[e]));
            } else {
              // query row qq = base + c(e) is visible iff lo <= base + c(e) < lim, where base
              // is this lane's first row relative to its key position; masked entries get
              // exp2(-inf)
              const int base = qpos - pos_k + 32 * sb + 8 * hh;
              const int lim = max(0, min(qpos + qn, hi_k) - pos_k);
#pragma unroll
              for (int e = 0; e < 16; ++e) {
                const int r = base + 16 * (e >> 3) + (e & 7);
                const bool vis = (unsigned)r < (unsigned)lim;
                p[e] = __builtin_amdgcn_exp2f(vis ? __builtin_fmaf(s[e], sl2, -lse_r[e]) : -INFINITY);
              }
            }
            pk[2 * sb] = to_bf16x8(p);
            pk[2 * sb + 1] = to_bf16x8(p + 8);
            lds_st16<2048 * sb>(pbuf, poff, pk[2 * sb]);
            lds_st16<2048 * sb + 1024>(pbuf, poff, pk[2 * sb + 1]);
          });
        }
        barrier_lds();  // P of this tile is in LDS
        // ---------------- phase 2: dV^T[dv][key] += dO^T[dv][q] P[q][key]; groups of four
        // dO^T fragments, one per 16 query rows; a group's products are issued before the
        // next group loads
        if (sees) {
          bf16x8 f[2][4];
          op_tr_x4<KV_BQ, 0, 0>(Os, o, f[0]);
          static_for<KV_BQ / 16>([&](auto g_) {
            constexpr int gq = decltype(g_)::value;
#pragma unroll
            for (int d = 0; d < DV / 32; ++d) acc[d] = mfma(f[gq & 1][d], pk[gq], acc[d]);
            if constexpr (gq + 1 < KV_BQ / 16) op_tr_x4<KV_BQ, 16 * (gq + 1), 0>(Os, o, f[(gq + 1) & 1]);
            sched_fence();
          });
        }
      } else {
        // ---------------- phase 1: dP - D = dO V^T - D of every sub-block
        f32x16 dp[KV_NSB];
        if (sees) {
          // the products accumulate onto -D of this lane's rows, 32*sb + 8*hh + {0..7, 16..23}
          static_for<KV_NSB>([&](auto sb_) {
            constexpr int sb = decltype(sb_)::value;
            f32x4 d0, d1, d2, d3;
            lds_x4_f32<KV_VEC * 4 + 128 * sb, KV_VEC * 4 + 128 * sb + 16, KV_VEC * 4 + 128 * sb + 64,
                       KV_VEC * 4 + 128 * sb + 80>(vec_s, 32 * hh, d0, d1, d2, d3);
            dp[sb] = f32x16{d0[0], d0[1], d0[2], d0[3], d1[0], d1[1], d1[2], d1[3],
                            d2[0], d2[1], d2[2], d2[3], d3[0], d3[1], d3[2], d3[3]};
          });
          // reads issued ahead as in role A's S
          const RowBases or_b = row_bases(Os, o);
          bf16x8 ob[DV / 16];
#pragma unroll
          for (int t2 = 0; t2 < DV / 16; ++t2) ob[t2] = op_b128<KV_BQ>(or_b, 0, t2);
          sched_fence();
          static_for<KV_NSB>([&](auto sb_) {
            constexpr int sb = decltype(sb_)::value;
#pragma unroll
            for (int t2 = 0; t2 < DV / 16; ++t2) {
              dp[sb] = mfma(ob[t2], bf[t2], dp[sb]);
              if constexpr (sb + 1 < KV_NSB) ob[t2] = op_b128<KV_BQ>(or_b, 32 * (sb + 1), t2);
            }
            sched_fence();
          });
        }
        barrier_lds();  // P of this tile is in LDS
        typedef __attribute__((address_space(1))) u32x4 gu32x4;
        auto store_ds = [&](int sb, bf16x8 d0, bf16x8 d1) {
          char* dst = a.ds + ds_off + (sb * 4 + pair) * DS_BLOCK_BYTES + lane * 16;
          __builtin_nontemporal_store(__builtin_bit_cast(u32x4, d0), (gu32x4*)(dst));
          __builtin_nontemporal_store(__builtin_bit_cast(u32x4, d1), (gu32x4*)(dst + DS_BLOCK_BYTES / 2));
        };
        // ---------------- phase 2: dS = P o (dP - D) of every sub-block first (its vector
        // work overlaps role A's dV products), then dK^T[c][key] += Q^T[c][q] dS[q][key]
        if (sees) {
          bf16x8 sf[KV_NSB][2], pr[KV_NSB][2];
          static_for<KV_NSB>([&](auto sb_) {
            constexpr int sb = decltype(sb_)::value;
            lds_x2_bf16<2048 * sb, 2048 * sb + 1024>(pbuf, poff, pr[sb][0], pr[sb][1]);
          });
          sched_fence();
          static_for<KV_BQ / 32>([&](auto sb_) {
            constexpr int sb = decltype(sb_)::value;
            float ds[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const float pv = (float)pr[sb][e >> 3][e & 7];
              ds[e] = pv * dp[sb][e];
            }
            sf[sb][0] = to_bf16x8(ds);
            sf[sb][1] = to_bf16x8(ds + 8);
            if constexpr (STORE_DS) {
              // this pair's 32 keys x sub-block sb's 32 queries, 2 KB: two 1 KB stores in the
              // register layout (lane 32h + m: key m, queries 16*half + 8h .. +7), non-temporal
              // (read once, by the dQ kernel)
              store_ds(sb, sf[sb][0], sf[sb][1]);
            }
          });
          static_for<KV_BQ / 32>([&](auto sb_) {
            constexpr int sb = decltype(sb_)::value;
            // groups of three Q^T column blocks
            bf16x8 f[2][3];
            op_tr_x3<KV_BQ, 32 * sb, 0>(Qs, o, f[0]);
            static_for<4>([&](auto g_) {
              constexpr int gq = decltype(g_)::value, half = gq >> 1, c0 = 3 * (gq & 1);
#pragma unroll
              for (int j = 0; j < 3; ++j) acc[c0 + j] = mfma(f[gq & 1][j], sf[sb][half], acc[c0 + j]);
              if constexpr (gq + 1 < 4)
                op_tr_x3<KV_BQ, 32 * sb + 16 * ((gq + 1) >> 1), 3 * ((gq + 1) & 1)>(Qs, o, f[(gq + 1) & 1]);
              sched_fence();
            });
          });
        } else if (STORE_DS && active) {  // dQ reads 64 keys at a time: the other pair's may be visible
#pragma unroll
          for (int sb = 0; sb < KV_NSB; ++sb) store_ds(sb, bf16x8{}, bf16x8{});
        }
      }
    }

    if (it.part >= 0) {
      char* p = part_at(a, kvl, it.part, KV_PART_BYTES);
      part_store(p + (ROLE == 0 ? pair * PART_WAVE_128 : 4 * PART_WAVE_128 + pair * PART_WAVE_192), lane_now(), acc);
      return;
    }
    barrier_lds();  // every wave is past its last tile
    const int64_t krow = (int64_t)(k_row0 + pair * 32) * a.Hkv + kv_head;
    if constexpr (ROLE == 0)
      rows_add<DV / 64>(smem + wave * ROWS_OUT_BYTES, lane_now(), acc, 1.0f, a.dv + krow * DV, a.Hkv * DV, kn_w);
    else
      rows_add<DQK / 64>(smem + wave * ROWS_OUT_BYTES, lane_now(), acc, a.scale, a.dk + krow * DQK, a.Hkv * DQK, kn_w);
  };
  if (role == 0) run(IntC<0>{});
  else run(IntC<1>{});
}

__global__ __launch_bounds__(512, 1) void bwd_dkdv_ds_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char smem_raw[KV_LDS];
  bwd_dkdv_body<true>(a, blockIdx.x, (lds_char*)smem_raw);
}

// The recompute backward: dK/dV, then dQ, in one launch.  The workgroups of dQ, which needs nothing
// from dK/dV, fill the CUs that the last ones of dK/dV leave idle; as two launches dQ waited for
// them.  dK/dV comes first because its workgroups are the longer ones (of 128 keys, and of all heads
// of a group).  Two launches and one: 1K rows x 16 heads 106 and 99 us, 2K 150 and 138, ragged 8K 434
// and 400, 16K on 2 K/V heads 675 and 618, ring of 64K with one head 1.82 and 1.73 ms; the same at
// 32K and 64K rows in one document (21.6 ms, 84 ms).  The two lists interleaved, both walked to
// the end together, lost where workgroups are long (64K: 79.3 to 83.2 ms): dK/dV's and dQ's tiles then
// share the L2s.  Up to seven places after dK/dV stay empty, so that dQ's heads keep their XCDs.
__global__ __launch_bounds__(512, 1) void bwd_recompute_kernel(AttnArgs q, AttnArgs kv) {
  __shared__ __attribute__((aligned(1024))) char smem_raw[DQ_LDS > KV_LDS ? DQ_LDS : KV_LDS];
  lds_char* smem = (lds_char*)smem_raw;
  const int nkv = kv.n_items * kv.kv_heads;
  const int b = blockIdx.x, q0 = (nkv + N_XCD - 1) / N_XCD * N_XCD;
  if (b < nkv) bwd_dkdv_body<false>(kv, b, smem);
  else if (b >= q0) bwd_dq_body(q, b - q0, smem);
}

// ------------------------------------------------------------------ dQ from stored dS
// Query-stationary like the dQ above, but reading the dS that bwd_dkdv_ds stored instead of
// recomputing S and dP: dQ^T[c][q] += K^T[c][key] dS^T[key][q], 384 of its 1024 FLOP
// per visible pair, and 2 bytes of dS read per pair (HBM-bound).  Eight waves x 32 query
// rows; keys walk the key items that the query tile's visible ranges touch, 64 keys (half
// an item) per tile.  Every 32-row query block coincides with one 32-row sub-block of each
// key item's query tiling (segments are 32-aligned on this path), so a wave finds its dS
// block from the item's ranges.
constexpr int DQS_BK = 64;                               // keys per tile
constexpr int DQS_KBYTES = DQS_BK * DQK * 2;             // 24 KB
constexpr int DQS_WAVE_BYTES = 2 * DS_BLOCK_BYTES;       // a wave's 32 queries x 64 keys of dS
constexpr int DQS_DBYTES = 8 * DQS_WAVE_BYTES;           // 32 KB
// K tiles (mostly L2 hits) are copied one tile ahead, the dS (read once, from HBM) two
// tiles ahead: 2 x 24 KB + 3 x 32 KB of LDS
constexpr int DQS_KSTAGES = 2, DQS_DSTAGES = 3;
constexpr int DQS_LDS = DQS_KSTAGES * DQS_KBYTES + DQS_DSTAGES * DQS_DBYTES;

// One tile of the walk (scalars): 64 keys of a key item, and where the wave's dS block for
// them sits (off < 0: the wave's rows do not see the item).  valid = 0 once the walk is over.
struct DsTile {
  int valid, krow0, kn;
  int64_t off;  // < 0: none of the wave's rows sees the keys
};

// The walk over the key items that a query item's ranges touch, in row order, 64 keys at a
// time.  The item records live in row order, so within a range the next item's record is
// the next one; they are read through the constant address space, which makes them scalar
// loads that the compiler waits for where they are used (never together with the copies in
// flight, as vector loads after the copies' memory-clobbering assembly would be).
struct DsWalk {
  int rr, r, end, kpos_r, j;  // range, next key row, the range's end, key position - key row, record
  int lo_first, q_last;       // document start of the wave's first row, position of its last (-1: no rows)
  i32x16 rec;
};

typedef const __attribute__((address_space(4))) i32x16 crec16;
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) i32x4 cint4;

// The item's ranges, a value type of scalars like TileRanges; x*: the record (krec) of the key item
// that holds the range's first row.
struct DsRanges {
  int nr, r0, p0, c0, x0, r1, p1, c1, x1, r2, p2, c2, x2, r3, p3, c3, x3;
};

__device__ __forceinline__ DsTile ds_next(const AttnArgs& a, const DsRanges R, DsWalk& w, int qrow) {
  DsTile d;
  d.valid = 0;
  if (w.r >= w.end) {  // the next range; ranges lie in segments of their own, so in other key items
    if (++w.rr >= R.nr) return d;
    int rr = R.r0, pp = R.p0, cc = R.c0, xx = R.x0;
    if (w.rr >= 1) { rr = R.r1; pp = R.p1; cc = R.c1; xx = R.x1; }
    if (w.rr >= 2) { rr = R.r2; pp = R.p2; cc = R.c2; xx = R.x2; }
    if (w.rr >= 3) { rr = R.r3; pp = R.p3; cc = R.c3; xx = R.x3; }
    w.r = rr;
    w.end = rr + cc;
    w.kpos_r = pp - rr;
    w.j = xx;
    w.rec = *(crec16*)(a.krec + w.j * ITEM_INTS);
  } else if (w.r >= w.rec[0] + w.rec[1]) {  // past this item: the next one in row order
    ++w.j;
    w.rec = *(crec16*)(a.krec + w.j * ITEM_INTS);
  }
  const int half = (w.r - w.rec[0]) >> 6;
  d.valid = 1;
  d.krow0 = w.rec[0] + 64 * half;
  d.kn = min(DQS_BK, w.rec[1] - 64 * half);
  w.r = d.krow0 + DQS_BK;
  // the sub-block of the item's query tiling that holds the wave's rows [qrow, qrow + 32)
  d.off = -1;
  const int kpos = d.krow0 + w.kpos_r;  // a key item lies in one segment: its rows' positions are consecutive
  if (kpos <= w.q_last && kpos + d.kn > w.lo_first) {
    int slot = w.rec[3];
#pragma unroll
    for (int k = 0; k < MAX_RANGES; ++k) {
      if (k >= w.rec[2]) break;
      const int row = w.rec[4 + 2 * k], cnt = w.rec[5 + 2 * k];
      if (qrow >= row && qrow < row + cnt) {
        const int u = (qrow - row) >> 5;
        const int sb = u % (KV_QTILE_ROWS / 32);
        d.off = (int64_t)(slot + u / (KV_QTILE_ROWS / 32)) * DS_TILE_BYTES + (sb * 4 + 2 * half) * DS_BLOCK_BYTES;
        break;
      }
      slot += (cnt + KV_QTILE_ROWS - 1) / KV_QTILE_ROWS;
    }
  }
  return d;
}

__global__ __launch_bounds__(512, 1) void bwd_dq_ds_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char smem_raw[DQS_LDS];
  lds_char* smem = (lds_char*)smem_raw;
  lds_char* dsmem = smem + DQS_KSTAGES * DQS_KBYTES;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 31, hh = lane >> 5;
  int hl, item;
  xcd_head_item(blockIdx.x, a.q_heads, a.n_items, hl, item);
  const int head = a.q_head0 + hl;
  const Item it(a.items, item);
  const bool wave_rows = 32 * wave < it.n;  // the wave's 32 query rows (all valid or none)
  const int qrow0 = it.row0 + 32 * wave;
  const i32x4 x = *(cint4*)(a.qslots + (int64_t)item * MAX_RANGES);
  const DsRanges R = {it.nr, it.r0, it.p0, it.c0, x[0], it.r1, it.p1, it.c1, x[1],
                      it.r2, it.p2, it.c2, x[2],  it.r3, it.p3, it.c3, x[3]};
  DsWalk walk;
  walk.rr = -1;
  walk.r = 0;
  walk.end = 0;
  walk.q_last = wave_rows ? it.pos0 + 32 * wave + 31 : -1;
  walk.lo_first = __builtin_amdgcn_readfirstlane(
      doc_edge<false>(a.cu, it.d0, it.d1, it.edge0, it.pos0 + (wave_rows ? 32 * wave : 0)));
  DsTile t0 = ds_next(a, R, walk, qrow0);
  if (!t0.valid) return;  // uniform over the workgroup
  const int kv_head = head / a.grp;
  const char* ds_head = a.ds + (int64_t)(head - a.q_head0) * a.ds_head_bytes;
  const int koff = dma_lane_off<DQK>(a.k_s, kv_head, wave, lane);
  // dS copy: LDS unit u = 4k + q8 (key k, queries 8*q8 .. +7) fetched from the stored
  // register layout (half q8/2, lane 32*(q8%2) + k)
  const int ds_voff = 1024 * ((lane >> 1) & 1) + 512 * (lane & 1) + 16 * (lane >> 2);
  // transpose read of the B operand: keys 8h' + 4v + j at query 16*(g%2) + i
  const int ds_rd = 512 * (lane >> 5) + 32 * ((lane >> 4) & 1) + 64 * ((lane >> 2) & 3) + 8 * (lane & 3);

  // no row of LDS is read that a copy has not written: a tile has 64 keys or 32 (segments are
  // 32-aligned), and of the latter only the first 32 are read

  // copies of tile d's K rows into K stage st (every wave its share)
  auto issue_k = [&](const DsTile& d, int st) {
    dma_tile<DQK, DQS_BK, 8>(smem + st * DQS_KBYTES, tile_rsrc(a.k, d.krow0, d.kn, a.k_s), koff, a.k_s, wave);
  };
  // this wave's dS block of tile d into dS stage st; returns the copy instructions issued
  // (0: the wave's rows do not see the tile's keys)
  auto issue_ds = [&](const DsTile& d, int st) -> int {
    if (d.off < 0) return 0;
    const int bytes = d.kn > 32 ? 2 * DS_BLOCK_BYTES : DS_BLOCK_BYTES;
    const u32x4 desc = tile_desc(ds_head, d.off, bytes);
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_addr(dsmem + st * DQS_DBYTES + wave * DQS_WAVE_BYTES));
    dma_cols<2, 256, 1024, true>(m0, desc, ds_voff);
    if (d.kn <= 32) return 2;
    dma_cols<2, 256, 1024, true>(m0 + 2048, desc, ds_voff + 2048);
    return 4;
  };

  f32x16 acc[DQK / 32];
#pragma unroll
  for (int c = 0; c < DQK / 32; ++c) acc[c] = f32x16{};
  OperandOffsets o = operand_offsets(lane);

  // issue order per wave: K(0) D(0) D(1) | K(1) D(2) | K(2) D(3) | ...: at the top of tile u
  // only D(u+1) (issued after K(u)) may still be in flight
  DsTile t1 = ds_next(a, R, walk, qrow0);
  issue_k(t0, 0);
  int n_cur = issue_ds(t0, 0);
  int n_1 = t1.valid ? issue_ds(t1, 1) : 0;
  DsTile t2;
  t2.valid = 0;
  if (t1.valid) t2 = ds_next(a, R, walk, qrow0);
  for (int u = 0;; ++u) {
    refresh(o);
    if (n_1 == 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    else if (n_1 == 2) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
    else wait_dma();
    barrier_lds();
    int n_2 = 0;
    if (t1.valid) issue_k(t1, (u + 1) % DQS_KSTAGES);
    if (t2.valid) n_2 = issue_ds(t2, (u + 2) % DQS_DSTAGES);
    if (n_cur > 0) {
      const lds_char* Ks = smem + (u % DQS_KSTAGES) * DQS_KBYTES;
      const lds_char* Ds = dsmem + (u % DQS_DSTAGES) * DQS_DBYTES + wave * DQS_WAVE_BYTES + ds_rd;
      auto kstep = [&](auto s_) {
        constexpr int s = decltype(s_)::value;
        constexpr int base = 2048 * (s >> 1) + 1024 * (s & 1);
        const bf16x8 b = join(lds_tr8(Ds + base), lds_tr8(Ds + base + 256));
        bf16x8 f[2][3];
        op_tr_x3<DQS_BK, 16 * s, 0>(Ks, o, f[0]);
        op_tr_x3<DQS_BK, 16 * s, 3>(Ks, o, f[1]);
#pragma unroll
        for (int j = 0; j < 3; ++j) acc[j] = mfma(f[0][j], b, acc[j]);
#pragma unroll
        for (int j = 0; j < 3; ++j) acc[3 + j] = mfma(f[1][j], b, acc[3 + j]);
      };
      kstep(IntC<0>{});
      kstep(IntC<1>{});
      if (n_cur == 4) {
        kstep(IntC<2>{});
        kstep(IntC<3>{});
      }
    }
    if (!t1.valid) break;
    t1 = t2;
    n_cur = n_1;
    n_1 = n_2;
    if (t2.valid) t2 = ds_next(a, R, walk, qrow0);
  }

  barrier_lds();  // every wave is past its last tile
  rows_add<DQK / 64>(smem + wave * ROWS_OUT_BYTES, lane_now(), acc, a.scale, a.dq + ((int64_t)qrow0 * a.H + head) * DQK,
                     a.H * DQK, wave_rows ? 32 : 0);
}

// ------------------------------------------------------------------ merges of split items
// One workgroup of one wave per 32 rows x 64 columns: the sum of the parts in their order, added
// to the accumulator.  DQ: three column groups of the eight waves' dQ rows of a query item;
// otherwise two of the four pairs' dV rows and three of their dK rows of a key item.
template <bool DQ> constexpr int merge_blocks() { return DQ ? 8 * (DQK / 64) : 4 * (DV / 64 + DQK / 64); }

template <bool DQ> __device__ __forceinline__ void bwd_merge_body(const AttnArgs& a, int b, lds_char* smem) {
  const int heads = DQ ? a.q_heads : a.kv_heads, lane = threadIdx.x;
  const int piece = b % merge_blocks<DQ>(), rest = b / merge_blocks<DQ>();
  const int hl = rest % heads;
  const int* mg = a.merges + (rest / heads) * 4;
  const bool dv = !DQ && piece < 4 * (DV / 64);
  const int k = DQ || dv ? piece : piece - 4 * (DV / 64), block = DQ ? k % 8 : k % 4, g = DQ ? k / 8 : k / 4;
  const int rows = min(32, mg[1] - 32 * block), n = mg[3];
  if (rows <= 0) return;
  const int64_t row0 = mg[0] + 32 * block;
  const int part_bytes = DQ ? DQ_PART_BYTES : KV_PART_BYTES;
  const char* p = part_at(a, hl, mg[2], part_bytes);
  float* out;
  int pitch;
  if constexpr (DQ) {
    p += block * PART_WAVE_192;
    out = a.dq + (row0 * a.H + a.q_head0 + hl) * DQK;
    pitch = a.H * DQK;
  } else {
    const int64_t at = row0 * a.Hkv + a.kv_head0 + hl;
    p += dv ? block * PART_WAVE_128 : 4 * PART_WAVE_128 + block * PART_WAVE_192;
    out = dv ? a.dv + at * DV : a.dk + at * DQK;
    pitch = a.Hkv * (dv ? DV : DQK);
  }
  f32x16 acc[2];
  parts_sum(p, part_bytes, n, g, lane, [](int) { return 1.0f; }, acc);
  rows_add<1>(smem, lane, acc, dv ? 1.0f : a.scale, out + 64 * g, pitch, rows);
}

// The first q_blocks workgroups merge dQ, the others dK and dV.
__global__ __launch_bounds__(64) void bwd_merge_kernel(AttnArgs q, AttnArgs kv, int q_blocks) {
  __shared__ __attribute__((aligned(1024))) char smem_raw[ROWS_OUT_BYTES];
  if ((int)blockIdx.x < q_blocks) bwd_merge_body<true>(q, blockIdx.x, (lds_char*)smem_raw);
  else bwd_merge_body<false>(kv, blockIdx.x - q_blocks, (lds_char*)smem_raw);
}

namespace {

// a over a list, whose parts lie at split.
AttnArgs list_args(const AttnArgs& a, const Launch& l, char* split) {
  AttnArgs b = a;
  b.items = l.units;
  b.n_items = l.n_units;
  b.merges = l.merges;
  b.n_parts = l.parts;
  b.split = split;
  return b;
}

template <class K>
hipError_t launch_list(K kernel, const char* name, const AttnArgs& a, int heads, hipStream_t stream) {
  if (a.n_items == 0) return hipSuccess;
  const int tok = prof_begin(name, stream);
  hipLaunchKernelGGL(kernel, dim3(a.n_items * heads), dim3(512), 0, stream, a);
  prof_end(tok, stream);
  return hipGetLastError();
}

// The merges of n_q split query items and n_kv split key items.
hipError_t launch_merges(const AttnArgs& q, int n_q, const AttnArgs& kv, int n_kv, hipStream_t stream) {
  const int q_blocks = n_q * q.q_heads * merge_blocks<true>(), kv_blocks = n_kv * kv.kv_heads * merge_blocks<false>();
  if (q_blocks + kv_blocks == 0) return hipSuccess;
  const int tok = prof_begin("bwd_merge", stream);
  hipLaunchKernelGGL(bwd_merge_kernel, dim3(q_blocks + kv_blocks), dim3(64), 0, stream, q, kv, q_blocks);
  prof_end(tok, stream);
  return hipGetLastError();
}

hipError_t launch_recompute(const AttnArgs& q, int q_merges, const AttnArgs& kv, int kv_merges, hipStream_t stream) {
  const int64_t nq = (int64_t)q.n_items * q.q_heads, nkv = (int64_t)kv.n_items * kv.kv_heads;
  if (nq + nkv == 0) return hipSuccess;
  const int tok = prof_begin("bwd_recompute", stream);
  const int64_t kv_blocks = nq > 0 ? (nkv + N_XCD - 1) / N_XCD * N_XCD : nkv;
  hipLaunchKernelGGL(bwd_recompute_kernel, dim3(unsigned(kv_blocks + nq)), dim3(512), 0, stream, q, kv);
  prof_end(tok, stream);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return launch_merges(q, q_merges, kv, kv_merges, stream);
}

}  // namespace

// kv_heads_per_pass = 0: recompute path over all heads.  kv_parts, dq_parts: where the parts of dK/dV
// and dQ go, for a list that has any.
// Otherwise the stored-dS path, in passes of that many K/V heads (the dS of one pass's query heads
// fits a.ds): bwd_dkdv_ds stores dS, then bwd_dq_ds reads it back.
hipError_t launch_attn_bwd(const AttnArgs& a, const Launch& q_whole, const Launch& dq, char* dq_parts, const Launch& kv,
                           char* kv_parts, int kv_heads_per_pass, hipStream_t stream) {
  const int64_t pairs = (int64_t)a.nq * a.H;
  const int64_t blocks = (pairs + 15) / 16 < (1 << 20) ? (pairs + 15) / 16 : (1 << 20);
  int tok = prof_begin("bwd_pre", stream);
  hipLaunchKernelGGL(bwd_pre_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, a.o, a.dO, a.lse, a.Dvec,
                     a.lse2, a.nq, a.H);
  prof_end(tok, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (kv_heads_per_pass > 0) {
    if (q_whole.n_units == 0 || kv.n_units == 0) return hipSuccess;
    for (int g0 = 0; g0 < a.Hkv; g0 += kv_heads_per_pass) {
      const int G = min(kv_heads_per_pass, a.Hkv - g0);
      AttnArgs b = list_args(a, kv, kv_parts);
      b.kv_head0 = g0;
      b.kv_heads = G;
      b.q_head0 = g0 * a.grp;
      b.q_heads = G * a.grp;
      if ((e = launch_list(bwd_dkdv_ds_kernel, "bwd_dkdv_ds", b, G, stream)) != hipSuccess) return e;
      if ((e = launch_merges(b, 0, b, kv.n_merges, stream)) != hipSuccess) return e;
      if ((e = launch_list(bwd_dq_ds_kernel, "bwd_dq_ds", list_args(b, q_whole, nullptr), G * a.grp, stream)) !=
          hipSuccess)
        return e;
    }
    return hipSuccess;
  }
  // a dispatch holds fewer than 2^32 lanes
  const bool turns = (int64_t)dq.n_units * a.H + (int64_t)kv.n_units * a.Hkv + N_XCD > (1 << 23);
  const AttnArgs q_args = list_args(a, dq, dq_parts), kv_args = list_args(a, kv, kv_parts);
  if (turns) {
    AttnArgs none = a;
    none.n_items = 0;
    if ((e = launch_recompute(none, 0, kv_args, kv.n_merges, stream)) != hipSuccess) return e;
    return launch_recompute(q_args, dq.n_merges, none, 0, stream);
  }
  return launch_recompute(q_args, dq.n_merges, kv_args, kv.n_merges, stream);
}

}  // namespace hydra
