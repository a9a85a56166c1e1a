// Forward partial of one ring step: O = softmax(scale * Q K^T, masked) V and its LSE.
//
// One workgroup = 8 waves = 256 query rows of one head; each wave owns 32 rows and keeps
// them in registers as MFMA B operands for the whole key loop.  Key/value tiles of 64 rows
// stream through two swizzled LDS stages (80 KB) filled by direct global->LDS copies:
// the copies of tile t+1 are in flight while tile t is computed, one barrier per
// tile.  Eight waves share every tile, which halves the L2->LDS traffic per FLOP against a
// 128-row workgroup; two waves per SIMD let one's softmax overlap the other's matrix work.
// Scores are computed transposed (S^T = K Q^T), so every lane holds one query and the
// softmax row reductions stay in-lane plus one exchange with the lane 32 away.
//
// The running max / sum update is the online softmax that FlashAttention uses (named in
// Sec. 1 and Sec. 3.5), with one liberty: the reference max m only moves when a tile's max
// exceeds it by more than 8 (log2 units), so O is rescaled rarely.  Every term is still
// exp2(s - m) for the same m in numerator and denominator, so the result is unchanged up to
// rounding (terms stay <= 2^8).  Only tiles that straddle a document start, the causal
// diagonal or the end of a range evaluate the mask (Sec. 2.2).
#include "kernels.h"
#include "prof.h"

namespace hydra {

constexpr int FWD_BK = FWD_TILE_ROWS;
constexpr int FWD_KBYTES = FWD_BK * DQK * 2;             // 24 KB
constexpr int FWD_STAGE = FWD_KBYTES + FWD_BK * DV * 2;  // 40 KB
constexpr int FWD_NSTAGE = 2;  // measured faster than three stages
constexpr int FWD_WAVES = 8;
constexpr int FWD_AHEAD = 6;  // operand reads of S in flight ahead of the products
constexpr float RESCALE_SLACK = 8.0f;

// Starts the copy of key/value tile k into LDS stage `stage`.
__device__ __forceinline__ void fwd_issue(lds_char* stage, const AttnArgs& a, const Tile k, int koff, int voff, int wave) {
  dma_tile<DQK, FWD_BK, FWD_WAVES>(stage, tile_rsrc(a.k, k.row0, k.n, a.k_s), koff, a.k_s, wave);
  dma_tile<DV, FWD_BK, FWD_WAVES>(stage + FWD_KBYTES, tile_rsrc(a.v, k.row0, k.n, a.v_s), voff, a.v_s, wave);
}

// LSE of the earlier steps for this lane's row m of a wave's rows (-inf past their end).
__device__ __forceinline__ float fwd_old_lse(const AttnArgs& a, int head, int q_row0, int q_n, int lane) {
  const int m = lane & 31;
  return m < q_n ? a.out_lse[(int64_t)head * a.nq + q_row0 + m] : -INFINITY;
}

// A wave's rows [q_row0, q_row0 + q_n), column groups G0 .. G0 + NG - 1 of 64, out: O = acc / l
// (and its bf16 copy), and with the first group the LSE from the running max and sum.  obuf:
// ROWS_OUT_BYTES of LDS of the wave's own.
// MERGE: O and LSE already hold the merge of the earlier ring steps (old_lse: that LSE), and this
// step's partial is merged into them here.  Written out on its own and merged by a second kernel,
// the partial costs a launch, its write and its read: 256K ring step, 32K rows x 16 heads, 170 us
// per step against 10 to 20 here.
template <bool MERGE, int G0, int NG>
__device__ __forceinline__ void fwd_out(const AttnArgs& a, uint16_t* o_bf16, lds_char* obuf, int head, int q_row0,
                                        int q_n, int lane, const f32x16 (&acc)[2 * NG], float m_run, float l_tot,
                                        float old_lse) {
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
  float lse = l_tot > 0.f ? (m_run + __builtin_log2f(l_tot)) * LN2 : -INFINITY;
  const int64_t base = ((int64_t)q_row0 * a.H + head) * DV;
  const int rows = max(q_n, 0), pitch = a.H * DV;
  const rows_rsrc ro = rows_buffer(a.out_o + base, rows, pitch * 4);
  const rows_rsrc rb = rows_buffer(o_bf16 + base, o_bf16 ? rows : 0, pitch * 2);
  float wa[8], wb[8];  // of the rows that this lane stores
  f32x4 old[NG][8];
  if constexpr (MERGE) {
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int i = 0; i < 8; ++i) old[g][i] = rows_old(ro, lane, i, pitch, G0 + g);
    sched_fence();
    float a_m, b_m;
    merge_weights(old_lse, lse, lse, a_m, b_m);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      wa[i] = __shfl(a_m, rows_row(lane, i), 64);
      wb[i] = __shfl(b_m, rows_row(lane, i), 64);
    }
  }
  if (G0 == 0 && lane < q_n) a.out_lse[(int64_t)head * a.nq + q_row0 + lane] = lse;
  static_for<NG>([&](auto g_) {
    constexpr int gi = decltype(g_)::value, g = G0 + gi;
    rows_stage<gi>(obuf, lane, acc, inv);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      f32x4 val = rows_read(obuf, lane, i);
      if constexpr (MERGE) {
#pragma unroll
        for (int e = 0; e < 4; ++e) val[e] = merge_value(wa[i], old[gi][i][e], wb[i], val[e]);
      }
      const int off = rows_row(lane, i) * pitch + rows_col(lane, i);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, val), ro, off * 4 + 256 * g, 0, 0);
      if (o_bf16)
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3])}, rb,
                                              off * 2 + 128 * g, 0, 0);
    }
  });
}

template <bool MERGE>
__global__ __launch_bounds__(64 * FWD_WAVES, 1) void attn_fwd_kernel(AttnArgs a, uint16_t* __restrict__ o_bf16) {
  // stage 0 | stage 1; before the loop the waves' Q rows from the start of stage 1, after it
  // their outputs
  constexpr int LDS_BYTES = FWD_STAGE + FWD_WAVES * own_bytes<DQK>();
  static_assert(LDS_BYTES >= FWD_NSTAGE * FWD_STAGE && LDS_BYTES >= FWD_WAVES * ROWS_OUT_BYTES, "LDS");
  __shared__ __attribute__((aligned(1024))) char smem_raw[LDS_BYTES];
  lds_char* smem = (lds_char*)smem_raw;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, known to the compiler
  const int m = lane & 31, hh = lane >> 5;
  int head, item;
  xcd_head_item(blockIdx.x, a.H, a.n_items, head, item);
  const Item it(a.items, item);
  const TileRanges kr = tile_ranges(it, FWD_BK);
  const int t0 = it.t0, n_tiles = (it.t1 < 0 ? kr.nt : it.t1) - t0;  // this unit's tiles
  // nothing to add to the earlier steps, which leaves only their bf16 copy (uniform)
  if (MERGE && n_tiles == 0 && !o_bf16) return;
  const int kv_head = head / a.grp;  // grouped K/V heads: contiguous groups of query heads
  const int koff = dma_lane_off<DQK>(a.k_s, kv_head, wave, lane);
  const int voff = dma_lane_off<DV>(a.v_s, kv_head, wave, lane);
  const float sl2 = a.scale * LOG2E;

  // this wave's rows: [q_row0, q_row0 + q_n) at positions from q_pos0 on (q_n <= 0: none)
  const int q_row0 = it.row0 + 32 * wave, q_pos0 = it.pos0 + 32 * wave, q_n = min(32, it.n - 32 * wave);
  const int q_last = q_n > 0 ? q_pos0 + q_n - 1 : -1;
  const bool q_valid = m < q_n;
  const int pos_q = q_valid ? q_pos0 + m : -1;  // -1: sees nothing

  lds_char* qbuf = smem + FWD_STAGE + wave * own_bytes<DQK>();
  own_rows_issue<DQK>(qbuf, a.q, q_row0, max(q_n, 0), a.q_s, head, lane);
  Tile cur = tile_at(kr, t0, FWD_BK);  // with no tile: of no rows
  fwd_issue(smem, a, cur, koff, voff, wave);

  // document starts: of this lane's row, of the wave's first and last row
  const int lo_q = doc_edge<false>(a.cu, it.d0, it.d1, it.edge0, q_pos0 + min(m, max(q_n, 1) - 1));
  const int lo_first = __builtin_amdgcn_readfirstlane(lo_q);
  const int lo_last = __builtin_amdgcn_readlane(lo_q, 31);  // rows past the end repeat the last one
  bf16x8 qf[DQK / 16];
  wait_dma();
  own_rows_read<DQK>(qbuf, lane, qf);

  f32x16 acc[DV / 32];
#pragma unroll
  for (int d = 0; d < DV / 32; ++d) acc[d] = f32x16{};
  float m_run = NEG_BIG, l_run[4] = {0.f, 0.f, 0.f, 0.f};

  OperandOffsets o = operand_offsets(lane);

  for (int t = 0; t < n_tiles; ++t) {
    refresh(o);
    const int kpos = cur.pos0, kn = cur.n;
    lds_char* Ks = smem + (t % FWD_NSTAGE) * FWD_STAGE;
    lds_char* Vs = Ks + FWD_KBYTES;
    wait_dma();  // tile t's copies, the only ones in flight
    if (kn < FWD_BK) clear_tail<DV, FWD_BK, FWD_WAVES>(Vs, kn, wave, lane_now());
    barrier_lds();
    if (t + 1 < n_tiles) {
      cur = tile_at(kr, t0 + t + 1, FWD_BK);
      fwd_issue(smem + ((t + 1) % FWD_NSTAGE) * FWD_STAGE, a, cur, koff, voff, wave);
    }
    // a wave none of whose rows sees the tile (the diagonal's upper half, another document)
    // leaves the matrix cores to the others
    if (kpos > q_last || kpos + kn <= lo_first) continue;

    f32x16 s[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      s[kb] = f32x16{};
#pragma unroll
      for (int t2 = 0; t2 < DQK / 16; ++t2)
        s[kb] = mfma(op_b128<FWD_BK>(Ks, o, 32 * kb, t2), qf[t2], s[kb]);
    }
    // operand reads six k-steps ahead of their products: left to itself the compiler runs one
    // to two ahead, and how far changes with the code around it (256K ring step 14.29 against
    // 14.51 ms, packed 32K 1.40 against 1.48 ms; eight ahead measures the same)
    __builtin_amdgcn_sched_group_barrier(0x100, FWD_AHEAD, 0);
#pragma unroll
    for (int j = 0; j < 2 * (DQK / 16) - FWD_AHEAD; ++j) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, FWD_AHEAD, 0);

    // per wave: in a window of short documents most 256-row tiles straddle a boundary, their
    // 32-row waves seldom
    const bool full = (kn == FWD_BK) && (lo_last <= kpos) && (kpos + FWD_BK - 1 <= q_pos0);
    if (!full) {
      // key kpos + key(e) is visible iff lo_q <= it <= pos_q and key(e) < kn, i.e. iff
      // 0 <= base + c(e) < lim with base = kpos - lo_q + 8*hh
      const int base = kpos - lo_q + 8 * hh;
      const int lim = max(0, min(pos_q + 1, kpos + kn) - lo_q);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int r = base + 32 * kb + 16 * (e >> 3) + (e & 7);
          s[kb][e] = (unsigned)r < (unsigned)lim ? s[kb][e] : -INFINITY;
        }
    }
    // row max as four independent chains that take two new values per step (one
    // three-input maximum each)
    float mx4[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x16& v = s[j >> 1];
      const int e0 = 8 * (j & 1);
      float t = fmax2(fmax2(v[e0], v[e0 + 1]), v[e0 + 2]);
      t = fmax2(fmax2(t, v[e0 + 3]), v[e0 + 4]);
      mx4[j] = fmax2(fmax2(t, v[e0 + 5]), v[e0 + 6]);
    }
    float mx = fmax2(fmax2(mx4[0], s[0][7]), s[0][15]);
    mx = fmax2(fmax2(mx, mx4[1]), s[1][7]);
    mx = fmax2(fmax2(mx, mx4[2]), s[1][15]);
    mx = fmax2(mx, mx4[3]);
    const float mxs = xhalf_max(mx) * sl2;  // -inf when nothing is visible
    if (__builtin_amdgcn_ballot_w64(mxs > m_run + RESCALE_SLACK) != 0) {
      const float m_new = mxs > m_run + RESCALE_SLACK ? mxs : m_run;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
#pragma unroll
      for (int j = 0; j < 4; ++j) l_run[j] *= alpha;
#pragma unroll
      for (int d = 0; d < DV / 32; ++d) acc[d] *= alpha;
    }
    const float neg_m = -m_run;

    // P = exp2(s*scale*log2e - m); the row sum is kept as four partial sums
    bf16x8 pf[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float p[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[j >> 1][8 * (j & 1) + e], sl2, neg_m));
      l_run[j] += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      pf[j] = to_bf16x8(p);
    }

    // O^T[dv][q] += V^T[dv][key] * P^T[key][q]; V^T fragments via LDS transpose reads.  The
    // products of key step st are issued before the fragments of step st+1 load.
    bf16x8 vf[2][DV / 32];
    op_tr_x4<FWD_BK, 0, 0>(Vs, o, vf[0]);
    static_for<4>([&](auto st_) {
      constexpr int st = decltype(st_)::value;
#pragma unroll
      for (int d = 0; d < DV / 32; ++d) acc[d] = mfma(vf[st & 1][d], pf[st], acc[d]);
      if constexpr (st + 1 < 4) op_tr_x4<FWD_BK, 16 * (st + 1), 0>(Vs, o, vf[(st + 1) & 1]);
    });
  }

  const float l_tot = xhalf_sum((l_run[0] + l_run[1]) + (l_run[2] + l_run[3]));
  barrier_lds();  // every wave is past its last tile
  if (it.part >= 0) {
    char* p = part_at(a, head, it.part, FWD_PART_BYTES) + wave * PART_WAVE_O;
    part_store(p, lane, acc);
    *reinterpret_cast<float2*>(p + PART_WAVE_128 + lane * 8) = make_float2(m_run, l_tot);
    return;
  }
  const float old_lse = MERGE ? fwd_old_lse(a, head, q_row0, q_n, lane) : 0.f;
  fwd_out<MERGE, 0, DV / 64>(a, o_bf16, smem + wave * ROWS_OUT_BYTES, head, q_row0, q_n, lane, acc, m_run, l_tot,
                             old_lse);
}

// Merges the parts of a split item: one workgroup of two waves per 32 rows, 64 columns each, in the
// order of the parts.
template <bool MERGE>
__global__ __launch_bounds__(128) void fwd_merge_kernel(AttnArgs a, uint16_t* __restrict__ o_bf16) {
  __shared__ __attribute__((aligned(1024))) char smem_raw[2 * ROWS_OUT_BYTES];
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wave = blockIdx.x % FWD_WAVES, rest = blockIdx.x / FWD_WAVES;
  const int head = rest % a.H;
  const int* mg = a.merges + (rest / a.H) * 4;
  const int q_n = min(32, mg[1] - 32 * wave), part0 = mg[2], n = mg[3];
  if (q_n <= 0) return;
  const char* p = part_at(a, head, part0, FWD_PART_BYTES) + wave * PART_WAVE_O;
  auto ml = [&](int j) {
    return *reinterpret_cast<const float2*>(p + (int64_t)j * FWD_PART_BYTES + PART_WAVE_128 + lane * 8);
  };
  float m = NEG_BIG, l = 0.f;
#pragma unroll 4
  for (int j = 0; j < n; ++j) m = fmax2(m, ml(j).x);
#pragma unroll 4
  for (int j = 0; j < n; ++j) l += __builtin_amdgcn_exp2f(ml(j).x - m) * ml(j).y;  // a part that saw nothing: l = 0
  f32x16 acc[2];
  parts_sum(p, FWD_PART_BYTES, n, g, lane, [&](int j) { return __builtin_amdgcn_exp2f(ml(j).x - m); }, acc);
  const int q_row0 = mg[0] + 32 * wave;
  lds_char* obuf = (lds_char*)smem_raw + g * ROWS_OUT_BYTES;
  float old_lse = 0.f;
  if constexpr (MERGE) {
    old_lse = fwd_old_lse(a, head, q_row0, q_n, lane);
    settle(old_lse);
    __syncthreads();  // both waves have read the LSE that the first one replaces
  }
  if (g == 0)
    fwd_out<MERGE, 0, 1>(a, o_bf16, obuf, head, q_row0, q_n, lane, acc, m, l, old_lse);
  else
    fwd_out<MERGE, 1, 1>(a, o_bf16, obuf, head, q_row0, q_n, lane, acc, m, l, old_lse);
}

template <bool MERGE>
hipError_t launch_fwd(const AttnArgs& a, const Launch& l, uint16_t* o_bf16, hipStream_t stream) {
  int tok = prof_begin("attn_fwd", stream);
  hipLaunchKernelGGL(attn_fwd_kernel<MERGE>, dim3(a.n_items * a.H), dim3(64 * FWD_WAVES), 0, stream, a, o_bf16);
  prof_end(tok, stream);
  if (hipError_t e = hipGetLastError(); e != hipSuccess || l.n_merges == 0) return e;
  tok = prof_begin("attn_fwd_merge", stream);
  hipLaunchKernelGGL(fwd_merge_kernel<MERGE>, dim3(l.n_merges * a.H * FWD_WAVES), dim3(128), 0, stream, a, o_bf16);
  prof_end(tok, stream);
  return hipGetLastError();
}

// merge: into the O and LSE that a.out_o and a.out_lse hold.
hipError_t launch_attn_fwd(const AttnArgs& args, const Launch& l, uint16_t* o_bf16, bool merge, hipStream_t stream) {
  if (l.n_units == 0) return hipSuccess;
  AttnArgs a = args;
  a.items = l.units;
  a.n_items = l.n_units;
  a.merges = l.merges;
  a.n_parts = l.parts;
  return merge ? launch_fwd<true>(a, l, o_bf16, stream) : launch_fwd<false>(a, l, o_bf16, stream);
}

}  // namespace hydra
