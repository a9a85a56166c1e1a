// Device-side building blocks shared by the gfx950 attention kernels.
//
// Matrix-core conventions (v_mfma_f32_32x32x16_bf16, wave64), lane l = 32*h + m:
//   A operand (32 x 16): lane holds A[m][8h .. 8h+7]
//   B operand (16 x 32): lane holds B[8h .. 8h+7][m]
//   C (32 x 32, 16 fp32 per lane): reg r holds C[8*(r/4) + 4h + r%4][m]
// A tile whose rows are read from LDS in the order pi(row) (bits 2 and 3 of the row
// index swapped) therefore produces C rows with reg r <-> row 16*(r/8) + 8h + r%8: each
// lane holds two runs of 8 consecutive rows, which is exactly the k-slice layout of the
// next contraction's B operand.  Scores computed that way feed P*V (and dS*K, dS*Q,
// P*dO) straight from registers, with no shuffle.
//
// ds_read_b64_tr_b16 (LDS transpose read): within each 16-lane group, lane i receives
// element (i % 4) of the 8-byte words addressed by lanes 4j + i/4, j = 0..3.  Pointing
// lane i at row (base_row + i/4), column (base_col + 4*(i%4)) of a row-major bf16 tile
// gives lane i the column (base_col + i) for rows base_row .. base_row+3: a transposed
// operand fragment without a transposed copy in memory.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "tiles.h"

namespace hydra {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;

constexpr int DQK = 192;
constexpr int DV = 128;
constexpr int ITEM_INTS = 16;
constexpr int MAX_RANGES = 4;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float NEG_BIG = -1.0e30f;  // finite running-max floor: keeps exp2 arguments NaN-free

__device__ __forceinline__ int pi_row(int m) { return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1); }

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// IEEE 754-2019 maximum (a NaN operand gives NaN; scores never are NaN).  Unlike fmax it
// needs no canonicalising v_max of each operand first: nested calls become v_maximum3_f32.
__device__ __forceinline__ float fmax2(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// Value held by the lane 32 positions away (m stays, h flips) and the max / sum with it.
__device__ __forceinline__ float xhalf_max(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmax2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  __bf16 x = (__bf16)a, y = (__bf16)b;
  return uint32_t(__builtin_bit_cast(uint16_t, x)) | (uint32_t(__builtin_bit_cast(uint16_t, y)) << 16);
}

// Eight fp32 values -> one bf16 operand fragment (round to nearest even, v_cvt_pk_bf16_f32).
__device__ __forceinline__ bf16x8 to_bf16x8(const float* v) {
  typedef float f32x8 __attribute__((ext_vector_type(8)));
  const f32x8 x = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
  return __builtin_convertvector(x, bf16x8);
}

__device__ __forceinline__ u32x4 ldg16(const void* p) { return *reinterpret_cast<const u32x4*>(p); }

// Start (END = false) or end (END = true) of the document that holds position pos, which lies
// in one of documents d0 .. d1; edge0 is that boundary of document d0.  A tile usually lies in
// one document (no load at all) or a few (their boundaries are scalar loads, the same for
// every lane); tiles over many short documents search per lane.
typedef const __attribute__((address_space(4))) int cint;
template <bool END>
__device__ __forceinline__ int doc_edge(const int* __restrict__ cu, int d0, int d1, int edge0, int pos) {
  int edge = edge0;
  if (d1 - d0 <= 8) {
    for (int d = d0 + 1; d <= d1; ++d) {
      const int b = ((cint*)cu)[d], e = END ? ((cint*)cu)[d + 1] : b;
      edge = pos >= b ? e : edge;
    }
  } else {
    int lo = d0, hi = d1 + 1;  // the largest d with cu[d] <= pos
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (cu[mid] <= pos) lo = mid; else hi = mid;
    }
    edge = cu[END ? lo + 1 : lo];
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(edge)::"memory");
  }
  return edge;
}

// ------------------------------------------------------------------ swizzled LDS tiles
// A tile of ROWS rows and DIM (128 or 192) bf16 columns is stored as DIM/64 column blocks of
// 64 elements; each block is ROWS rows of 128 bytes, unpadded, so that one 1 KB direct-to-LDS
// instruction covers 8 whole rows.  Within a row the 16-byte chunk c (0..7) lives at chunk
// c ^ swz(r), which spreads both the 16-byte operand reads (16 rows, one chunk) and the
// transpose reads (4 rows x 4 chunks) over all 64 LDS banks.  swz(r) only looks at bits
// 1..3 of r, so every read below is a per-lane constant plus a compile-time offset.
__device__ __forceinline__ int swz(int r) { return (((r >> 1) & 1) << 2) | ((r >> 2) & 3); }

template <int ROWS> constexpr int block_bytes() { return ROWS * 128; }

// Lane-constant parts of the operand reads of a 32x32x16 MFMA from such tiles.
//   b128[j]: 16-byte read of row pi(m), chunk 2j + h within a column block (k-step t uses
//            j = t & 3, block t >> 2)
//   tr[v][k]: transpose read at row (v ? 4 : 0) + 8h + i/4, column 32*cb + 16*(g&1) + 4*(i&3)
//            with k = cb & 1 (block cb >> 1)
// Callers add row_block*128 (row_block a multiple of 16) and block*block_bytes as immediates.
struct OperandOffsets {
  int b128[4];
  int tr[2][2];
};

__device__ __forceinline__ OperandOffsets operand_offsets(int lane) {
  const int m = lane & 31, h = lane >> 5, g = lane >> 4, gi = lane & 15;
  OperandOffsets o;
  const int ra = pi_row(m);
#pragma unroll
  for (int j = 0; j < 4; ++j) o.b128[j] = ra * 128 + (((2 * j + h) ^ swz(ra)) << 4);
  const int rt = 8 * h + (gi >> 2);
  const int cl = 2 * (g & 1) + ((gi & 3) >> 1);  // chunk within 4, plus the 8-byte half below
  const int w = (gi & 1) << 3;
#pragma unroll
  for (int v = 0; v < 2; ++v)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int r = rt + 4 * v;
      o.tr[v][k] = r * 128 + (((4 * k + cl) ^ swz(r)) << 4) + w;
    }
  return o;
}

// Makes the offsets opaque at the top of each tile iteration, in place: otherwise the
// compiler hoists every (offset + immediate) sum out of the tile loop, one register each,
// instead of folding the immediate into the read's offset field.  In place, so that no
// second copy of the offsets stays live across the loop.
__device__ __forceinline__ void refresh(OperandOffsets& o) {
#pragma unroll
  for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(o.b128[j]));
#pragma unroll
  for (int v = 0; v < 2; ++v)
#pragma unroll
    for (int k = 0; k < 2; ++k) asm volatile("" : "+v"(o.tr[v][k]));
}

__device__ __forceinline__ bf16x8 lds_ld16(const lds_char* base, int off) {
  return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(base + off);
}

// This lane's four read addresses of b128 operands in a tile (row pi(m), one per 16-byte
// chunk of a 64-column block), opaque to the compiler: every read is then base + an
// immediate offset (column block, row block), with no address add per read.  Left to
// itself the compiler addresses the reads of a phase from its last read, with negative
// offsets that the unsigned offset field of an LDS read cannot hold.
struct RowBases {
  const lds_char* p[4];
};

__device__ __forceinline__ RowBases row_bases(const lds_char* tile, const OperandOffsets& o) {
  RowBases r;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    r.p[j] = tile + o.b128[j];
    asm volatile("" : "+v"(r.p[j]));
  }
  return r;
}

// k-step t of a b128 operand at rows row_block + pi(m) of a ROWS-row tile.
template <int ROWS>
__device__ __forceinline__ bf16x8 op_b128(const lds_char* tile, const OperandOffsets& o, int row_block, int t) {
  return lds_ld16(tile, o.b128[t & 3] + (t >> 2) * block_bytes<ROWS>() + row_block * 128);
}

// The same read from opaque bases.
template <int ROWS>
__device__ __forceinline__ bf16x8 op_b128(const RowBases& r, int row_block, int t) {
  return lds_ld16(r.p[t & 3], (t >> 2) * block_bytes<ROWS>() + row_block * 128);
}

// ------------------------------------------------------------------ LDS operand reads
// Plain LDS loads and the transpose-read builtin: the compiler schedules them ahead of their
// uses and waits for exactly the reads it needs.  It never sees the direct-to-LDS copies
// (those are inline assembly, below), so it never waits for a copy still in flight; the
// kernels wait for their copies explicitly and publish them with a barrier.

template <int N> struct IntC { static constexpr int value = N; };

// Calls f(IntC<0>{}) .. f(IntC<N-1>{}) (compile-time loop index).
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(IntC<I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ uint32_t lds_addr(const lds_char* p) { return (uint32_t)(uintptr_t)p; }

// The same (wave-uniform) LDS address, opaque to the compiler.  Without it the compiler
// addresses one tile's reads as offsets from another tile's base, and the negative ones do
// not fit the unsigned offset field of an LDS read, so each costs its own address add.
__device__ __forceinline__ const lds_char* lds_opaque(const lds_char* p) {
  asm volatile("" : "+s"(p));
  return p;
}

__device__ __forceinline__ bf16x8 join(i16x4 lo, i16x4 hi) {
  typedef short i16x8 __attribute__((ext_vector_type(8)));
  i16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ i16x4 lds_tr8(const lds_char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p));
}

// Transposed operand fragments for column blocks CB0 .. CB0+N-1 of rows ROWB .. ROWB+15 of
// a ROWS-row tile (lane pattern of OperandOffsets::tr).
template <int ROWS, int ROWB, int CB0, int N>
__device__ __forceinline__ void op_tr(const lds_char* tile, const OperandOffsets& o, bf16x8 (&f)[N]) {
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const lds_char* b = tile + ((CB0 + n) >> 1) * block_bytes<ROWS>() + ROWB * 128;
    f[n] = join(lds_tr8(b + o.tr[0][(CB0 + n) & 1]), lds_tr8(b + o.tr[1][(CB0 + n) & 1]));
  }
}
template <int ROWS, int ROWB, int CB0>
__device__ __forceinline__ void op_tr_x4(const lds_char* tile, const OperandOffsets& o, bf16x8 (&f)[4]) {
  op_tr<ROWS, ROWB, CB0, 4>(tile, o, f);
}
template <int ROWS, int ROWB, int CB0>
__device__ __forceinline__ void op_tr_x3(const lds_char* tile, const OperandOffsets& o, bf16x8 (&f)[3]) {
  op_tr<ROWS, ROWB, CB0, 3>(tile, o, f);
}

// Four 16-byte LDS reads at base + lane_off + I0..I3.
template <int I0, int I1, int I2, int I3>
__device__ __forceinline__ void lds_x4_f32(const lds_char* base, int lane_off, f32x4& a, f32x4& b, f32x4& c,
                                           f32x4& d) {
  typedef const __attribute__((address_space(3))) f32x4* P;
  const lds_char* p = base + lane_off;
  a = *reinterpret_cast<P>(p + I0);
  b = *reinterpret_cast<P>(p + I1);
  c = *reinterpret_cast<P>(p + I2);
  d = *reinterpret_cast<P>(p + I3);
}

// Two 16-byte LDS reads at base + lane_off + I0, I1.
template <int I0, int I1>
__device__ __forceinline__ void lds_x2_bf16(const lds_char* base, int lane_off, bf16x8& a, bf16x8& b) {
  a = lds_ld16(base + lane_off, I0);
  b = lds_ld16(base + lane_off, I1);
}

// 16-byte LDS store of an operand fragment.
template <int I0>
__device__ __forceinline__ void lds_st16(lds_char* base, int lane_off, bf16x8 v) {
  *reinterpret_cast<__attribute__((address_space(3))) bf16x8*>(base + lane_off + I0) = v;
}

// Keeps the instruction scheduler from moving anything across this point (used between
// the groups of a software-pipelined loop so that reads are not all hoisted to its top,
// which would need registers for every group at once).
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// Makes the compiler treat x as freshly produced here: a value loaded before a tile loop
// and passed through settle() right after its load is waited for at that point, not at its
// first use inside the loop (where the wait would also cover every copy in flight).
template <class T> __device__ __forceinline__ void settle(T& x) { asm volatile("" : "+v"(x)); }

typedef int i32x16 __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------------ direct global -> LDS copies
// Copies are inline assembly, invisible to the compiler's wait insertion (see above).  A
// buffer descriptor is built per tile with its base at the tile's first row and its record
// count ending at the tile's last valid row, so rows past the end are out of range for the
// hardware bounds check and never touch memory (all of the offset travels in the VGPR
// operand, which is what the check covers) (the kernels mask those rows and clear them in
// LDS, clear_tail).  Each copy instruction
// writes 16 (or 4) bytes per lane at LDS address M0 + 16*lane (4*lane).
__device__ __forceinline__ u32x4 tile_desc(const void* base, int64_t byte_off, int bytes) {
  const uint64_t b = (uint64_t)(uintptr_t)base + (uint64_t)byte_off;
  u32x4 d;
  d[0] = __builtin_amdgcn_readfirstlane((uint32_t)b);
  d[1] = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) & 0xffffu;  // stride 0
  d[2] = __builtin_amdgcn_readfirstlane((uint32_t)bytes);                // record count (bytes)
  d[3] = 0x00020000u;
  return d;
}
// Rows [row0, row0 + valid) of a token-major tensor whose rows are `pitch` elements apart.
__device__ __forceinline__ u32x4 tile_rsrc(const uint16_t* g, int64_t row0, int valid, int pitch) {
  return tile_desc(g, row0 * pitch * 2, valid * pitch * 2);
}

// N copies of 16 bytes per lane, at global offsets voff + STEP * j and LDS addresses
// m0v + LSTEP * j, in one statement.  The instruction's immediate offset moves both addresses,
// so M0 advances by the difference; no copy needs an address add of its own, and the wait
// states between the descriptor's last scalar write (v_readfirstlane) and its first use are paid
// once, not per copy (M0 itself needs one state before an LDS copy reads it).  STREAM: bytes read
// exactly once (the stored dS): the non-temporal hint keeps them from displacing lines that
// other workgroups read again (the K tiles of the same head).
#define HYDRA_DMA_FIRST(hint) "s_mov_b32 m0, %1\n\ts_nop 4\n\tbuffer_load_dwordx4 %0, %2, 0 offen " hint "lds\n\t"
#define HYDRA_DMA_NEXT(off, hint) \
  "s_add_u32 m0, m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %2, 0 offen offset:%c" off " " hint "lds\n\t"
template <int N, int STEP, int LSTEP, bool STREAM = false>
__device__ __forceinline__ void dma_cols(uint32_t m0v, u32x4 desc, int voff) {
  static_assert((N == 2 || N == 3) && (N - 1) * STEP < 4096, "immediate offsets");
  if constexpr (N == 3)
    asm volatile(HYDRA_DMA_FIRST("") HYDRA_DMA_NEXT("4", "") HYDRA_DMA_NEXT("5", "")
                 :
                 : "v"(voff), "s"(m0v), "s"(desc), "n"(LSTEP - STEP), "n"(STEP), "n"(2 * STEP)
                 : "memory", "m0", "scc");
  else if constexpr (STREAM)
    asm volatile(HYDRA_DMA_FIRST("nt ") HYDRA_DMA_NEXT("4", "nt ")
                 :
                 : "v"(voff), "s"(m0v), "s"(desc), "n"(LSTEP - STEP), "n"(STEP)
                 : "memory", "m0", "scc");
  else
    asm volatile(HYDRA_DMA_FIRST("") HYDRA_DMA_NEXT("4", "")
                 :
                 : "v"(voff), "s"(m0v), "s"(desc), "n"(LSTEP - STEP), "n"(STEP)
                 : "memory", "m0", "scc");
}
__device__ __forceinline__ void dma4(uint32_t m0v, u32x4 desc, int voff) {
  asm volatile(
      "s_mov_b32 m0, %1\n\t"
      "s_nop 4\n\t"
      "buffer_load_dword %0, %2, 0 offen lds"
      :
      : "v"(voff), "s"(m0v), "s"(desc)
      : "memory", "m0");
}

// Per-lane byte offset (tile-independent) for dma_tile with NW = 4 or 8 waves.  Lane L of
// wave w writes bytes [16L, 16L+16) of each 1 KB instruction, which holds rows 8j..8j+7 of
// one column block, j = w + NW*i; it fetches the logical chunk the swizzle places there
// (rows 8j + L/8 have bits 1..3 = (L/8 >> 1) and (j & 1) == (w & 1) for every i).
template <int DIM> __device__ __forceinline__ int dma_lane_off(int pitch, int head, int wave, int lane) {
  const int q = lane >> 3;
  const int lc = (lane & 7) ^ ((((q >> 1) & 1) << 2) | ((wave & 1) << 1) | (q >> 2));
  return ((8 * wave + q) * pitch + head * DIM + lc * 8) * 2;
}

// Copies a ROWS x DIM tile (NW waves, rows 8j .. 8j+7 of each column block per 1 KB
// instruction, j = wave + NW*i).  `wave` must be wave-uniform.
template <int DIM, int ROWS, int NW = 4>
__device__ __forceinline__ void dma_tile(lds_char* lds, u32x4 desc, int voff, int pitch, int wave) {
  constexpr int NINS = ROWS / 8;  // per column block
  static_assert(NINS % NW == 0, "tile must split evenly over the waves");
  const uint32_t base = __builtin_amdgcn_readfirstlane(lds_addr(lds) + wave * 1024);
  // opaque, so that the sums below are not kept in registers through the tile loop
  if constexpr (NINS > NW) asm volatile("" : "+v"(voff));
#pragma unroll
  for (int i = 0; i < NINS / NW; ++i)
    dma_cols<DIM / 64, 128, block_bytes<ROWS>()>(base + NW * i * 1024, desc, voff + 8 * NW * i * pitch * 2);
}

// A wave's own 32 rows x DIM, loaded once before its tile loop: copied into LDS by rows (one
// instruction covers 8 rows x 128 contiguous bytes) and read from there as operand fragments.
// Loading the fragments straight from global memory costs far more: each instruction then
// touches 32 rows, and the 96 of a workgroup took about 6000 cycles.  The 16-byte chunk c of a
// row's 64-column block lies at chunk c ^ (row & 7), which spreads both the copy and the reads
// over the banks.  buf: OWN_BYTES<DIM> of LDS that only this wave uses.  Rows past `valid`
// stay as they were in LDS: the caller masks them or does not store them.
template <int DIM> constexpr int own_bytes() { return 32 * DIM * 2; }
template <int DIM>
__device__ __forceinline__ void own_rows_issue(lds_char* buf, const uint16_t* g, int64_t row0, int valid, int pitch,
                                               int head, int lane) {
  const u32x4 desc = tile_rsrc(g, row0, valid, pitch);
  const uint32_t base = __builtin_amdgcn_readfirstlane(lds_addr(buf));
  const int q = lane >> 3;
  const int voff = (q * pitch + head * DIM + (((lane & 7) ^ q) << 3)) * 2;
#pragma unroll
  for (int i = 0; i < 4; ++i) dma_cols<DIM / 64, 128, 4096>(base + i * 1024, desc, voff + 8 * i * pitch * 2);
}
// f[t]: columns 16 t + 8 h .. + 7 of row m.  After the wave has waited for its copies.
template <int DIM>
__device__ __forceinline__ void own_rows_read(const lds_char* buf, int lane, bf16x8 (&f)[DIM / 16]) {
  const int m = lane & 31, h = lane >> 5;
#pragma unroll
  for (int t = 0; t < DIM / 16; ++t)
    f[t] = lds_ld16(buf, (t >> 2) * 4096 + m * 128 + (((2 * (t & 3) + h) ^ (m & 7)) << 4));
#pragma unroll
  for (int t = 0; t < DIM / 16; ++t) settle(f[t]);
}

// ------------------------------------------------------------------ accumulators -> rows
// Writes a wave's 32 rows x 64*G accumulated columns (acc[c] of column block c, transposed: the
// lane holds row m) to memory through 8 KB of LDS of its own, 64 columns at a time, so that one
// instruction stores 4 rows x 256 contiguous bytes.  Stored straight from the accumulators an
// instruction covers 32 bytes of each of 32 rows, and the output of a forward workgroup took
// 8000 cycles.  16-byte chunk c of a row lies at chunk c ^ (row & 15).  The caller has seen
// every wave past its last read of the LDS that holds buf.
constexpr int ROWS_OUT_BYTES = 32 * 256;

// Between LDS accesses of a wave whose lanes exchange data: the lanes of a wave access LDS in program
// order, and this keeps the compiler, which sees one lane's addresses, from changing that order.  It
// is no instruction.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <int G, int N>
__device__ __forceinline__ void rows_stage(lds_char* buf, int lane, const f32x16 (&acc)[N], float scale) {
  const int m = lane & 31, h = lane >> 5;
  wave_lds_order();  // after the reads of the group before
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const f32x16& x = acc[2 * G + d];
      const f32x4 v = {x[4 * rr] * scale, x[4 * rr + 1] * scale, x[4 * rr + 2] * scale, x[4 * rr + 3] * scale};
      *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(buf + m * 256 +
                                                                   (((8 * d + 2 * rr + h) ^ (m & 15)) << 4)) = v;
    }
  wave_lds_order();  // before rows_read
}
// Row and first column (of the 64) of the 16 bytes that this lane handles in step i of 8.
__device__ __forceinline__ int rows_row(int lane, int i) { return 4 * i + (lane >> 4); }
__device__ __forceinline__ int rows_col(int lane, int i) { return ((lane & 15) ^ (rows_row(lane, i) & 15)) * 4; }
__device__ __forceinline__ f32x4 rows_read(const lds_char* buf, int lane, int i) {
  return *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(buf + i * 1024 + lane * 16);
}

// A wave's output rows as a buffer of `valid` rows, `pitch_bytes` apart: the hardware's bounds
// check drops the rows past the end, with no branch per row.  All of an access's offset travels in
// its address operand and its immediate, which that check covers whatever the row count.
typedef __amdgpu_buffer_rsrc_t rows_rsrc;
__device__ __forceinline__ rows_rsrc rows_buffer(void* out, int valid, int pitch_bytes) {
  const uint64_t p = (uint64_t)(uintptr_t)out;
  // readfirstlane returns a signed int: widened as such, a low half with its top bit set would
  // fill the high half with ones
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)((uint64_t)hi << 32 | lo), 0, valid * pitch_bytes,
                                           0x00020000);
}

// The 16 bytes that this lane stores in step i, before the sum: column group g of 64.  All groups'
// loads are issued before the first is used: one workgroup runs on a CU, and nothing else hides
// the memory's latency at its end.
__device__ __forceinline__ f32x4 rows_old(rows_rsrc rs, int lane, int i, int pitch, int g) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                       rs, (rows_row(lane, i) * pitch + rows_col(lane, i)) * 4 + 256 * g, 0, 0));
}

// out[row][col] += scale * acc, rows [0, valid), `pitch` elements apart.
template <int NG>
__device__ __forceinline__ void rows_add(lds_char* buf, int lane, const f32x16 (&acc)[2 * NG], float scale, float* out,
                                         int pitch, int valid) {
  const rows_rsrc rs = rows_buffer(out, valid, pitch * 4);
  f32x4 old[NG][8];
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int i = 0; i < 8; ++i) old[g][i] = rows_old(rs, lane, i, pitch, g);
  sched_fence();
  static_for<NG>([&](auto g_) {
    constexpr int g = decltype(g_)::value;
    rows_stage<g>(buf, lane, acc, scale);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, old[g][i] + rows_read(buf, lane, i)), rs,
                                             (rows_row(lane, i) * pitch + rows_col(lane, i)) * 4 + 256 * g, 0, 0);
  });
}

// Exact merge of two partials of a row with log-sums La and Lb: weights w_x = e^(Lx - L) of their
// outputs, and L.  Two empty partials (-inf) give weights 0 and -inf, with no NaN.
__device__ __forceinline__ void merge_weights(float La, float Lb, float& L, float& wa, float& wb) {
  const float M = fmaxf(La, Lb);
  wa = 0.f;
  wb = 0.f;
  L = -INFINITY;
  if (M != -INFINITY) {
    const float ea = expf(La - M), eb = expf(Lb - M);
    const float tot = ea + eb;
    L = M + logf(tot);
    wa = ea / tot;
    wb = eb / tot;
  }
}
// A weight of 0 drops its partial, whatever that holds.
__device__ __forceinline__ float merge_value(float wa, float oa, float wb, float ob) {
  return (wa > 0.f ? wa * oa : 0.f) + (wb > 0.f ? wb * ob : 0.f);
}

// A wave's accumulators to and from its place in a part (see tiles.h).
template <int N> __device__ __forceinline__ void part_store(char* p, int lane, const f32x16 (&acc)[N]) {
#pragma unroll
  for (int d = 0; d < N; ++d)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr)
      *reinterpret_cast<f32x4*>(p + (4 * d + rr) * 1024 + lane * 16) =
          f32x4{acc[d][4 * rr], acc[d][4 * rr + 1], acc[d][4 * rr + 2], acc[d][4 * rr + 3]};
}
// Column blocks 2 g and 2 g + 1 of n parts, `part_bytes` apart, summed in the order of the parts
// with weights w(j).  Four parts' loads are in flight at a time.
template <class W>
__device__ __forceinline__ void parts_sum(const char* p, int part_bytes, int n, int g, int lane, W&& w, f32x16 (&acc)[2]) {
#pragma unroll
  for (int d = 0; d < 2; ++d) acc[d] = f32x16{};
  constexpr int AHEAD = 4;
  for (int j0 = 0; j0 < n; j0 += AHEAD) {
    f32x4 v[AHEAD][8];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
#pragma unroll
      for (int i = 0; i < 8; ++i)  // past the last part: that part again, not added
        v[u][i] = *reinterpret_cast<const f32x4*>(p + (int64_t)min(j0 + u, n - 1) * part_bytes + (8 * g + i) * 1024 +
                                                  lane * 16);
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      if (j0 + u >= n) break;
      const float x = w(j0 + u);
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i >> 2][4 * (i & 3) + e] += x * v[u][i][e];
    }
  }
}

// 64 fp32 values (valid of them in range) -> LDS, one wave.
__device__ __forceinline__ void dma_vec64(lds_char* lds, const float* g, int valid, int lane) {
  dma4(__builtin_amdgcn_readfirstlane(lds_addr(lds)), tile_desc(g, 0, valid * 4), lane * 4);
}

__device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Workgroup barrier for the tile loops: this wave's LDS reads are finished and every wave
// has arrived.  Copies into LDS are waited for explicitly (wait_dma / vmcnt) before it;
// unlike __syncthreads it does not also wait for the copies still in flight for later tiles.
__device__ __forceinline__ void barrier_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// This lane's index, computed afresh: code outside the tile loop (or rare in it) that uses it
// keeps no register alive through the loop.
__device__ __forceinline__ int lane_now() {
  int ones = -1;
  asm volatile("" : "+s"(ones));
  return __builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0));
}

// Zeroes rows >= n of a short tile that dma_tile<DIM, ROWS, NW> copied, each wave the rows of
// its own copies, after it has waited for them: a masked entry's P or dS is 0, and 0 times
// whatever LDS held in those rows need not be.
template <int DIM, int ROWS, int NW>
__device__ __forceinline__ void clear_tail(lds_char* tile, int n, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < ROWS / 8 / NW; ++i) {
    const int r = 8 * (wave + NW * i) + (lane >> 3);
    if (r < n) continue;
#pragma unroll
    for (int b = 0; b < DIM / 64; ++b)
      *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(tile + b * block_bytes<ROWS>() + r * 128 +
                                                                  (lane & 7) * 16) = u32x4{0u, 0u, 0u, 0u};
  }
}

// Workgroups are dispatched round-robin over the 8 XCDs (workgroup b runs on XCD b % 8), each
// with its own L2.  When the heads of a launch are a multiple of 8, each XCD takes whole heads
// one after another (its j-th workgroup: head (b % 8) * H / 8 + j / n_items, item j % n_items,
// heaviest first), so the workgroups running together on an XCD stream the same head's
// other-side tiles through its L2.  Otherwise the items of a head alternate over the XCDs
// (head b % H, item b / H).
constexpr int N_XCD = 8;
__device__ __forceinline__ void xcd_head_item(int b, int n_heads, int n_items, int& head, int& item) {
  if (n_heads % N_XCD == 0) {
    const int x = b % N_XCD, j = b / N_XCD;
    head = x * (n_heads / N_XCD) + j / n_items;
    item = j % n_items;
  } else {
    head = b % n_heads;
    item = b / n_heads;
  }
}

// A work item's launch record (see tiles.h), read once into scalar registers.
// Plain scalar members only: an array here would be placed in scratch memory and indexed
// dynamically.
struct Item {
  int row0, pos0, n, nr;
  int r0, p0, c0, r1, p1, c1, r2, p2, c2, r3, p3, c3;
  int edge0, d0, d1;  // document boundary of the first row, documents of the first and the last row
  int ds_slot;        // key items: first dS slot
  int t0, t1, part;   // tiles of the walk (t1 < 0: to its end), part of a split item or -1

  __device__ __forceinline__ Item(const int* items, int idx) {
    const int* s = items + (int64_t)idx * REC_INTS;
    row0 = __builtin_amdgcn_readfirstlane(s[0]);
    pos0 = __builtin_amdgcn_readfirstlane(s[1]);
    n = __builtin_amdgcn_readfirstlane(s[2]);
    nr = __builtin_amdgcn_readfirstlane(s[3]);
    r0 = __builtin_amdgcn_readfirstlane(s[4]);
    p0 = __builtin_amdgcn_readfirstlane(s[5]);
    c0 = nr > 0 ? __builtin_amdgcn_readfirstlane(s[6]) : 0;
    r1 = __builtin_amdgcn_readfirstlane(s[7]);
    p1 = __builtin_amdgcn_readfirstlane(s[8]);
    c1 = nr > 1 ? __builtin_amdgcn_readfirstlane(s[9]) : 0;
    r2 = __builtin_amdgcn_readfirstlane(s[10]);
    p2 = __builtin_amdgcn_readfirstlane(s[11]);
    c2 = nr > 2 ? __builtin_amdgcn_readfirstlane(s[12]) : 0;
    r3 = __builtin_amdgcn_readfirstlane(s[13]);
    p3 = __builtin_amdgcn_readfirstlane(s[14]);
    c3 = nr > 3 ? __builtin_amdgcn_readfirstlane(s[15]) : 0;
    edge0 = __builtin_amdgcn_readfirstlane(s[REC_EDGE]);
    d0 = __builtin_amdgcn_readfirstlane(s[REC_DOC0]);
    d1 = __builtin_amdgcn_readfirstlane(s[REC_DOC1]);
    ds_slot = __builtin_amdgcn_readfirstlane(s[REC_SLOT]);
    t0 = __builtin_amdgcn_readfirstlane(s[REC_T0]);
    t1 = __builtin_amdgcn_readfirstlane(s[REC_T1]);
    part = __builtin_amdgcn_readfirstlane(s[REC_PART]);
  }
};

// The ranges of a work item cut into tiles of B rows (the last tile of a range may be short).
// A value type of scalars: pass it by value and never take its address, so that it stays in
// scalar registers (a select between fields of a struct in memory becomes a scratch load
// with a dynamic index).
struct TileRanges {
  int r0, p0, c0, r1, p1, c1, r2, p2, c2, r3, p3, c3;
  int f1, f2, f3, nt;  // first tile of ranges 1..3, total tiles
};

__device__ __forceinline__ TileRanges tile_ranges(const Item& it, int B) {
  TileRanges R;
  R.r0 = it.r0; R.p0 = it.p0; R.c0 = it.c0;
  R.r1 = it.r1; R.p1 = it.p1; R.c1 = it.c1;
  R.r2 = it.r2; R.p2 = it.p2; R.c2 = it.c2;
  R.r3 = it.r3; R.p3 = it.p3; R.c3 = it.c3;
  R.f1 = (R.c0 + B - 1) / B;
  R.f2 = R.f1 + (R.c1 + B - 1) / B;
  R.f3 = R.f2 + (R.c2 + B - 1) / B;
  R.nt = R.f3 + (R.c3 + B - 1) / B;
  return R;
}

// Rows [row0, row0 + n) at global positions [pos0, pos0 + n).
struct Tile {
  int row0, pos0, n;
};

// Tile t < R.nt.  The kernels look a tile up once, when they start its copy, and carry it to the
// iteration that computes it: scalar work in the loops costs time of its own (all waves wait for
// the slowest at the tile's barrier).
__device__ __forceinline__ Tile tile_at(const TileRanges R, int t, int B) {
  int rr = R.r0, pp = R.p0, cc = R.c0, ff = 0;
  if (t >= R.f1) { rr = R.r1; pp = R.p1; cc = R.c1; ff = R.f1; }
  if (t >= R.f2) { rr = R.r2; pp = R.p2; cc = R.c2; ff = R.f2; }
  if (t >= R.f3) { rr = R.r3; pp = R.p3; cc = R.c3; ff = R.f3; }
  const int off = (t - ff) * B;
  return {rr + off, pp + off, min(B, cc - off)};
}

struct AttnArgs {
  const uint16_t* q;   // [nq][H][192]
  const uint16_t* k;   // [nk][Hkv][192]
  const uint16_t* v;   // [nk][Hkv][128]
  const uint16_t* o;   // bwd: final O bf16 [nq][H][128]
  const uint16_t* dO;  // bwd: [nq][H][128]
  const float* lse;    // bwd: final LSE [H][nq]
  float* out_o;        // fwd: O partial fp32
  float* out_lse;      // fwd: LSE partial
  float* dq;           // bwd accumulators
  float* dk;
  float* dv;
  float* Dvec;         // bwd: [H][nq] -rowsum(dO * O)
  float* lse2;         // bwd: [H][nq] final LSE * log2(e)
  const int* items;    // work items
  const int* cu;       // document boundaries
  int n_items;
  int H;               // query heads
  int Hkv;             // K/V heads; query head h uses K/V head h / grp
  int grp;             // H / Hkv
  int nq, nk;
  int q_s, k_s, v_s;   // elements between consecutive token rows of q, k, v (dO, O: dense)
  float scale;         // softmax scale
  // heads of one launch: K/V heads kv_head0 .. +kv_heads (key-stationary kernel), query heads
  // q_head0 .. +q_heads (query-stationary kernels)
  int kv_head0, kv_heads;
  int q_head0, q_heads;
  // stored-dS backward: dS blocks of the launch's query heads, ds_head_bytes apart; the key
  // items in row order as records (row0, rows, ranges, first slot, ranges); of each query item
  // the record of the key item that holds each range's first row
  char* ds;
  int64_t ds_head_bytes;
  const int* krec;
  const int* qslots;
  // split launches: the parts of all heads, parts per head, and the split items (merges)
  char* split;
  int n_parts;
  const int* merges;
};

// Part `part` of the launch's head `hl`.
__device__ __forceinline__ char* part_at(const AttnArgs& a, int hl, int part, int part_bytes) {
  return a.split + ((int64_t)hl * a.n_parts + part) * part_bytes;
}

// A launch list on the device (host side of a launch).
struct Launch {
  const int* units;
  int n_units;
  const int* merges;
  int n_merges, parts;
};

}  // namespace hydra
