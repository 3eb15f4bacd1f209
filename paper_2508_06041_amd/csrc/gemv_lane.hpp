// Any-precision GEMV for gfx950, one row per lane: y[o] = sum_c LUT_k[o][code_k(o,c)] * x[c]   (paper Sec. 3:
// the linear operation of a decode step; Sec. 2.2: the k-bit model is the top k planes of the parent).
//
// Layout: a plane is cut into tiles of 64 rows x 128 columns; lane l of a wavefront owns row
// 64 rb + l of the tile and reads its four 32-column words with one 128-bit load, so a wavefront load is 1 KiB
// of contiguous memory per plane.  Words are permuted and rotated as in layout_device.hpp.
//
// Why rows on lanes: every lane looks its weights up in its own row's table.  The tables of the 64 rows are
// interleaved in LDS (entry e of row l at byte e * 256 + l * 4), so lane l only ever touches bank l mod 32 and
// lookups are free of bank conflicts whatever the table size; the two-weight tables of k = 3 and k = 4, which
// cost 4 - 6 LDS cycles per lookup when a whole wavefront shares one row's table, cost 2.
// The activations are the same for all lanes.
// One right-hand side (the decode step): with every tile a lane fetches one dword of them (256 bytes per
// wavefront); before the tile is decoded the wavefront parks them in a private LDS slot.  A wavefront with at
// most four tiles per row block (rows up to 4096 columns) parks them once for its whole run instead.
// Every lane reads back 16 bytes per word (lane l takes the pairs 4 (l mod 4) .. + 3) and the multiply-add
// v_dot2c_f32_f16 reads the pair it needs from the right lane of its quad with a DPP quad broadcast: 16 registers
// hold the 64 pairs of a tile, fp32 accumulation in the lane.
// Several right-hand sides (a small dense contraction: 64 rows x up to 4 samples per wavefront), and one in some launches
// of its own (gemv_lone), run on the matrix pipe instead: v_mfma_f32_4x4x4_16b_f16 works on 16 blocks of four lanes; with the A operand of one block
// broadcast to all blocks (cbsz = 4, abid = Q) lane L gets
//     acc[i] += sum_n A(lane 4 Q + i)[n] * B(lane L)[n],  n = 0 .. 3,  i = 0 .. 3.
// (Five to eight right-hand sides: two matrix instructions per looked-up chunk, each with its four samples.)
// B = four looked-up weights of the lane's own row; A = the four activations that go with them, held by the
// lanes of quad Q: lane 4 Q + i holds sample i's chunk, acc[i] is sample i's sum.  Quad Q of the wavefront holds
// two of the tile's 32 chunks of four activations (LaneRawX says which), so 4 registers carry a tile's activations and
// every lookup serves four (eight) samples: up to eight right-hand sides share a pass over the planes.  They are loaded with the
// tile in that form.  (Parked in LDS sample by sample and read back, as one right-hand side is, they cost a tile of four samples
// four LDS writes and two reads per lane, at k = 4 two reads, a write and a wait for each sample more.  us per call, parked -> loaded:
// 14336 x 4096 B = 4, k = 6 15.6 -> 14.5, B = 2, k = 3 7.9 -> 7.4, B = 8, k = 3 10.4 -> 8.4; 20000 x 4096 B = 3, k = 4 15.7 -> 13.5; 4096 x
// 14336 B = 8, k = 3 11.8 -> 11.3.)
// Each lane accumulates its own row: no cross-lane reduction.  A workgroup is eight wavefronts that split the
// columns of the same 64 rows and share the tables; their eight partial sums per row meet in LDS.
//
//   k <= 4   : two weights per lookup, tables of 64 / 256 fp16 pairs per row (16 / 64 KiB per workgroup); k = 1, 2 are
//              k = 3 without the planes that are not read
//   k >= 5   : one weight per lookup (table of 2^k entries per row, 8 .. 64 KiB), two results packed into one
//              register of the B operand
// One kernel serves every bitwidth from 1 to 8: a workgroup reads the bitwidth of its job (a value, or the word a
// selector wrote in device memory) and branches to the code of that bitwidth.  Every branch of the kernels for large
// launches (G = 1) stays within 128 vector registers and the workgroup's LDS is sized for the largest tables (64 KiB), so
// two workgroups share a compute unit whatever the bitwidth.  The host looks at a bitwidth that a call names to choose the
// launch; what a workgroup then runs, and with it the order of the additions, is the same if the device says it.
// Small launches give a workgroup 64 / G rows, G = 2, 4, 8 (gemv_narrow).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "gemv_common.hpp"
#include "layout.hpp"
#include "layout_device.hpp"

namespace dpllm {

constexpr int kLaneWaves = 8;            // wavefronts per workgroup
constexpr int kLaneThreads = 64 * kLaneWaves;

template <int K>
struct LaneDecode {
  static constexpr bool pair = K <= 4;                        // two weights per lookup
  static constexpr int entries = K <= 3 ? 64 : K == 4 ? 256 : (1 << K);
  static constexpr int table_bytes = entries * 256;           // 64 lanes interleaved, 4 bytes per lane and entry
  static constexpr int share = entries / kLaneWaves;          // entries a wavefront builds per row block
  // k <= 3: the bits of an entry number that carry a code; the byte of a merged word holds [a2 a1 a0 b2 b1 b0 . .]
  // above two bits of other weights, and with k < 3 planes the low bits of a and b are not there
  static constexpr uint32_t pair_mask = K == 3 ? 0x3fu : K == 2 ? 0x36u : 0x24u;
  // single-weight schemes: the byte of column `col` is its code; which of the eight merged words, which byte
  static constexpr int d = 8 - K;
  __host__ __device__ static constexpr int top(int col) { return (col_to_pos(col) + d) & 31; }
  __host__ __device__ static constexpr int word(int col) { return top(col) & 7; }
  __host__ __device__ static constexpr int rot(int c) { return (c + 1) & 7; }
  __host__ __device__ static constexpr int byte(int col) { return ((top(col) - rot(word(col))) & 31) >> 3; }
};
constexpr int kLaneRedBytes = kLaneWaves * 64 * 4;            // the partial sums of the eight wavefronts, per sample
constexpr int kLaneKeepTiles = 4;                             // a wavefront with so few tiles per row block keeps their activations in LDS
constexpr int kLaneTableBytes = 65536;                        // the largest tables: k = 4 (pairs) and k = 8
static_assert(LaneDecode<2>::table_bytes <= kLaneTableBytes && LaneDecode<3>::table_bytes <= kLaneTableBytes && LaneDecode<4>::table_bytes <= kLaneTableBytes &&
              LaneDecode<5>::table_bytes <= kLaneTableBytes && LaneDecode<6>::table_bytes <= kLaneTableBytes &&
              LaneDecode<7>::table_bytes <= kLaneTableBytes && LaneDecode<8>::table_bytes <= kLaneTableBytes, "tables fit");
// G column groups per wavefront (see below); bytes from one group's parked activations to the next: 64 more than a
// tile's 256, so that the groups' reads of the same word fall on different banks
constexpr int kLaneGroupStride = 320;
// NB: 1 right-hand side per pass on the vector pipe, 4 or 8 on the matrix pipe, 2: one on the matrix pipe.
__host__ __device__ constexpr int lane_samples(int nb) { return nb == 2 ? 1 : nb; }
__host__ __device__ constexpr int lane_sets(int nb) { return nb == 8 ? 2 : 1; }   // of four samples
// One right-hand side: a slot per wavefront for the parked activations of its tiles (G of them); with one group four more
// for the tiles it keeps across row blocks.  Several right-hand sides read their activations from memory in the form they are used in.
template <int NB, int G>
__host__ __device__ constexpr int lane_x_bytes() {
  return NB > 1 ? 0 : G > 1 ? G * kLaneGroupStride : 256 + kLaneKeepTiles * 256;
}
// Tables, partial sums, activation slots, and (one sample: the decode step) room for the selectors.  At k = 4
// and G = 1 the 256 bytes a wavefront needs to re-pair the activations of one sample are borrowed from the partial sums, which are not in
// use between the barrier that opens a row block and the stores that close it (its own partial sums).
// Eight samples: their partial sums take the place of the tables, which are done with by then (at G = 1 two barriers
// more per row block keep two workgroups per compute unit).
template <int NB>
__host__ __device__ constexpr int lane_red_offset() { return NB == 8 ? 0 : kLaneTableBytes; }
template <int NB>
__host__ __device__ constexpr int lane_x_offset() { return NB == 8 ? kLaneTableBytes : kLaneTableBytes + lane_samples(NB) * kLaneRedBytes; }
template <int NB, int G>
__host__ __device__ constexpr int lane_lds_bytes() {
  return lane_x_offset<NB>() + kLaneWaves * lane_x_bytes<NB, G>() + (NB == 1 ? kSelSharedBytes : 0);
}
static_assert(8 * kLaneRedBytes <= LaneDecode<3>::table_bytes, "room for the sums of eight samples");
static_assert(lane_lds_bytes<8, 1>() <= 81920 && lane_lds_bytes<4, 1>() <= 81920 && lane_lds_bytes<1, 1>() <= 81920, "two workgroups per compute unit");
static_assert(lane_lds_bytes<1, 8>() <= 163840 && lane_lds_bytes<4, 8>() <= 163840 && lane_lds_bytes<8, 4>() <= 163840,
              "one workgroup per compute unit (such a launch has no more of them)");

// x pair held by lane Q of the quad, times the looked-up pair, added to acc
template <int Q>
__device__ __forceinline__ void dot2_quad(float& acc, uint32_t xreg, uint32_t wpair) {
  static_assert(Q >= 0 && Q < 4, "quad lane");
  if constexpr (Q == 0) asm("v_dot2c_f32_f16_dpp %0, %1, %2 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(xreg), "v"(wpair));
  if constexpr (Q == 1) asm("v_dot2c_f32_f16_dpp %0, %1, %2 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(xreg), "v"(wpair));
  if constexpr (Q == 2) asm("v_dot2c_f32_f16_dpp %0, %1, %2 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(xreg), "v"(wpair));
  if constexpr (Q == 3) asm("v_dot2c_f32_f16_dpp %0, %1, %2 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(xreg), "v"(wpair));
}

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// acc[i] += sum_n x(lane 4 Q + i)[n] * w[n]: x = four fp16 (what this lane holds matters to the lanes whose Q is
// this lane's quad), w = the four weights {w0.lo, w0.hi, w1.lo, w1.hi} of this lane's row.  With G groups Q counts
// the quads of the lane's own group: 16 / G of them share an operand.
template <int Q, int G>
__device__ __forceinline__ void mfma_chunk(f32x4& acc, uint64_t x, uint32_t w0, uint32_t w1) {
  static_assert(Q >= 0 && Q < 16 / G, "quad of the group");
  constexpr int cbsz = G == 1 ? 4 : G == 2 ? 3 : G == 4 ? 2 : 1;
  const uint64_t w = (uint64_t)w0 | ((uint64_t)w1 << 32);
  acc = __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(f16x4, x), __builtin_bit_cast(f16x4, w), acc, cbsz, Q, 0);
}

// The lane's partial sums.  One sample: four fp32 sums that take turns.  Four samples: two sets of four (sum i
// of a set = sample i) that take turns, so that no matrix instruction waits for the one before it and no chain of
// additions holds more than half of the columns.  Eight: two such sets for samples 0 .. 3 and two for 4 .. 7.
template <int NB>
struct LaneAcc;
template <>
struct LaneAcc<1> {
  float v[4];
  __device__ __forceinline__ void zero() { v[0] = v[1] = v[2] = v[3] = 0.f; }
  // between a step and sum(): a dot product's result may be read by another kind of vector instruction three wait states later;
  // the compiler keeps that distance behind instructions it knows, not behind inline asm
  __device__ __forceinline__ void settle() { asm("s_nop 2" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3])); }
  __device__ __forceinline__ float sum(int) const { return (v[0] + v[1]) + (v[2] + v[3]); }
};
template <>
struct LaneAcc<2> {
  f32x4 v[2];
  __device__ __forceinline__ void zero() { v[0] = v[1] = f32x4{0.f, 0.f, 0.f, 0.f}; }
  __device__ __forceinline__ void settle() {}
  __device__ __forceinline__ float sum(int) const { return v[0][0] + v[1][0]; }   // (four times the same)
};
template <>
struct LaneAcc<4> {
  f32x4 v[2];
  __device__ __forceinline__ void zero() { v[0] = v[1] = f32x4{0.f, 0.f, 0.f, 0.f}; }
  __device__ __forceinline__ void settle() {}
  __device__ __forceinline__ float sum(int b) const { return v[0][b] + v[1][b]; }
};

template <>
struct LaneAcc<8> {
  f32x4 v[4];
  __device__ __forceinline__ void zero() { v[0] = v[1] = v[2] = v[3] = f32x4{0.f, 0.f, 0.f, 0.f}; }
  __device__ __forceinline__ void settle() {}
  __device__ __forceinline__ float sum(int b) const { return v[2 * (b >> 2)][b & 3] + v[2 * (b >> 2) + 1][b & 3]; }
};

// LDS address of entry (byte N of t) in the lane's table column: byte 2 = which table (lanecol's), byte 1 = the entry,
// byte 0 = lane * 4
template <int N>
__device__ __forceinline__ uint32_t lane_entry_addr(uint32_t t, uint32_t lanecol) {
  constexpr uint32_t sel = 0x0c020000u | ((4u + N) << 8);   // {0, lanecol.byte2, t.byteN, lanecol.byte0}
  return __builtin_amdgcn_perm(t, lanecol, sel);
}

// The same for an entry byte whose two high bits are not part of the entry number: byte 1 of addr = byte N of t
// with those bits cleared, in one sub-dword instruction; the other bytes of addr keep what they hold (lane * 4,
// put there once).  mask: 0x3f in a register.
template <int N>
__device__ __forceinline__ void lane_entry_addr_masked(uint32_t t, uint32_t mask, uint32_t& addr) {
  static_assert(N >= 0 && N < 4, "byte");
  if constexpr (N == 0) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_0 src1_sel:DWORD" : "+v"(addr) : "v"(t), "v"(mask));
  if constexpr (N == 1) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_1 src1_sel:DWORD" : "+v"(addr) : "v"(t), "v"(mask));
  if constexpr (N == 2) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_2 src1_sel:DWORD" : "+v"(addr) : "v"(t), "v"(mask));
  if constexpr (N == 3) asm("v_and_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:DWORD" : "+v"(addr) : "v"(t), "v"(mask));
}

__device__ __forceinline__ uint32_t lds_u32(const char* lds, uint32_t addr) { return *reinterpret_cast<const uint32_t*>(lds + addr); }

// ---- a tile: the lane's row, 128 columns, and the lane's part of the activations -------------------------------
// One sample: a dword of the tile's 128 activations per lane (and group), parked in LDS before the tile is decoded.
// Several: sixteen bytes per lane, group and four samples, which the lanes exchange for the operands of the matrix instructions
// (LaneX::settle); nothing is parked.  The 32 chunks of a tile (four activations each, 8 j + 2 q + half: see mfma_chunk) go in twos,
// an eight of columns each, to the P = 16 / G quads of a group: quad n has the eights n, n + P, ..; its lane 4 n + i needs those of sample i.
// They are loaded by lane i P + n of the group instead, so that neighbouring lanes read neighbouring memory: four lanes of a quad
// in four vectors cost the vector cache about 90 cycles a load (3400 x 14336 k = 5, four column groups, eight samples that way 20.6 us, five,
// with four lanes in one vector in every second load, 16.6).
// At k = 4 a chunk is two pairs of columns (see nibble_pair_col_hi): merged words q = 0 and 3 of word j take the odd and the
// even ones of its columns 0 .. 7 and 16 .. 23, q = 2 and 1 those of columns 8 .. 15 and 24 .. 31.  A lane gets both eights and
// picks halves.
template <int K, int NB, int G>
struct LaneRawX {
  static constexpr int P = 16 / G;
  static constexpr int kLoads = G;
  u32x4 v[lane_sets(NB)][kLoads];
  // what lane `lane` loads: of which sample (of four), and the column of load r inside the tile
  static __device__ __forceinline__ int sample(int lane) { return lane % (4 * P) / P; }
  static __device__ __forceinline__ int column(int lane, int r) {
    const int n = lane % P;
    if constexpr (K == 4 && G == 2) return 32 * (n >> 1) + 8 * (n & 1) + 16 * r;
    if constexpr (K == 4 && G > 2) return 8 * G * n + 8 * r;
    return 8 * (r * P + n);
  }
  // the lane whose loads quad n of the lane's group needs for its own sample (as the address of a bpermute)
  static __device__ __forceinline__ int source(int lane, int n) { return 4 * ((lane & -(4 * P)) + (lane & 3) * P + n); }
};
// One sample on the matrix pipe: every lane loads the eights of its own quad (four lanes the same).
template <int K>
struct LaneRawX<K, 2, 1> {
  static constexpr int P = 16;
  static constexpr int kLoads = K == 4 ? 2 : 1;
  u32x4 v[1][kLoads];
  static __device__ __forceinline__ int sample(int) { return 0; }
  static __device__ __forceinline__ int column(int lane, int r) {
    const int n = lane >> 2;
    return K == 4 ? 32 * (n >> 2) + 8 * ((n ^ n >> 1) & 1) + 16 * r : 8 * n;
  }
};
template <int K, int G>
struct LaneRawX<K, 1, G> {
  uint32_t v[1][G];
};

template <int K, int NB, int G = 1>
struct LaneTile {
  u32x4 w[K];
  LaneRawX<K, NB, G> x;
};

// the lane's dword of the 128 activations of tile cc (address clamped to the row).  Columns past the end of a
// ragged row hold zero codes, whose centroid is not zero: their activations must read as 0, which lane_mask_x
// sees to when the value is used.  (Masking right after the load would make the wavefront wait for the load,
// and with it for every tile load issued before it, at the point of issue.)
__device__ __forceinline__ uint32_t lane_load_x(const GemvJob& job, int cc, int lane) {
  const int c = cc * 128 + lane * 2, last = job.ncw * 32 - 2;
  return *reinterpret_cast<const DPLLM_GLOBAL uint32_t*>(as_global(job.x) + min(c, last));
}
__device__ __forceinline__ uint32_t lane_mask_x(const GemvJob& job, int cc, int lane, uint32_t v) {
  return cc * 128 + lane * 2 <= job.ncw * 32 - 2 ? v : 0u;
}

// Several samples: asks for the lane's part of the activations of tile `tile` (clamped to the row).  rows[s]: the vector of
// the lane's sample among 4 s .. 4 s + 3; a group with fewer than NB samples re-reads its last one (the sums are not stored).
template <int K, int NB, int G>
__device__ __forceinline__ void lane_load_raw(LaneRawX<K, NB, G>& x, const DPLLM_GLOBAL uint16_t* const (&rows)[lane_sets(NB)], int tile, int ncw, int lane) {
#pragma unroll
  for (int r = 0; r < LaneRawX<K, NB, G>::kLoads; ++r) {
    const int c = min(tile * 128 + LaneRawX<K, NB, G>::column(lane, r), ncw * 32 - 8);
#pragma unroll
    for (int s = 0; s < lane_sets(NB); ++s) x.v[s][r] = *reinterpret_cast<const DPLLM_GLOBAL u32x4*>(rows[s] + c);
  }
}
// columns past the end of a ragged row (eight are inside or outside together) read as 0
template <int K, int NB, int G>
__device__ __forceinline__ void lane_mask_raw(LaneRawX<K, NB, G>& x, int tile, int ncw, int lane) {
#pragma unroll
  for (int r = 0; r < LaneRawX<K, NB, G>::kLoads; ++r) {
    const bool inside = tile * 128 + LaneRawX<K, NB, G>::column(lane, r) < ncw * 32;
#pragma unroll
    for (int s = 0; s < lane_sets(NB); ++s) x.v[s][r] = inside ? x.v[s][r] : u32x4{0u, 0u, 0u, 0u};
  }
}
template <int K, int NB, int G>
__device__ __forceinline__ void lane_sample_rows(const GemvJob& job, int lane, const DPLLM_GLOBAL uint16_t* (&rows)[lane_sets(NB)]) {
#pragma unroll
  for (int s = 0; s < lane_sets(NB); ++s)
    rows[s] = as_global(job.x) + (size_t)min(4 * s + LaneRawX<K, NB, G>::sample(lane), job.nsamples - 1) * job.ncw * 32;
}

// Loads are never predicated, which keeps the compiler's outstanding-load counts exact.  `real` = false (ring
// slots past the end of the run): the K loads still issue, but all from the first 16 bytes of the activation
// vector, which is hot in L2, so they cost no HBM traffic; the values are never decoded.
template <int K, int NB>
__device__ __forceinline__ void lane_load_tile(LaneTile<K, NB>& t, const GemvJob& job, int rb, int cc, int lane, bool real) {
  const DPLLM_GLOBAL u32x4* planes = as_global(reinterpret_cast<const u32x4*>(job.arena)) + ((size_t)rb * job.ncc + cc) * 64 + lane;
  const DPLLM_GLOBAL u32x4* p = real ? planes : as_global(reinterpret_cast<const u32x4*>(job.x));
  const size_t stride = real ? (size_t)job.plane_stride_u4 : 0;
#pragma unroll
  for (int b = 0; b < K; ++b) t.w[b] = load_stream(p + (size_t)b * stride);
}

// Parks a tile's activations in LDS in the form the lanes read back: 64 dwords, dword 16 j + n = pair n of word
// j; chunk g of the tile (dwords 2 g, 2 g + 1) goes with the lookups of pairs 2 (g mod 8), + 1 of word g / 8.
// k != 4: the natural pairs (2i, 2i+1), so the lane's dword goes straight to `ready`.
// k = 4: the pairs (x[col_hi], x[col_lo]) of merged word q, byte m (see nibble_pair_col_hi / _lo), cut from a
// natural copy in `scratch`.
template <int K>
__device__ __forceinline__ void lane_park_x(uint32_t x, int lane, char* scratch, char* ready) {
  if constexpr (K == 4) {
    *reinterpret_cast<uint32_t*>(scratch + lane * 4) = x;
    lds_order();
    const int j = lane >> 4, q = (lane >> 2) & 3, m = lane & 3, mr = (m + 3) & 3;
    const int ca = q == 0 ? 17 + 2 * m : q == 1 ? 8 + 2 * m : q == 2 ? 25 + 2 * m : 2 * m;
    const int cb = q == 0 ? 1 + 2 * m : q == 1 ? 24 + 2 * mr : q == 2 ? 9 + 2 * m : 16 + 2 * mr;
    const uint32_t lo = *reinterpret_cast<const uint16_t*>(scratch + (j * 32 + ca) * 2);
    const uint32_t hi = *reinterpret_cast<const uint16_t*>(scratch + (j * 32 + cb) * 2);
    *reinterpret_cast<uint32_t*>(ready + lane * 4) = lo | (hi << 16);
  } else {
    *reinterpret_cast<uint32_t*>(ready + lane * 4) = x;
  }
  lds_order();
}

// ---- entry words of one 32-column word -----------------------------------------------------------------------
// k = 3: four words of four bytes (8 a + b) + 64 (two bits of other weights, cleared when the address is formed),
// the pairs (2i, 2i+1), i = 4 jj + n (word 3 is left rotated by one byte: its pair n sits in byte n + 1)
// k = 1, 2: the same words without the planes that are not read (the bits in their places are cleared too)
template <int K>
__device__ __forceinline__ void lane_entries3(const uint32_t (&w)[K], uint32_t (&T)[4], const MergeMasks<3>& M) {
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    uint32_t o = w[0];
    if constexpr (K == 2) o = bfi_v(M.m[2 * jj], w[0], w[1]);
    if constexpr (K == 3) o = bfi_v(M.m[2 * jj], w[0], bfi_v(M.m[2 * jj + 1], w[1], w[2]));
    T[jj] = jj == 3 ? o : __builtin_rotateright32(o, 2 * jj + 2);   // jj = 3: a whole byte, taken care of by the byte index
  }
}

// two-weight schemes: eight lookups from entry words JA, JA + 1 (S: byte shift of word 3, see lane_entries3)
// k = 3 (S = 1): a[] = eight address registers holding lane * 4, mask = 0x3f
template <int JA, int S>
__device__ __forceinline__ void lane_issue_pairs(const uint32_t (&T)[4], uint32_t lanecol, const char* lds, uint32_t (&v)[8],
                                                 uint32_t (&a)[8], uint32_t mask) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t t = T[JA + h];
    if constexpr (S == 1) {
      if (JA + h == 3) {
        lane_entry_addr_masked<1>(t, mask, a[4 * h + 0]);
        lane_entry_addr_masked<2>(t, mask, a[4 * h + 1]);
        lane_entry_addr_masked<3>(t, mask, a[4 * h + 2]);
        lane_entry_addr_masked<0>(t, mask, a[4 * h + 3]);
      } else {
        lane_entry_addr_masked<0>(t, mask, a[4 * h + 0]);
        lane_entry_addr_masked<1>(t, mask, a[4 * h + 1]);
        lane_entry_addr_masked<2>(t, mask, a[4 * h + 2]);
        lane_entry_addr_masked<3>(t, mask, a[4 * h + 3]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * h + i] = lds_u32(lds, a[4 * h + i]);
    } else {
      v[4 * h + 0] = lds_u32(lds, lane_entry_addr<0>(t, lanecol));
      v[4 * h + 1] = lds_u32(lds, lane_entry_addr<1>(t, lanecol));
      v[4 * h + 2] = lds_u32(lds, lane_entry_addr<2>(t, lanecol));
      v[4 * h + 3] = lds_u32(lds, lane_entry_addr<3>(t, lanecol));
    }
  }
}

// One sample: the eight lookups of entry words JA, JA + 1 are the pairs 4 JA .. 4 JA + 7 of the word, which the
// lanes JA, JA + 1 of the quad hold in x.  Last lookup first: LDS answers in issue order, so one counter wait
// covers the eight.
template <int JA>
__device__ __forceinline__ void lane_consume_pairs(const uint32_t (&v)[8], const u32x4& x, float (&acc)[4]) {
  dot2_quad<JA + 1>(acc[3], x.w, v[7]);
  dot2_quad<JA + 1>(acc[2], x.z, v[6]);
  dot2_quad<JA + 1>(acc[1], x.y, v[5]);
  dot2_quad<JA + 1>(acc[0], x.x, v[4]);
  dot2_quad<JA>(acc[3], x.w, v[3]);
  dot2_quad<JA>(acc[2], x.z, v[2]);
  dot2_quad<JA>(acc[1], x.y, v[1]);
  dot2_quad<JA>(acc[0], x.x, v[0]);
}

// single-weight schemes: the eight lookups of columns 8 JJ .. 8 JJ + 7
template <int K, int JJ>
__device__ __forceinline__ void lane_issue_singles(const uint32_t (&R)[8], uint32_t lanecol, const char* lds, uint32_t (&v)[8]) {
  using D = LaneDecode<K>;
#define DPLLM_LANE_LOOKUP(N)                                                                        \
  {                                                                                                 \
    constexpr int ce = 8 * JJ + 2 * N, co = ce + 1;                                                 \
    v[2 * N] = lds_u32(lds, lane_entry_addr<D::byte(ce)>(R[D::word(ce)], lanecol));                 \
    v[2 * N + 1] = lds_u32(lds, lane_entry_addr<D::byte(co)>(R[D::word(co)], lanecol));             \
  }
  DPLLM_LANE_LOOKUP(0) DPLLM_LANE_LOOKUP(1) DPLLM_LANE_LOOKUP(2) DPLLM_LANE_LOOKUP(3)
#undef DPLLM_LANE_LOOKUP
}

// a table entry is an fp16 in the low half of a dword: two of them pack into one fp16 pair.  One sample: columns
// 8 JJ .. + 7 of the word are the pairs lane JJ of the quad holds
template <int JJ>
__device__ __forceinline__ void lane_consume_singles(const uint32_t (&v)[8], const u32x4& x, float (&acc)[4]) {
  dot2_quad<JJ>(acc[3], x.w, v[6] | (v[7] << 16));
  dot2_quad<JJ>(acc[2], x.z, v[4] | (v[5] << 16));
  dot2_quad<JJ>(acc[1], x.y, v[2] | (v[3] << 16));
  dot2_quad<JJ>(acc[0], x.x, v[0] | (v[1] << 16));
}

// k = 1, 2 use the masks of k = 3
template <int K>
using LaneMasks = MergeMasks<(K < 3 ? 3 : K)>;

// The merge tree with its masks in vector registers (full-rate instructions).  Two workgroups per compute unit (ROOM: one) leave k = 7, 8
// no registers to spare for fifteen masks; they keep them in the instructions there.  us per call with one workgroup, masks in the
// instructions -> in registers: 2500 x 6688 k = 7 9.3 -> 8.7, 4096 x 4096 k = 7 7.2 -> 6.9, 4096 x 11008 k = 7 13.6 -> 12.6, k = 8 14.1 ->
// 13.8, 8192 x 8192 k = 7 16.4 -> 15.7.  Nor do they leave any at k = 6 with eight samples, whose operands take sixteen more: with masks in
// registers that code spilled three, and every launch of its kernel came with scratch memory (us per call of eight, then -> now: 9000 x 11008
// k = 6 31.2 -> 29.3, 14336 x 4096 k = 6 16.0 -> 15.2, k = 3 9.7 -> 9.5).
template <int K, int NB, bool ROOM>
__device__ __forceinline__ void lane_merge_fields(const uint32_t (&w)[K], uint32_t (&R)[8], const LaneMasks<K>& M) {
  if constexpr (K <= (NB == 8 ? 5 : 6) || ROOM) merge_byte_fields_v<K, LaneDecode<K>::d>(w, R, M);
  else merge_byte_fields<K, LaneDecode<K>::d>(w, R);
}

// ---- one tile -------------------------------------------------------------------------------------------------
// Lookups run in chunks of eight; the next chunk's lookups are issued before the current chunk's multiply-adds.
// One sample: mine is where this lane finds its part of its tile's parked activations, the 16 bytes of its quad
// lane in word 0 (slot + 16 * (lane mod 4)), those of word j 64 j bytes on.
template <int K, int NB, int G>
struct LaneX {   // several samples: operands of the matrix instructions
  uint64_t a[lane_sets(NB)][2 * G];   // a[s][h]: the h-th chunk of the lane's quad (see LaneRawX), of sample 4 s + lane mod 4
  // which quad of the group and which of its operands holds chunk c
  static constexpr int quad(int c) {
    if constexpr (K == 4) {
      const int j = c >> 3, q = (c >> 1) & 3, t = (q ^ q >> 1) & 1;
      return G == 1 ? c >> 1 : G == 2 ? 2 * j + t : G == 4 ? j : j >> 1;
    }
    return (c >> 1) % (16 / G);
  }
  static constexpr int operand(int c) {
    if constexpr (K == 4) {
      const int j = c >> 3, q = (c >> 1) & 3, t = (q ^ q >> 1) & 1, even = q & 1, half = c & 1;
      return G == 1 ? half : G == 2 ? 2 * even + half : G == 4 ? 4 * t + 2 * even + half : 8 * (j & 1) + 4 * t + 2 * even + half;
    }
    return 2 * ((c >> 1) / (16 / G)) + (c & 1);
  }
  // lo and hi: columns 8 t .. + 7 and 16 + 8 t .. + 7 of a word.  Odd columns: pair m = (hi[2 m + 1], lo[2 m + 1]); even ones: pair m =
  // (lo[2 m], hi[2 ((m + 3) mod 4)])
  static __device__ __forceinline__ void odd_pairs(uint64_t (&o)[2], const u32x4& lo, const u32x4& hi) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      o[i] = (uint64_t)__builtin_amdgcn_perm(lo[2 * i + 1], hi[2 * i + 1], 0x07060302u) << 32 | __builtin_amdgcn_perm(lo[2 * i], hi[2 * i], 0x07060302u);
  }
  static __device__ __forceinline__ void even_pairs(uint64_t (&o)[2], const u32x4& lo, const u32x4& hi) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      o[i] = (uint64_t)__builtin_amdgcn_perm(hi[2 * i], lo[2 * i + 1], 0x05040100u) << 32 | __builtin_amdgcn_perm(hi[(2 * i + 3) & 3], lo[2 * i], 0x05040100u);
  }
  static __device__ __forceinline__ u32x4 pull(int from, const u32x4& v) {
    return u32x4{(uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)v.x), (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)v.y),
                 (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)v.z), (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)v.w)};
  }
  __device__ __forceinline__ void settle(const LaneRawX<K, NB, G>& raw, int lane) {
    using Raw = LaneRawX<K, NB, G>;
    const int n = (lane >> 2) % Raw::P;          // the lane's quad in its group
#pragma unroll
    for (int s = 0; s < lane_sets(NB); ++s) {
      if constexpr (K == 4 && G == 1) {
        // quad 4 j + q: q = 0, 2 take odd columns, 1, 3 even ones
        const bool even = n & 1;
        u32x4 lo = raw.v[s][0], hi = raw.v[s][Raw::kLoads - 1];
        if constexpr (NB > 2) {
          const int at = Raw::source(lane, (n & ~3) + ((n ^ n >> 1) & 1));
          lo = pull(at, raw.v[s][0]);
          hi = pull(at + 8, raw.v[s][0]);
        }
        const uint32_t sel = even ? 0x01000504u : 0x07060302u;   // even: the low half of the pair comes from lo
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const uint32_t h0 = even ? +hi[(2 * i + 3) & 3] : +hi[2 * i], h1 = even ? +hi[2 * i] : +hi[2 * i + 1];
          a[s][i] = (uint64_t)__builtin_amdgcn_perm(lo[2 * i + 1], h1, sel) << 32 | __builtin_amdgcn_perm(lo[2 * i], h0, sel);
        }
      } else {
        u32x4 v[G];
#pragma unroll
        for (int r = 0; r < G; ++r) {
          if constexpr (NB > 2) v[r] = pull(Raw::source(lane, n), raw.v[s][r]);
          else v[r] = raw.v[s][r];
        }
        if constexpr (K == 4) {
          // G = 2: (odd, even) of one t; G = 4: of t = 0, 1 (loads 0, 2 and 1, 3); G = 8: of two words
#pragma unroll
          for (int u = 0; u < G / 2; ++u) {
            const int at = G == 2 ? 0 : 4 * (u >> 1) + (u & 1);
            const u32x4 &lo = v[at], &hi = v[at + (G == 2 ? 1 : 2)];
            uint64_t o[2], e[2];
            odd_pairs(o, lo, hi);
            even_pairs(e, lo, hi);
            a[s][4 * u] = o[0]; a[s][4 * u + 1] = o[1];
            a[s][4 * u + 2] = e[0]; a[s][4 * u + 3] = e[1];
          }
        } else {
#pragma unroll
          for (int r = 0; r < G; ++r) {
            a[s][2 * r] = (uint64_t)v[r].y << 32 | v[r].x;
            a[s][2 * r + 1] = (uint64_t)v[r].w << 32 | v[r].z;
          }
        }
      }
    }
  }
  __device__ __forceinline__ void load() {}   // (nothing is read back)
  __device__ __forceinline__ void load_word(int) {}
};
template <int K, int G>
struct LaneX<K, 1, G> {
  u32x4 q[4];   // q[j][m] = pair 4 (lane mod 4) + m of word j
  const char* mine;
  __device__ __forceinline__ void load() {
#pragma unroll
    for (int j = 0; j < 4; ++j) load_word(j);
  }
  __device__ __forceinline__ void load_word(int j) { q[j] = *reinterpret_cast<const u32x4*>(mine + j * 64); }
};
// chunk C of the tile for four samples or eight (chunks take turns in the two accumulator sets of four samples)
template <int C, int K, int NB, int G>
__device__ __forceinline__ void lane_mac_chunk(uint32_t w0, uint32_t w1, const LaneX<K, NB, G>& x, LaneAcc<NB>& acc) {
  constexpr int Q = LaneX<K, NB, G>::quad(C), h = LaneX<K, NB, G>::operand(C);
  mfma_chunk<Q, G>(acc.v[C & 1], x.a[0][h], w0, w1);
  if constexpr (NB == 8) mfma_chunk<Q, G>(acc.v[2 + (C & 1)], x.a[1][h], w0, w1);
}

// the eight lookups of entry words JA, JA + 1 of word J: chunks 8 J + 2 JA .. + 3
template <int JA, int J, int K, int G>
__device__ __forceinline__ void lane_mac_pairs(const uint32_t (&v)[8], const LaneX<K, 1, G>& x, LaneAcc<1>& acc) {
  lane_consume_pairs<JA>(v, x.q[J], acc.v);
}
template <int JA, int J, int K, int NB, int G>
__device__ __forceinline__ void lane_mac_pairs(const uint32_t (&v)[8], const LaneX<K, NB, G>& x, LaneAcc<NB>& acc) {
  lane_mac_chunk<8 * J + 2 * JA + 3>(v[6], v[7], x, acc);
  lane_mac_chunk<8 * J + 2 * JA + 2>(v[4], v[5], x, acc);
  lane_mac_chunk<8 * J + 2 * JA + 1>(v[2], v[3], x, acc);
  lane_mac_chunk<8 * J + 2 * JA + 0>(v[0], v[1], x, acc);
}
// the lookups of columns 8 JJ .. + 7 of word J: chunks 8 J + 2 JJ, + 1
template <int JJ, int J, int K, int G>
__device__ __forceinline__ void lane_mac_singles(const uint32_t (&v)[8], const LaneX<K, 1, G>& x, LaneAcc<1>& acc) {
  lane_consume_singles<JJ>(v, x.q[J], acc.v);
}
template <int JJ, int J, int K, int NB, int G>
__device__ __forceinline__ void lane_mac_singles(const uint32_t (&v)[8], const LaneX<K, NB, G>& x, LaneAcc<NB>& acc) {
  lane_mac_chunk<8 * J + 2 * JJ + 1>(v[4] | (v[5] << 16), v[6] | (v[7] << 16), x, acc);
  lane_mac_chunk<8 * J + 2 * JJ + 0>(v[0] | (v[1] << 16), v[2] | (v[3] << 16), x, acc);
}

// words: how many of the lane's four words lie inside the row, ragged: not all four in every lane (wave-uniform).  The
// activations of the others are zero, but their codes are zero too, and an infinite centroid of that code would make
// 0 x inf; k <= 2 clears what those lookups return.
// LAZY: spent(tw) runs as soon as the planes tw (and what the activations were loaded into) may be asked for anew; one sample's
// activations are read back a word at a time, which takes 8 registers instead of 16.  ROOM as in lane_merge_fields.
struct LaneNothing {
  template <class Planes>
  __device__ __forceinline__ void operator()(Planes&) const {}
};
template <int K, int NB, int G, bool LAZY = false, bool ROOM = (G > 1), int H = K, class Spent = LaneNothing>
__device__ __forceinline__ void lane_compute(u32x4 (&tw)[H], uint32_t lanecol, const char* lds, LaneX<K, NB, G>& x,
                                             LaneAcc<NB>& acc, uint32_t (&addr)[8], uint32_t mask, const LaneMasks<K>& M, int words, bool ragged,
                                             Spent spent = LaneNothing{}) {
  auto clear = [&](uint32_t (&v)[8], int j) {
    if constexpr (K <= 2) {
      if (ragged) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = j < words ? v[i] : 0u;
      }
    }
  };
  uint32_t va[8], vb[8];
  if constexpr (LAZY) x.load_word(0);
  else x.load();
  using J0 = std::integral_constant<int, 0>;
  using J1 = std::integral_constant<int, 1>;
  using J2 = std::integral_constant<int, 2>;
  using J3 = std::integral_constant<int, 3>;
  if constexpr (LaneDecode<K>::pair) {
    uint32_t T[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t w[K];
#pragma unroll
      for (int b = 0; b < K; ++b) w[b] = tw[b][j];
      if constexpr (K <= 3) lane_entries3<K>(w, T[j], M);
      else merge_nibble_pairs_v(w, T[j], M);
    }
    if constexpr (LAZY) {
      sched_fence();
      spent(tw);
      sched_fence();
    }
    lane_issue_pairs<0, K <= 3>(T[0], lanecol, lds, va, addr, mask);
    auto word = [&](auto jc) {
      constexpr int j = decltype(jc)::value;
      if constexpr (LAZY && j + 1 < 4) x.load_word(j + 1);
      lane_issue_pairs<2, K <= 3>(T[j], lanecol, lds, vb, addr, mask);
      sched_fence();
      clear(va, j);
      lane_mac_pairs<0, j>(va, x, acc);
      sched_fence();
      if constexpr (j + 1 < 4) lane_issue_pairs<0, K <= 3>(T[j + 1], lanecol, lds, va, addr, mask);
      sched_fence();
      clear(vb, j);
      lane_mac_pairs<2, j>(vb, x, acc);
      sched_fence();
    };
    word(J0{}); word(J1{}); word(J2{}); word(J3{});
  } else {
    uint32_t R[2][8];
    u32x4 mine[K];
#pragma unroll
    for (int b = 0; b < K; ++b) mine[b] = tw[b];
    if constexpr (LAZY) {
#pragma unroll
      for (int b = 0; b < K; ++b) asm volatile("" : "+v"(mine[b]));
      spent(tw);
      sched_fence();
    }
    {
      uint32_t w[K];
#pragma unroll
      for (int b = 0; b < K; ++b) w[b] = mine[b][0];
      lane_merge_fields<K, NB, ROOM>(w, R[0], M);
    }
    lane_issue_singles<K, 0>(R[0], lanecol, lds, va);
    auto word = [&](auto jc) {
      constexpr int j = decltype(jc)::value;
      if constexpr (j + 1 < 4) {
        uint32_t w[K];
#pragma unroll
        for (int b = 0; b < K; ++b) w[b] = mine[b][j + 1];
        lane_merge_fields<K, NB, ROOM>(w, R[(j + 1) & 1], M);
      }
      if constexpr (LAZY && j + 1 < 4) x.load_word(j + 1);
      lane_issue_singles<K, 1>(R[j & 1], lanecol, lds, vb);
      sched_fence();
      lane_mac_singles<0, j>(va, x, acc);
      sched_fence();
      lane_issue_singles<K, 2>(R[j & 1], lanecol, lds, va);
      sched_fence();
      lane_mac_singles<1, j>(vb, x, acc);
      sched_fence();
      lane_issue_singles<K, 3>(R[j & 1], lanecol, lds, vb);
      sched_fence();
      lane_mac_singles<2, j>(va, x, acc);
      sched_fence();
      if constexpr (j + 1 < 4) lane_issue_singles<K, 0>(R[(j + 1) & 1], lanecol, lds, va);
      sched_fence();
      lane_mac_singles<3, j>(vb, x, acc);
      sched_fence();
    };
    word(J0{}); word(J1{}); word(J2{}); word(J3{});
  }
}

// ---- tables -------------------------------------------------------------------------------------------------
// The lane's row of the k-bit table (the part this wavefront builds entries from), fetched one row block ahead.
//   k <= 4: the whole row (2^k fp16); k >= 5: entries [share * wave, + share)
template <int K>
struct LaneLut {
  static constexpr int kDwords = K <= 4 ? (1 << K) / 2 : LaneDecode<K>::share / 2;
  uint32_t v[kDwords];
};

// row: the row's start in the table
template <int K>
__device__ __forceinline__ void lane_fetch_lut_at(LaneLut<K>& L, const DPLLM_GLOBAL char* row_start, int wave) {
  const DPLLM_GLOBAL uint32_t* row = reinterpret_cast<const DPLLM_GLOBAL uint32_t*>(row_start);
  const DPLLM_GLOBAL uint32_t* src = K <= 4 ? row : row + wave * LaneLut<K>::kDwords;
  if constexpr (LaneLut<K>::kDwords >= 4) {
#pragma unroll
    for (int i = 0; i < LaneLut<K>::kDwords / 4; ++i) {
      const u32x4 q = reinterpret_cast<const DPLLM_GLOBAL u32x4*>(src)[i];
      L.v[4 * i] = q.x; L.v[4 * i + 1] = q.y; L.v[4 * i + 2] = q.z; L.v[4 * i + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < LaneLut<K>::kDwords; ++i) L.v[i] = src[i];
  }
}
template <int K>
__device__ __forceinline__ void lane_fetch_lut(LaneLut<K>& L, const DPLLM_GLOBAL uint16_t* lut_base, int row_number, int wave) {
  lane_fetch_lut_at<K>(L, reinterpret_cast<const DPLLM_GLOBAL char*>(lut_base + ((size_t)row_number << K)), wave);
}

// half h (0 = low) of dword d, for a wavefront-uniform h
__device__ __forceinline__ uint32_t half_of(uint32_t d, int h) { return h ? d >> 16 : d & 0xffffu; }

template <int K>
__device__ __forceinline__ void lane_build_table(const LaneLut<K>& L, int wave, uint32_t lanecol, char* lds) {
  if constexpr (K <= 2) {
    // wavefront w < 2^k writes the entries (a = w, b): (LUT[a], LUT[b])
    if (wave < (1 << K)) {
      const uint32_t la = half_of(K == 2 && wave >= 2 ? +L.v[LaneLut<K>::kDwords - 1] : +L.v[0], wave & 1);
#pragma unroll
      for (int b = 0; b < (1 << K); ++b) {
        const uint32_t hb = (b & 1) ? (L.v[b >> 1] & 0xffff0000u) : (L.v[b >> 1] << 16);
        const uint32_t entry = (uint32_t)wave << (6 - K) | (uint32_t)b << (3 - K);
        *reinterpret_cast<uint32_t*>(lds + entry * 256 + lanecol) = la | hb;
      }
    }
  } else if constexpr (K == 3) {
    // wavefront w writes the entries (a = w, b = 0..7): (LUT[a], LUT[b])
    const uint32_t v0 = L.v[0], v1 = L.v[1], v2 = L.v[2], v3 = L.v[3];
    const uint32_t lw = wave < 2 ? +v0 : wave < 4 ? +v1 : wave < 6 ? +v2 : +v3;
    const uint32_t la = half_of(lw, wave & 1);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint32_t hb = (b & 1) ? (L.v[b >> 1] & 0xffff0000u) : (L.v[b >> 1] << 16);
      *reinterpret_cast<uint32_t*>(lds + (uint32_t)(wave * 8 + b) * 256 + lanecol) = la | hb;
    }
  } else if constexpr (K == 4) {
    // wavefront w writes the entries (a = 2 w + s, b = 0..15), s = 0, 1
    uint32_t lw = L.v[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) lw = wave == i ? +L.v[i] : +lw;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const uint32_t la = s ? lw >> 16 : lw & 0xffffu;
#pragma unroll
      for (int b = 0; b < 16; ++b) {
        const uint32_t hb = (b & 1) ? (L.v[b >> 1] & 0xffff0000u) : (L.v[b >> 1] << 16);
        *reinterpret_cast<uint32_t*>(lds + (uint32_t)((wave * 2 + s) * 16 + b) * 256 + lanecol) = la | hb;
      }
    }
  } else {
    // wavefront w writes its share of the entries, an fp16 in the low half of a dword
    constexpr int share = LaneDecode<K>::share;
#pragma unroll
    for (int e = 0; e < share; ++e) {
      const uint32_t v = (e & 1) ? L.v[e >> 1] >> 16 : L.v[e >> 1] & 0xffffu;
      *reinterpret_cast<uint32_t*>(lds + (uint32_t)(wave * share + e) * 256 + lanecol) = v;
    }
  }
}

// Tiles in registers per wavefront: one being decoded, one in flight.  A third measured equal or up to 1.3 %
// slower in launches that fill the chip (with sixteen wavefronts on a compute unit the memory system has enough
// requests either way), and three or four tiles in flight did not help launches of a few hundred workgroups
// either (one dependency level of a chained step: 9.2 -> 10.3 us for q, k, v of a 7B block): those are bound by
// the chain launch -> job record -> selector results -> tables and first tiles -> decode, not by the number of
// requests in flight.
constexpr int kLaneDepth = 2;

// One workgroup: row blocks block, block + nblocks, ... of a job; its wavefront w takes the column tiles
// [w ncc / 8, (w + 1) ncc / 8) in every row block.  Tile loads run kLaneDepth - 1 tiles ahead, also across row
// blocks; past the end of the run the ring is refilled with dummy loads (see lane_load_tile).
template <int K, int NB>
__device__ __forceinline__ void gemv_lane(const GemvJob& job, uint32_t lut_at, int block, int tid, char* lds) {
  constexpr int D = kLaneDepth;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const uint32_t lanecol = (uint32_t)lane * 4;  // the lane's column of the interleaved tables
  float* red = reinterpret_cast<float*>(lds + lane_red_offset<NB>());
  char* ready = lds + lane_x_offset<NB>() + wave * lane_x_bytes<NB, 1>();   // (one sample) the parked tile
  char* repair = reinterpret_cast<char*>(red) + wave * 256;   // k = 4: room to re-pair a tile's activations (see lane_lds_bytes)
  const int c0 = wave * job.ncc / kLaneWaves, c1 = (wave + 1) * job.ncc / kLaneWaves;
  const int nrb = job.nrq;                     // row blocks of the job
  const int step = job.nblocks;
  const DPLLM_GLOBAL uint16_t* lut_base = as_global(reinterpret_cast<const uint16_t*>(job.arena + (size_t)lut_at * kAlign));
  const bool idle = c0 >= c1;                  // fewer tiles than wavefronts: this one only helps with the tables
  // the table rows of the next row block travel one block ahead, except at k >= 7, where their 8 - 16 registers
  // would cost the second workgroup per compute unit
  constexpr bool kLutAhead = K <= 6;
  LaneTile<K, NB> ring[D];
  LaneLut<K> L;
  // few tiles per row block: their activations are parked once, for every row block of the run.  Their loads
  // go out first and are parked after the first table rows and tiles have been asked for, so that the
  // workgroup starts with one memory round trip, not two (k = 4 has no registers to spare for that: there the
  // tiles are asked for after the activations have been parked)
  constexpr bool kEarlyX = K != 4;
  const bool keep = NB == 1 && c1 - c0 <= kLaneKeepTiles;
  char* kept = ready + 256;
  const DPLLM_GLOBAL uint16_t* xrows[lane_sets(NB)];
  if constexpr (NB > 1) lane_sample_rows<K, NB, 1>(job, lane, xrows);
  uint32_t xkeep[kLaneKeepTiles];
  if (keep) {
    if constexpr (kEarlyX) {
#pragma unroll
      for (int i = 0; i < kLaneKeepTiles; ++i) xkeep[i] = lane_load_x(job, min(c0 + i, job.ncc - 1), lane);
    } else {
      for (int cc = c0; cc < c1; ++cc)
        lane_park_x<K>(lane_mask_x(job, cc, lane, lane_load_x(job, cc, lane)), lane, repair, kept + (cc - c0) * 256);
    }
  }
  if constexpr (kLutAhead) lane_fetch_lut<K>(L, lut_base, block * 64 + lane, wave);
  int lrb = block, lcc = c0;                   // load cursor
  bool more = true;                            // the load cursor is still inside the run
  auto load_next = [&](LaneTile<K, NB>& t) {
    if constexpr (NB > 1) lane_load_raw(t.x, xrows, lcc, job.ncw, lane);
    lane_load_tile<K, NB>(t, job, lrb, lcc, lane, more);
    if constexpr (NB == 1) {
      if (!keep) t.x.v[0][0] = lane_load_x(job, lcc, lane);
    }
    if (++lcc >= c1) {
      lcc = c0;
      if (lrb + step < nrb) lrb += step; else more = false;
    }
  };
  if (!idle) {
#pragma unroll
    for (int i = 0; i < D - 1; ++i) load_next(ring[i]);
  }
  if (kEarlyX && keep) {
#pragma unroll
    for (int i = 0; i < kLaneKeepTiles; ++i)
      if (c0 + i < c1) lane_park_x<K>(lane_mask_x(job, c0 + i, lane, xkeep[i]), lane, repair, kept + i * 256);
  }
  LaneAcc<NB> acc;
  acc.zero();
  LaneMasks<K> M;
  if constexpr (K <= 6) M.init();
  uint32_t addr[8], mask = LaneDecode<K>::pair ? LaneDecode<K>::pair_mask : 0;   // k <= 3: address registers of the lookups (see lane_issue_pairs)
#pragma unroll
  for (int i = 0; i < 8; ++i) addr[i] = lanecol;
  int rb = block, cc = c0;                     // compute cursor
  auto open_block = [&]() {
    if constexpr (!kLutAhead) lane_fetch_lut<K>(L, lut_base, rb * 64 + lane, wave);
    lane_build_table<K>(L, wave, lanecol, lds);
    if constexpr (kLutAhead) lane_fetch_lut<K>(L, lut_base, (rb + step < nrb ? rb + step : rb) * 64 + lane, wave);
    lds_barrier();
  };
  auto close_block = [&]() {
    if constexpr (NB == 8) lds_barrier();   // the tables are done with
    if constexpr (NB == 1) {   // the wait of LaneAcc<1>::settle, once a block (7B step 503 us with and without; with settle() 492 for 490)
      sched_fence();
      asm volatile("s_nop 2");
      sched_fence();
    }
#pragma unroll
    for (int b = 0; b < lane_samples(NB); ++b) red[(b * kLaneWaves + wave) * 64 + lane] = acc.sum(b);
    acc.zero();
    lds_barrier();
    const bool storer = wave < lane_samples(NB) && (lane_samples(NB) == 1 || wave < job.nsamples);   // wavefront b stores sample b
    float s = 0.f;
    if (storer) {
#pragma unroll
      for (int w = 0; w < kLaneWaves; ++w) s += red[(wave * kLaneWaves + w) * 64 + lane];
    }
    const int o = rb * 64 + lane;
    if (storer && o < job.out) as_global(job.y)[(size_t)wave * job.out + o] = __builtin_bit_cast(uint16_t, (_Float16)s);
    if constexpr (NB == 8) lds_barrier();   // the next tables may be built
  };
  open_block();
  if (idle) {
    for (;;) {
      close_block();
      rb += step;
      if (rb >= nrb) return;
      open_block();
    }
  }
  for (;;) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      load_next(ring[(s + D - 1) % D]);
      const bool ragged = cc * 4 + 4 > job.ncw;
      LaneX<K, NB, 1> x;
      if constexpr (NB == 1) {
        x.mine = kept + (cc - c0) * 256;
        if (!keep) {
          lane_park_x<K>(lane_mask_x(job, cc, lane, ring[s].x.v[0][0]), lane, repair, ready);
          x.mine = ready;
        }
        x.mine += (lane & 3) * 16;
      } else {
        if (ragged) lane_mask_raw(ring[s].x, cc, job.ncw, lane);
        x.settle(ring[s].x, lane);
      }
      lane_compute<K, NB, 1>(ring[s].w, lanecol, lds, x, acc, addr, mask, M, job.ncw - cc * 4, ragged);
      if (++cc >= c1) {
        close_block();
        rb += step;
        if (rb >= nrb) return;
        cc = c0;
        open_block();
      }
    }
  }
}

// Launches that would leave the chip idle with 64 rows per workgroup (a 4096-row linear has 64 such blocks for 256
// compute units): a workgroup takes a block of 64 / G rows, and each of its wavefronts G neighbouring column tiles of
// them at a time: lane l works on row l mod (64 / G) of the block and on the tile of group l / (64 / G).  Every lane
// still has a column of its own in the interleaved tables (the G lanes of a row hold G copies of its table), so the
// lookups stay free of bank conflicts and the decode is the same code.  The sums of a row meet inside the workgroup:
// nothing is handed over between workgroups (sharing 64 rows between workgroups that split the columns, with a
// device-scope release, ticket and acquire at the end, cost 2 - 3 us of 10).
// What bounds it is one chain of latencies, not bandwidth: 4096 x 4096 at k = 4 on 256 workgroups, us after the first
// workgroup's entry: table rows here 1.4 - 1.7, tables built 2.0, first tile here 2.5, its 128 columns decoded 3.4,
// stored 4.2; another 1.3 around the kernel.  So the loads are asked for in the order they are needed, the activations
// are parked while the rest is on its way, and one workgroup per compute unit may use all its registers.
// One set of planes: a step's planes are merged first, and the next step's are asked for into the same registers before the lookups.
// Two sets in turns ask earlier but make the loop two bodies of code, which a launch this short runs through a few times at most: us per
// launch in a graph, two sets -> one: 1024 x 4096 k = 3 3.64 -> 3.56; 4096 x 4096 k = 4 B = 4 6.1 -> 5.6; 2500 x 6688 k = 7 9.0 -> 8.5; 4096 x
// 11008 k = 2 7.5 -> 6.9; 8192 x 8192 k = 4 9.8 -> 8.6, k = 8 17.5 -> 16.3; 4096 x 14336 B = 8 k = 3 12.2 -> 11.1.  (Two sets, each asked for
// anew as soon as it is merged: 5.4 where one takes 5.2, 9.4 for 8.5, 17.6 for 16.0.)
// us per launch, columns split between workgroups -> now: 4096 x 4096 k = 4 10.9 -> 5.1, k = 8 14.6 -> 8.0; 4096 x 11008
// k = 3 12.2 -> 7.3; 1024 x 4096 k = 3 7.3 -> 3.5.
template <int N>
__device__ __forceinline__ void load_dwords(uint32_t (&v)[N], const DPLLM_GLOBAL uint32_t* p) {
  if constexpr (N == 2) {
    const u32x2 q = *reinterpret_cast<const DPLLM_GLOBAL u32x2*>(p);
    v[0] = q.x; v[1] = q.y;
  } else {
#pragma unroll
    for (int i = 0; i < N; i += 4) {
      const u32x4 q = *reinterpret_cast<const DPLLM_GLOBAL u32x4*>(p + i);
      v[i] = q.x; v[i + 1] = q.y; v[i + 2] = q.z; v[i + 3] = q.w;
    }
  }
}

// the planes of the lane's tile (number `tile`, clamped to the row); real as in lane_load_tile
template <int K, int NB, int G>
__device__ __forceinline__ void narrow_load_planes(LaneTile<K, NB, G>& t, const GemvJob& job, const DPLLM_GLOBAL u32x4* rows, int tile, bool real) {
  const DPLLM_GLOBAL u32x4* p = real ? rows + (size_t)min(tile, job.ncc - 1) * 64 : as_global(reinterpret_cast<const u32x4*>(job.x));
  const size_t stride = real ? (size_t)job.plane_stride_u4 : 0;
#pragma unroll
  for (int b = 0; b < K; ++b) t.w[b] = load_stream(p + (size_t)b * stride);
}

// One sample: the lane's dwords G lane .. + G - 1 of the activations of step sc (G tiles).  They are 2 G columns; rows are
// whole 32-column words, so they are all inside the row or all past it.
template <int K, int G>
__device__ __forceinline__ void narrow_load_x(LaneTile<K, 1, G>& t, const GemvJob& job, int sc, int lane) {
  const int c = min(sc * G * 128 + lane * 2 * G, job.ncw * 32 - 2 * G);
  load_dwords<G>(t.x.v[0], reinterpret_cast<const DPLLM_GLOBAL uint32_t*>(as_global(job.x) + c));
}

// The sum over the G lanes of a row (64 / G lanes apart), in every one of them.  The swaps exchange two registers,
// so the value goes in twice, in registers of its own (the copy is opaque: left to itself the compiler hands the
// instruction one register twice, which then holds what it held).
template <int G>
__device__ __forceinline__ float sum_groups(float s) {
  if constexpr (G >= 8) s += __shfl_xor(s, 8, 64);
  auto copy = [](float v) { uint32_t r; asm("v_mov_b32 %0, %1" : "=v"(r) : "v"(v)); return r; };
  if constexpr (G >= 4) {
    const auto q = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, s), copy(s), false, false);
    s = __builtin_bit_cast(float, (uint32_t)q[0]) + __builtin_bit_cast(float, (uint32_t)q[1]);
  }
  const auto q = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, s), copy(s), false, false);
  return __builtin_bit_cast(float, (uint32_t)q[0]) + __builtin_bit_cast(float, (uint32_t)q[1]);
}

// parks the G tiles' activations of one sample (see lane_park_x): group g's at ready + kLaneGroupStride g
template <int K, int G>
__device__ __forceinline__ void narrow_park(const uint32_t (&x)[G], bool inside, int lane, char* ready) {
  constexpr int per = 64 / G;   // lanes that hold one tile's dwords
  char* mine = ready + (lane / per) * kLaneGroupStride + (lane % per) * 4 * G;
#pragma unroll
  for (int i = 0; i < G; ++i) *reinterpret_cast<uint32_t*>(mine + 4 * i) = inside ? x[i] : 0u;
  lds_order();
  if constexpr (K == 4) {       // re-paired in place: everything is read before anything is written
    const int j = lane >> 4, q = (lane >> 2) & 3, m = lane & 3, mr = (m + 3) & 3;
    const int ca = q == 0 ? 17 + 2 * m : q == 1 ? 8 + 2 * m : q == 2 ? 25 + 2 * m : 2 * m;
    const int cb = q == 0 ? 1 + 2 * m : q == 1 ? 24 + 2 * mr : q == 2 ? 9 + 2 * m : 16 + 2 * mr;
    uint32_t v[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const uint32_t lo = *reinterpret_cast<const uint16_t*>(ready + g * kLaneGroupStride + (j * 32 + ca) * 2);
      const uint32_t hi = *reinterpret_cast<const uint16_t*>(ready + g * kLaneGroupStride + (j * 32 + cb) * 2);
      v[g] = lo | (hi << 16);
    }
    lds_order();
#pragma unroll
    for (int g = 0; g < G; ++g) *reinterpret_cast<uint32_t*>(ready + g * kLaneGroupStride + lane * 4) = v[g];
    lds_order();
  }
}

// one workgroup: block number `block` of 64 / G rows
template <int K, int NB, int G>
__device__ __forceinline__ void gemv_narrow(const GemvJob& job, uint32_t lut_at, int block, int tid, char* lds) {
  constexpr int rows = 64 / G;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int row = block * rows + lane % rows, group = lane / rows;
  const uint32_t lanecol = (uint32_t)lane * 4;
  float* red = reinterpret_cast<float*>(lds + lane_red_offset<NB>());
  char* ready = lds + lane_x_offset<NB>() + wave * lane_x_bytes<NB, G>();   // (one sample)
  const int nsc = (job.ncc + G - 1) / G;
  const int c0 = wave * nsc / kLaneWaves, c1 = (wave + 1) * nsc / kLaneWaves;
  const DPLLM_GLOBAL u32x4* plane_rows = as_global(reinterpret_cast<const u32x4*>(job.arena)) + (size_t)(row / 64) * job.ncc * 64 + row % 64;
  const DPLLM_GLOBAL uint16_t* xrows[lane_sets(NB)];
  if constexpr (NB > 1) lane_sample_rows<K, NB, G>(job, lane, xrows);
  auto load_x = [&](LaneTile<K, NB, G>& t, int sc) {
    if constexpr (NB > 1) lane_load_raw(t.x, xrows, sc * G + group, job.ncw, lane);
    else narrow_load_x(t, job, sc, lane);
  };
  // first the activations of the first step (hot in L2: parked while the rest is on its way), then the table rows and
  // the planes
  LaneLut<K> L;
  LaneTile<K, NB, G> tile;
  const bool some = c0 < c1;                   // fewer steps than wavefronts: some only help with the tables
  auto park = [&](const LaneTile<K, NB, G>& t, int sc) {
    if constexpr (NB == 1) narrow_park<K, G>(t.x.v[0], sc * G * 128 + lane * 2 * G < job.ncw * 32, lane, ready);
  };
  if (some) load_x(tile, c0);
  lane_fetch_lut<K>(L, as_global(reinterpret_cast<const uint16_t*>(job.arena + (size_t)lut_at * kAlign)), row, wave);
  if (some) {
    narrow_load_planes<K, NB, G>(tile, job, plane_rows, c0 * G + group, true);
    sched_fence();
    park(tile, c0);
  }
  LaneAcc<NB> acc;
  acc.zero();
  float done[lane_samples(NB)];   // the sums before the last step, where lanes may be without a tile
#pragma unroll
  for (int b = 0; b < lane_samples(NB); ++b) done[b] = 0.f;
  LaneMasks<K> M;
  M.init();
  uint32_t addr[8], mask = LaneDecode<K>::pair ? LaneDecode<K>::pair_mask : 0;   // k <= 3 (see lane_issue_pairs)
#pragma unroll
  for (int i = 0; i < 8; ++i) addr[i] = lanecol;
  lane_build_table<K>(L, wave, lanecol, lds);
  lds_barrier();
#pragma unroll 1
  for (int cc = c0; cc < c1; ++cc) {
    if (cc != c0) park(tile, cc);
#pragma unroll
    for (int b = 0; b < lane_samples(NB); ++b) done[b] = acc.sum(b);
    const int at = cc * G + group;
    const bool ragged = (cc + 1) * G * 4 > job.ncw;
    LaneX<K, NB, G> x;
    if constexpr (NB == 1) {
      x.mine = ready + group * kLaneGroupStride + (lane & 3) * 16;
    } else {
      if (ragged) lane_mask_raw(tile.x, at, job.ncw, lane);
      x.settle(tile.x, lane);
    }
    lane_compute<K, NB, G, true>(tile.w, lanecol, lds, x, acc, addr, mask, M, job.ncw - at * 4, ragged, [&](u32x4 (&)[K]) {
      load_x(tile, cc + 1);
      narrow_load_planes<K, NB, G>(tile, job, plane_rows, (cc + 1) * G + group, cc + 1 < c1);
    });
    acc.settle();
  }
  // the last step may have fewer than G tiles: a lane without one (it decoded another tile) drops what it added there
  const bool whole = (c1 - 1) * G + group < job.ncc;
  if constexpr (NB == 8) lds_barrier();   // the tables, which the sums take the place of, are done with
#pragma unroll
  for (int b = 0; b < lane_samples(NB); ++b) red[(b * kLaneWaves + wave) * 64 + lane] = whole ? acc.sum(b) : done[b];
  lds_barrier();
  if (wave < lane_samples(NB) && (lane_samples(NB) == 1 || wave < job.nsamples)) {   // wavefront b stores sample b
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kLaneWaves; ++w) s += red[(wave * kLaneWaves + w) * 64 + lane];
    s = sum_groups<G>(s);
    if (group == 0 && row < job.out) as_global(job.y)[(size_t)wave * job.out + row] = __builtin_bit_cast(uint16_t, (_Float16)s);
  }
}

template <int NB, int G>
__device__ __forceinline__ double* lane_sel_shared(char* lds) { return reinterpret_cast<double*>(lds + lane_lds_bytes<NB, G>() - kSelSharedBytes); }

// One workgroup of a launch of its own.  Which code a bitwidth runs is settled here and not by the host, so that a call leaves the same
// bits whether it names the bitwidth or the device does, and whichever pairs are attached.
// One right-hand side, blocks of 64 rows: on the matrix pipe, four equal sums a lane, which spares parking the activations and a fifth of the
// vector instructions.  us per call, vector / matrix pipe: 9000 x 4096 k = 2 7.3 / 6.8, k = 4 8.8 / 7.8, k = 5 10.8 / 10.9, k = 7 12.9 / 13.2; 14336 x
// 4096 k = 4 9.0 / 8.3, k = 5 11.2 / 11.1, k = 8 14.9 / 15.0; 28672 x 4096 k = 4 13.4 / 12.9, k = 8 23.5 / 23.6; more tiles than a wavefront keeps
// the activations of (4096 columns) parks them for every row block, so there it pays at every bitwidth (planes side by side): 14336 x 14336 k = 2 21.9 /
// 16.0, k = 4 22.0 / 18.3, k = 5 30.5 / 28.6, k = 8 37.2 / 35.5; 16384 x 8192 k = 3 11.7 / 10.2, k = 6 20.9 / 19.6; 28672 x 8192 k = 6 34.8 / 34.0.  With several
// column groups it costs a per cent more than it saves; in a step, whose wavefronts are four to a SIMD, 2 % more (7B, 3 and 4 bits).
// A batch at k = 4 in a launch for eight column groups: four of them, in the first half of the workgroups (see pick_groups).
// Five to eight samples in a launch for one pass with four or two column groups: up to k = 4 two passes of four, each in half of the workgroups,
// which take half of the groups (see launch_gemv; with two groups on rows of many tiles one pass all the same).
constexpr int kLaneWideTiles = 4 * kLaneWaves;
template <int NB, int G>
__host__ __device__ constexpr int lane_lone_lds_bytes() {
  return NB == 8 && G > 1 && lane_lds_bytes<4, G / 2>() > lane_lds_bytes<NB, G>() ? lane_lds_bytes<4, G / 2>() : lane_lds_bytes<NB, G>();
}
template <int K, int G>
__device__ __forceinline__ void gemv_two_passes(const GemvJob& job, uint32_t lut_at, int block, int tid, char* lds) {
  GemvJob half = job;
  half.nblocks = (job.out + 64 / G - 1) / (64 / G);
  const int pass = block >= half.nblocks;
  half.x += (size_t)pass * 4 * job.ncw * 32;
  half.y += (size_t)pass * 4 * job.out;
  half.nsamples = pass ? job.nsamples - 4 : 4;
  block -= pass * half.nblocks;
  if (block >= half.nblocks) return;
  if constexpr (G == 1) gemv_lane<K, 4>(half, lut_at, block, tid, lds);
  else gemv_narrow<K, 4, G>(half, lut_at, block, tid, lds);
}
template <int K, int NB, int G>
__device__ __forceinline__ void gemv_lone(const GemvJob& job, uint32_t lut_at, int block, int tid, char* lds) {
  if constexpr (NB == 1 && G == 1) {
    static_assert(lane_lds_bytes<2, 1>() <= lane_lds_bytes<1, 1>(), "room for either");
    if constexpr (K >= 5) {
      if (job.ncc <= kLaneWaves * kLaneKeepTiles) return gemv_lane<K, 1>(job, lut_at, block, tid, lds);
    }
    gemv_lane<K, 2>(job, lut_at, block, tid, lds);
  } else if constexpr (G == 1) {
    gemv_lane<K, NB>(job, lut_at, block, tid, lds);
  } else if constexpr (NB == 4 && G == 8 && K == 4) {
    if (block * 16 < job.out) gemv_narrow<K, NB, 4>(job, lut_at, block, tid, lds);
  } else if constexpr (NB == 8 && G == 4 && K <= 4) {
    gemv_two_passes<K, 2>(job, lut_at, block, tid, lds);
  } else {
    if constexpr (NB == 8 && G == 2 && K <= 4) {
      if (job.ncc < kLaneWideTiles) return gemv_two_passes<K, 1>(job, lut_at, block, tid, lds);
    }
    if (block * (64 / G) < job.out) gemv_narrow<K, NB, G>(job, lut_at, block, tid, lds);
  }
}

// lut_at(K as a constant): where the K-bit tables start in the arena, in units of kAlign bytes.  LONE: a launch of its own.
template <int NB, int G, bool LONE, class At>
__device__ __forceinline__ void gemv_lane_width(const GemvJob& job, int k, At lut_at, int block, int tid, char* lds) {
  auto run = [&](auto kc) {
    constexpr int K = decltype(kc)::value;
    if constexpr (LONE) gemv_lone<K, NB, G>(job, lut_at(kc), block, tid, lds);
    else if constexpr (G == 1) gemv_lane<K, NB>(job, lut_at(kc), block, tid, lds);
    else gemv_narrow<K, NB, G>(job, lut_at(kc), block, tid, lds);
  };
  switch (k) {
    case 1: run(std::integral_constant<int, 1>{}); break;
    case 2: run(std::integral_constant<int, 2>{}); break;
    case 3: run(std::integral_constant<int, 3>{}); break;
    case 4: run(std::integral_constant<int, 4>{}); break;
    case 5: run(std::integral_constant<int, 5>{}); break;
    case 6: run(std::integral_constant<int, 6>{}); break;
    case 7: run(std::integral_constant<int, 7>{}); break;
    default: run(std::integral_constant<int, 8>{}); break;
  }
}

// The bitwidth of the job: its own value, the word a selector left in device memory, or the decision taken here
// from the partial products in the slots, left by workgroups of this launch or of an earlier one (every workgroup of the job repeats the same
// fixed-order sums, so all arrive at the same bits; the job's first workgroup writes bitwidth and estimate out).  A value
// outside [kmin, p] is not served: the workgroup returns and y keeps what it held.
template <int G>
__device__ __forceinline__ void gemv_lane_block(const GemvJob& job, int block, int tid, char* lds, const SelParams* active,
                                                int polls) {   // active == nullptr: no decisions here
  constexpr int NB = 1;
  if (block * (64 / G) >= job.out) return;   // (no row of the job is this workgroup's)
  int k = job.k;
  if (job.has_fin && active != nullptr) {
    static_assert(kSelMaxRank * sizeof(double) <= kLaneTableBytes, "room where the tables will be");
    const SelParams P = load_record(active + job.fin.linear);
    k = selector_gather(job.fin, P, polls, block, tid, lane_sel_shared<NB, G>(lds), reinterpret_cast<double*>(lds), block == 0);
    k = __builtin_amdgcn_readfirstlane(k);
  } else if (job.k_dev != nullptr) {
    k = __builtin_amdgcn_readfirstlane(*as_global(job.k_dev));
  }
  if (k < job.kmin || k > job.p) return;
  gemv_lane_width<NB, G, false>(job, k, [&](auto kc) { return job.lut_at[decltype(kc)::value - 1]; }, block, tid, lds);
}

// One linear, for several right-hand sides in groups of NB that share one pass over the planes (group g reads x + g * NB * in
// and writes y + g * NB * out; workgroups [g * nblocks, (g + 1) * nblocks) serve it).  All that a workgroup needs comes as plain arguments,
// fourteen dwords, which fit the registers that are set with the launch: nothing is loaded from the argument memory, and the host writes
// 56 bytes instead of 320.  us per call of a loop in Python, with a record by value for what is not needed first -> now: 1024 x 4096 k = 3
// 4.4 -> 4.05, 11008 x 4096 k = 4 8.8 -> 8.7; an estimate and a GEMV of 4096 x 4096, both so, 10.2 -> 9.7, in a graph 9.7 -> 9.6.
// bits: LaneBits; lut: where the tables start in the arena, in units of kAlign bytes, less row blocks << (k - 1) where k_dev says the bitwidth (a
// block's tables of k bits are so many units, and those of fewer bits lie in front).
struct LaneBits {
  int k, kmin, p, nrhs;                      // the bitwidth unless k_dev says it; those the linear serves; right-hand sides
  __host__ __device__ uint32_t pack() const { return (uint32_t)(k | kmin << 4 | p << 8 | nrhs << 12); }
  static __host__ __device__ LaneBits unpack(uint32_t v) { return {(int)(v & 15), (int)(v >> 4 & 15), (int)(v >> 8 & 15), (int)(v >> 12)}; }
};
template <int NB, int G>
__global__ void __launch_bounds__(kLaneThreads, G == 1 ? 4 : 2) gemv_lane_kernel(const char* arena, const uint16_t* x, uint16_t* y, const int32_t* k_dev,
                                                                                uint32_t plane_stride_u4, uint32_t lut, uint32_t bits, int out,
                                                                                int ncw, int nblocks) {
  __shared__ __attribute__((aligned(256))) char lds[lane_lone_lds_bytes<NB, G>()];
  // the lookup addresses are formed as (entry << 8) | (lane << 2): the tables must start at LDS address 0
  if ((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds != 0u) return;
  const LaneBits b = LaneBits::unpack(bits);
  const int group = NB == 1 ? 0 : blockIdx.x / nblocks;
  GemvJob job{};
  job.arena = arena;
  job.x = x + (size_t)group * NB * ncw * 32;
  job.y = y + (size_t)group * NB * out;
  job.plane_stride_u4 = plane_stride_u4;
  job.out = out;
  job.ncw = ncw;
  job.ncc = (ncw + 3) / 4;
  job.nrq = (out + 63) / 64;
  job.nblocks = nblocks;
  job.nsamples = min(NB, b.nrhs - group * NB);
  const int block = blockIdx.x - group * nblocks;
  int k = b.k;
  if (k_dev != nullptr) {
    k = load_record(k_dev);
    if (k < b.kmin || k > b.p) return;
    lut += (uint32_t)job.nrq << (k - 1);
  }
  gemv_lane_width<NB, G, true>(job, k, [&](auto) { return lut; }, block, threadIdx.x, lds);
}

// The linears of a dependency level of a decode step: block b < nblocks belongs to job block_jobs[b]; blocks past them
// help with the selectors only.  active: the table of selector parameters, for launches that take the decisions of their
// jobs here; else nullptr.  ntasks: selector work of the launch (see selector_tasks), 0 if an earlier one did it.
template <int G>
__global__ void __launch_bounds__(kLaneThreads, G == 1 ? 4 : 2) gemv_step_kernel(const SelTask* tasks, const GemvJob* jobs, const int32_t* block_jobs,
                                                                                const SelParams* active, int ntasks, int task_groups,
                                                                                int nblocks, int polls) {
  __shared__ __attribute__((aligned(256))) char lds[lane_lds_bytes<1, G>()];
  if ((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds != 0u) return;
  const int b = blockIdx.x;
  selector_tasks(tasks, ntasks, task_groups, b, threadIdx.x, lane_sel_shared<1, G>(lds));
  if (b >= nblocks) return;
  const GemvJob job = load_record(jobs + load_record(block_jobs + b));
  gemv_lane_block<G>(job, b - job.block_start, threadIdx.x, lds, active, polls);
}

}  // namespace dpllm
