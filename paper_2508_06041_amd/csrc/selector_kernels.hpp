// Precision selector kernels (paper Sec. 3: the layer takes h when the relative error exceeds its threshold
// T, else l; Sec. 5.1: the error is estimated as ||G x|| with G = A (W_h - W_l) precomputed, or as
// alpha ||x|| + beta).  One launch serves a list of selector jobs; the bitwidth lands in device memory, where
// the GEMV kernels read it.
//
// What a linear's selector is (candidate pair, estimator kind, G, alpha, beta, T) depends on the target
// precision the model runs under (Algorithm 1 hands out one threshold list per target; Sec. 5.1 keeps one G per
// candidate pair): a table on the device holds the parameters of every target, and the kernels read a copy of the
// active target's row.  A switch of target is one small kernel (selector_activate_kernel) that copies the row and
// writes the tasks of the small launches; the launches stay what they are, and none of them has to look the
// target up before it can look its parameters up (a round trip to memory of 0.6 us in every launch of a chained step).
//
// A projection job reads 0.5 - 3.5 MB of G.  It is cut into parts of 16 rows of G (one workgroup of four
// wavefronts, four rows per wavefront sharing the activation loads) by a chunk of columns: the whole row when
// the launch has enough parts to fill the chip, down to 512 columns when it serves a few linears only (a part
// that streams a whole row alone takes 10 - 30 us).  A part leaves the fp64 partial dot products of its rows in
// workspace slots of its own, and that is all it does.  Linears whose estimator is the linear regression need
// sum x^2 only: the jobs of a launch that read the same input vector form a group with one extra part, which
// adds up x^2 once and leaves it in the slot of every member that asks for it.
//
// Who takes the estimate and the decision (the choice for a step: runs_selectors and kPrologueMaxBlocks in dpllm_api.hip):
//   - the selectors of a step alone, and in front of large GEMV launches: selector_decide_kernel, in
//     a launch of its own behind the parts (the end of one launch and the start of the next order the two at device
//     scope);
//   - one estimate (dpllm_estimate): the workgroup of the part launch that started last (selector_estimate_kernel);
//   - in GEMV launches of up to two rounds of workgroups: every workgroup, before it starts (selector_gather), from the
//     slots of its own linear;
//   - in the small launches of a chained step, whose selectors are little work (selector_tasks, selector_gather): every
//     workgroup of the GEMV launch
//     first works off its share of the launch's selectors, a row of G times a slice of the columns, and leaves the
//     partial dot product in its slot; then every workgroup collects the slots of its own linear, adds them up and
//     decides.  A slot is its own flag: it holds kSelEmpty (a NaN no writer stores) until the value is there, and both
//     sides use relaxed atomics on that one 64-bit word, so nothing rests on the order of two memory locations and no
//     fence is needed (a device-scope release writes back the die's whole L2: 126 us instead of 30 for the 224
//     selectors of a 7B step).  A fill kernel empties the slots at the start of the step.  The wait is bounded: a
//     workgroup that has polled often enough computes the missing products itself, so no workgroup depends on
//     another one being scheduled.  What the way costs (7B block, q, k, v: 192 workgroups, us after the first one's
//     entry): task record here 0.8, product stored 2.6, all slots seen 3.8, bitwidth known 4.3; the launches of their own
//     cost 3.8 for the parts, 1.6 between launches and 1.6 for the decision in the GEMV prologue.  Chained step of 32
//     blocks 1888 -> 1428 us, of 16 8B blocks with selectors ahead 1060 -> 940.  Tried on top of it: asking for the
//     planes and tables of the level while the selectors work (the traffic delays the hand-over by more than it saves:
//     1605 us with the first tiles, 1460 with the table rows alone), longer pauses between polls (no change).
//
// The estimate and the compare are taken in fp64: fp16 x fp16 products are exact in fp32, their sums run in fp64.  Every
// order of additions is fixed, so a decision is reproducible and workgroups that repeat it get the same bits, but the
// orders differ: the columns of a row are cut differently for parts and tasks, selector_finish adds the squares of the rows
// in 64 lanes, selector_gather in 512.  Estimates of dpllm_estimate, of DPLLM_STEP_SELECT and of a whole step agree to about
// 1e-13 relative; a decision differs between them, or from an ideal-arithmetic one, only when |e - T| is below that.
#pragma once
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdint>

namespace dpllm {

constexpr int kSelPartThreads = 256;
constexpr int kSelPartWaves = kSelPartThreads / 64;
constexpr int kSelRowsPerWave = 4;   // rows of G a wavefront carries at once (they share the activation loads)
constexpr int kSelDepth = 2;         // column tiles in registers: one being accumulated, one in flight (two in flight measured slower: 32 against 28 us for the 224 selectors of a 7B step)
constexpr int kSelPartRows = kSelPartWaves * kSelRowsPerWave;
constexpr int kSelMaxRank = 1024;
constexpr int kSelMaxChunks = 32;    // column chunks of a job
constexpr int kSelChunkStep = 512;   // columns a wavefront covers per tile: chunks are multiples of it

// What the selector of one linear is under one target.  kind: 0 none (always l), 1 projection, 2 linear regression
struct alignas(64) SelParams {   // (aligned: one scalar load)
  const uint16_t* G;   // fp16 [r][in] (projection kind)
  float T, alpha, beta;
  int32_t r, l, h, kind;
};

// The target-independent part of a selector job.
struct SelJob {
  const uint16_t* x;   // fp16 [in]: the vector the selector reads
  float* e_out;
  int32_t* k_out;
  double* ws;          // [nchunks][ws_rows] partial dot products (projection), or [0] = sum x^2 (linear regression)
  int32_t in;
  int32_t linear;      // row of the job's linear in the parameter table
  int32_t nchunks, chunk_cols;  // projection part p covers rows [16 (p / nchunks), + 16), columns [chunk_cols (p % nchunks), + chunk_cols)
  int32_t ws_rows;     // rows of one chunk's slots in ws (the largest rank of the linear's pairs, rounded up to 16)
  int32_t row_each;    // a lone estimate: parts of four rows, one to a wavefront (see selector_estimate_kernel)
};
struct SelPart {
  int32_t job;     // index into the job table of the launch
  int32_t part;    // projection part number inside the job; -1: the group part of the group whose first member is `job`
  int32_t linear;  // the job's row in the parameter table (so that job record and parameters load side by side)
  int32_t count;   // group part: members of the group; they are members[first .. first + count) of the launch's member
  int32_t first;   //   table (indices into the job table), all reading the same vector
  int32_t pad;
};

__host__ __device__ inline int sel_rowgroups_of(int kind, int r) {
  return kind == 1 ? (r + kSelPartRows - 1) / kSelPartRows : 0;
}

// a partial dot product nobody has written yet; a computed NaN with these bits is stored as another NaN
constexpr uint64_t kSelEmpty = ~0ull;
__device__ __forceinline__ double sel_storable(double v) {
  return __builtin_bit_cast(uint64_t, v) == kSelEmpty ? __builtin_bit_cast(double, 0x7ff8000000000000ull) : v;
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// v of this half (16 or 32 lanes) plus v of the other one.  The swaps exchange two registers, so the value goes in
// twice, in registers of its own (the copies are opaque: left to itself the compiler passes one register twice).
template <int LANES>
__device__ __forceinline__ double swap_add_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  uint32_t lo2, hi2;
  asm("v_mov_b32 %0, %1" : "=v"(lo2) : "v"(lo));
  asm("v_mov_b32 %0, %1" : "=v"(hi2) : "v"(hi));
  if constexpr (LANES == 16) {
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo2, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi2, false, false);
    return __builtin_bit_cast(double, (uint64_t)b[0] << 32 | a[0]) + __builtin_bit_cast(double, (uint64_t)b[1] << 32 | a[1]);
  } else {
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo2, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi2, false, false);
    return __builtin_bit_cast(double, (uint64_t)b[0] << 32 | a[0]) + __builtin_bit_cast(double, (uint64_t)b[1] << 32 | a[1]);
  }
}
// the sum over the wavefront, in every lane: pairs, quads, groups of 8 and 16 with DPP moves, then across the rows
__device__ __forceinline__ double wave_sum_f64(double v) {
  v += dpp_f64<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_f64<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_f64<0x141>(v);   // row_half_mirror
  v += dpp_f64<0x140>(v);   // row_mirror
  v = swap_add_f64<16>(v);
  return swap_add_f64<32>(v);
}

typedef uint32_t sel_u32x4 __attribute__((ext_vector_type(4)));

template <int ROWS>
struct SelTile {
  sel_u32x4 g[ROWS];
  uint4 x;
};

// columns [c, c + 8) of the wavefront's rows and of x; c is clamped by the caller, so the loads are
// unconditional and the next tile can be in flight while the current one is accumulated
// (pointers taken from a job record are generic; global-address-space loads keep them on the vector-memory path)
#define DPLLM_SEL_GLOBAL __attribute__((address_space(1)))
template <int ROWS>
__device__ __forceinline__ void sel_load(SelTile<ROWS>& t, const uint16_t* const (&rows)[ROWS], const uint16_t* x, int c) {
#pragma unroll
  for (int i = 0; i < ROWS; ++i)
    t.g[i] = __builtin_nontemporal_load((const DPLLM_SEL_GLOBAL sel_u32x4*)(rows[i] + c));
  const sel_u32x4 xv = *(const DPLLM_SEL_GLOBAL sel_u32x4*)(x + c);
  t.x = make_uint4(xv.x, xv.y, xv.z, xv.w);
}

template <int ROWS>
__device__ __forceinline__ void sel_accumulate(const SelTile<ROWS>& t, bool valid, double (&acc)[ROWS]) {
  const __half* xh = reinterpret_cast<const __half*>(&t.x);
  double xd[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) xd[i] = valid ? (double)__half2float(xh[i]) : 0.0;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const __half* gh = reinterpret_cast<const __half*>(&t.g[r]);
    // an fp16 x fp16 product is exact in fp64, so the fused multiply-add rounds once, like an fp64 add of the
    // exact product
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[r] = fma((double)__half2float(gh[i]), xd[i], acc[r]);
  }
}

// LDS of a selector workgroup / of the finishing step
struct SelShared {
  double sq[kSelMaxRank + 1];   // [kSelMaxRank]: the total
};

// What the finishing step needs of a selector job (a copy of it travels in the GEMV job record).  Slot [chunk]
// [row] of ws holds the partial dot product of a row.
struct SelFinish {
  const double* ws;
  float* e_out;
  int32_t* k_out;
  const uint16_t* x;
  int32_t in, linear, nchunks, ws_rows, chunk_cols;   // chunk c: columns [chunk_cols c, + chunk_cols) inside the row
  int32_t copies;      // of the slots, [copy][chunk][row] (1 or kSelCopies)
  int32_t task_first, task_rows;   // the selector's tasks: entries of the table from task_first on, [row][chunk] (0 rows: none)
  int32_t x_handed;    // SelTask::x_handed of them
  int32_t squares;     // linear regression: row 0 of the tasks adds up x^2
};
__host__ __device__ inline SelFinish sel_finish_of(const SelJob& j) {
  return SelFinish{j.ws, j.e_out, j.k_out, j.x, j.in, j.linear, j.nchunks, j.ws_rows, j.chunk_cols, 1, 0, 0, 0, 0};
}

// The estimate from what the selector launch left in the workspace, and the decision; called by all `nthreads`
// (a multiple of 64, at least 64) threads of a workgroup (it holds workgroup barriers), every thread returns the
// bitwidth.  write: thread 0 also stores the estimate and the bitwidth.  The partial products were written by an
// earlier launch.  Order of the additions (fixed, so that every workgroup that repeats them gets the same bits):
// per row of G its chunks in chunk order; the squares of rows t, t + 64, t + 128, ... in that order in lane t of
// the first wavefront; the 64 lane sums by a butterfly.  Loads are issued in batches ahead of the additions that
// consume them.
__device__ __forceinline__ int selector_finish(const SelFinish& f, const SelParams* prow, int tid, int nthreads, double* sq, bool write) {
  const DPLLM_SEL_GLOBAL double* ws = (const DPLLM_SEL_GLOBAL double*)f.ws;
  // the first batch of partial products is asked for before the parameters, so that both arrive together (what
  // the batch means is known once the parameters are here: slot 0 may also be sum x^2)
  double v[8];
  const int t0 = min(tid, f.ws_rows - 1);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = ws[(size_t)min(i, f.nchunks - 1) * f.ws_rows + t0];
  const SelParams P = *prow;
  double e = 0.0;
  if (P.kind == 1) {
    for (int t = tid; t < P.r; t += nthreads) {
      double g = 0.0;
      for (int c0 = 0; c0 < f.nchunks; c0 += 8) {
        if (c0 > 0 || t != tid) {
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] = ws[(size_t)min(c0 + i, f.nchunks - 1) * f.ws_rows + t];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) g += c0 + i < f.nchunks ? v[i] : 0.0;
      }
      sq[t] = g * g;
    }
    __syncthreads();
    if (tid < 64) {
      double part = 0.0;
      for (int t = tid; t < P.r; t += 64) part += sq[t];
      part = wave_sum_f64(part);
      if (tid == 0) sq[kSelMaxRank] = part;
    }
    __syncthreads();
    e = sqrt(sq[kSelMaxRank]);
    __syncthreads();                              // sq may be reused by the caller
  } else if (P.kind == 2) {
    e = (double)P.alpha * sqrt(ws[0]) + (double)P.beta;
  }
  // strictly exceeding T selects h; +inf pins l, -inf pins h; no estimator: always l
  const int k = (P.kind != 0 && e > (double)P.T) ? P.h : P.l;
  if (write && tid == 0) {
    *f.e_out = (float)e;
    *f.k_out = k;
  }
  return k;
}

// The group part: sum x^2, added up once for the jobs of the launch that read the same vector and left in the
// slot of every member whose estimator under the active target is the linear regression.
__device__ __forceinline__ void selector_group_part(const SelJob* jobs, const int32_t* members, int count, const SelParams* params,
                                                    const SelJob& lone, const SelParams& one, int tid, SelShared& sh) {
  const int wave = tid >> 6, lane = tid & 63;
  const SelJob& head = jobs ? jobs[members[0]] : lone;
  int need = 0;
  if (jobs) {
    for (int i = tid; i < count; i += kSelPartThreads) need |= params[jobs[members[i]].linear].kind == 2;
  } else {
    need = one.kind == 2;
  }
  if (!__syncthreads_or(need)) return;
  double acc = 0.0;
  for (int c = tid * 8; c < head.in; c += kSelPartThreads * 8) {
    const sel_u32x4 xv = *(const DPLLM_SEL_GLOBAL sel_u32x4*)(head.x + c);
    const __half* xh = reinterpret_cast<const __half*>(&xv);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float v = __half2float(xh[i]);
      acc += (double)(v * v);  // exact square in fp32
    }
  }
  acc = wave_sum_f64(acc);
  if (lane == 0) sh.sq[wave] = acc;
  __syncthreads();
  double tot = 0.0;
  for (int w = 0; w < kSelPartWaves; ++w) tot += sh.sq[w];
  if (jobs) {
    for (int i = tid; i < count; i += kSelPartThreads) {
      const SelJob& j = jobs[members[i]];
      if (params[j.linear].kind == 2) j.ws[0] = tot;
    }
  } else if (tid == 0) {
    lone.ws[0] = tot;
  }
}

// What a wavefront does of a projection part: the products of ROWS rows from row0 on (clamped to r - 1; surplus rows are dropped)
// and columns [cb, ce) of x, chunk ch.  ONE: in a launch for one row a wavefront.
template <bool ONE, int ROWS>
__device__ __forceinline__ void selector_part_products(const SelJob& job, const SelParams& P, int row0, int ch, int wave, int lane, double (&rowsum)[ROWS]) {
  const int cb = ch * job.chunk_cols, ce = min(job.in, cb + job.chunk_cols);
  const uint16_t* rows[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) rows[i] = P.G + (size_t)min(row0 + i, P.r - 1) * job.in;
  double acc[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) acc[i] = 0.0;
  const int last = ce - 8;              // in % 32 == 0 and chunks are multiples of 512, so every 8-column group is whole
  const int nit = (ce - cb + kSelChunkStep - 1) / kSelChunkStep;
  // Rows of G are a power-of-two number of bytes apart in the common shapes, so wavefronts that all walk the
  // columns from the start would hit the same few memory channels at any moment: every wavefront starts its
  // (circular) walk at a different 1 KiB column chunk.  (A row starts where it does in a launch of parts of four rows a wavefront:
  // the same order of additions, the same bits.)
  const unsigned walk = ONE ? (unsigned)((row0 / kSelPartRows * job.nchunks + ch) * kSelPartWaves + row0 % kSelPartRows / kSelRowsPerWave)
                            : blockIdx.x * kSelPartWaves + wave;
  int it = (int)(walk * 5u % (unsigned)nit);   // tile being loaded
  int ca = cb + it * kSelChunkStep + lane * 8;                                // first column of the tile being accumulated
  SelTile<ROWS> ring[kSelDepth];
#pragma unroll
  for (int d = 0; d < kSelDepth - 1; ++d) {
    sel_load(ring[d], rows, job.x, min(cb + it * kSelChunkStep + lane * 8, last));
    it = it + 1 == nit ? 0 : it + 1;
  }
  for (int k = 0; k < nit; k += kSelDepth) {
#pragma unroll
    for (int d = 0; d < kSelDepth; ++d) {
      // loads past the end of the walk re-read a tile that is never accumulated (uniform, unconditional issue)
      sel_load(ring[(d + kSelDepth - 1) % kSelDepth], rows, job.x, min(cb + it * kSelChunkStep + lane * 8, last));
      it = it + 1 == nit ? 0 : it + 1;
      if (k + d < nit) sel_accumulate(ring[d], ca <= last, acc);
      ca = ca + kSelChunkStep >= cb + nit * kSelChunkStep ? ca + kSelChunkStep - nit * kSelChunkStep : ca + kSelChunkStep;
    }
  }
#pragma unroll
  for (int i = 0; i < ROWS; ++i) rowsum[i] = sel_storable(wave_sum_f64(acc[i]));
}

// One projection part of 16 rows: wavefront w owns rows 16 rg + 4 w .. + 3
__device__ __forceinline__ void selector_proj_part(const SelJob& job, const SelParams& P, int part, int tid) {
  const int wave = tid >> 6, lane = tid & 63;
  if (P.kind != 1) return;                                    // this target estimates the linear otherwise
  const int rg = part / job.nchunks, ch = part - rg * job.nchunks;
  if (rg * kSelPartRows >= P.r) return;                       // the pair of this target has fewer rows of G
  const int row0 = rg * kSelPartRows + wave * kSelRowsPerWave;
  double rowsum[kSelRowsPerWave];
  selector_part_products<false>(job, P, row0, ch, wave, lane, rowsum);
  DPLLM_SEL_GLOBAL double* ws = (DPLLM_SEL_GLOBAL double*)job.ws;
#pragma unroll
  for (int i = 0; i < kSelRowsPerWave; ++i)
    if (lane == 0) ws[(size_t)ch * job.ws_rows + row0 + i] = rowsum[i];
}

// ---- the selectors of a small GEMV launch, worked off by its own workgroups --------------------------------------
// One row of a projection times a slice of the columns: what a workgroup does at a time.
struct alignas(64) SelTask {
  const uint16_t* g;   // the slice of the row of G; nullptr: nothing to do under the active target (selector_activate_kernel)
  const uint16_t* x;   // the same columns of the vector
  uint64_t* slot;      // where the partial dot product goes, kSelCopies times,
  int32_t copy_stride; //   slots apart
  int32_t cols;        // length of the slice
  int32_t x_handed;    // gemv_chain_kernel only: x lies in a mailbox
};
// Records that no kernel of the launch writes, read at an address that is the same for the whole workgroup: from the
// constant address space they come with one scalar load (through a generic pointer every field is a vector load of its
// own, waited for where it is first used: four round trips of 0.5 us before the row of G was asked for).
template <class T>
__device__ __forceinline__ T load_record(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole dwords");
  struct Raw { uint32_t w[sizeof(T) / 4]; };
  const __attribute__((address_space(4))) uint32_t* q = (const __attribute__((address_space(4))) uint32_t*)(uintptr_t)p;
  Raw r;
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 4; ++i) r.w[i] = q[i];
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 4; ++i) asm volatile("" : "+s"(r.w[i]));   // all of it here, not each field where it is used
  return __builtin_bit_cast(T, r);
}
constexpr int kSelTaskGroups = 256;     // workgroups the tasks of a launch are cut for: one per compute unit
constexpr int kSelTaskCols = 4096;      // a slice this long keeps eight wavefronts busy with one load each
// Every product is stored this many times and every workgroup reads the copy of its own number modulo that (its die's,
// as workgroups are dealt out to the dies): 256 workgroups that poll the same four lines wait for one another.  Chained
// 7B step with 1, 2, 8, 16 copies: 1539, 1473, 1428, 1430 us.
constexpr int kSelCopies = 8;
constexpr int kSelSharedBytes = 256;    // LDS of selector_tasks and selector_gather

// chunks w, w + 8, ... of 512 columns of a slice, in the lane's eight columns of each; the wavefront's sum in every lane
__device__ __forceinline__ double selector_chunks_dot(const uint16_t* row, const uint16_t* x, int cols, int w, int lane) {
  constexpr int step = 8 * kSelChunkStep;
  const DPLLM_SEL_GLOBAL uint16_t* g = (const DPLLM_SEL_GLOBAL uint16_t*)row;
  const DPLLM_SEL_GLOBAL uint16_t* xg = (const DPLLM_SEL_GLOBAL uint16_t*)x;
  const int last = cols - 8;            // cols is a multiple of 32: eight columns are inside or outside together
  auto load = [&](const DPLLM_SEL_GLOBAL uint16_t* p, int c) { return *(const DPLLM_SEL_GLOBAL sel_u32x4*)(p + min(c, last)); };
  int c = w * kSelChunkStep + lane * 8;
  sel_u32x4 ga = load(g, c), xa = load(xg, c);
  double acc = 0.0;
  for (int c0 = w * kSelChunkStep; c0 < cols; c0 += step) {
    const sel_u32x4 gv = ga, xv = xa;
    const bool valid = c <= last;
    c += step;
    if (c0 + step < cols) {
      ga = load(g, c);
      xa = load(xg, c);
    }
    if (valid) {
      const __half* gh = reinterpret_cast<const __half*>(&gv);
      const __half* xh = reinterpret_cast<const __half*>(&xv);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc = fma((double)__half2float(gh[i]), (double)__half2float(xh[i]), acc);
    }
  }
  return wave_sum_f64(acc);
}

// barrier of a workgroup that shares data through LDS only: loads and stores in flight stay in flight
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The launch's share of selector work: workgroup b < groups runs tasks b, b + groups, ...  By a workgroup of eight
// wavefronts; sh: kSelSharedBytes of LDS, [0, 16)
__device__ __forceinline__ void selector_tasks(const SelTask* tasks, int count, int groups, int block, int tid, double* sh) {
  if (block >= groups) return;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  int turn = 0;   // the tasks take turns in two sets of eight partial sums, so that one barrier per task is enough
  for (int t = block; t < count; t += groups) {
    const SelTask k = load_record(tasks + t);
    if (k.g == nullptr) continue;
    const double v = selector_chunks_dot(k.g, k.x, k.cols, wave, lane);
    if (lane == 0) sh[turn + wave] = v;
    lds_barrier();
    if (tid < kSelCopies) {
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < 8; ++w) sum += sh[turn + w];
      __hip_atomic_store((DPLLM_SEL_GLOBAL uint64_t*)k.slot + (size_t)tid * k.copy_stride, __builtin_bit_cast(uint64_t, sel_storable(sum)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    turn ^= 8;
  }
}

// The estimate and the decision from the slots of the linear, by the 512 threads of a workgroup; every thread returns
// the bitwidth.  sh: kSelSharedBytes of LDS, [16, 32); spare: kSelMaxRank doubles of LDS, free again on return.
__device__ __forceinline__ int selector_gather(const SelFinish& f, const SelParams& P, int polls, int block, int tid, double* sh, double* spare, bool write) {
  constexpr int threads = 512, waves = threads / 64, batch = 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  double e = 0.0;
  if (P.kind == 1) {
    const DPLLM_SEL_GLOBAL uint64_t* slots = (const DPLLM_SEL_GLOBAL uint64_t*)f.ws + (size_t)(block & (f.copies - 1)) * f.nchunks * f.ws_rows;
    // row t in thread t mod 512: its slices in order, squared; the rows of a thread in order, the threads of a
    // wavefront, the wavefronts in order
    double part = 0.0;
    bool lack = false;
    for (int t = tid; t < P.r; t += threads) {
      double g = 0.0;
      for (int c0 = 0; c0 < f.nchunks; c0 += batch) {
        uint64_t v[batch];
        for (int left = polls;; --left) {
          bool all = true;
#pragma unroll
          for (int i = 0; i < batch; ++i)
            v[i] = __hip_atomic_load(slots + (size_t)min(c0 + i, f.nchunks - 1) * f.ws_rows + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
          for (int i = 0; i < batch; ++i) all = all && v[i] != kSelEmpty;
          if (__all(all) || left <= 0) break;
          __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int i = 0; i < batch; ++i) {
          lack = lack || v[i] == kSelEmpty;
          if (c0 + i < f.nchunks) g += __builtin_bit_cast(double, v[i]);
        }
      }
      part += g * g;
    }
    part = wave_sum_f64(part);
    // a wavefront that lacks a product says so with a word of its own (the sum of squares may be any double)
    uint32_t* lacks = reinterpret_cast<uint32_t*>(sh + 16 + waves);
    const bool wave_lacks = __any(lack);
    if (lane == 0) {
      sh[16 + wave] = part;
      lacks[wave] = wave_lacks;
    }
    lds_barrier();
    double sum = 0.0;
    uint32_t lacking = 0;
#pragma unroll
    for (int w = 0; w < waves; ++w) {
      sum += sh[16 + w];
      lacking |= lacks[w];
    }
    if (__builtin_amdgcn_readfirstlane(lacking)) {
      // the same sums in the same order, all of them here
      for (int t = wave; t < P.r; t += waves) {
        double g = 0.0;
        for (int c = 0; c < f.nchunks; ++c) {
          const size_t at = (size_t)c * f.chunk_cols;
          const int cols = min(f.chunk_cols, f.in - c * f.chunk_cols);
          double s = 0.0;
          for (int w = 0; w < 8; ++w) s += w * kSelChunkStep < cols ? selector_chunks_dot(P.G + (size_t)t * f.in + at, f.x + at, cols, w, lane) : 0.0;
          g += sel_storable(s);
        }
        if (lane == 0) spare[t] = g;
      }
      lds_barrier();
      sum = 0.0;
      for (int w = 0; w < waves; ++w) {
        double mine = 0.0;
        for (int t = w * 64 + lane; t < P.r; t += threads) mine += spare[t] * spare[t];
        sum += wave_sum_f64(mine);
      }
      lds_barrier();
    }
    e = sqrt(sum);
  } else if (P.kind == 2 && f.copies == 1) {
    e = (double)P.alpha * sqrt(((const DPLLM_SEL_GLOBAL double*)f.ws)[0]) + (double)P.beta;   // an earlier launch's group part
  } else if (P.kind == 2) {
    // sum x^2 of the linear's own vector: no hand-over; the first kSelPartWaves wavefronts, as selector_group_part does
    if (wave < kSelPartWaves) {
      double acc = 0.0;
      for (int c = tid * 8; c < f.in; c += kSelPartThreads * 8) {
        const sel_u32x4 xv = *(const DPLLM_SEL_GLOBAL sel_u32x4*)(f.x + c);
        const __half* xh = reinterpret_cast<const __half*>(&xv);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float v = __half2float(xh[i]);
          acc += (double)(v * v);
        }
      }
      acc = wave_sum_f64(acc);
      if (lane == 0) sh[16 + wave] = acc;
    }
    lds_barrier();
    double tot = 0.0;
#pragma unroll
    for (int w = 0; w < kSelPartWaves; ++w) tot += sh[16 + w];
    e = (double)P.alpha * sqrt(tot) + (double)P.beta;
  }
  const int k = (P.kind != 0 && e > (double)P.T) ? P.h : P.l;
  if (write && tid == 0) {
    *f.e_out = (float)e;
    *f.k_out = k;
  }
  return k;
}

// parts == nullptr: the single job `one_job` with the parameters `one`; workgroup b is its projection part b, or
// (linear regression: one workgroup) its group part.  Else workgroup b serves parts[b] of the launch's job table
// under the parameters `active` (members: the launch's table of group members).
__global__ void __launch_bounds__(kSelPartThreads) __attribute__((amdgpu_waves_per_eu(5))) selector_part_kernel(const SelJob* __restrict__ jobs, const SelPart* __restrict__ parts,
                                                                         const int32_t* __restrict__ members,
                                                                         const SelParams* __restrict__ active,
                                                                         SelJob one_job, SelParams one) {
  __shared__ SelShared sh;
  if (parts == nullptr) {
    if (one.kind == 1 && one_job.row_each) {
      const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, rg = blockIdx.x / one_job.nchunks, ch = blockIdx.x - rg * one_job.nchunks;
      const int row = rg * kSelPartWaves + wave;
      double sum[1];
      selector_part_products<true>(one_job, one, row, ch, wave, lane, sum);
      if (lane == 0 && row < one.r) ((DPLLM_SEL_GLOBAL double*)one_job.ws)[(size_t)ch * one_job.ws_rows + row] = sum[0];
    } else if (one.kind == 1) selector_proj_part(one_job, one, blockIdx.x, threadIdx.x);
    else selector_group_part(nullptr, nullptr, 1, nullptr, one_job, one, threadIdx.x, sh);
    return;
  }
  const SelPart p = parts[blockIdx.x];
  if (p.part < 0) {
    selector_group_part(jobs, members + p.first, p.count, active, one_job, one, threadIdx.x, sh);
  } else {
    const SelParams P = active[p.linear];
    const SelJob job = jobs[p.job];
    selector_proj_part(job, P, p.part, threadIdx.x);
  }
}

// The estimates and decisions of a selector launch, where no GEMV launch follows that takes them itself:
// workgroup b finishes jobs[b] under the parameters `active` (jobs == nullptr: the single job `one_job` with the
// parameters `one`).  Launched after selector_part_kernel on the same stream.
constexpr int kSelDecideThreads = 128;
__global__ void __launch_bounds__(kSelDecideThreads) selector_decide_kernel(const SelJob* __restrict__ jobs, const SelParams* __restrict__ active,
                                                                            SelJob one_job, SelParams one) {
  __shared__ SelShared sh;
  if (jobs == nullptr) {
    selector_finish(sel_finish_of(one_job), &one, threadIdx.x, kSelDecideThreads, sh.sq, true);
    return;
  }
  const SelJob job = jobs[blockIdx.x];
  selector_finish(sel_finish_of(job), active + job.linear, threadIdx.x, kSelDecideThreads, sh.sq, true);
}

// One estimate in one launch.  The workgroups are parts of the projection, four rows of G by a chunk of columns; the last one
// collects the products of all and decides.  A product travels in two 64-bit words, half of it and the number of the call (tag) in
// each: a word says itself whose it is, so no order of memory locations and no fence is needed (relaxed atomics on both sides), and
// what another call has left is never taken.  Who has collected a product empties its words again, for a graph that replays the
// call under the same number.  Workgroups start in order, and no more than one per launch ever waits, so those it waits for find a
// place whatever else the chip is doing: the wait ends.  Nothing rests on that: it is bounded, and who gives up computes all
// products itself, with the same bits.  What it gave up on may still come and stay; that matters to a replay of the same captured
// call only, which has its number again: a captured call that gives up leaves its number in the mark of the set of slots, and who
// finds its own there (or that several calls have given up) computes for itself too.  (A wait is given up where calls of one model
// overlap, which the header rules out: their products overwrite one another.)  Launches take turns in kEstRing sets of slots.
// What bounds it is a chain of latencies: launch, rows of G and x, the sum over a wavefront, store and collection.
// us of a dpllm_estimate in a graph, with a launch for the parts and one for the decision / one for both: rank 64 of 4096 columns 4.6 / 3.9, of 8192
// 5.1 / 4.5, of 11008 5.7 / 4.7, rank 256 of 4096 5.4 / 4.8, of 11008 7.2 / 5.8, linear regression 3.7 / 2.0; rank 512 of 8192, where rows go four to a
// wavefront, 8.7 / 9.1: beyond the lanes of the workgroup that collects there are two.  14 linears of 7B with a GEMV each: 190 -> 169 (161 with
// products of one word, which what an overlap left behind could pass for), 157 now.
constexpr int kEstRing = 16;
constexpr int kEstRows = 1;             // rows of G of a wavefront
constexpr int kEstPartRows = kSelPartWaves * kEstRows;
constexpr int kEstMaxRank = kSelPartThreads;
constexpr int kEstChunks = 12;          // column chunks of an estimate, at most: as many as are collected at a time
constexpr int kEstPolls = 1 << 20;      // of about a microsecond
constexpr uint32_t kEstAll = ~0u;       // a mark: several captured calls have given up

// Row t of the products, the sum of its chunks (at most CHUNKS, all asked for at once) in order.  A chunk's slots are the lower halves
// of its rows, then the upper ones.  false: given up, or the slots are not relied on.  What lies past the last chunk adds nothing and empties the
// last one's slots again: a branch for each chunk costs more (rank 64 of 4096 columns 4.20 us with, 4.13 without, 11008 5.18 / 5.06, 28672 6.54 / 6.38).
template <int CHUNKS>
__device__ __forceinline__ bool selector_collect(DPLLM_SEL_GLOBAL uint64_t* slots, uint32_t tag, int nchunks, int ws_rows, int t, bool marked, int polls, double& g) {
  uint64_t lo[CHUNKS], hi[CHUNKS];
  auto slot = [&](int i) { return slots + (uint32_t)(min(i, nchunks - 1) * ws_rows * 2) + t; };   // (those past the last: it again)
  for (;;) {
    bool all = true;
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      lo[i] = __hip_atomic_load(slot(i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      hi[i] = __hip_atomic_load(slot(i) + ws_rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) all = all && (uint32_t)(lo[i] >> 32) == tag && (uint32_t)(hi[i] >> 32) == tag;
    if (__all(all)) break;
    if (marked || --polls < 0) return false;
    __builtin_amdgcn_s_sleep(1);
  }
  g = 0.0;
#pragma unroll
  for (int i = 0; i < CHUNKS; ++i) {
    g += i < nchunks ? __builtin_bit_cast(double, hi[i] << 32 | (uint32_t)lo[i]) : 0.0;
    __hip_atomic_store(slot(i), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(slot(i) + ws_rows, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return !marked;
}

// What all workgroups need, and what the last one does where it is on its way, comes as plain arguments that are set in registers with the
// launch (see gemv_lane_kernel): fourteen dwords, so the small ones are packed.  The bound of the wait is loaded from the argument memory while
// the first look at the products is on its way.
struct EstShape {
  int words, nchunks, ws_rows;               // 32-column words of the vector (16 bits); chunks; rows of a chunk's slots (a multiple of 16, up to 496)
  __host__ __device__ uint32_t pack() const { return (uint32_t)(words | nchunks << 16 | ws_rows / kSelPartRows << 22); }
  static __host__ __device__ EstShape unpack(uint32_t v) { return {(int)(v & 0xffff), (int)(v >> 16 & 63), (int)(v >> 22 & 31) * kSelPartRows}; }
};
constexpr int kEstMaxWords = 65535 / 16 * 16;   // (whole chunks of 512 columns in 12 bits)
struct EstPair {
  int chunk_cols, r, kind, captured, l, h;   // a multiple of 512; up to kEstMaxRank; SelParams; whether a graph holds the call
  __host__ __device__ uint32_t pack() const {
    return (uint32_t)(chunk_cols / kSelChunkStep | r << 12 | kind << 21 | captured << 23) | (uint32_t)l << 24 | (uint32_t)h << 28;
  }
  static __host__ __device__ EstPair unpack(uint32_t v) {
    return {(int)(v & 0xfff) * kSelChunkStep, (int)(v >> 12 & 0x1ff), (int)(v >> 21 & 3), (int)(v >> 23 & 1), (int)(v >> 24 & 15), (int)(v >> 28)};
  }
};
// A set of slots is a header of kEstHeader 64-bit words, whose first dword is its mark, and the slots (ws).
constexpr int kEstHeader = 16;
__global__ void __launch_bounds__(kSelPartThreads) selector_estimate_kernel(const uint16_t* G, const uint16_t* x, uint64_t* ws, float* e_out, int32_t* k_out,
                                                                           uint32_t shape, uint32_t pair, uint32_t tag, float T, int polls, float alpha,
                                                                           float beta) {
  __shared__ SelShared sh;
  __shared__ int here[kSelPartWaves];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const EstShape S = EstShape::unpack(shape);
  const EstPair Q = EstPair::unpack(pair);
  const int in = S.words * 32, nchunks = S.nchunks, ws_rows = S.ws_rows, r = Q.r, kind = Q.kind;
  SelParams P{};
  P.G = G; P.r = r; P.kind = kind;
  SelJob job{};
  job.x = x; job.in = in; job.nchunks = nchunks; job.chunk_cols = Q.chunk_cols;
  double e = 0.0;
  if (kind == 1) {
    static_assert(kEstRows == 1 && kEstMaxRank <= kSelPartThreads, "a product a wavefront, a row a lane");
    DPLLM_SEL_GLOBAL uint64_t* slots = (DPLLM_SEL_GLOBAL uint64_t*)ws;
    DPLLM_SEL_GLOBAL uint32_t* mark = (DPLLM_SEL_GLOBAL uint32_t*)(slots - kEstHeader);
    const int rg = blockIdx.x / nchunks, ch = blockIdx.x - rg * nchunks, row = rg * kEstPartRows + wave;
    double g[1];
    selector_part_products<true>(job, P, row, ch, wave, lane, g);
    if (lane == 0 && row < r) {
      const uint64_t v = __builtin_bit_cast(uint64_t, g[0]);
      DPLLM_SEL_GLOBAL uint64_t* slot = slots + (size_t)ch * ws_rows * 2 + row;
      __hip_atomic_store(slot, (uint64_t)tag << 32 | (uint32_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(slot + ws_rows, (uint64_t)tag << 32 | v >> 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (blockIdx.x + 1 != gridDim.x) return;
    const uint32_t found = Q.captured ? __hip_atomic_load(mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    const bool marked = found == tag || found == kEstAll;
    bool all = true;
    if (wave * 64 < r) {
      all = nchunks <= 8 ? selector_collect<8>(slots, tag, nchunks, ws_rows, min(tid, r - 1), marked, polls, g[0])
                         : selector_collect<kEstChunks>(slots, tag, nchunks, ws_rows, min(tid, r - 1), marked, polls, g[0]);
      sh.sq[tid] = g[0] * g[0];
    }
    if (lane == 0) here[wave] = all;
    __syncthreads();
    if (!(here[0] && here[1] && here[2] && here[3])) {
      static_assert(kSelPartWaves == 4, "flags");
      __syncthreads();
      if (tid == 0 && Q.captured) {
        uint32_t was = 0u;
        if (!__hip_atomic_compare_exchange_strong(mark, &was, tag, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) && was != tag)
          __hip_atomic_store(mark, kEstAll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      for (int t = wave; t < r; t += kSelPartWaves) {
        double sum = 0.0;
        for (int c = 0; c < nchunks; ++c) {
          selector_part_products<true>(job, P, t, c, wave, lane, g);
          sum += g[0];
        }
        if (lane == 0) sh.sq[t] = sum * sum;
      }
      __syncthreads();
    }
    if (tid >= 64) return;
    // as selector_finish does: the same bits
    double part = 0.0;
    for (int t = tid; t < r; t += 64) part += sh.sq[t];
    e = sqrt(wave_sum_f64(part));
  } else if (kind == 2) {
    // as selector_group_part does
    double acc = 0.0;
    for (int c = tid * 8; c < in; c += kSelPartThreads * 8) {
      const sel_u32x4 xv = *(const DPLLM_SEL_GLOBAL sel_u32x4*)(x + c);
      const __half* xh = reinterpret_cast<const __half*>(&xv);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float v = __half2float(xh[i]);
        acc += (double)(v * v);  // exact square in fp32
      }
    }
    acc = wave_sum_f64(acc);
    if (lane == 0) sh.sq[wave] = acc;
    __syncthreads();
    double tot = 0.0;
    for (int w = 0; w < kSelPartWaves; ++w) tot += sh.sq[w];
    e = (double)alpha * sqrt(tot) + (double)beta;
  }
  if (tid == 0) {
    *e_out = (float)e;
    *k_out = kind != 0 && e > (double)T ? Q.h : Q.l;
  }
}

}  // namespace dpllm
