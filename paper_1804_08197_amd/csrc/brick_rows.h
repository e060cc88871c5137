// brick_rows.h -- how the kernels that write or scan whole bricks share a
// slot out over threads.
//
// The unit is a row of four voxels along x: row r (0..15) of 4x4x4 block q,
// the blocks of a slot counted x fastest, M = ceil(S / 4) to an edge in both
// slot layouts. Item i = 16 q + r: sixteen consecutive lanes hold one block,
// a wave four blocks along x. In a micro-block slot row i is the four voxels
// at element 4 i, so a wave reads or writes one run of 512 (uint16) or 256
// (uint8) bytes; in a linear slot a workgroup's sixteen blocks cover the
// same sixteen rows over 128 bytes. Everything about a row (its place in the
// level, whether it holds apron voxels) is decided once per four voxels, with
// quotients from a reciprocal instead of 64-bit divisions per voxel.
#pragma once

#include <algorithm>

#include "sg_internal.h"

namespace sg {

// floor(x / d) exactly for 0 <= x < 2^21 (inv = rcp(d)): the reciprocal is
// within one ulp, so the product is off by less than 2^-22 of its value,
// and (x + 1/2) / d lies at least 1 / (2 d) from an integer. A slot of the
// largest brick (256) has 65^3 < 2^19 blocks.
__device__ __forceinline__ int quot_exact(int x, float inv) {
  return (int)(((float)x + 0.5f) * inv);
}

struct Row {
  int bx, x, y, z;  // block column; stored index of the first voxel, and the row
};
// inv_m, inv_mm: reciprocals of M and M M.
__device__ __forceinline__ Row row_at(int i, int M, float inv_m, float inv_mm) {
  const int q = i >> 4, bz = quot_exact(q, inv_mm), t = q - bz * M * M,
            by = quot_exact(t, inv_m), bx = t - by * M;
  return Row{bx, 4 * bx, 4 * by + (i & 3), 4 * bz + ((i >> 2) & 3)};
}

// Four voxels, as read: packed into one (uint8) or two (uint16) words, x
// fastest from the low end.
template <typename T>
struct Vox4 {
  uint32_t w[sizeof(T)];
  __device__ __forceinline__ uint32_t get(int k) const {
    return sizeof(T) == 1 ? (w[0] >> (8 * k)) & 0xFFu : (w[k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
  }
  __device__ __forceinline__ void set(int k, uint32_t v) {
    const int b = sizeof(T) == 1 ? 8 * k : 16 * (k & 1);
    uint32_t& d = w[sizeof(T) == 1 ? 0 : k >> 1];
    d = (d & ~((sizeof(T) == 1 ? 0xFFu : 0xFFFFu) << b)) | (v << b);
  }
};
// Rows per thread in flight: a thread's loads of a batch are issued together
// (with one row at a time 2048 threads per CU keep 4 MB in flight over the
// chip, which measured 1.5 to 2 TB/s).
constexpr int kRowBatch = 4;

// Workgroups per brick for `bricks` bricks of `items` rows: enough for
// about 4096 workgroups in all (16 per CU), each with at least one batch
// of rows per thread, and one per brick (no merging of ranges) from 4096
// bricks on.
inline int groups_per_brick(int64_t bricks, int items) {
  const int64_t want = (4096 + bricks - 1) / std::max<int64_t>(bricks, 1);
  const int64_t most = std::max<int64_t>(1, items / (256 * kRowBatch));
  return (int)std::max<int64_t>(1, std::min(want, most));
}

// The workgroups (256 threads) of a launch over n bricks of M blocks an edge:
// `per` to a brick, or `pack`: bricks of 2 and 4 (M = 1 and 2) share
// workgroups, one row to a thread: all 16 and 128 rows, or the 4 and 32 that
// hold core voxels (`core`). With a workgroup each, most of its threads had
// nothing to do, and a 256^3 volume in bricks of 4 took 437, 66 and 667 us to
// upload, build and commit (343, 44 and 499 with one thread per voxel; 316, 43
// and 384 so).
struct Shares {
  bool pack;
  int per, n;
  unsigned grid;
};
__host__ __device__ constexpr int pack_log(int M, bool core) {  // log2 threads to a brick
  return M == 1 ? (core ? 2 : 4) : (core ? 5 : 7);
}
inline Shares brick_shares(int64_t n, int M, bool core = false) {
  Shares s;
  s.n = (int)n;
  s.pack = M <= 2;
  s.per = s.pack ? 1 : groups_per_brick(n, M * M * M * 16);
  s.grid = (unsigned)(s.pack ? ((n << pack_log(M, core)) + 255) / 256 : n * s.per);
  return s;
}
// A thread's part in such a launch: brick j (at or beyond n: none), workgroup
// `part` of those that share it, thread `lane` of `threads` on the brick, and
// which of the workgroup's bricks it is.
struct Part {
  int64_t j;
  int part, lane, threads, sub;
};
template <bool PACK, bool CORE = false>
__device__ __forceinline__ Part brick_part(int per, int M) {
  if (PACK) {
    const int log = pack_log(M, CORE), sub = (int)(threadIdx.x >> log);
    return Part{((int64_t)blockIdx.x << (8 - log)) + sub, 0, (int)(threadIdx.x & ((1u << log) - 1)),
                1 << log, sub};
  }
  return Part{(int64_t)(blockIdx.x / (unsigned)per), (int)(blockIdx.x % (unsigned)per),
              (int)threadIdx.x, 256, 0};
}
template <bool PACK, bool CORE = false>
constexpr int kMostBricks = PACK ? 256 >> pack_log(1, CORE) : 1;  // to a workgroup
// Row k of those of a brick of 2 or 4 that hold core voxels: its number among
// all rows.
__device__ __forceinline__ int core_row_number(int k, int M) {
  const int bx = k & (M - 1), t = k >> (M - 1), y = 1 + (t & (2 * M - 1)), z = 1 + (t >> M);
  return 16 * (((z >> 2) * M + (y >> 2)) * M + bx) + 4 * (z & 3) + (y & 3);
}

// Element offset of a row's first voxel in the slot.
template <bool MB>
__device__ __forceinline__ int64_t row_offset(const Row& w, int i, int S, int Sx) {
  return MB ? (int64_t)4 * i : ((int64_t)w.z * S + w.y) * Sx + w.x;
}
// Rows of a slot are read and written in 4-byte words (linear rows start on
// 4-byte boundaries, see kRowAlignBytes) or one 4- or 8-byte word
// (micro-blocks). A linear row's last word may lie past the row stride: it
// is left alone (its voxels read as 0; none of them is below S).
template <typename T, bool MB>
__device__ __forceinline__ Vox4<T> load_row(const T* slot, const Row& w, int i, int S, int Sx) {
  const T* p = slot + row_offset<MB>(w, i, S, Sx);
  Vox4<T> o;
  if (sizeof(T) == 1) {
    o.w[0] = *reinterpret_cast<const uint32_t*>(p);
  } else if (MB) {
    const uint2 ab = *reinterpret_cast<const uint2*>(p);
    o.w[0] = ab.x;
    o.w[sizeof(T) - 1] = ab.y;
  } else {
    o.w[0] = reinterpret_cast<const uint32_t*>(p)[0];
    o.w[sizeof(T) - 1] = w.x + 2 < Sx ? reinterpret_cast<const uint32_t*>(p)[1] : 0u;
  }
  return o;
}
// Four voxels at p, at a row boundary of the slot, none beyond its end.
template <typename T, bool MB>
__device__ __forceinline__ Vox4<T> four_at(const T* p) {
  Vox4<T> o;
  if (sizeof(T) > 1 && MB) {
    const uint2 ab = *reinterpret_cast<const uint2*>(p);
    o.w[0] = ab.x;
    o.w[sizeof(T) - 1] = ab.y;
  } else {
#pragma unroll
    for (int k = 0; k < (int)sizeof(T); ++k) o.w[k] = reinterpret_cast<const uint32_t*>(p)[k];
  }
  return o;
}
template <typename T, bool MB>
__device__ __forceinline__ void store_row(T* slot, const Row& w, int i, int S, int Sx,
                                          const Vox4<T>& o) {
  T* p = slot + row_offset<MB>(w, i, S, Sx);
  if (sizeof(T) == 1) {
    *reinterpret_cast<uint32_t*>(p) = o.w[0];
  } else if (MB) {
    *reinterpret_cast<uint2*>(p) = make_uint2(o.w[0], o.w[sizeof(T) - 1]);
  } else {
    reinterpret_cast<uint32_t*>(p)[0] = o.w[0];
    if (w.x + 2 < Sx) reinterpret_cast<uint32_t*>(p)[1] = o.w[sizeof(T) - 1];
  }
}

// The largest value over the sixteen lanes of a block, in every one of them
// (lane swaps inside a 16-lane row; all sixteen lanes active).
__device__ __forceinline__ uint32_t row16_max(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false));   // xor 1
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false));   // xor 2
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false));  // half mirror
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false));  // mirror
  return v;
}

// The first `left` voxels of a row folded into a minimum and a maximum.
// Interior rows (left >= 4) fold two packed uint16 at a time.
template <typename T>
__device__ __forceinline__ void row_range(const Vox4<T>& o, int left, uint32_t& lo, uint32_t& hi) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  if (sizeof(T) == 2 && left >= 4) {
    const u16x2 a = __builtin_bit_cast(u16x2, o.w[0]), b = __builtin_bit_cast(u16x2, o.w[sizeof(T) - 1]);
    const u16x2 mn = __builtin_elementwise_min(a, b), mx = __builtin_elementwise_max(a, b);
    lo = min(lo, min((uint32_t)mn.x, (uint32_t)mn.y));
    hi = max(hi, max((uint32_t)mx.x, (uint32_t)mx.y));
    return;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (k < left) {
      lo = min(lo, o.get(k));
      hi = max(hi, o.get(k));
    }
}

// A workgroup's (256 threads) share of a brick's value range, into range[0]
// (minimum) and range[1] (maximum): stored when the workgroup holds the whole
// brick, else merged with atomics (they start at ~0 and 0; minima and maxima
// do not depend on the order). With PACK every brick of the workgroup is
// whole: range is the thread's own brick's, NULL beyond the last.
template <bool PACK>
__device__ __forceinline__ void range_out(uint32_t lo, uint32_t hi, uint32_t* range, bool whole,
                                          const Part& p) {
  if (PACK && p.threads == 16) {  // the same for the whole workgroup
    hi = row16_max(hi);
    lo = ~row16_max(~lo);
    if (p.lane == 0 && range) {
      range[0] = lo;
      range[1] = hi;
    }
    return;
  }
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, m));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, m));
  }
  __shared__ uint32_t part[2][4];
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    part[0][wave] = lo;
    part[1][wave] = hi;
  }
  __syncthreads();
  if (PACK) {  // two waves a brick
    if (p.lane != 0 || !range) return;
    range[0] = min(part[0][wave], part[0][wave + 1]);
    range[1] = max(part[1][wave], part[1][wave + 1]);
    return;
  }
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    lo = min(lo, part[0][k]);
    hi = max(hi, part[1][k]);
  }
  if (whole) {
    range[0] = lo;
    range[1] = hi;
  } else {
    atomicMin(range, lo);
    atomicMax(range + 1, hi);
  }
}

}  // namespace sg
