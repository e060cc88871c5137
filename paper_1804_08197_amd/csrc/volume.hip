// volume.hip -- brick pool, page table, uploads, pyramid, aprons, value
// ranges and empty-node flags (the one-time per-volume work, and the
// per-transfer-function refresh).
//
// Pool layout: one slot per (timepoint, channel, node); a slot stores the
// node's brick as (B+2)^3 voxels, the core at offset (1, 1, 1) and a
// one-voxel apron around it holding the clamped neighbour values, in the
// volume's slot layout (slot_index): linear rows, x fastest, padded to a
// multiple of 4 bytes (row stride Sx), or 4^3-voxel micro-blocks
// (Sec 5.2: blocks of a multi-resolution pyramid; Sec 4.2: chunks resident
// in a GPU cache). With the apron, any trilinear sample inside a node reads
// only that node's slot.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "brick_rows.h"

namespace sg {

namespace {

__device__ __forceinline__ int32_t clampi(int32_t v, int32_t lo, int32_t hi) {
  return v < lo ? lo : (v > hi ? hi : v);
}

template <typename T>
__device__ __forceinline__ T* slot_ptr(uint8_t* pool, int64_t slot_bytes,
                                       int32_t slot) {
  return reinterpret_cast<T*>(pool + (int64_t)slot * slot_bytes);
}

struct LevelGeom {
  int32_t n[3];      // level dims
  int32_t g[3];      // brick grid
  int64_t node_off;  // first node index of the level
};
struct Levels {
  int32_t n[kMaxLevels][3];
  int32_t g[kMaxLevels][3];
  int64_t node_off[kMaxLevels];
};

// A row of a destination brick that holds core voxels: stored y and z in
// [1, B]. The rows' apron columns (stored x = 0 and B + 1) are written with
// whatever voxel is at hand; commit fills every apron before anything reads
// one.
__device__ __forceinline__ bool core_row(const Row& w, int B) {
  return w.y >= 1 && w.y <= B && w.z >= 1 && w.z <= B && w.x <= B;
}

// Upload: scatter n brick cores (x fastest) into their slots, one thread per
// stored row of four voxels (see brick_rows.h). Bound by memory. A stored row
// holds core voxels x - 1 .. x + 2 (x a multiple of four): WIDE reads the aligned voxels
// x .. x + 3 with one load and voxel x - 1 with another (cores of at least
// four voxels an edge at a row-aligned address); otherwise voxel by voxel.
// 512^3 uint16 in micro-block slots: 167 us (3.2 TB/s read and written; 426
// with one thread per voxel, 260 with one row in flight and 2-byte loads).
template <typename T, bool MB, bool WIDE, bool PACK>
__global__ __launch_bounds__(256) void upload_kernel(uint8_t* __restrict__ pool,
                                                     int64_t slot_bytes, const int32_t* page,
                                                     LevelGeom lg, const int32_t* coords,
                                                     const T* __restrict__ src, int n, int per,
                                                     int logB, int S, int Sx, int M) {
  constexpr int kBatch = PACK ? 1 : kRowBatch;
  const int B = 1 << logB, items = M * M * M * 16;
  const Part p = brick_part<PACK, true>(per, M);
  const int64_t j = p.j;
  if (j >= n) return;
  const float inv_m = __builtin_amdgcn_rcpf((float)M), inv_mm = __builtin_amdgcn_rcpf((float)(M * M));
  const int32_t* c = coords + 3 * (int64_t)j;
  const int64_t node = lg.node_off + ((int64_t)c[2] * lg.g[1] + c[1]) * lg.g[0] + c[0];
  T* dst = slot_ptr<T>(pool, slot_bytes, page[node]);
  src += j << (3 * logB);
  const int first = PACK ? core_row_number(p.lane, M) : p.part * 256 * kBatch + p.lane;
  for (int i0 = first; i0 < items; i0 += PACK ? items : per * 256 * kBatch) {
    Row w[kBatch];
    Vox4<T> o[kBatch];
    uint32_t before[kBatch];
    bool on[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + 256 * u;
      w[u] = row_at(i, M, inv_m, inv_mm);
      on[u] = i < items && core_row(w[u], B);
      if (!on[u]) continue;
      const T* q = src + ((((w[u].z - 1) << logB) + (w[u].y - 1)) << logB);
      const int x = w[u].x;
      if (WIDE) {
        o[u] = Vox4<T>{};
        if (x < B) {
          if (sizeof(T) == 1) {
            o[u].w[0] = *reinterpret_cast<const uint32_t*>(q + x);
          } else {
            const uint2 ab = *reinterpret_cast<const uint2*>(q + x);
            o[u].w[0] = ab.x;
            o[u].w[sizeof(T) - 1] = ab.y;
          }
        }
        before[u] = q[max(x - 1, 0)];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) o[u].set(k, q[clampi(x + k - 1, 0, B - 1)]);
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (!on[u]) continue;
      if (WIDE) {  // one voxel to the right
        if (sizeof(T) == 1) {
          o[u].w[0] = (o[u].w[0] << 8) | before[u];
        } else {
          o[u].w[sizeof(T) - 1] = (o[u].w[sizeof(T) - 1] << 16) | (o[u].w[0] >> 16);
          o[u].w[0] = (o[u].w[0] << 16) | before[u];
        }
      }
      store_row<T, MB>(dst, w[u], i0 + 256 * u, S, Sx, o[u]);
    }
  }
}

// Pyramid: core voxel g of level L+1 = (sum of children 2g + delta, clamped
// to level L, + 4) >> 3. Children are read from level-L cores. One thread
// per destination row of four voxels; a voxel's eight children lie in one
// source brick (2g and 2g + 1 share a brick: its edge is even), whose slot
// is one of the eight under the destination brick, and the child's offset
// in the slot is a sum of one part per axis. A stored row holds the core
// voxels x - 1 .. x + 2: the children of the last three are read as whole
// rows of four, those of the first (in the blocks before, maybe in another
// brick) one by one, as are all of them at the level's far end. The row
// beyond the core's end has one core voxel; the other three are apron.
// Three levels of 512^3 uint16: 178 us (226 with a 2-byte load per child, 400
// with one thread, eight node look-ups and 64-bit divisions per voxel).
template <typename T, bool MB, bool PACK>
__global__ __launch_bounds__(256) void downsample_kernel(uint8_t* pool, int64_t slot_bytes,
                                                         const int32_t* page, LevelGeom src,
                                                         LevelGeom dst, int n, int per, int logB,
                                                         int S, int Sx, int M) {
  const int B = 1 << logB, mask = B - 1, items = M * M * M * 16;
  const float inv_m = __builtin_amdgcn_rcpf((float)M), inv_mm = __builtin_amdgcn_rcpf((float)(M * M));
  const Part p = brick_part<PACK, true>(per, M);
  const int64_t j = p.j;
  const uint32_t row = (uint32_t)j / (uint32_t)dst.g[0];
  const int b[3] = {(int)((uint32_t)j - row * (uint32_t)dst.g[0]), (int)(row % (uint32_t)dst.g[1]),
                    (int)(row / (uint32_t)dst.g[1])};
  // the source slots under this brick (indices clamped into the grid: those
  // beyond it are never the brick of a child)
  __shared__ int32_t under[kMostBricks<PACK, true>][8];
  int32_t* const slots = under[p.sub];
  for (int k = p.lane; k < 8 && j < n; k += p.threads) {
    const int sx = min(2 * b[0] + (k & 1), src.g[0] - 1), sy = min(2 * b[1] + ((k >> 1) & 1), src.g[1] - 1),
              sz = min(2 * b[2] + (k >> 2), src.g[2] - 1);
    slots[k] = page[src.node_off + ((int64_t)sz * src.g[1] + sy) * src.g[0] + sx];
  }
  __syncthreads();
  if (j >= n) return;
  T* out = slot_ptr<T>(pool, slot_bytes, page[dst.node_off + j]);
  // the parts of slot_index per axis (stored index = core index + 1)
  auto fx = [&](int h) { const int x = (h & mask) + 1; return MB ? ((x >> 2) << 6) + (x & 3) : x; };
  auto fy = [&](int h) {
    const int y = (h & mask) + 1;
    return MB ? (((y >> 2) * M) << 6) + ((y & 3) << 2) : y * Sx;
  };
  auto fz = [&](int h) {
    const int z = (h & mask) + 1;
    return MB ? (((z >> 2) * M * M) << 6) + ((z & 3) << 4) : z * S * Sx;
  };
  const int first = PACK ? core_row_number(p.lane, M) : p.part * 256 + p.lane;
  for (int i = first; i < items; i += PACK ? items : per * 256) {
    const Row w = row_at(i, M, inv_m, inv_mm);
    if (!core_row(w, B)) continue;
    const int gy = min(b[1] * B + w.y - 1, dst.n[1] - 1), gz = min(b[2] * B + w.z - 1, dst.n[2] - 1);
    const int y0 = 2 * gy, y1 = min(2 * gy + 1, src.n[1] - 1);
    const int z0 = 2 * gz, z1 = min(2 * gz + 1, src.n[2] - 1);
    const int oct = (((z0 >> logB) & 1) << 2) | (((y0 >> logB) & 1) << 1);
    const int r00 = fy(y0) + fz(z0), r10 = fy(y1) + fz(z0), r01 = fy(y0) + fz(z1),
              r11 = fy(y1) + fz(z1);
    Vox4<T> o{};
    auto one = [&](int k) {
      const int gx = min(b[0] * B + clampi(w.x + k - 1, 0, B - 1), dst.n[0] - 1);
      const int x0 = 2 * gx, x1 = min(2 * gx + 1, src.n[0] - 1);
      const T* q = slot_ptr<T>(pool, slot_bytes, slots[oct | ((x0 >> logB) & 1)]);
      const int a = fx(x0), c = fx(x1);
      const uint32_t sum = (uint32_t)q[r00 + a] + q[r00 + c] + q[r10 + a] + q[r10 + c] +
                           q[r01 + a] + q[r01 + c] + q[r11 + a] + q[r11 + c];
      o.set(k, (sum + 4u) >> 3);
    };
    one(0);
    const int cx = b[0] * B + w.x;  // voxels 1 .. 3 are the level's cx .. cx + 2
    if (B >= 8 && w.x < B && 2 * cx + 5 < src.n[0]) {
      const int h = (2 * w.x) & mask;  // their children: stored h + 1 .. h + 6
      const T* q = slot_ptr<T>(pool, slot_bytes, slots[oct | (((2 * cx) >> logB) & 1)]) +
                   (MB ? (h >> 2) << 6 : h);
      const int next = MB ? 64 : 4;
      const int rows[4] = {r00, r10, r01, r11};
      Vox4<T> c[4][2];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < 2; ++u) c[r][u] = four_at<T, MB>(q + rows[r] + u * next);
      uint32_t s1 = 4u, s2 = 4u, s3 = 4u;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s1 += c[r][0].get(1) + c[r][0].get(2);
        s2 += c[r][0].get(3) + c[r][1].get(0);
        s3 += c[r][1].get(1) + c[r][1].get(2);
      }
      o.set(1, s1 >> 3);
      o.set(2, s2 >> 3);
      o.set(3, s3 >> 3);
    } else if (w.x < B) {
      one(1);
      one(2);
      one(3);
    }
    store_row<T, MB>(out, w, i, S, Sx, o);
  }
}

// Aprons of every brick of a (channel, timepoint), all levels in one launch:
// every stored voxel that is not an in-extent core voxel receives the value
// of the clamped level index, read from the owning brick's core (cores are
// only read here, so no brick waits for another). A brick that lies in the
// level's extent needs its six faces only, S x S voxels each, one thread per
// voxel (edges and corners are written by two or three faces, with the same
// value); a brick cut by the far faces walks all of its rows. Also resets
// the ranges that range_kernel merges into. Four levels of 512^3 uint16: 96
// us in one launch (332 in four, one thread walking the 66 voxels of each
// stored row); fused with range_kernel the two took 221 us instead of 164:
// most waves hold an apron row, so most paid for the fill.
template <typename T, bool MB, bool PACK>
__global__ __launch_bounds__(256) void apron_kernel(uint8_t* pool, int64_t slot_bytes,
                                                    const int32_t* page, const NodeInfo* info,
                                                    Levels lv, uint32_t* range, int n, int per,
                                                    int logB, int S, int Sx, int M) {
  const int B = 1 << logB, mask = B - 1, items = M * M * M * 16;
  const Part p = brick_part<PACK>(per, M);
  const int64_t node = min(p.j, (int64_t)n - 1);
  const NodeInfo ni = info[node];
  const int L = ni.level;
  const int n0 = lv.n[L][0], n1 = lv.n[L][1], n2 = lv.n[L][2];
  const int g0 = ni.b[0] * B - 1, g1 = ni.b[1] * B - 1, g2 = ni.b[2] * B - 1;  // of stored (0,0,0)
  T* own = slot_ptr<T>(pool, slot_bytes, page[node]);
  // the slots of the 3x3x3 bricks around this one (clamped into the grid:
  // one beyond it never owns a clamped voxel)
  __shared__ int32_t around[kMostBricks<PACK>][27];
  int32_t* const near = around[p.sub];
  for (int k = p.lane; k < 27; k += p.threads) {
    const int x = clampi(ni.b[0] + k % 3 - 1, 0, lv.g[L][0] - 1),
              y = clampi(ni.b[1] + (k / 3) % 3 - 1, 0, lv.g[L][1] - 1),
              z = clampi(ni.b[2] + k / 9 - 1, 0, lv.g[L][2] - 1);
    near[k] = page[lv.node_off[L] + ((int64_t)z * lv.g[L][1] + y) * lv.g[L][0] + x];
  }
  __syncthreads();
  if (p.j >= n) return;
  if (p.part == 0 && p.lane == 0) {
    range[2 * node] = 0xFFFFFFFFu;
    range[2 * node + 1] = 0u;
  }
  // stored voxel (x, y, z) of this brick from the brick that owns it
  auto from = [&](int x, int y, int z) -> const T* {
    const int cx = clampi(g0 + x, 0, n0 - 1), cy = clampi(g1 + y, 0, n1 - 1),
              cz = clampi(g2 + z, 0, n2 - 1);
    const int k = 9 * ((cz >> logB) - ni.b[2] + 1) + 3 * ((cy >> logB) - ni.b[1] + 1) +
                  (cx >> logB) - ni.b[0] + 1;
    return slot_ptr<T>(pool, slot_bytes, near[k]) +
           slot_index((cx & mask) + 1, (cy & mask) + 1, (cz & mask) + 1, S, Sx, MB ? M : 0);
  };
  if (g0 + B < n0 && g1 + B < n1 && g2 + B < n2) {
    const int face = S * S;
    const float inv_f = __builtin_amdgcn_rcpf((float)face), inv_s = __builtin_amdgcn_rcpf((float)S);
    for (int i = p.part * 256 + p.lane; i < 6 * face; i += per * p.threads) {
      const int f = quot_exact(i, inv_f), r = i - f * face, v = quot_exact(r, inv_s), u = r - v * S;
      const int edge = (f & 1) ? S - 1 : 0;
      // faces 0, 1 across x, 2, 3 across y, 4, 5 across z; u runs along the
      // face's faster axis
      const int x = f < 2 ? edge : u, y = f < 2 ? u : (f < 4 ? edge : v), z = f < 4 ? v : edge;
      own[slot_index(x, y, z, S, Sx, MB ? M : 0)] = *from(x, y, z);
    }
    return;
  }
  const float inv_m = __builtin_amdgcn_rcpf((float)M), inv_mm = __builtin_amdgcn_rcpf((float)(M * M));
  for (int i = p.part * 256 + p.lane; i < items; i += per * 256) {
    const Row w = row_at(i, M, inv_m, inv_mm);
    if (w.y >= S || w.z >= S) continue;
    const bool row_core = w.y >= 1 && w.y <= B && w.z >= 1 && w.z <= B && g1 + w.y < n1 &&
                          g2 + w.z < n2;
    if (row_core && w.x >= 1 && w.x + 3 <= B && g0 + w.x + 3 < n0) continue;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int x = w.x + k;
      if (x >= S || (row_core && x >= 1 && x <= B && g0 + x < n0)) continue;
      own[slot_index(x, w.y, w.z, S, Sx, MB ? M : 0)] = *from(x, w.y, w.z);
    }
  }
}

// One pass over every brick of a (channel, timepoint) once its apron is in
// place: the largest value of every 4x4x4 block of the slot (bmax, or NULL)
// and the brick's value range over every stored voxel (core and apron). One
// thread per stored row of four voxels; bound by reading the pool once.
// Four levels of 512^3 uint16: 68 us (5.4 TB/s; 555 with one workgroup per
// brick and a division per voxel); one 128^3 uint8 brick took 3.1 ms so.
template <typename T, bool MB, bool PACK>
__global__ __launch_bounds__(256) void range_kernel(const uint8_t* __restrict__ pool,
                                                    int64_t slot_bytes, const int32_t* page,
                                                    uint32_t* range, uint8_t* bmax,
                                                    int64_t bmax_stride, int n, int per, int S,
                                                    int Sx, int M) {
  constexpr int kBatch = PACK ? 1 : kRowBatch;
  const int items = M * M * M * 16;
  const Part p = brick_part<PACK>(per, M);
  const bool any = !PACK || p.j < n;
  const int64_t node = any ? p.j : 0;
  const float inv_m = __builtin_amdgcn_rcpf((float)M), inv_mm = __builtin_amdgcn_rcpf((float)(M * M));
  const int32_t slot = page[node];
  const T* own = reinterpret_cast<const T*>(pool + (int64_t)slot * slot_bytes);
  T* bm = bmax ? reinterpret_cast<T*>(bmax + (int64_t)slot * bmax_stride) : nullptr;
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  // (the same trip count for every lane: blocks are folded across lanes)
  for (int i0 = p.part * 256 * kBatch; i0 < items; i0 += per * 256 * kBatch) {
    Row w[kBatch];
    Vox4<T> o[kBatch];
    bool on[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + 256 * u + p.lane;
      w[u] = row_at(i, M, inv_m, inv_mm);
      on[u] = any && i < items && w[u].y < S && w[u].z < S;
      o[u] = Vox4<T>{};
      if (on[u]) o[u] = load_row<T, MB>(own, w[u], i, S, Sx);
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + 256 * u + p.lane;
      uint32_t rmax = 0u;
      if (on[u]) row_range(o[u], S - w[u].x, lo, rmax);
      hi = max(hi, rmax);
      if (PACK) continue;  // (no block maxima)
      rmax = row16_max(rmax);
      if (bm && i < items && (i & 15) == 0) bm[i >> 4] = (T)rmax;
    }
  }
  range_out<PACK>(lo, hi, any ? range + 2 * node : nullptr, per == 1, p);
}

// Of a brick's regions of three to four blocks an edge, about the size of a
// wave's slab, the maximum that a quarter stay at or below (dark): under a
// table that is transparent up to there the ray caster asks of each slab in
// the brick whether it holds anything. Where fewer regions are, asking costs
// more than the slabs stepped over save (every fiftieth 4^3 block opaque, at
// random, and a quarter of the regions free of them: 1431 us a frame without
// asking, 1419 with; every tenth, none free: 1421 and 1544). It is a guess at
// what pays and decides nothing else, so bricks of 128 and 256 are taken in
// six regions to an edge and by every second and fourth row of blocks.
// One workgroup per brick, or one wave for bricks of 16 and 32. Bound by
// latency: the block maxima are read once, a round's loads together, and
// folded into the regions' in LDS; one wave searches them, a ballot for every
// 64, without barriers. 8 us for 585 bricks of 64, 27 for 37449 of 16.
template <typename T>
__global__ __launch_bounds__(512) void dark_kernel(const uint8_t* bmax, int64_t bmax_stride,
                                                   const int32_t* slots, const int32_t* entries,
                                                   int count, int threads, int M, uint32_t* dark) {
  extern __shared__ uint32_t dark_smem[];  // the regions of each of the workgroup's bricks
  constexpr int kLoads = 5;
  const int sub = (int)threadIdx.x / threads, tid = (int)threadIdx.x % threads;
  const int j = (int)(blockIdx.x * (blockDim.x / threads)) + sub;
  const T* bm = reinterpret_cast<const T*>(bmax + (int64_t)slots[min(j, count - 1)] * bmax_stride);
  const int G = dark_regions(M), n = G * G * G;
  const int every = (M + 16) / 17, my = (M + every - 1) / every, blocks = M * my * my;
  const float inv_m = __builtin_amdgcn_rcpf((float)M), inv_p = __builtin_amdgcn_rcpf((float)(M * my));
  uint32_t* const top = dark_smem + sub * n;
  for (int r = tid; r < n; r += threads) top[r] = 0u;
  __syncthreads();
  for (int i0 = tid; i0 < blocks; i0 += threads * kLoads) {
    uint32_t v[kLoads];
    int at[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int i = min(i0 + threads * u, blocks - 1);
      const int sz = quot_exact(i, inv_p), t = i - sz * M * my, sy = quot_exact(t, inv_m);
      const int z = sz * every, y = sy * every, x = t - sy * M;
      v[u] = bm[(z * M + y) * M + x];
      auto part = [&](int c) { return quot_exact(c * G, inv_m); };  // region of block c of an axis
      at[u] = (part(z) * G + part(y)) * G + part(x);
    }
#pragma unroll
    for (int u = 0; u < kLoads; ++u)
      if (i0 + threads * u < blocks) atomicMax(top + at[u], v[u]);
  }
  __syncthreads();
  if (tid >= 64 || j >= count) return;  // whole waves
  const int lane = tid, need = (n + 3) / 4;
  constexpr int kTops = (kDarkRegions * kDarkRegions * kDarkRegions + 63) / 64;
  uint32_t v[kTops];
#pragma unroll
  for (int k = 0; k < kTops; ++k) v[k] = lane + 64 * k < n ? top[lane + 64 * k] : 0xFFFFFFFFu;
  uint32_t lo = 0u, hi = sizeof(T) == 1 ? 255u : 65535u;
  while (lo < hi) {  // the same in every lane
    const uint32_t mid = (lo + hi) / 2;
    int c = 0;
#pragma unroll
    for (int k = 0; k < kTops; ++k) c += __popcll(__ballot(v[k] <= mid));
    if (c >= need) hi = mid; else lo = mid + 1;
  }
  if (lane == 0) dark[entries ? entries[j] : j] = lo;
}

// Skip flags (one thread per (timepoint, node)). Bit 0 (transparent): for
// every channel the extinction of every table entry from floor(u_min) - 1
// to floor(u_max) + 2 is zero, u being the continuous table index of the
// node's min / max value. Bit 1 (dark): the same entries emit no colour.
// The one-entry guard band on each side keeps the flags exact for samples
// whose index is rounded in single precision. next[c][0][k] / next[c][1][k]:
// the first entry from k on with extinction / with colour (tf_n: none), so
// a node takes two reads instead of a walk over the entries (38 -> 3.4 us
// for 585 nodes and 256 entries). Bits 2 and 3: in some channel fewer than a
// quarter of the node's regions (see dark_kernel) stay at or below the largest
// value without extinction (colour), so its slabs are not tested.
__global__ void empty_kernel(const uint32_t* range, const uint32_t* dark, const int32_t* next,
                             const int32_t* dim, int tf_n, const double* lo, const double* hi, int C,
                             int64_t nodes, int64_t total, uint8_t* empty) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    int64_t t = i / nodes, node = i - t * nodes;
    bool clear = true, unlit = true, no_clear = false, no_unlit = false;
    for (int c = 0; c < C; ++c) {
      const int64_t dk = dark[(t * C + c) * nodes + node];
      no_clear |= dk > dim[2 * c];
      no_unlit |= dk > dim[2 * c + 1];
      const uint32_t* r = range + 2 * ((t * C + c) * nodes + node);
      double umin = (((double)r[0] - lo[c]) / (hi[c] - lo[c])) * (double)(tf_n - 1);
      double umax = (((double)r[1] - lo[c]) / (hi[c] - lo[c])) * (double)(tf_n - 1);
      int64_t klo = (int64_t)floor(umin) - 1;
      int64_t khi = (int64_t)floor(umax) + 2;
      klo = klo < 0 ? 0 : (klo > tf_n - 1 ? tf_n - 1 : klo);
      khi = khi < 0 ? 0 : (khi > tf_n - 1 ? tf_n - 1 : khi);
      const int32_t* nx = next + (int64_t)c * 2 * tf_n;
      // (an empty interval, khi < klo: nothing can show)
      if (nx[klo] <= khi) clear = false;
      if (nx[tf_n + klo] <= khi) unlit = false;
    }
    empty[i] = (uint8_t)((clear ? 1 : 0) | (unlit ? 2 : 0) | (no_clear ? 4 : 0) |
                         (no_unlit ? 8 : 0));
  }
}

LevelGeom geom(const Volume* v, int L) {
  LevelGeom g;
  for (int a = 0; a < 3; ++a) {
    g.n[a] = v->ldims[L][a];
    g.g[a] = v->grid[L][a];
  }
  g.node_off = v->node_off[L];
  return g;
}

int blocks_for(int64_t work, int per_block = 256) {
  int64_t b = (work + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > 262144) b = 262144;
  return (int)b;
}

const int32_t* page_at(const Volume* v, int c, int t) {
  return v->page + ((int64_t)t * v->d.channels + c) * v->nodes;
}

}  // namespace

sg_status launch_upload(Volume* v, int c, int t, int level, int n,
                        const int32_t* dcoords, const void* dsrc,
                        hipStream_t s) {
  const LevelGeom lg = geom(v, level);
  const Shares sh = brick_shares(n, v->Mb, true);
  const bool wide = v->B >= 4 && reinterpret_cast<uintptr_t>(dsrc) % (4 * v->bpv) == 0;
#define SG_UPLOAD(T, MB, WIDE, PACK)                                                           \
  hipLaunchKernelGGL((upload_kernel<T, MB, WIDE, PACK>), dim3(sh.grid), dim3(256), 0, s,       \
                     v->pool, v->slot_bytes, page_at(v, c, t), lg, dcoords, (const T*)dsrc,    \
                     sh.n, sh.per, v->logB, v->S, v->Sx, v->Mb)
#define SG_UPLOAD_W(T, MB, WIDE) \
  do { if (sh.pack) SG_UPLOAD(T, MB, WIDE, true); else SG_UPLOAD(T, MB, WIDE, false); } while (0)
#define SG_UPLOAD_T(T)                                                           \
  do {                                                                           \
    if (v->M) {                                                                  \
      if (wide) SG_UPLOAD_W(T, true, true); else SG_UPLOAD_W(T, true, false);    \
    } else {                                                                     \
      if (wide) SG_UPLOAD_W(T, false, true); else SG_UPLOAD_W(T, false, false);  \
    }                                                                            \
  } while (0)
  if (v->bpv == 1) SG_UPLOAD_T(uint8_t); else SG_UPLOAD_T(uint16_t);
#undef SG_UPLOAD_T
#undef SG_UPLOAD_W
#undef SG_UPLOAD
  SG_HIP(hipGetLastError());
  return SG_OK;
}

// A statement for the volume's voxel type T, slot layout MB and sharing PACK.
#define SG_BRICKS(STATEMENT)                                                                   \
  do {                                                                                         \
    if (v->bpv == 1) {                                                                         \
      if (v->M) { if (sh.pack) STATEMENT(uint8_t, true, true); else STATEMENT(uint8_t, true, false); }       \
      else { if (sh.pack) STATEMENT(uint8_t, false, true); else STATEMENT(uint8_t, false, false); }          \
    } else {                                                                                   \
      if (v->M) { if (sh.pack) STATEMENT(uint16_t, true, true); else STATEMENT(uint16_t, true, false); }     \
      else { if (sh.pack) STATEMENT(uint16_t, false, true); else STATEMENT(uint16_t, false, false); }        \
    }                                                                                          \
  } while (0)

sg_status launch_downsample(Volume* v, int c, int t, int level_dst,
                            hipStream_t s) {
  const LevelGeom src = geom(v, level_dst - 1), dst = geom(v, level_dst);
  const Shares sh = brick_shares((int64_t)dst.g[0] * dst.g[1] * dst.g[2], v->Mb, true);
#define SG_DOWN(T, MB, PACK)                                                                   \
  hipLaunchKernelGGL((downsample_kernel<T, MB, PACK>), dim3(sh.grid), dim3(256), 0, s, v->pool, \
                     v->slot_bytes, page_at(v, c, t), src, dst, sh.n, sh.per, v->logB, v->S,   \
                     v->Sx, v->Mb)
  SG_BRICKS(SG_DOWN);
#undef SG_DOWN
  SG_HIP(hipGetLastError());
  return SG_OK;
}

sg_status launch_commit(Volume* v, int c, int t, hipStream_t s) {
  const int64_t first = ((int64_t)t * v->d.channels + c) * v->nodes;
  uint32_t* r = v->range + 2 * first;
  Levels lv{};
  for (int L = 0; L < v->L; ++L) {
    for (int a = 0; a < 3; ++a) {
      lv.n[L][a] = v->ldims[L][a];
      lv.g[L][a] = v->grid[L][a];
    }
    lv.node_off[L] = v->node_off[L];
  }
  const Shares sh = brick_shares(v->nodes, v->Mb);
#define SG_COMMIT(T, MB, PACK)                                                                 \
  do {                                                                                         \
    hipLaunchKernelGGL((apron_kernel<T, MB, PACK>), dim3(sh.grid), dim3(256), 0, s, v->pool,   \
                       v->slot_bytes, page_at(v, c, t), v->info, lv, r, sh.n, sh.per, v->logB, \
                       v->S, v->Sx, v->Mb);                                                    \
    hipLaunchKernelGGL((range_kernel<T, MB, PACK>), dim3(sh.grid), dim3(256), 0, s, v->pool,   \
                       v->slot_bytes, page_at(v, c, t), r, v->bmax, v->bmax_stride, sh.n,      \
                       sh.per, v->S, v->Sx, v->Mb);                                            \
  } while (0)
  SG_BRICKS(SG_COMMIT);
#undef SG_COMMIT
#undef SG_BRICKS
  launch_dark(v, (int)v->nodes, page_at(v, c, t), nullptr, v->dark + first, s);
  SG_HIP(hipGetLastError());
  return SG_OK;
}

void launch_dark(Volume* v, int n, const int32_t* slots, const int32_t* entries, uint32_t* dark,
                 hipStream_t s) {
  if (!v->bmax) return;  // slabs are not tested
  const int G = dark_regions(v->Mb), threads = v->Mb <= 9 ? 64 : 512,
            bricks = v->Mb <= 9 ? 4 : 1;
  const dim3 grid((unsigned)((n + bricks - 1) / bricks));
  const size_t lds = (size_t)bricks * G * G * G * 4;
  if (v->bpv == 1)
    hipLaunchKernelGGL(dark_kernel<uint8_t>, grid, dim3(threads * bricks), lds, s, v->bmax, v->bmax_stride,
                       slots, entries, n, threads, v->Mb, dark);
  else
    hipLaunchKernelGGL(dark_kernel<uint16_t>, grid, dim3(threads * bricks), lds, s, v->bmax, v->bmax_stride,
                       slots, entries, n, threads, v->Mb, dark);
}

// The largest voxel value whose table index fma(x, scale, bias) is at most
// `last` (-1: none): the index never falls as the value rises.
static int32_t largest_below(float scale, float bias, float last, int32_t top) {
  if (!std::isfinite(scale) || !std::isfinite(bias) || !(bias <= last)) return -1;
  int32_t lo = 0, hi = top;  // fma(lo) <= last
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) / 2;
    if (std::fmaf((float)mid, scale, bias) <= last) lo = mid; else hi = mid - 1;
  }
  return lo;
}

sg_status launch_empty(Volume* v, hipStream_t s) {
  const int C = v->d.channels, n = v->tf_n;
  // tables: TF [C][n+1][4] floats, then lo[C], hi[C] doubles, then
  // next[C][2][n] (see empty_kernel), then dim[C][2] (see RenderArgs)
  const TfLayout at = tf_layout(C, n);
  std::vector<uint8_t> blob((size_t)at.bytes);
  float* f = reinterpret_cast<float*>(blob.data());
  int32_t* next = reinterpret_cast<int32_t*>(blob.data() + at.next);
  int32_t* dim = reinterpret_cast<int32_t*>(blob.data() + at.dim);
  for (int c = 0; c < C; ++c) {
    const std::vector<float>& h = v->tf_host[c];
    float* o = f + (int64_t)c * (n + 1) * 4;
    std::memcpy(o, h.data(), h.size() * sizeof(float));
    std::memcpy(o + 4 * n, h.data() + 4 * (n - 1), 4 * sizeof(float));
    int32_t* nx = next + (int64_t)c * 2 * n;
    int32_t opaque = n, bright = n;
    bool tame = true;  // differences of entries stay finite
    for (int k = n - 1; k >= 0; --k) {
      if (h[4 * k + 3] != 0.0f) opaque = k;
      if (h[4 * k] != 0.0f || h[4 * k + 1] != 0.0f || h[4 * k + 2] != 0.0f) bright = k;
      nx[k] = opaque;
      nx[n + k] = bright;
      for (int q = 0; q < 4; ++q) tame = tame && std::fabs(h[4 * k + q]) < 1e37f;
    }
    // up to the last entry before the first one with extinction (colour),
    // every interpolated value is exactly zero
    float scale, bias;
    tf_window(v, c, &scale, &bias);
    const int32_t top = v->bpv == 1 ? 255 : 65535;
    dim[2 * c] = tame && opaque > 0 ? largest_below(scale, bias, (float)(opaque - 1), top) : -1;
    dim[2 * c + 1] = tame && bright > 0 ? largest_below(scale, bias, (float)(bright - 1), top) : -1;
  }
  double* lohi = reinterpret_cast<double*>(blob.data() + at.lohi);
  for (int c = 0; c < C; ++c) {
    lohi[c] = v->tf_lo[c];
    lohi[C + c] = v->tf_hi[c];
  }
  sg_status st = stage_to_device(v, blob.data(), (int64_t)blob.size(), v->tf, s);
  if (st != SG_OK) return st;
  const uint8_t* dev = reinterpret_cast<const uint8_t*>(v->tf);
  const double* dlo = reinterpret_cast<const double*>(dev + at.lohi);
  const int32_t* dnext = reinterpret_cast<const int32_t*>(dev + at.next);
  const int32_t* ddim = reinterpret_cast<const int32_t*>(dev + at.dim);
  int64_t total = (int64_t)v->d.timepoints * v->nodes;
  hipLaunchKernelGGL(empty_kernel, dim3(blocks_for(total)), dim3(256), 0, s, v->range, v->dark,
                     dnext, ddim, n, dlo, dlo + C, C, v->nodes, total, v->empty);
  SG_HIP(hipGetLastError());
  return SG_OK;
}

sg_status commit(Volume* v, hipStream_t s) {
  bool any = false;
  for (int t = 0; t < v->d.timepoints; ++t)
    for (int c = 0; c < v->d.channels; ++c) {
      uint8_t& p = v->pending[(int64_t)t * v->d.channels + c];
      if (!p) continue;
      sg_status st = launch_commit(v, c, t, s);
      if (st != SG_OK) return st;
      p = 0;
      any = true;
    }
  if (any) v->empty_dirty = true;
  bool all_tf = true;
  for (int c = 0; c < v->d.channels; ++c) all_tf = all_tf && v->tf_set[c];
  if (all_tf && (v->empty_dirty || v->tf_dirty)) {
    sg_status st = launch_empty(v, s);
    if (st != SG_OK) return st;
    v->empty_dirty = false;
    v->tf_dirty = false;
  }
  return SG_OK;
}

}  // namespace sg
