// bricks.hip -- the import step of an out-of-core volume on the device:
// the resolution pyramid of a linear level array and whole bricks (core plus
// a one-voxel apron) cut out of a level, in the form sg_cache_put stores
// (Sec 4.1: the volume is stored as chunks at several resolutions, made once
// at import; Sec 4.2: chunks move whole between the CPU and GPU caches).
//
// Both calls work on plain device arrays of the volume's voxel type, x
// fastest, indexed [z][y][x]; they need no volume handle and run on the
// current device.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "brick_rows.h"

namespace sg {

namespace {

struct Dims {
  int64_t n[3];
};

// One coarser level: voxel g = (sum of the 2x2x2 children 2g + delta, each
// child index clamped to the finer level, + 4) >> 3 (the pyramid rule of
// the resident volume's builder, on a linear array).
//
// A thread makes two voxels of a row from four voxels of each of four source
// rows, one load a row where the four lie in the level at an address aligned
// to them, else voxel by voxel. A workgroup takes `rows` rows of a piece of
// `piece` pairs (`cols` pieces to a row): 2048 pairs, or fewer so that some
// 2048 workgroups share a small level (whole rows in windows of 2048 pairs
// left 100000x8x8 to 16 of them, 115 us against 14). Bound by reading the
// source once: three levels of 700x512x420 uint16 106 us (122 in whole rows).
template <typename T>
__device__ __forceinline__ void four_voxels(const T* row, int64_t x, int64_t n, bool wide,
                                            uint32_t (&v)[4]) {
  const T* p = row + x;
  if (x + 4 <= n && (reinterpret_cast<uintptr_t>(p) & (4 * sizeof(T) - 1)) == 0) {
    if (sizeof(T) == 1) {
      const uint32_t a = *reinterpret_cast<const uint32_t*>(p);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = (a >> (8 * k)) & 0xFFu;
    } else {
      const uint2 a = *reinterpret_cast<const uint2*>(p);
      v[0] = a.x & 0xFFFFu;
      v[1] = a.x >> 16;
      v[2] = a.y & 0xFFFFu;
      v[3] = a.y >> 16;
    }
  } else {
    v[0] = row[min(x, n - 1)];
    v[1] = row[min(x + 1, n - 1)];
    v[2] = v[3] = 0u;
    if (wide) {  // more than one voxel a row to make (the same in every thread)
      v[2] = row[min(x + 2, n - 1)];
      v[3] = row[min(x + 3, n - 1)];
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void pyramid_level_kernel(const T* __restrict__ src, Dims s,
                                                            T* __restrict__ dst, Dims d, int rows,
                                                            int piece, int cols) {
  const int64_t r0 = (int64_t)(blockIdx.x / (unsigned)cols) * rows, all = d.n[1] * d.n[2];
  const int c0 = (int)(blockIdx.x % (unsigned)cols) * piece, half = (int)((d.n[0] + 1) / 2);
  const int here = (int)min((int64_t)rows, all - r0), n1 = (int)d.n[1];
  const bool wide = d.n[0] > 1;
  const int64_t z0 = r0 / n1;  // of the window's first row
  const int y0 = (int)(r0 - z0 * n1);
  const float inv_p = __builtin_amdgcn_rcpf((float)piece), inv_y = __builtin_amdgcn_rcpf((float)n1);
  for (int i = threadIdx.x; i < here * piece; i += 256) {
    const int dr = quot_exact(i, inv_p), pair = c0 + i - dr * piece;
    if (pair >= half) continue;
    const int dz = quot_exact(y0 + dr, inv_y);
    const int64_t row = r0 + dr, x = 2 * (int64_t)pair, z = z0 + dz, y = y0 + dr - dz * n1;
    const int64_t y1 = min(2 * y + 1, s.n[1] - 1), z1 = min(2 * z + 1, s.n[2] - 1);
    const T *a = src + (2 * z * s.n[1] + 2 * y) * s.n[0], *b = src + (2 * z * s.n[1] + y1) * s.n[0],
            *c = src + (z1 * s.n[1] + 2 * y) * s.n[0], *e = src + (z1 * s.n[1] + y1) * s.n[0];
    const bool both = x + 1 < d.n[0];
    uint32_t va[4], vb[4], vc[4], ve[4];
    four_voxels(a, 2 * x, s.n[0], wide, va);
    four_voxels(b, 2 * x, s.n[0], wide, vb);
    four_voxels(c, 2 * x, s.n[0], wide, vc);
    four_voxels(e, 2 * x, s.n[0], wide, ve);
    uint32_t o[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
      o[k] = (va[2 * k] + va[2 * k + 1] + vb[2 * k] + vb[2 * k + 1] + vc[2 * k] + vc[2 * k + 1] +
              ve[2 * k] + ve[2 * k + 1] + 4u) >> 3;
    T* q = dst + row * d.n[0] + x;
    if (sizeof(T) == 2 && both && (reinterpret_cast<uintptr_t>(q) & 3) == 0) {
      *reinterpret_cast<uint32_t*>(q) = o[0] | (o[1] << 16);
    } else {
      q[0] = (T)o[0];
      if (both) q[1] = (T)o[1];
    }
  }
}

// Brick regions: region j holds level voxels B b_j - 1 .. B b_j + B per
// axis, indices clamped to the level, as an S^3 block (S = B + 2), x
// fastest. The brick coordinates of a launch travel in its arguments (three
// 21-bit fields each): no copy and no wait.
//
// A brick's S x S rows are shared by `per` workgroups in windows; a thread
// makes four voxels of a row (the last of a row may be two: S is even) with
// one load and one store, at whatever address the row starts (the compiler
// picks the instructions from the types' alignment), kQuads of them in
// flight; at the level's ends in x it reads voxel by voxel. SMALL: the S
// planes a brick spans hold fewer than 2^31 voxels and S n_y < 2^24, so a
// row's offset from the brick's first plane is 32-bit arithmetic with 24-bit
// products (beside one scalar base); otherwise 64-bit.
//
// Bound by memory. A row of 66 uint16 voxels is 132 bytes at an odd voxel,
// so it pulls two or three 128-byte lines, which its neighbours in x need
// too, so neighbouring bricks go to one XCD and its L2. 812 bricks of 64^3
// uint16 (five launches): 239 us (740 with one thread and two 64-bit
// divisions per voxel, plus a copy of the coordinates and a wait per call);
// two voxels or eight to a thread ran at 272 and 410 us (a row of 66 leaves
// an eight mostly outside).
constexpr int kLaunchBricks = 448;  // 3.5 KiB of arguments
struct BrickList {
  uint64_t b[kLaunchBricks];
};
constexpr int kQuads = 4;

uint64_t pack_brick(const int32_t* c) {
  return (uint64_t)c[0] | ((uint64_t)c[1] << 21) | ((uint64_t)c[2] << 42);
}
// Stored voxel (0, 0, 0) of a packed brick (coordinates below 2^20, see
// check_dims).
__device__ __forceinline__ void brick_origin(uint64_t packed, int B, int& g0, int& g1, int& g2) {
  g0 = B * (int)(packed & 0x1FFFFF) - 1;
  g1 = B * (int)((packed >> 21) & 0x1FFFFF) - 1;
  g2 = B * (int)(packed >> 42) - 1;
}
// Four voxels of a level's row of n0 from voxel gx on, indices clamped.
template <typename T>
__device__ __forceinline__ void read_quad(const T* row, int gx, int n0, uint32_t (&v)[4]) {
  // (any alignment: the compiler picks the load from it)
  typedef T Quad __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  if (gx >= 0 && gx + 4 <= n0) {
    const Quad q = *reinterpret_cast<const Quad*>(row + gx);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = q[k];
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = row[min(max(gx + k, 0), n0 - 1)];
  }
}
// ... stored, the first two of them at the end of a row of 4 q + 2.
template <typename T>
__device__ __forceinline__ void store_quad(T* o, const uint32_t (&v)[4], bool two) {
  typedef T Quad __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  if (!two) {
    Quad q;
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = (T)v[k];
    *reinterpret_cast<Quad*>(o) = q;
  } else {
    o[0] = (T)v[0];
    o[1] = (T)v[1];
  }
}

template <typename T, bool SMALL>
__global__ __launch_bounds__(256) void region_kernel(const T* __restrict__ level, Dims d,
                                                     BrickList list, int n, int B, int per,
                                                     T* __restrict__ out) {
  // workgroup w runs on XCD w % 8: the same rows of eight consecutive bricks
  // (neighbours in x, as a rule) are taken by one XCD in turn
  const int turn = (int)(blockIdx.x >> 3), unit = (turn >> 3) * 8 + (int)(blockIdx.x & 7);
  const int j = (unit / per) * 8 + (turn & 7), part = unit % per;
  if (j >= n) return;
  const int S = B + 2, quads = (S + 3) / 4, rows = S * S;
  int g0, g1, g2;
  brick_origin(list.b[j], B, g0, g1, g2);
  const int n0 = (int)d.n[0], n1 = (int)d.n[1], n2 = (int)d.n[2];
  const int zb = max(g2, 0);  // (a brick's core starts inside the level)
  const T* base = level + (int64_t)zb * n1 * n0;
  out += (int64_t)j * rows * S;
  const int chunk = (rows + per - 1) / per, first = part * chunk, last = min(rows, first + chunk);
  // (a window's items and a brick's rows stay below 2^21, see quot_exact)
  const int window = (1 << 20) / quads;
  const float inv_q = __builtin_amdgcn_rcpf((float)quads), inv_s = __builtin_amdgcn_rcpf((float)S);
  for (int r0 = first; r0 < last; r0 += window) {
    const int items = min(window, last - r0) * quads;
    for (int i0 = threadIdx.x; i0 < items; i0 += 256 * kQuads) {
      uint32_t v[kQuads][4];
      int at[kQuads];
      bool two[kQuads];
#pragma unroll
      for (int u = 0; u < kQuads; ++u) {
        const int i = min(i0 + 256 * u, items - 1);
        const int dr = quot_exact(i, inv_q), r = r0 + dr, x = 4 * (i - dr * quads);
        const int z = quot_exact(r, inv_s), y = r - z * S;
        const int gy = min(max(g1 + y, 0), n1 - 1), gz = min(max(g2 + z, 0), n2 - 1) - zb;
        at[u] = r * S + x;
        two[u] = x + 2 >= S;
        const T* row;
        if (SMALL)
          row = base + __umul24(__umul24(gz, n1) + gy, n0);
        else
          row = base + ((int64_t)gz * n1 + gy) * n0;
        read_quad(row, g0 + x, n0, v[u]);
      }
#pragma unroll
      for (int u = 0; u < kQuads; ++u) {
        if (i0 + 256 * u >= items) break;
        store_quad(out + at[u], v[u], two[u]);
      }
    }
  }
}

// Many small bricks (of 2, 4 and 8): `group` consecutive ones to a workgroup,
// about a thousand quads, their coordinates in device memory. A launch of 448
// costs the host more than the device (512^3 uint16 in bricks of 8: 3461 us in
// 586 launches, 1627 in one; 2026 with one thread per voxel), and a
// brick of 2 has 16 quads for a workgroup's 256 threads. Eight workgroups in a
// row run on one XCD, whose L2 holds the lines that neighbours in x share.
// SMALL: the level's rows and voxels are counted in 24 and 31 bits.
template <typename T, bool SMALL>
__global__ __launch_bounds__(256) void region_group_kernel(const T* __restrict__ level, Dims d,
                                                           const uint64_t* __restrict__ list,
                                                           int n, int B, int group,
                                                           T* __restrict__ out) {
  const int w = (int)blockIdx.x, g = (w & ~63) | ((w & 7) << 3) | ((w >> 3) & 7);
  const int64_t j0 = (int64_t)g * group;
  if (j0 >= n) return;
  const int here = (int)min((int64_t)group, n - j0);
  const int S = B + 2, quads = (S + 3) / 4, rows = S * S, per = rows * quads, items = here * per;
  const int n0 = (int)d.n[0], n1 = (int)d.n[1], n2 = (int)d.n[2];
  const float inv_p = __builtin_amdgcn_rcpf((float)per), inv_q = __builtin_amdgcn_rcpf((float)quads),
              inv_s = __builtin_amdgcn_rcpf((float)S);
  out += j0 * rows * S;
  for (int i0 = threadIdx.x; i0 < items; i0 += 256 * kQuads) {
    uint32_t v[kQuads][4];
    int at[kQuads];
    bool two[kQuads];
#pragma unroll
    for (int u = 0; u < kQuads; ++u) {
      const int i = min(i0 + 256 * u, items - 1);
      const int b = quot_exact(i, inv_p), k = i - b * per, r = quot_exact(k, inv_q),
                x = 4 * (k - r * quads), z = quot_exact(r, inv_s), y = r - z * S;
      int g0, g1, g2;
      brick_origin(list[j0 + b], B, g0, g1, g2);
      const int gy = min(max(g1 + y, 0), n1 - 1), gz = min(max(g2 + z, 0), n2 - 1);
      at[u] = (b * rows + r) * S + x;
      two[u] = x + 2 >= S;
      const T* row = SMALL ? level + __umul24(__umul24(gz, n1) + gy, n0)
                           : level + ((int64_t)gz * n1 + gy) * n0;
      read_quad(row, g0 + x, n0, v[u]);
    }
#pragma unroll
    for (int u = 0; u < kQuads; ++u) {
      if (i0 + 256 * u >= items) break;
      store_quad(out + at[u], v[u], two[u]);
    }
  }
}

// Select the caller's current device explicitly for this thread, as every
// other entry point does for its volume's device, before any launch.
sg_status current_device(int* dev) {
  SG_HIP(hipGetDevice(dev));
  SG_HIP(hipSetDevice(*dev));
  return SG_OK;
}

sg_status check_dims(const int32_t* dims, const char* where) {
  if (!dims) return fail(SG_ERR_INVALID_ARG, std::string(where) + ": NULL dims");
  for (int a = 0; a < 3; ++a)
    if (dims[a] < 1 || dims[a] > (1 << 20))
      return fail(SG_ERR_INVALID_ARG, std::string(where) + ": dims must be in [1, 2^20]");
  return SG_OK;
}

// One launch of region_group_kernel over all n bricks.
sg_status group_regions(int32_t dtype, Dims d, const void* level, int32_t brick, int32_t n,
                        const int32_t* coords, void* out, hipStream_t s) {
  std::vector<uint64_t> packed((size_t)n);
  for (int32_t i = 0; i < n; ++i) packed[(size_t)i] = pack_brick(coords + 3 * (int64_t)i);
  uint64_t* list = nullptr;
  SG_HIP(hipMallocAsync((void**)&list, packed.size() * 8, s));
  hipError_t e = hipMemcpyAsync(list, packed.data(), packed.size() * 8, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);  // the copy has read `packed`
  if (e == hipSuccess) {
    const bool small = d.n[1] * d.n[2] < (1 << 24) && d.n[0] < (1 << 24) &&
                       d.n[0] * d.n[1] * d.n[2] < ((int64_t)1 << 31);
    const void* k = dtype == SG_U8
                        ? (small ? reinterpret_cast<const void*>(region_group_kernel<uint8_t, true>)
                                 : reinterpret_cast<const void*>(region_group_kernel<uint8_t, false>))
                        : (small ? reinterpret_cast<const void*>(region_group_kernel<uint16_t, true>)
                                 : reinterpret_cast<const void*>(region_group_kernel<uint16_t, false>));
    const int S = brick + 2;
    int group = 1024 / (S * S * ((S + 3) / 4)) + 1, nb = n;
    const int64_t groups = ((int64_t)n + group - 1) / group;
    void* pa[] = {&level, &d, &list, &nb, &brick, &group, &out};
    e = hipLaunchKernel(k, dim3((unsigned)((groups + 63) / 64 * 64)), dim3(256), pa, 0, s);
  }
  const hipError_t f = hipFreeAsync(list, s);
  SG_HIP(e);
  SG_HIP(f);
  return SG_OK;
}

}  // namespace

}  // namespace sg

using namespace sg;

extern "C" sg_status sg_pyramid_level(int32_t dtype, const int32_t src_dims[3], const void* src,
                                      void* dst, void* hip_stream) {
  sg_status st = check_dims(src_dims, "sg_pyramid_level");
  if (st != SG_OK) return st;
  if (dtype != SG_U8 && dtype != SG_U16)
    return fail(SG_ERR_INVALID_ARG, "sg_pyramid_level: dtype must be SG_U8 or SG_U16");
  if (!src || !dst) return fail(SG_ERR_INVALID_ARG, "sg_pyramid_level: NULL src or dst");
  Dims s, d;
  for (int a = 0; a < 3; ++a) {
    s.n[a] = src_dims[a];
    d.n[a] = (src_dims[a] + 1) / 2;
  }
  const int64_t total = d.n[0] * d.n[1] * d.n[2];
  const int64_t bpv = dtype == SG_U8 ? 1 : 2;
  const uint8_t* sb = static_cast<const uint8_t*>(src);
  const uint8_t* db = static_cast<const uint8_t*>(dst);
  if (db < sb + s.n[0] * s.n[1] * s.n[2] * bpv && sb < db + total * bpv)
    return fail(SG_ERR_INVALID_ARG, "sg_pyramid_level: dst overlaps src");
  int dev = 0;
  if ((st = current_device(&dev)) != SG_OK) return st;
  // the launch's own status (not the thread's last-error state, which may
  // hold an earlier call's error)
  const void* sp = src;
  void* dp = dst;
  const int64_t half = (d.n[0] + 1) / 2, pairs = half * d.n[1] * d.n[2];
  const int64_t window = std::min<int64_t>(2048, std::max<int64_t>(256, pairs / 2048));
  int cols = (int)((half + window - 1) / window), piece = (int)((half + cols - 1) / cols);
  int rows = (int)std::max<int64_t>(1, window / piece);
  void* pa[] = {&sp, &s, &dp, &d, &rows, &piece, &cols};
  const int64_t groups = (d.n[1] * d.n[2] + rows - 1) / rows * cols;
  const void* k = dtype == SG_U8 ? reinterpret_cast<const void*>(pyramid_level_kernel<uint8_t>)
                                 : reinterpret_cast<const void*>(pyramid_level_kernel<uint16_t>);
  SG_HIP(hipLaunchKernel(k, dim3((unsigned)groups), dim3(256), pa, 0, (hipStream_t)hip_stream));
  return SG_OK;
}

extern "C" sg_status sg_brick_regions(int32_t dtype, const int32_t dims[3], const void* level,
                                      int32_t brick, int32_t n, const int32_t* coords, void* out,
                                      void* hip_stream) {
  sg_status st = check_dims(dims, "sg_brick_regions");
  if (st != SG_OK) return st;
  if (dtype != SG_U8 && dtype != SG_U16)
    return fail(SG_ERR_INVALID_ARG, "sg_brick_regions: dtype must be SG_U8 or SG_U16");
  if (brick < 2 || brick > 256 || (brick & (brick - 1)) != 0)
    return fail(SG_ERR_INVALID_ARG, "sg_brick_regions: brick must be a power of two in [2, 256]");
  if (n < 0) return fail(SG_ERR_INVALID_ARG, "sg_brick_regions: n must be >= 0");
  if (n == 0) return SG_OK;
  if (!level || !coords || !out)
    return fail(SG_ERR_INVALID_ARG, "sg_brick_regions: NULL level, coords or out");
  for (int32_t i = 0; i < n; ++i)
    for (int a = 0; a < 3; ++a) {
      const int32_t g = (dims[a] + brick - 1) / brick;
      if (coords[3 * i + a] < 0 || coords[3 * i + a] >= g)
        return fail(SG_ERR_INVALID_ARG, "sg_brick_regions: brick coordinate outside the grid");
    }
  Dims d;
  for (int a = 0; a < 3; ++a) d.n[a] = dims[a];
  const int64_t S = brick + 2;
  int dev = 0;
  if ((st = current_device(&dev)) != SG_OK) return st;
  const int64_t bpv = dtype == SG_U8 ? 1 : 2;
  const void* lvl = level;
  const bool small = S * d.n[1] < (1 << 24) && S * d.n[0] * d.n[1] < ((int64_t)1 << 31) &&
                     d.n[0] < (1 << 24);
  const void* k =
      dtype == SG_U8 ? (small ? reinterpret_cast<const void*>(region_kernel<uint8_t, true>)
                              : reinterpret_cast<const void*>(region_kernel<uint8_t, false>))
                     : (small ? reinterpret_cast<const void*>(region_kernel<uint16_t, true>)
                              : reinterpret_cast<const void*>(region_kernel<uint16_t, false>));
  // From seven launches on, small bricks go in one, with a copy of their
  // coordinates and a wait for it (about 50 us; a launch 11 us), unless the
  // stream is being captured.
  if (brick <= 8 && n > 7 * kLaunchBricks) {
    hipStream_t s = (hipStream_t)hip_stream;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
    if (cap == hipStreamCaptureStatusNone) return group_regions(dtype, d, level, brick, n, coords, out, s);
  }
  BrickList list;
  for (int32_t i0 = 0; i0 < n; i0 += kLaunchBricks) {
    const int m = std::min<int32_t>(kLaunchBricks, n - i0);
    for (int i = 0; i < m; ++i) list.b[i] = pack_brick(coords + 3 * (int64_t)(i0 + i));
    int per = groups_per_brick(m, (int)(S * S * ((S + 3) / 4) * kRowBatch / kQuads));
    int nb = m;
    const int64_t units = (int64_t)((m + 7) / 8) * per;  // dealt to the XCDs in turn
    void* o = static_cast<uint8_t*>(out) + (int64_t)i0 * S * S * S * bpv;
    void* pa[] = {&lvl, &d, &list, &nb, &brick, &per, &o};
    SG_HIP(hipLaunchKernel(k, dim3((unsigned)((units + 7) / 8 * 64)), dim3(256), pa, 0,
                           (hipStream_t)hip_stream));
  }
  return SG_OK;
}
