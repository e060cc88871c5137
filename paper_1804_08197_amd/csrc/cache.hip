// cache.hip -- out-of-core brick cache (Sec 4.2: a GPU cache of chunks that
// keeps as many as it can and drops the least recently used; Sec 5.2: blocks
// missing from the cache are requested and their parent rendered instead;
// Sec 5.4: time series streamed through the cache).
//
// The pool holds cache_slots bricks. The host mirrors the page table
// ((t, c, node) -> slot or -1) and the slot owners. Renders stamp the slots
// of the nodes they use with a frame number (cut-map kernel) and append
// missing children to a request list. A put that finds no free slot reads
// the stamps back and evicts the oldest slots through a min-heap, never a
// top-level node's (the traversal starts there). Bricks arrive whole (core
// and apron), so no neighbour is needed to store one.
#include <algorithm>
#include <functional>
#include <queue>
#include <vector>

#include "brick_rows.h"

namespace sg {

namespace {

// Store n regions ((B+2)^3 voxels, x fastest) in their slots, one thread per
// stored row of four voxels (see brick_rows.h), and take the largest value
// of every 4x4x4 block (bmax, or NULL) and each brick's value range in the
// same pass, while the voxels are in registers. Bound by memory. A region's
// rows have an even length: WIDE (uint16 at a 4-byte address) reads a row's
// two words; otherwise the source is read voxel by voxel. Up to 144 bricks
// of 64^3 uint16 per put: 28 us on average (61 + 344 us when storing and
// taking the ranges were two kernels, with 64-bit divisions per voxel and
// one workgroup per brick).
template <typename T, bool MB, bool WIDE, bool PACK>
__global__ __launch_bounds__(256) void put_kernel(uint8_t* __restrict__ pool, int64_t slot_bytes,
                                                  const int32_t* slots, const int32_t* entries,
                                                  const T* __restrict__ src, uint32_t* range,
                                                  uint8_t* bmax, int64_t bmax_stride, int n,
                                                  int per, int S, int Sx, int M) {
  constexpr int kBatch = PACK ? 1 : kRowBatch;
  const int items = M * M * M * 16;
  const Part p = brick_part<PACK>(per, M);
  const bool any = !PACK || p.j < n;
  const int64_t j = any ? p.j : 0;
  const float inv_m = __builtin_amdgcn_rcpf((float)M), inv_mm = __builtin_amdgcn_rcpf((float)(M * M));
  const int32_t slot = slots[j];
  T* dst = reinterpret_cast<T*>(pool + (int64_t)slot * slot_bytes);
  T* bm = bmax ? reinterpret_cast<T*>(bmax + (int64_t)slot * bmax_stride) : nullptr;
  src += j * (int64_t)S * S * S;
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
      if (!on[u]) continue;
      const T* from = src + ((int64_t)w[u].z * S + w[u].y) * S + w[u].x;
      if (WIDE) {
        const uint32_t* q = reinterpret_cast<const uint32_t*>(from);
        if (w[u].x < S) o[u].w[0] = q[0];
        if (w[u].x + 2 < S) o[u].w[sizeof(T) - 1] = q[1];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (w[u].x + k < S) o[u].set(k, from[k]);
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + 256 * u + p.lane;
      uint32_t rmax = 0u;
      if (on[u]) {
        row_range(o[u], S - w[u].x, lo, rmax);
        store_row<T, MB>(dst, w[u], i, S, Sx, o[u]);
      }
      hi = max(hi, rmax);
      if (PACK) continue;  // (no block maxima)
      rmax = row16_max(rmax);
      if (bm && i < items && (i & 15) == 0) bm[i >> 4] = (T)rmax;
    }
  }
  range_out<PACK>(lo, hi, any ? range + 2 * (int64_t)entries[j] : nullptr, per == 1, p);
}

// The small tables of a put: a freshly stored brick counts as used now
// (stamp), its range starts empty, and the page table takes its new entries.
__global__ void put_tables_kernel(uint32_t* stamp, const int32_t* slots, const int32_t* entries,
                                  int n, uint32_t frame, uint32_t* range, int32_t* page,
                                  const int32_t* idx, const int32_t* val, int np) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    stamp[slots[i]] = frame;
    const int64_t e = entries[i];
    range[2 * e] = 0xFFFFFFFFu;
    range[2 * e + 1] = 0u;
  }
  if (i < np) page[idx[i]] = val[i];
}

// Clear the flag bits of the listed entries (the list holds every set bit
// unless it overflowed).
__global__ void clear_requests_kernel(uint32_t* flags, const uint32_t* list,
                                      const uint32_t* count, int cap) {
  const uint32_t n = min(*count, (uint32_t)cap);
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t e = list[i];
    atomicAnd(flags + (e >> 5), ~(1u << (e & 31)));
  }
}

__global__ void clear_all_kernel(uint32_t* flags, int64_t words) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < words;
       i += (int64_t)gridDim.x * blockDim.x)
    flags[i] = 0u;
}

__global__ void zero_count_kernel(uint32_t* count) {
  if (threadIdx.x == 0) *count = 0u;
}

int64_t entry_of(const Volume* v, int t, int c, int64_t node) {
  return ((int64_t)t * v->d.channels + c) * v->nodes + node;
}

bool is_top(const Volume* v, int64_t entry) {
  const int64_t node = entry % v->nodes;
  return node >= v->node_off[v->L - 1];
}

}  // namespace

bool top_level_resident(const Volume* v, int t) {
  if (!v->cache) return true;
  for (int c = 0; c < v->d.channels; ++c)
    for (int64_t n = v->node_off[v->L - 1]; n < v->nodes; ++n)
      if (v->page_host[(size_t)entry_of(v, t, c, n)] < 0) return false;
  return true;
}

}  // namespace sg

using namespace sg;

namespace {

// Room for n entries of a call's tables.
sg_status put_meta_room(Volume* v, int64_t n) {
  if (n <= v->put_meta_cap) return SG_OK;
  if (v->put_meta) SG_HIP(hipFree(v->put_meta));  // (waits for what uses it)
  if (v->put_meta_host) SG_HIP(hipHostFree(v->put_meta_host));
  v->put_meta = v->put_meta_host = nullptr;
  v->put_meta_cap = 0;
  const int64_t cap = std::max<int64_t>(2 * n, 16384);
  if (hipMalloc((void**)&v->put_meta, (size_t)cap * 4) != hipSuccess ||
      hipHostMalloc((void**)&v->put_meta_host, (size_t)cap * 4, hipHostMallocDefault) !=
          hipSuccess) {
    (void)hipGetLastError();
    return fail(SG_ERR_OUT_OF_MEMORY, "sg_cache_put: allocation of the put's tables failed");
  }
  v->put_meta_cap = cap;
  return SG_OK;
}

// Room for the regions of up to n bricks (*batch: how many fit at a time),
// fewer where memory is short. Kept from put to put: a buffer taken from the
// stream's pool for each put went back to the system at the next
// synchronisation, and mapping up to 83 MB anew took 0.3 ms of a put.
sg_status put_stage_room(Volume* v, int64_t region, int64_t n, int64_t* batch) {
  int64_t want = std::min(n, std::max<int64_t>(1, kPutStage / region));
  if (want * region > v->put_stage_cap) {
    if (v->put_stage) SG_HIP(hipFree(v->put_stage));  // (waits for what uses it)
    v->put_stage = nullptr;
    v->put_stage_cap = 0;
    while (hipMalloc((void**)&v->put_stage, (size_t)(want * region)) != hipSuccess) {
      (void)hipGetLastError();
      v->put_stage = nullptr;
      if (want == 1)
        return fail(SG_ERR_OUT_OF_MEMORY, "sg_cache_put: allocation of the staging buffer failed");
      want /= 2;
    }
    v->put_stage_cap = want * region;
  }
  *batch = std::min(n, v->put_stage_cap / region);
  return SG_OK;
}

// Copy k regions from b0 on to the staging buffer.
sg_status send_regions(Volume* v, int64_t region, int64_t b0, int64_t k, const void* src,
                       const void* const* srcs, hipStream_t s) {
  if (!srcs) {
    SG_HIP(hipMemcpyAsync(v->put_stage, (const uint8_t*)src + region * b0, (size_t)(region * k),
                          hipMemcpyHostToDevice, s));
    return SG_OK;
  }
  // one copy per run of regions that lie back to back in the source
  for (int64_t i = 0; i < k;) {
    int64_t j = i + 1;
    while (j < k && (const uint8_t*)srcs[b0 + j] == (const uint8_t*)srcs[b0 + j - 1] + region) ++j;
    SG_HIP(hipMemcpyAsync(v->put_stage + region * i, srcs[b0 + i], (size_t)(region * (j - i)),
                          hipMemcpyDefault, s));
    i = j;
  }
  return SG_OK;
}

// Store the regions at dsrc in their slots.
void launch_put(Volume* v, int n, const int32_t* d_slot, const int32_t* d_ent, const void* dsrc,
                hipStream_t s) {
  const Shares sh = brick_shares(n, v->Mb);
  const bool wide = v->bpv == 2 && reinterpret_cast<uintptr_t>(dsrc) % 4 == 0;
#define SG_PUT(T, MB, WIDE, PACK)                                                              \
  hipLaunchKernelGGL((put_kernel<T, MB, WIDE, PACK>), dim3(sh.grid), dim3(256), 0, s, v->pool, \
                     v->slot_bytes, d_slot, d_ent, (const T*)dsrc, v->range, v->bmax,          \
                     v->bmax_stride, sh.n, sh.per, v->S, v->Sx, v->Mb)
#define SG_PUT_W(T, WIDE)                                                                      \
  do {                                                                                         \
    if (v->M) { if (sh.pack) SG_PUT(T, true, WIDE, true); else SG_PUT(T, true, WIDE, false); } \
    else { if (sh.pack) SG_PUT(T, false, WIDE, true); else SG_PUT(T, false, WIDE, false); }    \
  } while (0)
  if (v->bpv == 1) SG_PUT_W(uint8_t, false);
  else if (wide) SG_PUT_W(uint16_t, true);
  else SG_PUT_W(uint16_t, false);
#undef SG_PUT_W
#undef SG_PUT
  launch_dark(v, n, d_slot, d_ent, v->dark, s);
}

// Both put entry points: the regions come from one buffer (src, host or
// device) or from one pointer per brick (srcs, any memory; each copied by
// its own DMA into the staging buffer).
sg_status put_impl(sg_volume* vol, int32_t channel, int32_t timepoint, int32_t level, int32_t n,
                   const int32_t* coords, const void* src, const void* const* srcs,
                   int32_t src_on_device, void* hip_stream) {
  if (!vol) return fail(SG_ERR_INVALID_ARG, "sg_cache_put: NULL volume");
  Volume* v = &vol->v;
  if (!v->cache) return fail(SG_ERR_UNSUPPORTED, "sg_cache_put: not a cache volume");
  if (channel < 0 || channel >= v->d.channels || timepoint < 0 ||
      timepoint >= v->d.timepoints || level < 0 || level >= v->L || n < 0)
    return fail(SG_ERR_INVALID_ARG, "sg_cache_put: channel/timepoint/level/n out of range");
  if (n == 0) return SG_OK;
  if (!coords || (!src && !srcs))
    return fail(SG_ERR_INVALID_ARG, "sg_cache_put: NULL coords or source");
  if (srcs)
    for (int32_t i = 0; i < n; ++i)
      if (!srcs[i]) return fail(SG_ERR_INVALID_ARG, "sg_cache_put_scattered: NULL region pointer");
  std::vector<int64_t> ent((size_t)n);
  for (int32_t i = 0; i < n; ++i) {
    for (int a = 0; a < 3; ++a)
      if (coords[3 * i + a] < 0 || coords[3 * i + a] >= v->grid[level][a])
        return fail(SG_ERR_INVALID_ARG, "sg_cache_put: brick coordinate outside the grid");
    const int64_t node = v->node_off[level] +
                         ((int64_t)coords[3 * i + 2] * v->grid[level][1] + coords[3 * i + 1]) *
                             v->grid[level][0] +
                         coords[3 * i];
    ent[(size_t)i] = entry_of(v, timepoint, channel, node);
  }
  {
    std::vector<int64_t> sorted = ent;
    std::sort(sorted.begin(), sorted.end());
    if (std::adjacent_find(sorted.begin(), sorted.end()) != sorted.end())
      return fail(SG_ERR_INVALID_ARG, "sg_cache_put: a brick appears twice");
  }
  DeviceGuard guard(v->d.device);
  if (!guard.ok) return fail(SG_ERR_DEVICE, "cannot select device");
  hipStream_t s = (hipStream_t)hip_stream;

  // a put waits for its copies and so cannot be recorded
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
  if (cap != hipStreamCaptureStatusNone)
    return fail(SG_ERR_DEVICE, "sg_cache_put: the stream is being captured");

  // room for what travels, before the tables change
  const int64_t region = (int64_t)v->S * v->S * v->S * v->bpv;
  const bool staged = srcs || !src_on_device;
  int64_t batch = n;  // bricks on their way at a time
  int need = 0;
  for (int64_t e : ent)
    if (v->page_host[(size_t)e] < 0) ++need;
  const bool evict = need > (int)v->free_slots.size();
  sg_status st = put_meta_room(v, std::max<int64_t>(6 * (int64_t)n, evict ? v->slots : 0));
  if (st != SG_OK) return st;
  if (staged && (st = put_stage_room(v, region, n, &batch)) != SG_OK) return st;
  // The stamps come back before the regions leave, and the regions leave
  // before the host chooses slots by the stamps. A put on another stream than
  // the last one finds that one's scratch free. (Two timepoints of 384x384x256
  // with two channels through a cache of one, 380 MB in 12 puts and 6 frames:
  // 13.4 -> 10.8 ms, of which the bus needs 6.7 and the kernels 3.0.)
  if (v->put_pending) SG_HIP(hipStreamWaitEvent(s, v->put_done, 0));
  v->put_pending = true;
  if (evict) {
    SG_HIP(hipMemcpyAsync(v->put_meta_host, v->stamp, (size_t)v->slots * 4, hipMemcpyDeviceToHost, s));
    SG_HIP(hipEventRecord(v->put_copied, s));
  }
  if (staged && (st = send_regions(v, region, 0, std::min<int64_t>(batch, n), src, srcs, s)) != SG_OK)
    return st;

  // slots: the brick's own if resident, else a free one, else the oldest
  // evictable one (min-heap over the stamps of the last renders)
  std::vector<int32_t> slot((size_t)n, -1);
  std::vector<int32_t> pidx, pval;  // page updates
  if (evict) {
    SG_HIP(hipEventSynchronize(v->put_copied));
    const uint32_t* stamp = reinterpret_cast<const uint32_t*>(v->put_meta_host);
    std::vector<char> keep((size_t)v->entries, 0);
    for (int64_t e : ent) keep[(size_t)e] = 1;
    typedef std::pair<uint32_t, int32_t> Item;  // (stamp, slot): oldest first
    std::priority_queue<Item, std::vector<Item>, std::greater<Item>> heap;
    for (int64_t sl = 0; sl < v->slots; ++sl) {
      const int64_t e = v->owner[(size_t)sl];
      if (e < 0 || keep[(size_t)e] || is_top(v, e)) continue;
      heap.push(Item(stamp[(size_t)sl], (int32_t)sl));
    }
    if ((int64_t)heap.size() + (int64_t)v->free_slots.size() < need) {
      SG_HIP(hipStreamSynchronize(s));  // the regions are on their way
      return fail(SG_ERR_OUT_OF_MEMORY,
                  "sg_cache_put: more bricks than the cache can free (top-level nodes are "
                  "never evicted)");
    }
    while (need > (int)v->free_slots.size()) {
      const int32_t sl = heap.top().second;
      heap.pop();
      const int64_t e = v->owner[(size_t)sl];
      v->page_host[(size_t)e] = -1;
      v->owner[(size_t)sl] = -1;
      pidx.push_back((int32_t)e);
      pval.push_back(-1);
      v->free_slots.push_back(sl);
      ++v->evictions;
    }
  }
  for (int32_t i = 0; i < n; ++i) {
    const int64_t e = ent[(size_t)i];
    int32_t sl = v->page_host[(size_t)e];
    if (sl < 0) {
      sl = v->free_slots.back();
      v->free_slots.pop_back();
      v->page_host[(size_t)e] = sl;
      v->owner[(size_t)sl] = e;
      pidx.push_back((int32_t)e);
      pval.push_back(sl);
    }
    slot[(size_t)i] = sl;
  }
  v->uploads += n;

  // device side: regions, page updates, ranges; only the copies are waited for
  const int np = (int)pidx.size();
  int32_t* const m = v->put_meta_host;
  std::copy(slot.begin(), slot.end(), m);
  for (int32_t i = 0; i < n; ++i) m[n + i] = (int32_t)ent[(size_t)i];
  std::copy(pidx.begin(), pidx.end(), m + 2 * n);
  std::copy(pval.begin(), pval.end(), m + 2 * n + np);
  const int32_t* d_slot = v->put_meta;
  const int32_t* d_ent = d_slot + n;
  const int32_t* d_pidx = d_ent + n;
  const int32_t* d_pval = d_pidx + np;
  for (int64_t b0 = 0; b0 < n; b0 += batch) {
    const int64_t k = std::min<int64_t>(batch, n - b0);
    const void* dsrc = staged ? v->put_stage : (const uint8_t*)src;
    if (staged && b0 > 0 && (st = send_regions(v, region, b0, k, src, srcs, s)) != SG_OK)
      return st;
    if (b0 == 0)
      SG_HIP(hipMemcpyAsync(v->put_meta, m, ((size_t)n + (size_t)np) * 8, hipMemcpyHostToDevice, s));
    if (b0 + k == n) SG_HIP(hipEventRecord(v->put_copied, s));
    if (b0 == 0)
      hipLaunchKernelGGL(put_tables_kernel, dim3((unsigned)((std::max(n, np) + 255) / 256)),
                         dim3(256), 0, s, v->stamp, d_slot, d_ent, n, v->frame, v->range, v->page,
                         d_pidx, d_pval, np);
    launch_put(v, (int)k, d_slot + b0, d_ent + b0, dsrc, s);
    SG_HIP(hipGetLastError());
  }
  SG_HIP(hipEventRecord(v->put_done, s));
  SG_HIP(hipEventSynchronize(v->put_copied));  // host buffers consumed before returning
  v->empty_dirty = true;
  return SG_OK;
}

}  // namespace

extern "C" sg_status sg_cache_put(sg_volume* vol, int32_t channel, int32_t timepoint,
                                  int32_t level, int32_t n, const int32_t* coords,
                                  const void* src, int32_t src_on_device, void* hip_stream) {
  return put_impl(vol, channel, timepoint, level, n, coords, src, nullptr, src_on_device,
                  hip_stream);
}

extern "C" sg_status sg_cache_put_scattered(sg_volume* vol, int32_t channel, int32_t timepoint,
                                            int32_t level, int32_t n, const int32_t* coords,
                                            const void* const* srcs, void* hip_stream) {
  if (!srcs && n > 0) return fail(SG_ERR_INVALID_ARG, "sg_cache_put_scattered: NULL srcs");
  return put_impl(vol, channel, timepoint, level, n, coords, nullptr, srcs, 0, hip_stream);
}

extern "C" sg_status sg_cache_requests(sg_volume* vol, uint64_t* ids, int32_t* timepoints,
                                       int32_t* n, void* hip_stream) {
  if (!vol || !n || *n < 0 || (*n > 0 && (!ids || !timepoints)))
    return fail(SG_ERR_INVALID_ARG, "sg_cache_requests: NULL argument or negative capacity");
  Volume* v = &vol->v;
  if (!v->cache) return fail(SG_ERR_UNSUPPORTED, "sg_cache_requests: not a cache volume");
  DeviceGuard guard(v->d.device);
  if (!guard.ok) return fail(SG_ERR_DEVICE, "cannot select device");
  hipStream_t s = (hipStream_t)hip_stream;
  // the count and the first of the list together; the rest only if there is more
  sg_status st = put_meta_room(v, 4096);
  if (st != SG_OK) return st;
  const int32_t first = (int32_t)std::min<int64_t>(4096, v->put_meta_cap - kReqHead);
  SG_HIP(hipMemcpyAsync(v->put_meta_host, v->req_count, ((size_t)kReqHead + (size_t)first) * 4,
                        hipMemcpyDeviceToHost, s));
  SG_HIP(hipStreamSynchronize(s));
  const uint32_t count = (uint32_t)v->put_meta_host[0];
  const int32_t m = (int32_t)std::min<uint32_t>(count, (uint32_t)kReqCap);
  if (m > *n) {
    *n = m;
    return fail(SG_ERR_INVALID_ARG, "sg_cache_requests: capacity too small");
  }
  std::vector<uint32_t> list((size_t)m);
  std::copy_n(v->put_meta_host + kReqHead, std::min(m, first), list.begin());
  if (m > first)
    SG_HIP(hipMemcpyAsync(list.data() + first, v->req_list + first, (size_t)(m - first) * 4,
                          hipMemcpyDeviceToHost, s));
  const int64_t words = ((int64_t)v->d.timepoints * v->nodes + 31) / 32;
  if (count > (uint32_t)kReqCap) {
    // the list overflowed: some set bits are not listed, so clear them all
    hipLaunchKernelGGL(clear_all_kernel, dim3((unsigned)std::min<int64_t>((words + 255) / 256,
                                                                          65536)),
                       dim3(256), 0, s, v->req_flags, words);
  } else {
    hipLaunchKernelGGL(clear_requests_kernel, dim3((unsigned)std::max(1, (m + 255) / 256)),
                       dim3(256), 0, s, v->req_flags, v->req_list, v->req_count, kReqCap);
  }
  hipLaunchKernelGGL(zero_count_kernel, dim3(1), dim3(64), 0, s, v->req_count);
  SG_HIP(hipGetLastError());
  SG_HIP(hipStreamSynchronize(s));
  std::vector<std::pair<int32_t, uint64_t>> out;
  for (int32_t i = 0; i < m; ++i) {
    const int64_t e = list[(size_t)i];
    const int32_t t = (int32_t)(e / v->nodes);
    const int64_t node = e - (int64_t)t * v->nodes;
    int L = 0;
    while (L + 1 < v->L && node >= v->node_off[L + 1]) ++L;
    const int64_t r = node - v->node_off[L];
    const int64_t x = r % v->grid[L][0], y = (r / v->grid[L][0]) % v->grid[L][1],
                  z = r / ((int64_t)v->grid[L][0] * v->grid[L][1]);
    out.emplace_back(t, ((uint64_t)L << 60) | ((uint64_t)x << 40) | ((uint64_t)y << 20) |
                            (uint64_t)z);
  }
  std::sort(out.begin(), out.end());
  for (int32_t i = 0; i < m; ++i) {
    timepoints[i] = out[(size_t)i].first;
    ids[i] = out[(size_t)i].second;
  }
  *n = m;
  return SG_OK;
}

extern "C" sg_status sg_cache_get_info(const sg_volume* vol, sg_cache_info* info) {
  if (!vol || !info) return fail(SG_ERR_INVALID_ARG, "sg_cache_get_info: NULL argument");
  const Volume* v = &vol->v;
  info->capacity = v->slots;
  info->resident = v->cache ? v->slots - (int64_t)v->free_slots.size() : v->slots;
  info->uploads = v->uploads;
  info->evictions = v->evictions;
  info->frame = v->frame;
  return SG_OK;
}

extern "C" sg_status sg_cache_resident(const sg_volume* vol, int32_t channel, int32_t timepoint,
                                       int32_t level, const int32_t b[3], int32_t* resident) {
  if (!vol || !b || !resident) return fail(SG_ERR_INVALID_ARG, "sg_cache_resident: NULL argument");
  const Volume* v = &vol->v;
  if (channel < 0 || channel >= v->d.channels || timepoint < 0 ||
      timepoint >= v->d.timepoints || level < 0 || level >= v->L)
    return fail(SG_ERR_INVALID_ARG, "sg_cache_resident: out of range");
  for (int a = 0; a < 3; ++a)
    if (b[a] < 0 || b[a] >= v->grid[level][a])
      return fail(SG_ERR_INVALID_ARG, "sg_cache_resident: brick outside the grid");
  if (!v->cache) {
    *resident = 1;
    return SG_OK;
  }
  const int64_t node =
      v->node_off[level] + ((int64_t)b[2] * v->grid[level][1] + b[1]) * v->grid[level][0] + b[0];
  *resident = v->page_host[(size_t)entry_of(v, timepoint, channel, node)] >= 0 ? 1 : 0;
  return SG_OK;
}
