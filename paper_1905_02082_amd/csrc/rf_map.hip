// Map maintenance kernels: initialisation, import/export (checkpoint), the
// frame block list, and zero-crossing surface extraction.
#include "rf_device.h"
#include "rf_internal.h"

namespace rf {

// What an initialised map's state is marked with: it then describes a pool of
// this size and form.
__host__ __device__ __forceinline__ uint32_t map_mark(const MapDev& m, int storage) {
  return 0x52464D01u ^ m.max_blocks * 0x9E3779B1u ^ (m.bucket_mask + (uint32_t)storage) * 0x85EBCA77u;
}

// Clears a map's arrays: the hash, the marks of the listing, the flood fill's
// tile flags, the counts of the tracking cache's pairs (without them its pairs
// are not read) and the voxels of every pool slot handed out since the last
// time; the others are still zero.  An arena whose state does not carry the
// mark (a new map) is cleared whole.  One launch, all stores 16 bytes wide:
// bound by what it writes.  Clearing the pool and the pairs whole, with a
// launch per array, took 179 us in eight kernels for the temporary model of ten
// 640x480 frames, now 33 in two (of the whole call, with the gaps between the
// launches, 1329 us became 1113).
__global__ __launch_bounds__(256) void clear_map_kernel(MapDev m, uint32_t num_buckets, int storage, int whole) {
  const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, n = (size_t)gridDim.x * blockDim.x;
  const uint4 z = make_uint4(0, 0, 0, 0);
  auto clear = [&](void* p, size_t bytes) {
    uint4* q = reinterpret_cast<uint4*>(p);
    for (size_t i = t0; i < (bytes + 15) / 16; i += n) q[i] = z;
  };
  const size_t used = whole || m.st->mark != map_mark(m, storage) ? m.max_blocks : min(m.st->n_blocks, m.max_blocks);
  clear(m.sdfw, used * 512 * (storage == RF_STORAGE_FP32 ? 8 : 4));
  clear(m.rgb, used * 512 * 4);
  for (size_t i = t0; i < num_buckets; i += n) m.buckets[i] = Bucket{kEmptyKey, kInvalidSlot, 0};
  // no bucket touched; every listing leaves the map so
  clear(touched_map(m), num_buckets);
  // the flood-fill tile flags start at zero, and every mask computation
  // leaves them so
  clear(m.dirty, (size_t)m.dirty_cap * 2 * 4);
  clear(m.tc_count, (size_t)kCacheLevels * m.tc_tiles * 4);
}

__global__ void init_state_kernel(DevState* st, uint32_t mark) {
  if (threadIdx.x == 0) {
    DevState s{};
    s.mark = mark;
    *st = s;
  }
}

// Imported blocks end the allocation epoch, so no tracking cache keeps an
// absent-block entry across an import.
__global__ void advance_epoch_kernel(DevState* st) {
  if (threadIdx.x == 0) advance_epoch(st);
}

void launch_map_init(const MapDev& m, uint32_t num_buckets, int storage, bool whole, hipStream_t s) {
  clear_map_kernel<<<4096, 256, 0, s>>>(m, num_buckets, storage, whole ? 1 : 0);
  init_state_kernel<<<1, 64, 0, s>>>(m.st, map_mark(m, storage));
}

__device__ __forceinline__ uint32_t live_blocks(const MapDev& m) { return min(m.st->n_blocks, m.max_blocks); }

template <int STORAGE>
__global__ __launch_bounds__(256) void export_kernel(MapDev m, int32_t* keys, float* sdf, float* w, uint8_t* rgb,
                                                     uint32_t cap, uint32_t* count) {
  const uint32_t n = live_blocks(m);
  if (blockIdx.x == 0 && threadIdx.x == 0) *count = n;
  for (uint32_t b = blockIdx.x; b < n && b < cap; b += gridDim.x) {
    if (keys && threadIdx.x == 0) {
      int x, y, z;
      unpack_key(m.block_keys[b], x, y, z);
      keys[3 * b] = x;
      keys[3 * b + 1] = y;
      keys[3 * b + 2] = z;
    }
    for (int l = threadIdx.x; l < 512; l += blockDim.x) {
      const uint32_t i = b * 512u + l;
      float s, ww;
      VoxelStore<STORAGE>::load(m, i, s, ww);
      if (sdf) sdf[i] = s;
      if (w) w[i] = ww;
      if (rgb) {
        const uchar4 c = m.rgb[i];
        rgb[3 * (size_t)i] = c.x;
        rgb[3 * (size_t)i + 1] = c.y;
        rgb[3 * (size_t)i + 2] = c.z;
      }
    }
  }
}

template <int STORAGE>
__global__ __launch_bounds__(256) void import_kernel(MapDev m, const int32_t* keys, const float* sdf, const float* w,
                                                     const uint8_t* rgb, uint32_t n) {
  __shared__ int s_slot;
  for (uint32_t b = blockIdx.x; b < n; b += gridDim.x) {
    if (threadIdx.x == 0) {
      const int h = insert_block(m, keys[3 * b], keys[3 * b + 1], keys[3 * b + 2]);
      const uint32_t slot = (h >= 0) ? m.buckets[h].slot : kInvalidSlot;
      s_slot = (slot < m.max_blocks) ? (int)slot : -1;
    }
    __syncthreads();
    const int slot = s_slot;
    if (slot >= 0) {
      for (int l = threadIdx.x; l < 512; l += blockDim.x) {
        const size_t src = (size_t)b * 512 + l;
        const uint32_t dst = (uint32_t)slot * 512u + l;
        VoxelStore<STORAGE>::store(m, dst, sdf[src], w[src]);
        m.rgb[dst] = make_uchar4(rgb[3 * src], rgb[3 * src + 1], rgb[3 * src + 2], 0);
      }
    }
    __syncthreads();
  }
}

__global__ void frame_blocks_kernel(MapDev m, int32_t* keys, uint32_t cap, uint32_t* count) {
  const uint32_t n = min(m.st->f_count, m.flist_cap);
  if (blockIdx.x == 0 && threadIdx.x == 0) *count = n;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n && i < cap; i += gridDim.x * blockDim.x) {
    int x, y, z;
    // compact free-space maps keep the whole-block test's outcome in bits 22-31
    unpack_key(m.buckets[m.flist[i] & (m.free_blocks ? 0x003FFFFFu : 0xFFFFFFFFu)].key, x, y, z);
    keys[3 * i] = x;
    keys[3 * i + 1] = y;
    keys[3 * i + 2] = z;
  }
}

__global__ void zero_u32_kernel(uint32_t* p) {
  if (threadIdx.x == 0) *p = 0;
}

template <int STORAGE>
__global__ __launch_bounds__(256) void surface_kernel(MapDev m, float* pts, uint32_t cap, uint32_t* count) {
  const uint32_t n = live_blocks(m);
  for (uint32_t b = blockIdx.x; b < n; b += gridDim.x) {
    int bx, by, bz;
    unpack_key(m.block_keys[b], bx, by, bz);
    for (int l = threadIdx.x; l < 512; l += blockDim.x) {
      const uint32_t i = b * 512u + l;
      float a, wa;
      VoxelStore<STORAGE>::load(m, i, a, wa);
      if (!(wa > 0.0f) || !(fabsf(a) < m.tau)) continue;
      const int lc[3] = {l & 7, (l >> 3) & 7, l >> 6};
      const int vi[3] = {8 * bx + lc[0], 8 * by + lc[1], 8 * bz + lc[2]};
#pragma unroll
      for (int ax = 0; ax < 3; ++ax) {
        uint32_t j;
        if (lc[ax] < 7) {
          j = i + (ax == 0 ? 1u : (ax == 1 ? 8u : 64u));
        } else {
          const int sl = find_slot(m, bx + (ax == 0), by + (ax == 1), bz + (ax == 2));
          if (sl < 0) continue;
          const int nl = (ax == 0 ? 0 : lc[0]) + 8 * (ax == 1 ? 0 : lc[1]) + 64 * (ax == 2 ? 0 : lc[2]);
          j = (uint32_t)sl * 512u + nl;
        }
        float c, wc;
        VoxelStore<STORAGE>::load(m, j, c, wc);
        if (!(wc > 0.0f) || !(fabsf(c) < m.tau)) continue;
        if ((a > 0.0f) == (c > 0.0f)) continue;
        const float tt = a / (a - c);
        const uint32_t k = atomicAdd(count, 1u);
        if (k < cap) {
          float* o = pts + 7 * (size_t)k;
          o[0] = (float)vi[0] * m.s;
          o[1] = (float)vi[1] * m.s;
          o[2] = (float)vi[2] * m.s;
          o[ax] = (float)vi[ax] * m.s + tt * m.s;
          const uchar4 col = m.rgb[i];
          o[3] = col.x;
          o[4] = col.y;
          o[5] = col.z;
          o[6] = (float)ax;
        }
      }
    }
  }
}

void launch_surface(const MapDev& m, int storage, float* pts, uint32_t cap, uint32_t* count, hipStream_t s) {
  zero_u32_kernel<<<1, 64, 0, s>>>(count);
  if (storage == RF_STORAGE_FP32) surface_kernel<RF_STORAGE_FP32><<<2048, 256, 0, s>>>(m, pts, cap, count);
  else surface_kernel<RF_STORAGE_FP16_U8><<<2048, 256, 0, s>>>(m, pts, cap, count);
}

// Free blocks of a compact free-space map: key and the weight their voxels
// read as, in no particular order (the buckets are scanned).  A workgroup takes
// kFreeScan buckets a thread at a time, all asked for together, and one atomic
// for the room of what it found: an atomic a wavefront and 64 buckets, all on
// one counter, took 54.8 us for 2^20 buckets, this 11.1.
constexpr int kFreeScan = 8;

__global__ __launch_bounds__(256) void export_free_kernel(MapDev m, uint32_t num_buckets, int32_t* keys, float* w,
                                                          uint32_t cap, uint32_t* count) {
  __shared__ uint32_t s_n, s_base;
  const int lane = threadIdx.x & 63;
  for (uint32_t h0 = blockIdx.x * (blockDim.x * kFreeScan); h0 < num_buckets; h0 += gridDim.x * (blockDim.x * kFreeScan)) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    Bucket b[kFreeScan];
    unsigned long long found[kFreeScan];
    uint32_t n = 0;
#pragma unroll
    for (int q = 0; q < kFreeScan; ++q) {
      const uint32_t h = h0 + q * blockDim.x + threadIdx.x;
      b[q] = m.buckets[min(h, num_buckets - 1u)];
    }
#pragma unroll
    for (int q = 0; q < kFreeScan; ++q) {
      const uint32_t h = h0 + q * blockDim.x + threadIdx.x;
      found[q] = __ballot(h < num_buckets && b[q].key != kEmptyKey && is_free_slot(b[q].slot));
      n += (uint32_t)__popcll(found[q]);
    }
    uint32_t at = 0;
    if (lane == 0 && n) at = atomicAdd(&s_n, n);  // LDS
    __syncthreads();
    if (threadIdx.x == 0 && s_n) s_base = atomicAdd(count, s_n);
    __syncthreads();
    at = s_base + (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
    for (int q = 0; q < kFreeScan; ++q) {
      const uint32_t i = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(found[q] >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)found[q], 0u));
      at += (uint32_t)__popcll(found[q]);
      if (!((found[q] >> lane) & 1ull) || i >= cap) continue;
      int x, y, z;
      unpack_key(b[q].key, x, y, z);
      keys[3 * (size_t)i] = x;
      keys[3 * (size_t)i + 1] = y;
      keys[3 * (size_t)i + 2] = z;
      if (w) w[i] = (float)(b[q].slot & 0xFFu);
    }
    __syncthreads();  // s_n and s_base are used again
  }
}

void launch_export_free(const MapDev& m, uint32_t num_buckets, int32_t* keys, float* w, uint32_t cap, uint32_t* count,
                        hipStream_t s) {
  zero_u32_kernel<<<1, 64, 0, s>>>(count);
  const uint32_t per = 256 * kFreeScan, grid = (num_buckets + per - 1) / per;
  export_free_kernel<<<grid < 2048 ? grid : 2048, 256, 0, s>>>(m, num_buckets, keys, w, cap, count);
}

void launch_frame_blocks(const MapDev& m, int32_t* keys, uint32_t cap, uint32_t* count, hipStream_t s) {
  frame_blocks_kernel<<<256, 256, 0, s>>>(m, keys, cap, count);
}

void launch_export(const MapDev& m, int storage, int32_t* keys, float* sdf, float* w, uint8_t* rgb, uint32_t cap,
                   uint32_t* count, hipStream_t s) {
  if (storage == RF_STORAGE_FP32) export_kernel<RF_STORAGE_FP32><<<2048, 256, 0, s>>>(m, keys, sdf, w, rgb, cap, count);
  else export_kernel<RF_STORAGE_FP16_U8><<<2048, 256, 0, s>>>(m, keys, sdf, w, rgb, cap, count);
}

void launch_import(const MapDev& m, int storage, const int32_t* keys, const float* sdf, const float* w,
                   const uint8_t* rgb, uint32_t n, hipStream_t s) {
  if (n == 0) return;
  const int grid = (int)(n < 4096 ? n : 4096);
  advance_epoch_kernel<<<1, 64, 0, s>>>(m.st);
  if (storage == RF_STORAGE_FP32) import_kernel<RF_STORAGE_FP32><<<grid, 256, 0, s>>>(m, keys, sdf, w, rgb, n);
  else import_kernel<RF_STORAGE_FP16_U8><<<grid, 256, 0, s>>>(m, keys, sdf, w, rgb, n);
}

}  // namespace rf
