// Virtual depth by ray casting the model (Sec. III-E, second option for
// invalid measurements), for gfx950.
//
// Along the pixel's ray the samples are taken at camera depths
// z_k = z_near + k step, step = tau / 2, at the back-projection of the pixel
// at z_k (Eq. 1) moved to the world by the pose; the virtual depth is the
// first crossing from a defined sample S_{k-1} > 0 to a defined sample
// S_k <= 0, z_{k-1} + step (S_{k-1} / (S_{k-1} - S_k)), or 0.  With
// only_invalid the pixels whose depth is not zero keep it (metres) and only
// the zeros are cast, getting the virtual depth or far_value.
//
// A workgroup takes a 16x16 pixel tile and collects the rays to cast.  What
// a ray costs is the chain of its samples (a hundred and more, each a round
// trip to the map), and nearly all of them lie in free space, where every
// sample is defined and positive.  Two ways round that chain, both with the
// decisions of sampling one by one:
//   few rays (holes of a frame): 32 lanes share a ray, each with a sample of
//     its own, and the first crossing of a batch is found by a ballot;
//   many rays: the blocks the tile's rays pass are looked up and tested once
//     per tile by whole wavefronts, and the samples in blocks known to hold
//     only observed, positive distances (or in no block) are stepped over
//     without reading them.  Each wavefront tests the beam of its 64 rays: a
//     slab of samples about one block long against the box of blocks it can
//     touch, 8 slabs at a time with 8 lanes on each (with one slab at a time
//     the tests' arithmetic, not the map, took most of the kernel: 8000 cycles
//     a slab).
// 640x480 at 1 cm voxels, all pixels: 820 -> 167 us; the kernel is now bound by
// the arithmetic of the tests and of the ~14 samples a ray still reads.
#include <type_traits>

#include "rf_device.h"
#include "rf_internal.h"

namespace rf {

constexpr int kRayTile = 16;        // tile edge (pixels)
constexpr int kRayThreads = kRayTile * kRayTile;
constexpr int kRayLanes = 32;       // lanes sharing a ray (few rays)
// Tiles with at most this many rays share lanes between them: testing the
// blocks of a tile costs the same for 5 rays as for 256.  640x480, 1 cm, holes
// at random, shared / tested: 2% of the pixels (5 rays a tile) 49 / 177 us, 10%
// 139 / 198, 20% 242 / 200, all 977 / 191 (one thread per ray before: 612, 721,
// 694, 734).
constexpr int kRaySparse = 40;
constexpr int kRayTable = 512;      // blocks of the tile's table
constexpr int kRayProbes = 16;
constexpr int kSlabLanes = 8;      // lanes on a slab of the beam
constexpr int kSlabs = 64 / kSlabLanes;
// Codes of the tile's table: a pool slot (>= 0, with kRayPositive when the
// block's 512 voxels are observed and positive), -1 absent, <= -2 a free
// block (as resolve_slot), or not known yet.
constexpr int kRayPending = (int)0x80000000;
constexpr int kRayPositive = 0x40000000;
__device__ __forceinline__ bool ray_positive(int c) { return c >= 0 ? (c & kRayPositive) != 0 : c < -2; }
__device__ __forceinline__ bool ray_absent(int c) { return c == -1 || c == -2; }  // -2: free, not yet observed

struct RayTable {
  unsigned long long* key;
  int* code;
  uint32_t* req;   // entries to be looked up
  uint32_t* nreq;
  uint32_t* used;

  // entry of block (x,y,z), added and asked for if it is new; -1 when the
  // table has no room near its home
  __device__ __forceinline__ int entry(int x, int y, int z) const {
    const unsigned long long k = pack_key(x, y, z);
    uint32_t h = hash3(x, y, z) & (kRayTable - 1);
#pragma unroll 1
    for (int i = 0; i < kRayProbes; ++i) {
      unsigned long long old = key[h];
      if (old == kEmptyKey) old = atomicCAS(&key[h], kEmptyKey, k);
      if (old == k) return (int)h;
      if (old == kEmptyKey) {
        req[atomicAdd(nreq, 1u)] = h;
        atomicAdd(used, 1u);
        return (int)h;
      }
      h = (h + 1) & (kRayTable - 1);
    }
    return -1;
  }
};

// Corner-block slots from the codes of a box of blocks (lower block b0, nx by
// ny blocks a layer).
struct BoxSlots {
  const int* code;
  int b0[3], nx, ny;
  bool direct;  // from the hash table instead
  __device__ __forceinline__ int at(int x, int y, int z) const {
    return code[((x - b0[0]) + nx * ((y - b0[1]) + ny * (z - b0[2]))) & 63];
  }
  // every corner of the cell lies in one block, and that is a positive one
  __device__ __forceinline__ bool inside_positive(const int i0[3]) const {
    return (i0[0] & 7) != 7 && (i0[1] & 7) != 7 && (i0[2] & 7) != 7 &&
           ray_positive(at(i0[0] >> 3, i0[1] >> 3, i0[2] >> 3));
  }
  __device__ __forceinline__ bool operator()(const MapDev& m, int bx, int by, int bz, int cross, int sl[8]) const {
    if (direct) return HashSlots()(m, bx, by, bz, cross, sl);
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int c = at(bx + (k & 1 & cross), by + ((k & 2 & cross) >> 1), bz + ((k & 4 & cross) >> 2));
      sl[k] = c >= 0 ? (c & ~kRayPositive) : c;
      ok = ok && c != -1;
    }
    return ok;
  }
};

// The test of a block by a whole wavefront, lanes reading 16 bytes at a time:
// positive when its 512 voxels are observed with a distance in
// [tau / 1024, 4 tau].  Interpolated values of such corners stay positive whatever the
// rounding (each of the seven interpolations is off by at most a few units
// of 2^-24 of the largest corner).
template <int STORAGE>
__device__ __forceinline__ bool block_positive(const MapDev& m, uint32_t slot, int lane) {
  constexpr int rec = STORAGE == RF_STORAGE_FP32 ? 8 : 4, nv = 512 * rec / (64 * 16);
  const float lo = m.tau * 0x1p-10f, hi = m.tau * 4.0f;
  const uint4* p = reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(m.sdfw) + (size_t)slot * (512 * rec));
  uint4 v[nv];
#pragma unroll
  for (int q = 0; q < nv; ++q) v[q] = p[lane + 64 * q];
  bool ok = true;
#pragma unroll
  for (int q = 0; q < nv; ++q) {
    const uint32_t r[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
    if constexpr (STORAGE == RF_STORAGE_FP32) {
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        const float s = __uint_as_float(r[j]), w = __uint_as_float(r[j + 1]);
        ok = ok && w > 0.0f && s >= lo && s <= hi;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float s = __half2float(__ushort_as_half((unsigned short)(r[j] & 0xFFFFu))) * m.tau;
        ok = ok && ((r[j] >> 16) & 0xFFu) != 0u && s >= lo && s <= hi;
      }
    }
  }
  return __all(ok) != 0;
}

// World point of the ray (ru, rv) at camera depth z.
__device__ __forceinline__ void ray_point(const float R[9], const float t[3], float ru, float rv, float z, float y[3]) {
  const float x[3] = {ru * z, rv * z, z};
  xform(R, t, x, y);
}

// FILL: only the pixels without a depth are cast (only_invalid); without it
// every tile is full and the shared-ray path is compiled out.
template <int DF, int STORAGE, bool FILL>
__global__ __launch_bounds__(kRayThreads, FILL ? 4 : 3) void raycast_kernel(MapDev m, FrameDev f, const double* pose,
                                                              float z_near, float z_far, float far_value, float* out) {
  __shared__ uint16_t s_ray[kRayThreads];   // the tile's rays (local pixel)
  __shared__ uint32_t s_nray, s_nreq, s_used;
  __shared__ unsigned long long s_key[kRayTable];
  __shared__ int s_code[kRayTable];
  __shared__ uint32_t s_req[kRayTable];
  __shared__ int s_box[kRayThreads / 64][64 * kSlabs];  // per wavefront and slab: codes of its box of blocks
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int tiles_x = (f.W + kRayTile - 1) / kRayTile;
  const int tu = (int)(blockIdx.x % tiles_x) * kRayTile, tv = (int)(blockIdx.x / tiles_x) * kRayTile;
  // wavefront = 8x8 pixels of the tile
  const int lu = (wave & 1) * 8 + (lane & 7), lv = (wave >> 1) * 8 + (lane >> 3);
  const bool inside = tu + lu < f.W && tv + lv < f.H;
  if (threadIdx.x == 0) s_nray = s_nreq = s_used = 0u;
  __syncthreads();
  {
    const int idx = inside ? (tv + lv) * f.W + tu + lu : 0;
    const float D = FILL ? load_depth<DF>(f, idx) : 0.0f;  // the depth is read only to fill it
    const bool cast = inside && !(FILL && D != 0.0f);
    if (inside && !cast) out[idx] = D;
    const unsigned long long bal = __ballot(cast);
    uint32_t base = 0;
    if (lane == 0 && bal) base = atomicAdd(&s_nray, (uint32_t)__popcll(bal));
    base = __shfl(base, 0);
    if (cast)
      s_ray[base + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u))] =
          (uint16_t)(lv * kRayTile + lu);
  }
  __syncthreads();
  const int n = (int)s_nray;
  if (n == 0) return;
  float R[9], t[3];
  load_pose_f(pose, R, t);
  const float step = 0.5f * m.tau;

  if (FILL && n <= kRaySparse) {
    const int sub = threadIdx.x & (kRayLanes - 1);
    // uniform per group of kRayLanes; the groups of a wavefront diverge only
    // between whole batches, and a group's shuffles stay inside it
    for (int r = threadIdx.x / kRayLanes; r < n; r += kRayThreads / kRayLanes) {
      const int l = s_ray[r];
      const int u = tu + (l & (kRayTile - 1)), v = tv + l / kRayTile;
      const float ru = ((float)u - f.cx) * f.ifx, rv = ((float)v - f.cy) * f.ify;
      float hit = 0.0f, carry = -1.0f;  // carry: S of the sample before the batch (-1 where undefined)
      for (int k0 = 0; z_near + (float)k0 * step <= z_far; k0 += kRayLanes) {
        const int k = k0 + sub;
        const float z = z_near + (float)k * step;
        float y[3], S = 0.0f, gS[3], Iv, gI[3];
        ray_point(R, t, ru, rv, z, y);
        const bool defined = z <= z_far && sample_map<STORAGE, false, false>(m, y, S, gS, Iv, gI);
        const float val = defined ? S : -1.0f;
        float prev = __shfl_up(val, 1, kRayLanes);
        if (sub == 0) prev = carry;
        carry = __shfl(val, kRayLanes - 1, kRayLanes);
        const bool cross = defined && S <= 0.0f && prev > 0.0f;
        const uint32_t cb = (uint32_t)(__ballot(cross) >> (lane & ~(kRayLanes - 1)));
        if (cb) {
          const float zp = z_near + (float)(k - 1) * step;
          hit = __shfl(zp + step * (prev / (prev - S)), __ffs((int)cb) - 1, kRayLanes);
          break;
        }
      }
      if (sub == 0) out[v * f.W + u] = FILL ? (hit > 0.0f ? hit : far_value) : hit;
    }
    return;
  }

  const RayTable tab{s_key, s_code, s_req, &s_nreq, &s_used};
  const bool mine = threadIdx.x < (unsigned)n;
  const int l = s_ray[mine ? threadIdx.x : 0];
  const int u = tu + (l & (kRayTile - 1)), v = tv + l / kRayTile;
  const float ru = ((float)u - f.cx) * f.ifx, rv = ((float)v - f.cy) * f.ify;
  // The wavefront's rays per unit of camera depth, axis by axis (its beam):
  // at depths [z0, z1] they lie within t + [min(dlo z), max(dhi z)].
  float dlo[3], dhi[3], mag[3];  // mag: sum of the magnitudes (bounds the rounding)
  {
    float ulo = mine ? ru : INFINITY, uhi = mine ? ru : -INFINITY, vlo = mine ? rv : INFINITY, vhi = mine ? rv : -INFINITY;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      ulo = fminf(ulo, __shfl_xor(ulo, o));
      uhi = fmaxf(uhi, __shfl_xor(uhi, o));
      vlo = fminf(vlo, __shfl_xor(vlo, o));
      vhi = fmaxf(vhi, __shfl_xor(vhi, o));
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      dlo[a] = (R[3 * a] * (R[3 * a] > 0.0f ? ulo : uhi) + R[3 * a + 1] * (R[3 * a + 1] > 0.0f ? vlo : vhi)) + R[3 * a + 2];
      dhi[a] = (R[3 * a] * (R[3 * a] > 0.0f ? uhi : ulo) + R[3 * a + 1] * (R[3 * a + 1] > 0.0f ? vhi : vlo)) + R[3 * a + 2];
      mag[a] = (fabsf(R[3 * a]) * fmaxf(fabsf(ulo), fabsf(uhi)) + fabsf(R[3 * a + 1]) * fmaxf(fabsf(vlo), fabsf(vhi))) +
               fabsf(R[3 * a + 2]);
    }
  }
  // the box of blocks that hold the corners of the beam's samples at depths
  // [z0, z1] (a margin of a fiftieth of a voxel and a millionth of the summed
  // magnitudes covers the rounding); false if it has more than 64 blocks
  auto box = [&](float z0, float z1, int b0[3], int& nx, int& ny, int& nb) -> bool {
    int d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float lo = (t[a] + fminf(dlo[a] * z0, dlo[a] * z1)) * m.is, hi = (t[a] + fmaxf(dhi[a] * z0, dhi[a] * z1)) * m.is;
      const float e = 0.02f + 1.0e-6f * ((fabsf(t[a]) + mag[a] * z1) * m.is);
      if (!(lo - e > -kMaxVoxelCoord && hi + e < kMaxVoxelCoord - 8.0f)) return false;
      b0[a] = (int)floorf(lo - e) >> 3;
      d[a] = (((int)floorf(hi + e) + 1) >> 3) - b0[a] + 1;
      if (d[a] > 64) return false;
    }
    nx = d[0];
    ny = d[1];
    nb = d[0] * d[1] * d[2];
    return nb <= 64;
  };
  auto block_of = [&](int i, const int b0[3], int nx, int ny, int b[3]) {
    const int q = i / nx;
    b[0] = b0[0] + i - q * nx;
    b[1] = b0[1] + q % ny;
    b[2] = b0[2] + q / ny;
  };
  // samples taken together: the beam over about one block's length
  const int slab = (int)fminf(fmaxf(8.0f * m.s / step + 0.5f, 1.0f), 16.0f);
  float hit = 0.0f, prev = 0.0f;
  // the sample before k: 0 undefined, 1 positive (not read), 2 its value is in prev
  int have = 0;
  bool alive = mine;
  bool going = __any(mine) != 0;  // uniform per wavefront
  int k = 0;                      // uniform per wavefront
  bool first = true, cleared = false;  // uniform
  int* code = s_box[wave];
#pragma unroll
  for (int j = 0; j < kSlabs; ++j) code[64 * j + lane] = -1;
  for (;;) {
    // an emptied table before the first round and whenever it has filled up;
    // never twice in a row, so what a wavefront waits for is there when it
    // goes on (or finds no room, and its rays read the map by themselves)
    if (first || (!cleared && s_used > (uint32_t)kRayTable / 2)) {
      __syncthreads();
      for (int i = threadIdx.x; i < kRayTable; i += kRayThreads) {
        s_key[i] = kEmptyKey;
        s_code[i] = kRayPending;
      }
      if (threadIdx.x == 0) s_used = 0u;
      first = false;
      cleared = true;
    } else {
      cleared = false;
    }
    __syncthreads();
    bool waiting = false;  // uniform per wavefront
    while (going && !waiting) {
      // a chunk of slabs at a time, kSlabLanes lanes on each: its box of blocks
      // and their codes (lanes striding over the box), in LDS for the samples
      const int k0 = k, js = lane / kSlabLanes;
      int b0[3], nx = 1, ny = 1, nb = 0;
      const bool fits = box(z_near + (float)(k0 + js * slab) * step, z_near + (float)(k0 + (js + 1) * slab - 1) * step,
                            b0, nx, ny, nb);
      bool room = fits, pend = false, pos = true, absent = true;
      for (int i = lane & (kSlabLanes - 1); room && i < nb; i += kSlabLanes) {
        int bb[3];
        block_of(i, b0, nx, ny, bb);
        const int e = tab.entry(bb[0], bb[1], bb[2]);
        room = e >= 0;
        const int c = room ? s_code[e] : kRayPending;
        pend = pend || c == kRayPending;
        pos = pos && c != kRayPending && ray_positive(c);
        absent = absent && ray_absent(c);
        code[js * 64 + i] = c;
      }
      const unsigned long long mroom = __ballot(!room), mpend = __ballot(pend), mpos = __ballot(!pos),
                               mabs = __ballot(!absent);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 1
      for (int j = 0; j < kSlabs && going; ++j) {
        if (!(z_near + (float)k * step <= z_far)) {
          going = false;
          break;
        }
        const unsigned long long of = ((1ull << kSlabLanes) - 1ull) << (j * kSlabLanes);
        const bool direct = (mroom & of) != 0ull;  // no room in the table or too large a box: from the map itself
        if (!direct && (mpend & of) != 0ull) {
          waiting = true;
          break;
        }
        if (!direct && ((mpos & of) == 0ull || (mabs & of) == 0ull)) {
          have = (mpos & of) == 0ull ? 1 : 0;
          k += slab;
          continue;
        }
        const int jl = j * kSlabLanes;
        BoxSlots slots{code + 64 * j,
                       {__builtin_amdgcn_readlane(b0[0], jl), __builtin_amdgcn_readlane(b0[1], jl),
                        __builtin_amdgcn_readlane(b0[2], jl)},
                       __builtin_amdgcn_readlane(nx, jl), __builtin_amdgcn_readlane(ny, jl), direct};
#pragma unroll 1
        for (int q = 0; q < slab; ++q, ++k) {
          const float z = z_near + (float)k * step, zp = z_near + (float)(k - 1) * step;
          if (!alive || !(z <= z_far)) continue;
          // a crossing from a sample that was stepped over reads that sample too
          float Sk = 0.0f;
          bool back = false;
          for (;;) {
            float y[3], fr[3], S = 0.0f, gS[3], Iv, gI[3];
            int i0[3];
            ray_point(R, t, ru, rv, back ? zp : z, y);
            bool defined = voxel_cell(m, y, i0, fr), pos = false;
            if (defined) {
              // samples inside a positive block are not read here either
              pos = !back && !direct && slots.inside_positive(i0);
              if (!pos) {
                float cs[8], cw[8];
                uint32_t cc[8];
                slots.direct = direct || back;
                defined = gather_corners<STORAGE, false, true>(m, i0, slots, cs, cw, cc) &&
                          interpolate<false, false>(m, cs, cw, cc, fr, S, gS, Iv, gI);
              }
            }
            if (back) {
              prev = S;
            } else if (!defined || pos) {
              have = defined ? 1 : 0;
              break;
            } else {
              Sk = S;
              if (have == 1 && S <= 0.0f) {
                back = true;
                continue;
              }
            }
            if (have != 0 && prev > 0.0f && Sk <= 0.0f) {
              hit = zp + step * (prev / (prev - Sk));
              alive = false;
            }
            prev = Sk;
            have = 2;
            break;
          }
        }
        going = __any(alive) != 0;
      }
      // ask for the next chunk too, unless the table is filling up
      if (waiting && s_used < (uint32_t)kRayTable / 2) {
        const int ka = k0 + (kSlabs + js) * slab;
        if (box(z_near + (float)ka * step, z_near + (float)(ka + slab - 1) * step, b0, nx, ny, nb)) {
          for (int i = lane & (kSlabLanes - 1); i < nb; i += kSlabLanes) {
            int bb[3];
            block_of(i, b0, nx, ny, bb);
            tab.entry(bb[0], bb[1], bb[2]);
          }
        }
      }
    }
    const int more = __syncthreads_or(waiting ? 1 : 0);
    if (!more) break;  // no wavefront waits: all have ended
    // look the asked-for blocks up, then test those with voxels
    const int nreq = (int)s_nreq;
    for (int i = threadIdx.x; i < nreq; i += kRayThreads) {
      const uint32_t e = s_req[i];
      const unsigned long long key = s_key[e];
      int x, yb, zb;
      unpack_key(key, x, yb, zb);
      const uint32_t h = hash3(x, yb, zb) & m.bucket_mask;
      s_code[e] = resolve_slot(m, m.buckets[h], key, h);
    }
    __syncthreads();
    if (threadIdx.x == 0) s_nreq = 0u;
    for (int i = wave; i < nreq; i += kRayThreads / 64) {
      const uint32_t e = s_req[i];
      const int c = s_code[e];
      if (c < 0) continue;  // uniform per wavefront
      if (block_positive<STORAGE>(m, (uint32_t)c, lane) && lane == 0) s_code[e] = c | kRayPositive;
    }
    __syncthreads();
  }
  if (mine) out[v * f.W + u] = FILL ? (hit > 0.0f ? hit : far_value) : hit;
}

void launch_raycast(const MapDev& m, const FrameDev& f, int depth_format, int storage, const double* pose,
                    float z_near, float z_far, float far_value, int only_invalid, float* out, hipStream_t s) {
  const dim3 g(((f.W + kRayTile - 1) / kRayTile) * ((f.H + kRayTile - 1) / kRayTile)), blk(kRayThreads);
  auto run = [&](auto df, auto st) {
    constexpr int D = decltype(df)::value, S = decltype(st)::value;
    if (only_invalid) raycast_kernel<D, S, true><<<g, blk, 0, s>>>(m, f, pose, z_near, z_far, far_value, out);
    else raycast_kernel<RF_DEPTH_U16, S, false><<<g, blk, 0, s>>>(m, f, pose, z_near, z_far, far_value, out);  // no depth is read
  };
  auto with_storage = [&](auto df) {
    if (storage == RF_STORAGE_FP32) run(df, std::integral_constant<int, RF_STORAGE_FP32>{});
    else run(df, std::integral_constant<int, RF_STORAGE_FP16_U8>{});
  };
  if (depth_format == RF_DEPTH_U16) with_storage(std::integral_constant<int, RF_DEPTH_U16>{});
  else with_storage(std::integral_constant<int, RF_DEPTH_F32>{});
}

}  // namespace rf
