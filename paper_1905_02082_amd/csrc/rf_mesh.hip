// Triangle mesh of the model's zero level set (the paper shows its models as
// meshes, Sec. I and Fig. 1) by marching tetrahedra, for gfx950.
//
// A cube of 8 voxel centres (lower corner v, corner k = dx + 2 dy + 4 dz at
// v + (dx, dy, dz)) is meshed when all 8 voxels exist, are observed (w > 0)
// and hold |sdf| < tau.  It is cut into the six tetrahedra (0, a, a|b, 7)
// along its diagonal, one per order of the axis bits; neighbouring cubes cut
// their shared faces alike, so the mesh is closed wherever the cubes are.
// Inside means sdf < 0.  One vertex alone on its side gives a triangle (the
// crossings of its three edges), two and two a quad (two triangles).  The
// crossing on edge (a, b), a the corner whose bits are a subset of b's, is
// P_a + t (P_b - P_a) with t = f_a / (f_a - f_b), so every tetrahedron and
// cube that shares a grid edge computes the same point.  Triangles face the
// positive (observed) side: a triangle whose normal has a negative dot
// product with n_in * sum(outside corners) - n_out * sum(inside corners) is
// reversed.
//
// Three launches, so that the output is compact without a contended
// counter: a count pass (triangles per workgroup), a one-workgroup scan, and
// a write pass in which every workgroup walks its blocks in the same order
// and places each tetrahedron's triangles by a prefix sum over the workgroup.
// Given the pool order of the blocks the output order is deterministic.
//
// Count: a wavefront per block, one lane per column of voxels; the slices'
// "in the band" and "inside" flags are ballots, 64-bit words in scalar
// registers, and a block without a voxel in the band (nearly all of free
// space) is done with them.  Otherwise the flags of the 217 voxels beyond the
// block's upper faces join, and the cubes of a slice are counted 64 at a time
// by bit operations.  Blocks with triangles are marked in a byte per pool
// slot, so that the write pass reads only those.
// Write: the block's 9^3 corner values go to LDS once, the tetrahedra that
// emit triangles are listed in order, and a thread takes one of them at a
// time (a block has tens of such cubes, hundreds of such tetrahedra).
// 36 k blocks, 5.1 M triangles: both passes 577 -> 178 us.  Bounds: the count
// reads every record of the map, the write pass the triangles' arithmetic.
#include "rf_device.h"
#include "rf_internal.h"

namespace rf {

constexpr int kMeshThreads = 512;  // one thread per voxel cube of a block

// Corner j of tetrahedron t: the chain 0, a, a|b, 7 with first axis bit
// a = 1 << (t / 2) and second b the lower (t even) or higher (t odd) of the
// other two bits: (0,1,3,7) (0,1,5,7) (0,2,3,7) (0,2,6,7) (0,4,5,7) (0,4,6,7).
__host__ __device__ constexpr int tet_corner(int t, int j) {
  return j == 0 ? 0
                : (j == 3 ? 7
                          : ((1 << (t >> 1)) |
                             (j == 1 ? 0
                                     : ((t & 1) ? ((7 & ~(1 << (t >> 1))) & ~((7 & ~(1 << (t >> 1))) & -(7 & ~(1 << (t >> 1)))))
                                                : ((7 & ~(1 << (t >> 1))) & -(7 & ~(1 << (t >> 1))))))));
}
static_assert(tet_corner(0, 2) == 3 && tet_corner(1, 2) == 5 && tet_corner(2, 2) == 3 && tet_corner(3, 2) == 6 &&
                  tet_corner(4, 2) == 5 && tet_corner(5, 2) == 6 && tet_corner(5, 1) == 4,
              "tetrahedra of the cube");

typedef unsigned long long u64;

// Marks of the blocks with triangles, a byte per pool slot, in the map's byte
// map of touched buckets: unused, and zero, outside an allocation (a slot has
// a bucket of its own, so the map is large enough).  The write pass clears
// what the count pass sets.
__device__ __forceinline__ uint8_t* mesh_marks(const MapDev& m) { return touched_map(m); }

// A voxel's value if it is observed and within the band, NaN otherwise (or
// without a slot).
template <int STORAGE>
__device__ __forceinline__ float band_value(const MapDev& m, int slot, int l) {
  float f, w;
  VoxelStore<STORAGE>::load(m, (uint32_t)(slot >= 0 ? slot : 0) * 512u + (uint32_t)l, f, w);
  return (slot >= 0 && w > 0.0f && fabsf(f) < m.tau) ? f : __uint_as_float(0x7FC00000u);
}

// Flags of the 9x9 corners of a slice for the 64 cubes at lower corner (x, y),
// bit x + 8 y: at (x, y), (x+1, y), (x, y+1), (x+1, y+1).  own: the 64 corners;
// px: the corners x = 8 (bit y), py: y = 8 (bit x), pxy: x = y = 8.
struct Slice {
  u64 c[4];
};
__device__ __forceinline__ Slice make_slice(u64 own, uint32_t px, uint32_t py, uint32_t pxy) {
  const u64 col7 = 0x8080808080808080ull;
  // spread px: bit y to bit 8 y + 7
  u64 sx = px & 0xFFu;
  sx = (sx | (sx << 28)) & 0x0000000F0000000Full;
  sx = (sx | (sx << 14)) & 0x0003000300030003ull;
  sx = ((sx | (sx << 7)) & 0x0101010101010101ull) << 7;
  Slice s;
  s.c[0] = own;
  s.c[1] = ((own >> 1) & ~col7) | sx;
  s.c[2] = (own >> 8) | ((u64)(py & 0xFFu) << 56);
  s.c[3] = ((s.c[2] >> 1) & ~col7) | (sx >> 8) | ((u64)(pxy & 1u) << 63);
  return s;
}

// This lane's share of the triangles of the cubes of block b (whole
// wavefront); f: the lane's column of its voxels.
template <int STORAGE>
__device__ __forceinline__ uint32_t block_triangles(const MapDev& m, uint32_t b, const float f[8], int lane) {
  u64 V[9], N[9], anyv = 0;
#pragma unroll
  for (int z = 0; z < 8; ++z) {
    V[z] = __ballot(f[z] == f[z]);
    N[z] = __ballot(f[z] < 0.0f);
    anyv |= V[z];
  }
  if (anyv == 0ull) return 0u;
  // the block's 7 upper neighbours (lane k: offset bits k)
  int bx, by, bz;
  unpack_key(m.block_keys[b], bx, by, bz);
  int sl = -1;
  if (lane >= 1 && lane < 8) sl = find_slot(m, bx + (lane & 1), by + ((lane >> 1) & 1), bz + (lane >> 2));
  const int i = lane & 7, j = lane >> 3;
  // upper faces, a voxel a lane: z = 8 at (x, y) = (i, j), x = 8 at (y, z),
  // y = 8 at (x, z); the edges and the corner share a load: lanes 0-7 x = y = 8
  // (z = i), 8-15 x = z = 8 (y = i), 16-23 y = z = 8 (x = i), 24 the corner
  const float fz = band_value<STORAGE>(m, __shfl(sl, 4), lane);
  const float fx = band_value<STORAGE>(m, __shfl(sl, 1), 8 * i + 64 * j);
  const float fy = band_value<STORAGE>(m, __shfl(sl, 2), i + 64 * j);
  const int es = __shfl(sl, j == 0 ? 3 : (j == 1 ? 5 : (j == 2 ? 6 : 7)));
  const float fe = band_value<STORAGE>(m, lane < 25 ? es : -1, j == 0 ? 64 * i : (j == 1 ? 8 * i : (j == 2 ? i : 0)));
  V[8] = __ballot(fz == fz);
  N[8] = __ballot(fz < 0.0f);
  const u64 vx = __ballot(fx == fx), nx = __ballot(fx < 0.0f), vy = __ballot(fy == fy), ny = __ballot(fy < 0.0f);
  const u64 ve = __ballot(fe == fe), ne = __ballot(fe < 0.0f);
  // lane i + 8 t counts tetrahedron t of the cubes of slice i: as scalar code,
  // slice after slice, the same operations made the kernel 2x as long
  int words[4] = {0, 0, 0, 0};  // lane z: V[z], N[z]
#pragma unroll
  for (int z = 0; z < 9; ++z) {
    if (lane != z) continue;
    words[0] = (int)V[z];
    words[1] = (int)(V[z] >> 32);
    words[2] = (int)N[z];
    words[3] = (int)(N[z] >> 32);
  }
  auto word = [&](int k, int z) {
    return ((u64)(uint32_t)__shfl(words[2 * k + 1], z) << 32) | (uint32_t)__shfl(words[2 * k], z);
  };
  auto slice = [&](int k, int z, u64 fxm, u64 fym, u64 fem) {
    const u64 own = word(k, z);
    return make_slice(own, (uint32_t)(z < 8 ? fxm >> (8 * z) : fem >> 8), (uint32_t)(z < 8 ? fym >> (8 * z) : fem >> 16),
                      (uint32_t)(fem >> (z < 8 ? z : 24)));
  };
  const Slice v0 = slice(0, i, vx, vy, ve), v1 = slice(0, i + 1, vx, vy, ve);
  const Slice n0 = slice(1, i, nx, ny, ne), n1 = slice(1, i + 1, nx, ny, ne);
  const u64 valid = (v0.c[0] & v0.c[1] & v0.c[2] & v0.c[3]) & (v1.c[0] & v1.c[1] & v1.c[2] & v1.c[3]);
  const u64 n[8] = {n0.c[0], n0.c[1], n0.c[2], n0.c[3], n1.c[0], n1.c[1], n1.c[2], n1.c[3]};
  u64 q = 0, r = 0;
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    q = j == t ? n[tet_corner(t, 1)] : q;
    r = j == t ? n[tet_corner(t, 2)] : r;
  }
  const u64 p = n[0], s = n[7];
  const u64 odd = p ^ q ^ r ^ s;                          // one corner alone: a triangle
  const u64 mixed = (p | q | r | s) & ~(p & q & r & s);  // two and two: two triangles
  return j < 6 ? (uint32_t)__popcll(valid & odd) + 2u * (uint32_t)__popcll(valid & mixed & ~odd) : 0u;
}

// Pass 1: triangles per workgroup -> scratch[g]; blocks with triangles marked.
constexpr int kCountThreads = 512;
template <int STORAGE>
__global__ __launch_bounds__(kCountThreads) void mesh_count_kernel(MapDev m, uint32_t* scratch) {
  __shared__ uint32_t s_sum;
  if (threadIdx.x == 0) s_sum = 0u;
  __syncthreads();
  const uint32_t n = min(m.st->n_blocks, m.max_blocks);
  const int lane = threadIdx.x & 63;
  uint8_t* marks = mesh_marks(m);
  uint32_t mine = 0;
  const uint32_t step = gridDim.x * (kCountThreads / 64);
  uint32_t b = blockIdx.x + gridDim.x * (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // the next block's records load while this one's flags are counted
  float sdf[8], w[8];
  auto load = [&](uint32_t q) {
#pragma unroll
    for (int z = 0; z < 8; ++z)
      VoxelStore<STORAGE>::load(m, (q < n ? q : 0u) * 512u + (uint32_t)(lane + 64 * z), sdf[z], w[z]);
  };
  if (b < n) load(b);
  for (; b < n; b += step) {
    float f[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) f[z] = (w[z] > 0.0f && fabsf(sdf[z]) < m.tau) ? sdf[z] : __uint_as_float(0x7FC00000u);
    if (b + step < n) load(b + step);
    const uint32_t c = block_triangles<STORAGE>(m, b, f, lane);
    mine += c;
    if (__ballot(c != 0u) != 0ull && lane == 0) marks[b] = 1;
  }
  if (mine) atomicAdd(&s_sum, mine);
  __syncthreads();
  if (threadIdx.x == 0) scratch[blockIdx.x] = s_sum;
}

// Pass 2 (one workgroup): exclusive offsets scratch[G + g] and the total.
__global__ __launch_bounds__(1024) void mesh_scan_kernel(uint32_t* scratch, int groups, uint32_t* count) {
  __shared__ uint32_t s_v[1024];
  const int t = threadIdx.x;
  const uint32_t x = t < groups ? scratch[t] : 0u;
  s_v[t] = x;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {  // inclusive Hillis-Steele scan
    const uint32_t y = t >= o ? s_v[t - o] : 0u;
    __syncthreads();
    s_v[t] += y;
    __syncthreads();
  }
  if (t < groups) scratch[groups + t] = s_v[t] - x;
  if (t == 1023) *count = s_v[1023];
}

// Corner values in LDS: corner (x, y, z), 0..8 each.
constexpr int kCorners = 9 * 9 * 9;
__device__ __forceinline__ int corner_at(int x, int y, int z) { return x + 9 * (y + 9 * z); }

// The corner that thread t < 217 loads beyond the block's upper faces: x = 8
// (64 of them), y = 8 (64), z = 8 (64), the edges (8 each), the corner.
__device__ __forceinline__ void halo_corner(int t, int& x, int& y, int& z) {
  const int q = t >> 6, i = t & 7, j = (t >> 3) & 7;
  x = q == 0 ? 8 : i;
  y = q == 0 ? i : (q == 1 ? 8 : j);
  z = q == 2 ? 8 : j;
  if (q == 3) {  // 0-7: x = y = 8, 8-15: x = z = 8, 16-23: y = z = 8, 24: the corner
    x = j == 2 ? i : 8;
    y = j == 1 ? i : 8;
    z = j == 0 ? i : 8;
  }
}

// What to do for a tetrahedron whose corners (0..3 along its chain) with sdf <
// 0 are the bits of `inside`: bits 4c..4c+3 the ends of crossing edge c (lower
// corner of the chain, then upper), bits 16-21 and 22-27 the first three
// inside and outside corners in chain order, bits 28-30 how many are inside.
// A corner alone has three crossing edges (the fourth entry repeats the
// third), two and two have four, in quad order.
__host__ __device__ constexpr uint32_t tet_case(uint32_t inside) {
  uint32_t in[4] = {0, 0, 0, 0}, out[4] = {0, 0, 0, 0}, ni = 0, no = 0;
  for (uint32_t j = 0; j < 4; ++j) {
    if ((inside >> j) & 1u) in[ni++] = j;
    else out[no++] = j;
  }
  uint32_t x = ni << 28;
  for (uint32_t j = 0; j < 3; ++j) x |= in[j] << (16 + 2 * j) | out[j] << (22 + 2 * j);
  for (uint32_t c = 0; c < 4; ++c) {
    uint32_t i = 0, o = 0;
    if (ni == 2) {
      i = in[c >= 2 ? 1 : 0];
      o = out[c == 1 || c == 2 ? 1 : 0];
    } else {
      i = ni == 1 ? in[0] : out[0];
      o = ni == 1 ? out[c < 3 ? c : 2] : in[c < 3 ? c : 2];
    }
    x |= (i < o ? i : o) << (4 * c) | (i < o ? o : i) << (4 * c + 2);
  }
  return x;
}
// The chain of tetrahedron t: corner j in bits 4j..4j+2.
__host__ __device__ constexpr uint32_t tet_chain(int t) {
  return (uint32_t)(tet_corner(t, 1) << 4 | tet_corner(t, 2) << 8 | 7 << 12);
}

// The triangles of a tetrahedron (chain, case) of the cube at voxel v; f: its
// corner 0's value in LDS.  No branch on the case: the selected corners are
// read from LDS and their positions picked per axis.
__device__ __forceinline__ void tet_write(const float* f, uint32_t chain, uint32_t tc, const int v[3], float s,
                                          float* tris, uint32_t next, uint32_t cap) {
  float p0[3], p1[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    p0[a] = (float)v[a] * s;
    p1[a] = (float)(v[a] + 1) * s;
  }
  auto corner = [&](uint32_t j) { return (chain >> (4 * j)) & 7u; };
  const uint32_t ni = (tc >> 28) & 7u, no = 4u - ni;
  const uint32_t ic[3] = {corner((tc >> 16) & 3u), corner((tc >> 18) & 3u), corner((tc >> 20) & 3u)};
  const uint32_t oc[3] = {corner((tc >> 22) & 3u), corner((tc >> 24) & 3u), corner((tc >> 26) & 3u)};
  float ref[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float so = 0.0f, si = 0.0f;
#pragma unroll
    for (uint32_t j = 0; j < 3; ++j) {
      const float xo = so + (((oc[j] >> a) & 1u) ? p1[a] : p0[a]), xi = si + (((ic[j] >> a) & 1u) ? p1[a] : p0[a]);
      so = j < no ? xo : so;
      si = j < ni ? xi : si;
    }
    ref[a] = (float)(int)ni * so - (float)(int)no * si;
  }
  float q[4][3];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint32_t kl = corner((tc >> (4 * c)) & 3u), kh = corner((tc >> (4 * c + 2)) & 3u);
    const float fl = f[(kl & 1u) + 9u * ((kl >> 1) & 1u) + 81u * (kl >> 2)];
    const float fh = f[(kh & 1u) + 9u * ((kh >> 1) & 1u) + 81u * (kh >> 2)];
    const float tt = fl / (fl - fh);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float pl = ((kl >> a) & 1u) ? p1[a] : p0[a], ph = ((kh >> a) & 1u) ? p1[a] : p0[a];
      q[c][a] = pl + tt * (ph - pl);
    }
  }
  const float e1[3] = {q[1][0] - q[0][0], q[1][1] - q[0][1], q[1][2] - q[0][2]};
  const float e2[3] = {q[2][0] - q[0][0], q[2][1] - q[0][1], q[2][2] - q[0][2]};
  const float nx = e1[1] * e2[2] - e1[2] * e2[1], ny = e1[2] * e2[0] - e1[0] * e2[2], nz = e1[0] * e2[1] - e1[1] * e2[0];
  const bool facing = (nx * ref[0] + ny * ref[1]) + nz * ref[2] >= 0.0f;
  float* o = tris + 9 * (size_t)next;
  if (next < cap) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      o[a] = q[0][a];
      o[3 + a] = facing ? q[1][a] : q[2][a];
      o[6 + a] = facing ? q[2][a] : q[1][a];
    }
  }
  if (ni == 2u && next + 1u < cap) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      o[9 + a] = q[0][a];
      o[12 + a] = facing ? q[2][a] : q[3][a];
      o[15 + a] = facing ? q[3][a] : q[2][a];
    }
  }
}

// Pass 3: every workgroup walks the blocks it marked in pass 1 in order and
// writes their triangles from its offset, cubes in voxel order, tetrahedra in
// order within a cube.
template <int STORAGE>
__global__ __launch_bounds__(kMeshThreads, 8) void mesh_write_kernel(MapDev m, const uint32_t* scratch, int groups,
                                                                  float* tris, uint32_t cap) {
  __shared__ uint32_t s_list[kMeshThreads];     // marked blocks of the chunk
  __shared__ uint32_t s_wave[kMeshThreads / 64];
  __shared__ int s_nb[2][8];                    // slots of a block and its upper neighbours
  __shared__ float s_fb[2][kCorners];
  // tetrahedra that emit: cube | tetrahedron << 9 | first triangle (in the block) << 12 | inside corners << 25
  __shared__ uint32_t s_tet[kMeshThreads * 6];
  __shared__ uint32_t s_case[16], s_chain[6];
  constexpr uint32_t kCase[16] = {tet_case(0),  tet_case(1),  tet_case(2),  tet_case(3), tet_case(4),  tet_case(5),
                                  tet_case(6),  tet_case(7),  tet_case(8),  tet_case(9), tet_case(10), tet_case(11),
                                  tet_case(12), tet_case(13), tet_case(14), tet_case(15)};
  constexpr uint32_t kChain[6] = {tet_chain(0), tet_chain(1), tet_chain(2), tet_chain(3), tet_chain(4), tet_chain(5)};
#pragma unroll
  for (uint32_t i = 0; i < 16; ++i)
    if (threadIdx.x == i) s_case[i] = kCase[i];
#pragma unroll
  for (uint32_t i = 0; i < 6; ++i)
    if (threadIdx.x == i) s_chain[i] = kChain[i];
  const uint32_t n = min(m.st->n_blocks, m.max_blocks);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint8_t* marks = mesh_marks(m);
  const float s = m.s;
  uint32_t base = scratch[groups + blockIdx.x];
  // exclusive prefix of x over the workgroup; total in *sum (a barrier before
  // s_wave is used again is up to the caller)
  auto prefix = [&](uint32_t x, uint32_t* sum) {
    uint32_t inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kMeshThreads / 64; ++w) {
      const uint32_t y = s_wave[w];
      before += w < wave ? y : 0u;
      total += y;
    }
    *sum = total;
    return before + inc - x;
  };
  auto find_neighbours = [&](uint32_t b, int* nb) {  // threads 0..7
    int bx, by, bz;
    unpack_key(m.block_keys[b], bx, by, bz);
    nb[tid] = tid == 0 ? (int)b : find_slot(m, bx + (tid & 1), by + ((tid >> 1) & 1), bz + (tid >> 2));
  };
  for (uint32_t c0 = 0; blockIdx.x + c0 * gridDim.x < n; c0 += kMeshThreads) {  // uniform
    const uint32_t b = blockIdx.x + (c0 + tid) * gridDim.x;
    const bool marked = b < n && marks[b] != 0;
    if (marked) marks[b] = 0;
    uint32_t nm;
    const uint32_t at = prefix(marked ? 1u : 0u, &nm);
    if (marked) s_list[at] = b;
    __syncthreads();
    // a block's corner values load while the block before it is written, and
    // the slots they need are found one block earlier still
    float fo = 0.0f, fh = 0.0f;
    int hx, hy, hz;
    halo_corner(tid < 217 ? tid : 0, hx, hy, hz);
    auto load = [&](const int* nb) {
      fo = band_value<STORAGE>(m, nb[0], tid);
      if (tid < 217)
        fh = band_value<STORAGE>(m, nb[(hx >> 3) | ((hy >> 3) << 1) | ((hz >> 3) << 2)],
                                 (hx & 7) + 8 * (hy & 7) + 64 * (hz & 7));
    };
    if (tid < 8 && nm) find_neighbours(s_list[0], s_nb[0]);
    __syncthreads();
    if (nm) load(s_nb[0]);
    if (tid < 8 && nm > 1) find_neighbours(s_list[1], s_nb[1]);
    for (uint32_t k = 0; k < nm; ++k) {
      float* s_f = s_fb[k & 1];
      s_f[corner_at(tid & 7, (tid >> 3) & 7, tid >> 6)] = fo;
      if (tid < 217) s_f[corner_at(hx, hy, hz)] = fh;
      int bx, by, bz;
      unpack_key(m.block_keys[s_list[k]], bx, by, bz);
      __syncthreads();  // the values and the next block's slots are there, the list of tetrahedra is free
      if (k + 1 < nm) load(s_nb[(k + 1) & 1]);
      if (tid < 8 && k + 2 < nm) find_neighbours(s_list[k + 2], s_nb[k & 1]);
      // the tetrahedra of this thread's cube that emit (3 bits: how many triangles each)
      const int cx = tid & 7, cy = (tid >> 3) & 7, cz = tid >> 6;
      uint32_t inside = 0;
      bool ok = true;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const float f = s_f[corner_at(cx + (c & 1), cy + ((c >> 1) & 1), cz + (c >> 2))];
        ok = ok && f == f;
        inside |= f < 0.0f ? 1u << c : 0u;
      }
      if (!ok) inside = 0u;
      uint32_t in[6], mine = 0;  // mine: tetrahedra << 16 | triangles
#pragma unroll
      for (int t = 0; t < 6; ++t) {
        in[t] = ((inside >> tet_corner(t, 0)) & 1u) | ((inside >> tet_corner(t, 1)) & 1u) << 1 |
                ((inside >> tet_corner(t, 2)) & 1u) << 2 | ((inside >> tet_corner(t, 3)) & 1u) << 3;
        const uint32_t some = in[t] != 0u && in[t] != 15u ? 0x10001u : 0u;
        mine += some + (__popc(in[t]) == 2 ? 1u : 0u);
      }
      uint32_t total;
      uint32_t off = prefix(mine, &total);
#pragma unroll
      for (int t = 0; t < 6; ++t) {
        if (in[t] == 0u || in[t] == 15u) continue;
        s_tet[off >> 16] = (uint32_t)tid | ((uint32_t)t << 9) | ((off & 0xFFFFu) << 12) | (in[t] << 25);
        off += 0x10001u + (__popc(in[t]) == 2 ? 1u : 0u);
      }
      __syncthreads();
      for (uint32_t e = tid; e < total >> 16; e += kMeshThreads) {
        const uint32_t x = s_tet[e];
        const int l = (int)(x & 511u), t = (int)((x >> 9) & 7u);
        const int lx = l & 7, ly = (l >> 3) & 7, lz = l >> 6;
        const int v[3] = {8 * bx + lx, 8 * by + ly, 8 * bz + lz};
        tet_write(s_f + corner_at(lx, ly, lz), s_chain[t], s_case[x >> 25], v, s, tris, base + ((x >> 12) & 0x1FFFu),
                  cap);
      }
      base += total & 0xFFFFu;
    }
    __syncthreads();  // the list is no longer read
  }
}

constexpr int kMeshGroups = kMeshScratch;

void launch_mesh(const MapDev& m, int storage, float* tris, uint32_t cap, uint32_t* count, hipStream_t s) {
  if (storage == RF_STORAGE_FP32) {
    mesh_count_kernel<RF_STORAGE_FP32><<<kMeshGroups, kCountThreads, 0, s>>>(m, m.mesh_scratch);
    mesh_scan_kernel<<<1, 1024, 0, s>>>(m.mesh_scratch, kMeshGroups, count);
    mesh_write_kernel<RF_STORAGE_FP32><<<kMeshGroups, kMeshThreads, 0, s>>>(m, m.mesh_scratch, kMeshGroups, tris, cap);
  } else {
    mesh_count_kernel<RF_STORAGE_FP16_U8><<<kMeshGroups, kCountThreads, 0, s>>>(m, m.mesh_scratch);
    mesh_scan_kernel<<<1, 1024, 0, s>>>(m.mesh_scratch, kMeshGroups, count);
    mesh_write_kernel<RF_STORAGE_FP16_U8><<<kMeshGroups, kMeshThreads, 0, s>>>(m, m.mesh_scratch, kMeshGroups, tris,
                                                                              cap);
  }
}

}  // namespace rf
