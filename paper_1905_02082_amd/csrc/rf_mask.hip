// Residual-based dynamics mask (Sec. III-C, Algorithm 1) for gfx950.
//
//   residual_kernel   r = S(T x)^2 per valid pixel, raw = r > gamma tau^2
//                     (with the tracking kernels: its corner blocks resolve
//                     through the tracking tile cache)
//   flood_seed        per 64x64 tile: 3x3 erosion (outside the image counts as
//                     0) -> seeds; the flood-fill rule for every pixel and its
//                     8 neighbours as 8 bits per pixel; seeds grown to the
//                     tile's fixpoint
//   flood_pass        the tiles that a neighbouring tile's growth may reach,
//                     in parallel
//   flood_finish      one workgroup per job re-runs such tiles, a wavefront on
//                     each, until none is left: growth is monotone, so the
//                     result is the unique least fixpoint the queue of
//                     Algorithm 1 reaches, with no grid-wide barrier
//   dilate            3x3 dilation -> final mask
// All passes take a batch of jobs (one map + frame each).
// The flood-fill rule: a neighbour n (8-neighbourhood) of a member p joins
// when |D(p) - D(n)| < theta D(p); invalid pixels carry D = 0 and so never
// join nor propagate.
//
// A tile is 64 rows of 64 bits, a lane per row, so a wavefront holds the
// members in one register pair and the rule in eight, and a fill along a row
// or a column takes six shift-and-mask steps (each step doubles the length of
// the runs filled) instead of one step per pixel.
#include "rf_device.h"
#include "rf_internal.h"

namespace rf {

typedef unsigned long long u64;

// What the fill keeps per frame.  Bits run along the frame's axis "u" (the
// image rows, or the columns of tall narrow frames, which would fill only
// part of a word); column strip tx holds bits u in [64 tx, 64 tx + 64) of
// every line v, as words tx nv + v.
struct FloodJob {
  u64* edge;    // 8 words per strip and line: bit u set when the pixel joins from its neighbour in that direction
  u64* member;  // a word per strip and line
  int nu, nv;   // frame size along the bits and across
  int su, sv;   // pixel strides
  int nx, ny;   // tiles
  int clear_from;  // first tile of the tracking cache's last level whose pairs the edges overwrite (-1: none)
};

struct FloodArgs {
  FloodJob job[kMaxBatch];
};

// Directions of the rule: the neighbour a pixel joins from.
enum { kL, kR, kU, kD, kUL, kUR, kDL, kDR };

// x of lane - s (or lane + s), 0 beyond the tile.
__device__ __forceinline__ u64 line_up(u64 x, int s) {
  const u64 y = __shfl_up(x, s, 64);
  return (int)(threadIdx.x & 63) >= s ? y : 0ull;
}
__device__ __forceinline__ u64 line_down(u64 x, int s) {
  const u64 y = __shfl_down(x, s, 64);
  return (int)(threadIdx.x & 63) + s < 64 ? y : 0ull;
}

// Members of a tile (lane = line) grown to the tile's fixpoint under the
// rule e.  Fills along the lines and columns go as far as they reach in one
// round; diagonal steps go one pixel a round.
__device__ __forceinline__ u64 grow_tile(u64 m, const u64 e[8]) {
  // e.g. after a step of s, pr[i] holds the pixels reached from s to the left
  u64 pl[6], pr[6], pu[6], pd[6];
  pl[0] = e[kL];
  pr[0] = e[kR];
  pu[0] = e[kU];
  pd[0] = e[kD];
#pragma unroll
  for (int i = 1; i < 6; ++i) {
    const int s = 1 << (i - 1);
    pl[i] = pl[i - 1] & (pl[i - 1] << s);
    pr[i] = pr[i - 1] & (pr[i - 1] >> s);
    pu[i] = pu[i - 1] & line_up(pu[i - 1], s);
    pd[i] = pd[i - 1] & line_down(pd[i - 1], s);
  }
  for (;;) {
    const u64 before = m;
    u64 a = m, b = m;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      a |= pl[i] & (a << (1 << i));
      b |= pr[i] & (b >> (1 << i));
    }
    m = a | b;
    a = b = m;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      a |= pu[i] & line_up(a, 1 << i);
      b |= pd[i] & line_down(b, 1 << i);
    }
    m = a | b;
    const u64 up = line_up(m, 1), dn = line_down(m, 1);
    m |= ((up << 1) & e[kUL]) | ((up >> 1) & e[kUR]) | ((dn << 1) & e[kDL]) | ((dn >> 1) & e[kDR]);
    if (__ballot(m != before) == 0ull) return m;
  }
}

// Marks the tiles that the new members of tile (tx, ty) touch (any of their
// pixels next to one may join; lane = line).
__device__ __forceinline__ void mark_neighbours(const FloodJob& F, int tx, int ty, u64 fresh, uint32_t* mark) {
  const u64 left = __ballot((fresh & 1ull) != 0ull), right = __ballot((fresh >> 63) != 0ull);
  const u64 any = __ballot(fresh != 0ull);
  const int lane = threadIdx.x & 63;
  // lane 0..8: tile offset (lane % 3 - 1, lane / 3 - 1)
  if (lane < 9 && lane != 4) {
    const int dx = lane % 3 - 1, dy = lane / 3 - 1;
    const u64 rows = dy < 0 ? 1ull : (dy > 0 ? 1ull << 63 : ~0ull);
    const u64 hit = (dx < 0 ? left : (dx > 0 ? right : any)) & rows;
    const int x = tx + dx, y = ty + dy;
    if (hit && x >= 0 && y >= 0 && x < F.nx && y < F.ny) mark[y * F.nx + x] = 1u;
  }
}

// One wavefront on tile (tx, ty): members that its halo lets in, grown to the
// fixpoint, written back, neighbours marked.  Another wavefront may be on a
// neighbouring tile: each writes only its own tile's words, and a new member
// on a border marks the neighbour, which then runs again.
__device__ void flood_tile(const FloodJob& F, int tx, int ty, uint32_t* mark) {
  const int lane = threadIdx.x & 63;
  const int v = ty * 64 + lane;
  const bool in = v < F.nv;
  const size_t w = (size_t)tx * F.nv + (in ? v : 0);
  u64 e[8];
  const ulonglong2* ep = reinterpret_cast<const ulonglong2*>(F.edge + 8 * w);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const ulonglong2 q = ep[i];
    e[2 * i] = in ? q.x : 0ull;
    e[2 * i + 1] = in ? q.y : 0ull;
  }
  // own line and the lines of the strips beside it; lanes 0 and 63 also hold
  // the lines above and below the tile
  const bool hl = tx > 0, hr = tx + 1 < F.nx;
  const bool edge_line = (lane == 0 && ty > 0) || (lane == 63 && v + 1 < F.nv);
  const size_t wv = edge_line ? (lane == 0 ? w - 1 : w + 1) : w;
  const u64 m0 = in ? F.member[w] : 0ull;
  const u64 lw = hl && in ? F.member[w - F.nv] >> 63 : 0ull;
  const u64 rw = hr && in ? F.member[w + F.nv] << 63 : 0ull;
  const u64 hv = edge_line ? F.member[wv] : 0ull;
  const u64 hvl = hl && edge_line ? F.member[wv - F.nv] >> 63 : 0ull;
  const u64 hvr = hr && edge_line ? F.member[wv + F.nv] << 63 : 0ull;
  u64 up = line_up(m0, 1), upl = line_up(lw, 1), upr = line_up(rw, 1);
  u64 dn = line_down(m0, 1), dnl = line_down(lw, 1), dnr = line_down(rw, 1);
  if (lane == 0) {
    up = hv;
    upl = hvl;
    upr = hvr;
  }
  if (lane == 63) {
    dn = hv;
    dnl = hvl;
    dnr = hvr;
  }
  u64 m = m0 | (((m0 << 1) | lw) & e[kL]) | (((m0 >> 1) | rw) & e[kR]) | (up & e[kU]) | (dn & e[kD]) |
          (((up << 1) | upl) & e[kUL]) | (((up >> 1) | upr) & e[kUR]) | (((dn << 1) | dnl) & e[kDL]) |
          (((dn >> 1) | dnr) & e[kDR]);
  if (__ballot(m != m0) == 0ull) return;  // nothing joins
  m = grow_tile(m, e);
  if (in) F.member[w] = m;
  mark_neighbours(F, tx, ty, m & ~m0, mark);
}

// Erosion, the rule's bits and the first growth of every tile; marks into
// flag buffer 0.  Eight wavefronts take 8 lines each, a lane per column.
template <int DF>
__global__ __launch_bounds__(512) void flood_seed_kernel(Batch b, FloodArgs A, float theta) {
  __shared__ u64 s_e[64][8];
  __shared__ u64 s_m[64];
  const int jb = batch_job(b, blockIdx.x);
  const Job& J = b.job[jb];
  const FrameDev& f = J.f;
  const FloodJob& F = A.job[jb];
  const float dmax = J.m.dmax;
  const int g = blockIdx.x - b.base[jb];
  const int tx = g % F.nx, ty = g / F.nx;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (g == 0 && F.clear_from >= 0) {
    // the tracking cache's tiles whose pairs the rule's bits replace hold none
    for (uint32_t i = F.clear_from + threadIdx.x; i < J.m.tc_tiles; i += blockDim.x)
      J.m.tc_count[(kCacheLevels - 1) * J.m.tc_tiles + i] = 0u;
  }
  constexpr int kLines = 8;  // lines per wavefront
  const int r0 = wave * kLines, v0 = ty * 64 + r0;
  const int u = tx * 64 + lane;
  const bool uin = u < F.nu, lin = u > 0 && u <= F.nu, rin = u + 1 < F.nu;  // the column, its left and right neighbours
  const int off = u * F.su;
  if (v0 < F.nv) {  // uniform per wavefront
    const uint8_t* raw = J.raw ? J.raw : J.mask_out;
    // every load first (one round trip): the raw mask and depth of the lines
    // and of the lines beside them, at columns u - 1, u, u + 1
    uint32_t rw[kLines + 2][3];
    float dp[kLines + 2][3];
#pragma unroll
    for (int i = 0; i < kLines + 2; ++i) {
      const int v = v0 - 1 + i;
      const bool vin = v >= 0 && v < F.nv;
      const int at = (vin ? v : v0) * F.sv + off;
      const int c0 = lin ? at - F.su : 0, c1 = uin ? at : 0, c2 = rin ? at + F.su : 0;
      rw[i][0] = raw[c0];
      rw[i][1] = raw[c1];
      rw[i][2] = raw[c2];
      dp[i][0] = load_depth<DF>(f, c0);
      dp[i][1] = load_depth<DF>(f, c1);
      dp[i][2] = load_depth<DF>(f, c2);
    }
#pragma unroll
    for (int i = 0; i < kLines + 2; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) asm volatile("" : "+v"(rw[i][c]), "+v"(dp[i][c]));
    u64 h[kLines + 2];  // per line: pixels whose left, own and right raw bits are set
    float td[kLines + 2][3];
#pragma unroll
    for (int i = 0; i < kLines + 2; ++i) {
      const int v = v0 - 1 + i;
      const bool vin = v >= 0 && v < F.nv;
      const bool in[3] = {vin && lin, vin && uin, vin && rin};
      const bool set = (rw[i][0] != 0) & (rw[i][1] != 0) & (rw[i][2] != 0) & in[0] & in[1] & in[2];
      h[i] = __ballot(set);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        dp[i][c] = (in[c] & (dp[i][c] > 0.0f) & (dp[i][c] <= dmax)) ? dp[i][c] : 0.0f;
        td[i][c] = theta * dp[i][c];
      }
    }
#pragma unroll
    for (int i = 1; i <= kLines; ++i) {
      const float dq = dp[i][1];
      const u64 ok = __ballot(dq > 0.0f);
      auto joins = [&](int q, int c) { return __ballot(fabsf(dp[q][c] - dq) < td[q][c]) & ok; };
      const u64 w[8] = {joins(i, 0),     joins(i, 2),     joins(i - 1, 1), joins(i + 1, 1),
                        joins(i - 1, 0), joins(i - 1, 2), joins(i + 1, 0), joins(i + 1, 2)};  // kL .. kDR
      if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) s_e[r0 + i - 1][k] = w[k];
        s_m[r0 + i - 1] = h[i - 1] & h[i] & h[i + 1];
      }
    }
  } else if (lane < kLines) {
#pragma unroll
    for (int i = 0; i < 8; ++i) s_e[r0 + lane][i] = 0ull;
    s_m[r0 + lane] = 0ull;
  }
  __syncthreads();
  // the rule's bits to memory, 16 bytes a thread
  const int lines = min(64, F.nv - ty * 64);
  ulonglong2* out = reinterpret_cast<ulonglong2*>(F.edge + 8 * ((size_t)tx * F.nv + ty * 64));
  for (int i = threadIdx.x; i < lines * 4; i += blockDim.x)
    out[i] = make_ulonglong2(s_e[i >> 2][2 * (i & 3)], s_e[i >> 2][2 * (i & 3) + 1]);
  if (wave != 0) return;
  const int v = ty * 64 + lane;
  u64 m = s_m[lane];
  if (J.eroded) {
    for (int r = 0; r < lines; ++r) {
      const u64 w = s_m[r];
      if (uin) J.eroded[(ty * 64 + r) * F.sv + off] = (uint8_t)((w >> lane) & 1ull);
    }
  }
  if (__ballot(m != 0ull) != 0ull) {
    u64 e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = s_e[lane][i];
    m = grow_tile(m, e);
    mark_neighbours(F, tx, ty, m, J.m.dirty);
  }
  if (v < F.nv) F.member[(size_t)tx * F.nv + v] = m;
}

// The tiles marked in flag buffer 0 (clearing their own flag), marking into
// buffer 1, so the pass does not read the flags it writes.
__global__ __launch_bounds__(64) void flood_pass_kernel(Batch b, FloodArgs A) {
  const int jb = batch_job(b, blockIdx.x);
  const MapDev& m = b.job[jb].m;
  const FloodJob& F = A.job[jb];
  const int g = blockIdx.x - b.base[jb];
  uint32_t* own = m.dirty + g;
  if (!*own) return;  // uniform
  __builtin_amdgcn_wave_barrier();
  if (threadIdx.x == 0) *own = 0u;
  flood_tile(F, g % F.nx, g / F.nx, m.dirty + m.dirty_cap);
}

// One workgroup per job: the marked tiles, a wavefront on each, until none is
// left (or the work cap).
constexpr int kFinishThreads = 1024;
__global__ __launch_bounds__(kFinishThreads) void flood_finish_kernel(Batch b, FloodArgs A, int buf) {
  __shared__ int s_list[1024];
  __shared__ int s_n;
  const Job& J = b.job[blockIdx.x];
  const MapDev& m = J.m;
  const FloodJob& F = A.job[blockIdx.x];
  const int ntiles = F.nx * F.ny;
  const int max_tiles_processed = 64 * ntiles + J.f.W * J.f.H;
  uint32_t* dirty = m.dirty + (size_t)buf * m.dirty_cap;
  int processed = 0;
  for (;;) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < ntiles; i += blockDim.x) {
      if (dirty[i]) {
        dirty[i] = 0;
        const int k = atomicAdd(&s_n, 1);
        if (k < 1024) s_list[k] = i;
        else dirty[i] = 1;  // no room this sweep: keep it for the next
      }
    }
    __syncthreads();
    const int n = min(s_n, 1024);
    __syncthreads();
    if (n == 0) break;
    for (int k = threadIdx.x >> 6; k < n; k += kFinishThreads / 64) {
      const int tile = s_list[k];
      flood_tile(F, tile % F.nx, tile / F.nx, dirty);
    }
    processed += n;
    if (processed > max_tiles_processed) {
      if (threadIdx.x == 0) atomicOr(&m.st->flags, (uint32_t)RF_FLAG_MASK_LIMIT);
      __syncthreads();
      for (int i = threadIdx.x; i < ntiles; i += blockDim.x) dirty[i] = 0;  // leave no flag behind
      break;
    }
    __syncthreads();
  }
}

// 3x3 dilation of the members into the mask (and, for callers that ask, the
// fill itself): a thread per 8 pixels of a line.
__global__ __launch_bounds__(256) void dilate_kernel(Batch b, FloodArgs A) {
  const int jb = batch_job(b, blockIdx.x);
  const Job& J = b.job[jb];
  const FloodJob& F = A.job[jb];
  const int per = F.nx * 8;  // groups of 8 bits a line
  const int i = (blockIdx.x - b.base[jb]) * blockDim.x + threadIdx.x;
  const int v = i / per, c = i % per, u = 8 * c;
  if (v >= F.nv || u >= F.nu) return;
  // bits u - 1 .. u + 8 of line y, the lowest at bit 0
  const int tx = c >> 3, sh = (c & 7) * 8;
  auto window = [&](int y) -> uint32_t {
    if (y < 0 || y >= F.nv) return 0u;
    const u64* p = F.member + (size_t)tx * F.nv + y;
    const u64 w = *p;
    uint32_t x = (uint32_t)(sh ? w >> (sh - 1) : w << 1) & 0x3FFu;
    if (sh == 0 && tx > 0) x |= (uint32_t)(p[-(ptrdiff_t)F.nv] >> 63);
    if (sh == 56) {
      x &= 0x1FFu;
      if (tx + 1 < F.nx) x |= (uint32_t)(p[F.nv] & 1ull) << 9;
    }
    return x;
  };
  const uint32_t mid = window(v);
  const uint32_t x = window(v - 1) | mid | window(v + 1);
  const uint32_t y = (x | (x >> 1) | (x >> 2)) & 0xFFu;
  auto put = [&](uint8_t* base, uint32_t bits) {
    uint8_t* o = base + (size_t)v * F.sv + (size_t)u * F.su;
    if (F.su == 1 && u + 8 <= F.nu && (reinterpret_cast<uintptr_t>(o) & 7) == 0) {
      // spread the 8 bits over the 8 bytes of a word
      u64 s = bits;
      s = (s | (s << 28)) & 0x0000000F0000000Full;
      s = (s | (s << 14)) & 0x0003000300030003ull;
      s = (s | (s << 7)) & 0x0101010101010101ull;
      *reinterpret_cast<u64*>(o) = s;
    } else {
      for (int k = 0; k < 8 && u + k < F.nu; ++k) o[(size_t)k * F.su] = (uint8_t)((bits >> k) & 1u);
    }
  };
  if (J.filled) put(J.filled, (mid >> 1) & 0xFFu);
  put(J.mask_out, y);
}

static int set_bases(Batch& b, const FloodArgs& A, int (*count)(const FloodJob&)) {
  int total = 0;
  for (int j = 0; j < b.n; ++j) {
    b.base[j] = total;
    total += count(A.job[j]);
  }
  b.base[b.n] = total;
  return total;
}

static int tile_count(const FloodJob& F) { return F.nx * F.ny; }
static int dilate_groups(const FloodJob& F) { return (F.nx * 8 * F.nv + 255) / 256; }

// Tall frames narrower than four words put their columns along the bits.
static void flood_axes(const FrameDev& f, FloodJob& F) {
  const bool rows = f.W >= 256 || f.W >= f.H;
  F.nu = rows ? f.W : f.H;
  F.nv = rows ? f.H : f.W;
  F.su = rows ? 1 : f.W;
  F.sv = rows ? f.W : 1;
  F.nx = (F.nu + 63) / 64;
  F.ny = (F.nv + 63) / 64;
}

size_t flood_edge_bytes(const FrameDev& f) {
  FloodJob F;
  flood_axes(f, F);
  return (size_t)F.nx * F.nv * 64;
}

// Bytes of the last level's pairs: 8192 a tile.  Every frame of up to
// max_pixels pixels fits: its bits take 64 bytes for each 64 pixels of a line or
// part of them, so a line of at least 64 pixels takes less than 2 bytes a
// pixel, where a map has 8192 for each 256 pixels, and the frames whose longer
// side is shorter take less than 4096, which the map's 64 spare tiles hold.
size_t flood_edge_room(uint32_t tc_tiles) {
  return (size_t)tile_refs(kCacheLevels - 1) * tc_tiles * sizeof(BlockRef);
}

size_t flood_member_bytes(const FrameDev& f) {
  FloodJob F;
  flood_axes(f, F);
  return (size_t)F.nx * F.nv * 8;
}

// Frames of more tiles than this (8 rounds of the drain's 16 wavefronts) get a
// parallel pass over the marked tiles before the drain.  With nothing to fill it
// costs 1 to 3 us.  Masks of frames with a third and two thirds of the view
// moving, means of three scenes, without / with: 640x480 (80 tiles) 47 / 48 and
// 51 / 51 us, 848x480 (112) 48 / 49 and 50 / 49, 960x540 (135) 50 / 49 and
// 55 / 51, 1024x640 (160) 57 / 56 and 59 / 55, 1280x720 (240) 60 / 56 and
// 65 / 60.
constexpr int kPassTiles = 128;

void launch_mask(Batch& b, int df, int st, const rf_mask_params& mp, void* edges, hipStream_t s) {
  FloodArgs A{};
  for (int j = 0; j < b.n; ++j) {
    const Job& J = b.job[j];
    FloodJob& F = A.job[j];
    flood_axes(J.f, F);
    F.member = reinterpret_cast<u64*>(J.m.md);
    F.clear_from = -1;
    if (edges) {
      F.edge = static_cast<u64*>(edges);
    } else {
      // The end of the tracking cache: its last level has pairs for as many
      // tiles as the finest, of which a frame uses one in 64, so the pairs of
      // the last tiles are free (thin frames may reach them: their counts are
      // cleared).  The caller has checked that the bits fit (flood_edge_room).
      const size_t bytes = (flood_edge_bytes(J.f) + 255) & ~(size_t)255;
      const size_t region = flood_edge_room(J.m.tc_tiles);
      char* end = reinterpret_cast<char*>(J.m.tcache + (size_t)tile_refs_before(kCacheLevels) * J.m.tc_tiles);
      F.edge = reinterpret_cast<u64*>(end - bytes);
      F.clear_from = (int)((region - bytes) / (tile_refs(kCacheLevels - 1) * sizeof(BlockRef)));
    }
  }
  launch_residual(b, df, st, mp.gamma, s);
  // the tile flags are all zero here: map initialisation zeroes them, and
  // every mask computation ends with both buffers empty (each parallel pass
  // clears the flags it consumes, the finish drains the last buffer)
  const int g = set_bases(b, A, tile_count);
  if (df == RF_DEPTH_U16) flood_seed_kernel<RF_DEPTH_U16><<<g, 512, 0, s>>>(b, A, mp.theta);
  else flood_seed_kernel<RF_DEPTH_F32><<<g, 512, 0, s>>>(b, A, mp.theta);
  int passes = 0;
  for (int j = 0; j < b.n; ++j)
    if (tile_count(A.job[j]) > kPassTiles) passes = 1;
  if (passes) flood_pass_kernel<<<g, 64, 0, s>>>(b, A);
  flood_finish_kernel<<<b.n, kFinishThreads, 0, s>>>(b, A, passes);
  dilate_kernel<<<set_bases(b, A, dilate_groups), 256, 0, s>>>(b, A);
}

}  // namespace rf
