// Direct registration to the TSDF (Sec. III-B, Eqs. 1-4) for gfx950.
//
// One launch per Gauss-Newton/LM iteration, one thread per pixel of the
// pyramid level (a workgroup covers a 16x16 pixel tile, so the voxels its
// wavefronts gather are close together).  A thread forms the depth residual S and the photometric
// residual Iv - I with their 6-DoF Jacobians in FP32 and, from them, its
// pixel's 29 normal-equation terms in FP64 (products of FP32 factors are exact
// in FP64); each wavefront adds its terms up in a fixed order, and the
// workgroup adds the wavefronts' sums to device-wide accumulators.
//
// The accumulators are fixed point (units of 2^-60) held as two chunks in
// 64-bit words, the low 48 bits and the signed rest, and summed with
// device-scope integer atomics: integer addition is associative, so the
// totals do not depend on the order in which workgroups finish
// (bit-reproducible), and the chunks need no carry chain, so every atomic is
// independent (the low chunk's sums keep 16 bits of headroom for carries).  Workgroups spread over kAccCopies
// copies of the accumulators (fewer atomics per address), which the reader
// sums exactly.  Nothing in a launch waits for the
// other workgroups: the solve of iteration j runs at the start of launch j+1,
// redundantly in every workgroup (all read the same completed totals and run
// the same instructions, so all obtain the same pose), overlapped with the
// pose-independent loads of the pixel (levels with more workgroups than two
// resident rounds solve in a one-workgroup launch instead, see
// kSeparateSolveTiles).  Accumulators rotate through three
// buffers (read j-1, write j, clear j+1) and the pose through two, so no
// launch reads what the same launch writes.  A one-workgroup finalize launch
// solves the last iteration and writes the caller's pose.
#include <type_traits>

#include "rf_device.h"
#include "rf_internal.h"

namespace rf {

constexpr double kFixScale = 0x1p60;
constexpr int kTermWords = 16;                     // one 128-byte line per term
constexpr int kCopyWords = kNE * kTermWords;       // one copy of the 29 accumulators
constexpr int kBufWords = kAccCopies * kCopyWords;  // one accumulator buffer
constexpr int kTerms = 14;                         // J_d(6) J_c(6) r_d r_c
constexpr int kTileW = kTrackBlock / 16;           // pixel tile: kTileW x 16

struct TrackArgs {
  int level;         // pyramid level evaluated by this launch (-1: none)
  float w_c;
  int min_valid;
  double lm_lambda;
  int solve;         // 1: first solve the system accumulated by the previous launch
  int prev_level;    // level of that previous evaluation
  int prev_first;    // it was the first iteration of its level
  int acc_read, acc_write, acc_clear;  // accumulator buffer indices (-1: none)
  int pose_read, pose_write;           // 0/1: pose scratch, 2: caller's pose (-1: none)
  int mode;          // 0: track; 1: write the normal equations of acc_read to out29; 2: solve only
  int adaptive;      // 1: Levenberg-Marquardt (accept / reject, adaptive lambda); 0: fixed lambda
  int state_read, state_write;         // Levenberg-Marquardt state buffers (0/1, -1: none)
};

__device__ __forceinline__ unsigned long long* acc_buf(const MapDev& m, int b) {
  return reinterpret_cast<unsigned long long*>(m.partials) + (size_t)b * kBufWords;
}
// The words an accumulator buffer actually uses: two chunks per term per copy
// (the rest of each 128-byte line is padding against false sharing: atomics on
// one line are served one after another).  Entry q of kUsedPairs.
constexpr int kUsedPairs = kAccCopies * kNE;
static_assert(kUsedPairs <= kTrackBlock, "a launch clears its share with one store a thread");
__device__ __forceinline__ ulonglong2* used_pair(unsigned long long* buf, int q) {
  return reinterpret_cast<ulonglong2*>(buf + (q / kNE) * kCopyWords + (q % kNE) * kTermWords);
}
__device__ __forceinline__ double* pose_buf(const MapDev& m, double* user, int b) {
  return b == 2 ? user : reinterpret_cast<double*>(m.partials) + (size_t)3 * kBufWords + 16 * b;
}
// Levenberg-Marquardt state: [0, 16) accepted pose, [16, 45) its normal
// equations, [45] lambda.
constexpr int kLmWords = 48;
__device__ __forceinline__ double* lm_state(const MapDev& m, int b) {
  return reinterpret_cast<double*>(m.partials) + (size_t)3 * kBufWords + 32 + kLmWords * b;
}

// Adds v to a term: v 2^60 truncated toward zero as a two's complement
// integer lo + hi 2^48 (lo unsigned 48-bit, hi signed 64-bit), two atomics
// (one where hi is 0).  The low chunks of a copy sum below 2^63 for up to 2^15
// workgroups (a 2^26-pixel frame's tiles over the copies), the high chunks of
// terms below 2^34 likewise.  A non-finite v, or |v| >= 2^34 (beyond that
// range), is not added: the low chunk's top bit, which its sum does not reach,
// is set instead, and its total then reads as NaN, which stops the registration
// pass (RF_FLAG_TRACK_RANGE).  Returns false in that case.
constexpr unsigned long long kRangeMark = 1ull << 63;
__device__ __forceinline__ bool fixed_add(unsigned long long* acc, double v) {
  double a = fabs(v) * kFixScale;
  if (!(a < 0x1p94)) {
    atomicOr(&acc[0], kRangeMark);
    return false;
  }
  const double hi_d = floor(a * 0x1p-48);
  unsigned long long hi = (unsigned long long)hi_d;
  unsigned long long lo = (unsigned long long)(a - hi_d * 0x1p48);
  if (v < 0.0) {
    hi = ~hi + (lo == 0ull ? 1ull : 0ull);
    lo = (0ull - lo) & 0xFFFFFFFFFFFFull;
  }
  if (lo) atomicAdd(&acc[0], lo);
  if (hi) atomicAdd(&acc[1], hi);
  return true;
}

// Totals of the terms over the accumulator copies, by a whole wavefront: lane
// l of each half reads half of the copies of term l mod 32, a pair of chunks a
// load, so the 232 lines are asked for by 4 loads (one lane a term took 24
// loads of a word each, half of a solve's 3000 cycles of waiting for them).
struct TermLoads {
  ulonglong2 acc[kAccCopies / 2];
};
static_assert(kAccCopies % 2 == 0 && kNE <= 32, "half a wavefront reads half of the copies");
__device__ __forceinline__ void load_terms(const unsigned long long* buf, int lane, TermLoads& L) {
  const unsigned long long* p = buf + (lane >> 5) * (kAccCopies / 2 * kCopyWords) + min(lane & 31, kNE - 1) * kTermWords;
#pragma unroll
  for (int c = 0; c < kAccCopies / 2; ++c) L.acc[c] = *reinterpret_cast<const ulonglong2*>(p + c * kCopyWords);
}
// The value of the lane 32 below or above.
__device__ __forceinline__ unsigned long long other_half(unsigned long long v) {
  const bool upper = threadIdx.x & 32;
  const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
  return ((unsigned long long)(upper ? h[0] : h[1]) << 32) | (upper ? l[0] : l[1]);
}
// Total of term lane mod 32 as FP64 (exact 128-bit integer sum, then
// conversion).  A term whose range mark is set in any copy totals NaN.
__device__ __forceinline__ double fixed_total(const TermLoads& L) {
  unsigned long long lo = 0, hi = 0, bad = 0;
#pragma unroll
  for (int c = 0; c < kAccCopies / 2; ++c) {
    const unsigned long long s0 = L.acc[c].x & ~kRangeMark;
    const long long s1 = (long long)L.acc[c].y;
    bad |= L.acc[c].x;
    // s1 2^48 + s0 as a 128-bit two's complement number, added to (hi, lo)
    const unsigned long long l1 = (unsigned long long)s1 << 48;
    const unsigned long long h1 = (unsigned long long)(s1 >> 16);
    const unsigned long long n = lo + l1;
    hi += h1 + (n < lo ? 1ull : 0ull);
    lo = n + s0;
    hi += (lo < n ? 1ull : 0ull);
  }
  const unsigned long long lo2 = other_half(lo), hi2 = other_half(hi);
  lo += lo2;
  hi += hi2 + (lo < lo2 ? 1ull : 0ull);
  bad |= other_half(bad);
  if (bad & kRangeMark) return __longlong_as_double(0x7FF8000000000000ll);
  const bool neg = (long long)hi < 0;
  if (neg) {
    lo = ~lo + 1ull;
    hi = ~hi + (lo == 0ull ? 1ull : 0ull);
  }
  const double mag = ((double)hi * 0x1p64 + (double)lo) * (1.0 / kFixScale);
  return neg ? -mag : mag;
}

__device__ __forceinline__ int tri_index(int i, int j) {  // H(i,j), i <= j, packed upper triangle
  return 6 * i - (i * (i - 1)) / 2 + (j - i);
}

// The solving wavefront of a workgroup: totals -> delta by elimination of
// [H + lambda diag H | -g] (no pivoting, H is symmetric positive semi-definite,
// so its upper triangle is enough) -> exp(delta^) T.  Writes the new pose
// (row-major 12 values) to s_T, in 32 bits to s_Tf if given, and the outcome to
// *s_state: 0 ok, RF_FLAG_TRACK_FEW_PIXELS or RF_FLAG_TRACK_SINGULAR (pose kept).
// A pivot of the elimination equals the squared Cholesky pivot, so the
// singularity test is the Cholesky one: pivot <= 1e-12 trace(H).
// Tin: the input pose in LDS; lane l < 16 forms element (l / 4, l % 4) of the new one.
//
// Every lane solves the whole system: a dependent chain, in which passing rows
// between lanes costs more than the arithmetic it would save (a row a lane took
// 96 lane reads and a branch a pivot; with the range test a ballot and the
// exponential applied as cross products, 3250 -> 2100 cycles from totals to
// pose).
__device__ __forceinline__ void solve_update_wave(const double* s_ne, const TrackArgs& a, const double* Tin,
                                                  double* s_T, float* s_Tf, int* s_state) {
  const int lane = threadIdx.x & 63;
  const double own = s_ne[lane < kNE ? lane : 0];
  double h[21], g[6];
#pragma unroll
  for (int k = 0; k < 21; ++k) h[k] = s_ne[k];
#pragma unroll
  for (int i = 0; i < 6; ++i) g[i] = -s_ne[21 + i];
  double tr = 0.0;
#pragma unroll
  for (int i = 0; i < 6; ++i) tr += h[tri_index(i, i)];
  asm volatile("" : "+v"(tr));  // its terms need not outlive the elimination
#pragma unroll
  for (int i = 0; i < 6; ++i) h[tri_index(i, i)] *= (1.0 + a.lm_lambda);
  bool singular = false;
  double inv[6];  // reciprocal pivots, reused by the back substitution
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const double piv = h[tri_index(k, k)];
    singular |= !(piv > 1e-12 * tr);
    inv[k] = rcp_f64(piv);
#pragma unroll
    for (int i = k + 1; i < 6; ++i) {
      const double fct = h[tri_index(k, i)] * inv[k];
#pragma unroll
      for (int c = i; c < 6; ++c) h[tri_index(i, c)] = fma(-fct, h[tri_index(k, c)], h[tri_index(i, c)]);
      g[i] = fma(-fct, g[k], g[i]);
      asm volatile("" : "+v"(g[i]));  // or the factors stay in registers until the end
    }
  }
  double x[6];
#pragma unroll
  for (int k = 5; k >= 0; --k) {
    double s = g[k];
#pragma unroll
    for (int j = 5; j > k; --j) s = fma(-h[tri_index(k, j)], x[j], s);
    x[k] = s * inv[k];
  }
  // solved before the branches below, so that the system's registers are free again
#pragma unroll
  for (int k = 0; k < 6; ++k) asm volatile("" : "+v"(x[k]));
  int state = 0;
  if (__ballot(!(own == own)) != 0ull) state = RF_FLAG_TRACK_RANGE;
  else if (__ballot(lane == 28 && own < (double)a.min_valid) != 0ull) state = RF_FLAG_TRACK_FEW_PIXELS;
  else if (__ballot(singular) != 0ull) state = RF_FLAG_TRACK_SINGULAR;
  const double tin[3] = {Tin[lane & 3], Tin[4 + (lane & 3)], Tin[8 + (lane & 3)]};
  double out = Tin[lane & 15];
  if (state == 0) {
    // exp of the twist (rho, phi) = x: R = I + A K + B K^2, t = (I + B K + C K^2) rho
    // with K v = phi x v, applied to the lane's column of the input pose
    const double p[3] = {x[3], x[4], x[5]};
    const double th2 = p[0] * p[0] + p[1] * p[1] + p[2] * p[2];
    double A, B, C;
    if (th2 < 1e-2) {
      // Taylor series of sin(th)/th, (1 - cos th)/th^2, (th - sin th)/th^3 in
      // th^2 (Horner); for th < 0.1 the first omitted term is below 1e-18
      A = fma(th2, fma(th2, fma(th2, fma(th2, fma(th2, -1.0 / 39916800.0, 1.0 / 362880.0), -1.0 / 5040.0),
                                1.0 / 120.0), -1.0 / 6.0), 1.0);
      B = fma(th2, fma(th2, fma(th2, fma(th2, fma(th2, -1.0 / 479001600.0, 1.0 / 3628800.0), -1.0 / 40320.0),
                                1.0 / 720.0), -1.0 / 24.0), 0.5);
      C = fma(th2, fma(th2, fma(th2, fma(th2, fma(th2, -1.0 / 6227020800.0, 1.0 / 39916800.0), -1.0 / 362880.0),
                                1.0 / 5040.0), -1.0 / 120.0), 1.0 / 6.0);
    } else {
      const double th = sqrt(th2), sn = sin(th), hs = sin(0.5 * th);
      A = sn / th;
      B = 2.0 * hs * hs / th2;
      C = (th - sn) / (th2 * th);
    }
    auto cross = [&](const double v[3], double o[3]) {
      o[0] = fma(p[1], v[2], -(p[2] * v[1]));
      o[1] = fma(p[2], v[0], -(p[0] * v[2]));
      o[2] = fma(p[0], v[1], -(p[1] * v[0]));
    };
    double c1[3], c2[3], d1[3], d2[3], o[3];
    cross(tin, c1);
    cross(c1, c2);
    cross(x, d1);  // x[0..2] = rho
    cross(d1, d2);
    const bool last = (lane & 3) == 3;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const double t = fma(C, d2[i], fma(B, d1[i], x[i]));
      o[i] = fma(B, c2[i], fma(A, c1[i], tin[i])) + (last ? t : 0.0);
    }
    out = lane < 4 ? o[0] : (lane < 8 ? o[1] : o[2]);
    if (lane >= 12) out = (lane == 15) ? 1.0 : 0.0;
  } else if (lane >= 12) {
    out = (lane == 15) ? 1.0 : 0.0;
  }
  if (lane < 16) s_T[lane] = out;
  if (s_Tf && lane < 12) s_Tf[lane] = (float)out;
  if (lane == 0) *s_state = state;
}

// What the solve reads from memory, asked for before the launch's other loads
// so that all of it takes one round trip.
template <bool LM>
struct SolveLoads {
  TermLoads terms;
  double pose;     // element lane mod 16 of the input pose (the candidate's)
  double st;       // Levenberg-Marquardt state
  int iters;       // the count that publishing adds to
};
template <bool LM>
__device__ __forceinline__ void solve_loads(const MapDev& m, double* user_pose, const TrackArgs& a,
                                            const rf_track_stats* stats, int lane, SolveLoads<LM>& L) {
  load_terms(acc_buf(m, a.acc_read), lane, L.terms);
  L.pose = pose_buf(m, user_pose, a.pose_read)[lane & 15];
  if (LM) L.st = lm_state(m, a.state_read)[lane < kLmWords ? lane : 0];
  L.iters = stats ? stats->iters : 0;
}

// The solve step shared by the tracking and finalize launches, run by the
// solving wavefront: reads the accumulated totals, solves, and (workgroup 0 only)
// publishes the pose, the statistics and, on a degenerate system, the stop
// flag.  Returns through LDS: s_T (new pose), *s_state.
//
// Levenberg-Marquardt (a.adaptive): the totals are those of the candidate
// pose the previous launch evaluated.  The first evaluation of a level is
// accepted as it is; a later one when it has at least min_valid residuals and
// a mean cost (cost / count) no larger than the accepted one's, which divides
// lambda by 10 (a rejection multiplies it by 10, at least 1e-4).  The step is
// then solved from the accepted pose and its normal equations; with
// final_only (the last decision of a pass) no step follows and the accepted
// pose is the result.  s_nc, s_st: LDS scratch of kLmWords doubles each.
template <bool LM>
__device__ __forceinline__ void solve_step(const MapDev& m, double* user_pose, const TrackArgs& a,
                                           rf_track_stats* stats, SolveLoads<LM>& L, double* s_ne, double* s_T,
                                           float* s_Tf, int* s_state, bool publish, bool stopped, bool final_only,
                                           double* s_nc, double* s_st) {
  const int lane = threadIdx.x & 63;
  const double* Tin = s_nc + kNE;
  double lam = a.lm_lambda;
  bool accept = true, first = true;
#pragma unroll
  for (int c = 0; c < kAccCopies / 2; ++c) asm volatile("" : "+v"(L.terms.acc[c].x), "+v"(L.terms.acc[c].y));
  asm volatile("" : "+v"(L.pose), "+v"(L.iters));
  const double tot = fixed_total(L.terms);
  if (!LM) {
    // the pose goes through LDS (fewer registers held across the solve)
    if (lane < 16) s_nc[kNE + lane] = L.pose;
    if (lane < kNE) s_ne[lane] = tot;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    asm volatile("" : "+v"(L.st));
    if (lane < kNE) s_nc[lane] = tot;
    if (lane < kLmWords) s_st[lane] = L.st;
    if (lane < 16) s_nc[kNE + lane] = L.pose;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    first = a.prev_first != 0;
    accept = first || (s_nc[28] >= (double)a.min_valid && s_nc[27] / s_nc[28] <= s_st[16 + 27] / s_st[16 + 28]);
    lam = s_st[45];
    if (!first) lam = accept ? lam / 10.0 : fmax(lam * 10.0, 1e-4);
    if (lane < kNE) s_ne[lane] = accept ? s_nc[lane] : s_st[16 + lane];
    if (!accept) Tin = s_st;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (final_only) {
    if (lane < 16) s_T[lane] = Tin[lane];
    if (lane == 0) *s_state = 0;
  } else {
    TrackArgs ta = a;
    ta.lm_lambda = lam;
    solve_update_wave(s_ne, ta, Tin, s_T, s_Tf, s_state);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (!publish || stopped) return;
  const int state = *s_state;
  if (lane < 16) {
    double* Tout = pose_buf(m, user_pose, a.pose_write);
    Tout[lane] = s_T[lane];
    if (state != 0 && a.pose_write != 2) pose_buf(m, user_pose, 1 - a.pose_write)[lane] = s_T[lane];
  }
  if (LM && a.state_write >= 0) {
    double* S = lm_state(m, a.state_write);
    if (lane < 16) S[lane] = Tin[lane];
    if (lane < kNE) S[16 + lane] = s_ne[lane];
    if (lane == 0) S[45] = lam;
  }
  if (lane == 0) {
    if (stats) {
      stats->cost = s_ne[27];
      stats->count = s_ne[28];
      if (a.prev_first && a.prev_level >= 0 && a.prev_level < 8)
        stats->level_count[a.prev_level] = LM ? s_nc[28] : s_ne[28];
      if (state != 0) stats->flags |= (uint32_t)state;
      else if (LM ? (accept && !first) : !final_only) stats->iters = L.iters + 1;
    }
    if (state != 0) {
      m.st->track_stop = 1;
      atomicOr(&m.st->flags, (uint32_t)state);
    }
  }
}

// Per-workgroup block cache in LDS: a direct-mapped window of win^3 blocks
// centred on the bounding box of the tile's cached blocks (one indexed read,
// no key to compare) and, for blocks outside it, a small open-addressing
// hash (linear probing).  Built from the tile's cached pairs before the first
// barrier, consulted before the hash table, extended with every pair the hash
// table resolves, and written back (the pairs used in this launch) for the
// next launch at this level and tile.  A slot still being written reads as
// kNoSlot, which a lookup treats as a miss, so concurrent inserts never
// yield a wrong slot.
constexpr int kNoSlot = (int)0x80000000;
constexpr int kMaxProbe = 8;   // a key is placed within 8 slots of its home or not cached
// Direct-mapped window of win^3 blocks around the tile's blocks.  A tile of the
// coarsest levels (64 pixels of a 640-pixel row and more) is up to 11 blocks wide at
// 0.5 cm; with 8 most of its lookups went on to the LDS hash and the table:
// with 16 a 640x480 step takes 965 us instead of 996 at 0.5 cm, 746 instead of
// 775 at 1 cm.  The finer levels' tiles fit 8, which clears faster.  Coarse
// voxels would fit 8 too, for little: a registration of 640x480 over four levels
// takes 344 us with 8 and 348 with 16 at 2 cm (160x120 285 both, 320x240 294 and
// 297), 355 both at 1.4 cm, but 481 and 398 at 1 cm, 534 and 455 at 0.6 cm.
__host__ __device__ constexpr int win_of(int slots) { return slots >= 512 ? 16 : 8; }
constexpr int kFarOrigin = 0x40000000;  // window origin that no block coordinate reaches

// SLOTS: LDS hash capacity (the tile's pair capacity at the launch's level).
template <int SLOTS>
struct TileCache {
  static constexpr int kWin = win_of(SLOTS);
  unsigned long long* key;  // SLOTS, kEmptyKey when free
  int* slot;                // SLOTS, kNoSlot until written
  uint8_t* used;            // SLOTS, 1 when looked up in this launch
  int* grid;                // kWin^3 window of block slots (kNoSlot: unknown)
  uint8_t* gused;           // kWin^3, 1 when looked up in this launch
  int* miss;                // set when a lookup went to the hash table
  int ax, ay, az;           // window origin (block coordinates)

  // window cell of block (x,y,z), or -1 outside the window
  __device__ __forceinline__ int cell(int x, int y, int z) const {
    const uint32_t dx = (uint32_t)(x - ax), dy = (uint32_t)(y - ay), dz = (uint32_t)(z - az);
    return (dx < (uint32_t)kWin && dy < (uint32_t)kWin && dz < (uint32_t)kWin) ? (int)(dx + kWin * (dy + kWin * dz)) : -1;
  }

  __device__ __forceinline__ void insert(int x, int y, int z, unsigned long long k, int sl, bool mark) const {
    uint32_t h = hash3(x, y, z) & (SLOTS - 1);
#pragma unroll 1
    for (int i = 0; i < kMaxProbe; ++i) {
      const unsigned long long old = atomicCAS(&key[h], kEmptyKey, k);
      if (old == kEmptyKey) {
        slot[h] = sl;
        if (mark) used[h] = 1;
        return;
      }
      if (old == k) {
        if (mark) used[h] = 1;
        return;
      }
      h = (h + 1) & (SLOTS - 1);
    }
  }

  __device__ __forceinline__ int find(int x, int y, int z, unsigned long long k) const {
    uint32_t h = hash3(x, y, z) & (SLOTS - 1);
#pragma unroll 1
    for (int i = 0; i < kMaxProbe; ++i) {
      const unsigned long long kk = key[h];
      if (kk == k) {
        const int sl = slot[h];
        if (sl != kNoSlot) used[h] = 1;
        return sl;
      }
      if (kk == kEmptyKey) break;
      h = (h + 1) & (SLOTS - 1);
    }
    return kNoSlot;
  }
};

// Slot resolution of sample_map through the tile cache: cached blocks cost
// an LDS probe; the others take the hash table (first probes of all missing
// corner blocks issued together) and are added to the cache.
//
// Almost every lookup finds all its corner blocks in the window, and those take
// eight reads at the corners' own cells: no key, no comparison, no choice among
// the distinct blocks' slots.  Their window cells are marked as used only when
// the tile's cache is written back (mark: the lower corner's cell, with the
// crossed block faces from bit 12; -1 without a lookup to mark), since most
// launches don't.  A lookup of separate tests per corner took 2700 of a
// workgroup's 18000 cycles.
template <int SLOTS>
struct CachedSlots {
  static constexpr int kWin = win_of(SLOTS);
  TileCache<SLOTS> c;
  int* mark;
  __device__ __forceinline__ bool operator()(const MapDev& m, int bx0, int by0, int bz0, int cross, int sl[8]) const {
    const uint32_t dx = (uint32_t)(bx0 - c.ax), dy = (uint32_t)(by0 - c.ay), dz = (uint32_t)(bz0 - c.az);
    const uint32_t ox = cross & 1, oy = (cross >> 1) & 1, oz = cross >> 2;
    static_assert((kWin & (kWin - 1)) == 0, "one test for all coordinates");
    const bool in = (dx | dy | dz | (dx + ox) | (dy + oy) | (dz + oz)) < (uint32_t)kWin;
    const int* g = c.grid + (in ? dx + kWin * (dy + kWin * dz) : 0u);
    const uint32_t ix = in ? ox : 0u, iy = in ? kWin * oy : 0u, iz = in ? kWin * kWin * oz : 0u;
#pragma unroll
    for (int k = 0; k < 8; ++k) sl[k] = g[(k & 1 ? ix : 0u) + (k & 2 ? iy : 0u) + (k & 4 ? iz : 0u)];
    int least = sl[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) least = min(least, sl[k]);
    if (in && least != kNoSlot) {  // kNoSlot is the lowest value
      *mark = (int)(g - c.grid) | cross << 12;
    } else {
      general(m, bx0, by0, bz0, cross, sl);
    }
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 8; ++k) ok &= sl[k] != -1;  // absent; free blocks (<= -2) read as (tau, count)
    return ok;
  }
  // blocks outside the window or not known yet
  __device__ __forceinline__ void general(const MapDev& m, int bx0, int by0, int bz0, int cross, int sl[8]) const {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      sl[k] = kNoSlot;
      if ((k & ~cross) != 0) continue;
      const int x = bx0 + (k & 1), y = by0 + ((k >> 1) & 1), z = bz0 + (k >> 2);
      const int cl = c.cell(x, y, z);
      if (cl >= 0) {
        sl[k] = c.grid[cl];
        if (sl[k] != kNoSlot) c.gused[cl] = 1;
      } else {
        sl[k] = c.find(x, y, z, pack_key(x, y, z));
      }
    }
    unsigned long long bkey[8];
    uint32_t bslot[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if ((k & ~cross) != 0 || sl[k] != kNoSlot) continue;
      const int x = bx0 + (k & 1), y = by0 + ((k >> 1) & 1), z = bz0 + (k >> 2);
      const Bucket* p = m.buckets + (hash3(x, y, z) & m.bucket_mask);
      bkey[k] = p->key;
      bslot[k] = p->slot;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if ((k & ~cross) != 0 || sl[k] != kNoSlot) continue;
      const int x = bx0 + (k & 1), y = by0 + ((k >> 1) & 1), z = bz0 + (k >> 2);
      Bucket b0;
      b0.key = bkey[k];
      b0.slot = bslot[k];
      const unsigned long long key = pack_key(x, y, z);
      sl[k] = resolve_slot(m, b0, key, hash3(x, y, z) & m.bucket_mask);
      *c.miss = 1;
      const int cl = c.cell(x, y, z);
      if (cl >= 0) {
        c.grid[cl] = sl[k];
        c.gused[cl] = 1;
      } else {
        c.insert(x, y, z, key, sl[k], true);
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if ((k & ~cross) != 0) sl[k] = sl[k & cross];
  }
};

// Marks the window cells of a lookup (CachedSlots::mark) as used.
template <int WIN>
__device__ __forceinline__ void mark_used(uint8_t* gused, int mark) {
  if (mark < 0) return;
  const int cl = mark & 4095, cross = mark >> 12;
  static_assert(WIN * WIN * WIN <= 4096, "cell and faces fit 15 bits");
#pragma unroll
  for (int k = 0; k < 8; ++k)
    gused[cl + (k & cross & 1) + WIN * ((k & cross) >> 1 & 1) + WIN * WIN * ((k & cross) >> 2)] = 1;
}

// LDS of a tile's cache and the wavefront that fills it: the tile's cached
// block pairs (tiles without a cache entry start from an empty table) placed
// in the direct-mapped window or in the LDS hash.  Entry 0 of a tile's pairs
// holds the window's origin, set when the pairs were written.
template <int SLOTS>
struct CacheLds {
  static constexpr int kWin = win_of(SLOTS), kWinCells = kWin * kWin * kWin;
  alignas(16) unsigned long long hk[SLOTS];
  alignas(16) int hs[SLOTS];
  alignas(16) uint8_t used[SLOTS];
  alignas(16) int grid[kWinCells];
  alignas(16) uint8_t gused[kWinCells];
  int org[3];
  int miss;
  int cnt;               // pairs loaded
  uint32_t nref;         // pairs written back
  uint32_t cells[2];     // their bounding box: the window's x and y, and z, in use (16 bits each),
  int lo[3], hi[3];      // and the blocks outside the window

  __device__ __forceinline__ TileCache<SLOTS> cache(int ax, int ay, int az) {
    return TileCache<SLOTS>{hk, hs, used, grid, gused, &miss, ax, ay, az};
  }
};

template <int SLOTS>
__device__ __forceinline__ void build_tile_cache(const BlockRef* tab, const uint32_t* tcount, bool cached, int nrefs,
                                                 uint32_t epoch, int lane, CacheLds<SLOTS>& L) {
  const BlockRef none{kEmptyKey, -1, 0u};
  constexpr int kLoads = SLOTS / 64;
  constexpr int kWinCells = CacheLds<SLOTS>::kWinCells;
  const int cnt = cached ? (int)min(*tcount, (uint32_t)(nrefs - 1)) : 0;
  BlockRef e[kLoads];
#pragma unroll
  for (int q = 0; q < kLoads; ++q) e[q] = (cached && lane + 64 * q < nrefs) ? tab[lane + 64 * q] : none;
  // clear with the widest stores
#pragma unroll
  for (int q = 0; q < SLOTS / 128; ++q)
    reinterpret_cast<ulonglong2*>(L.hk)[lane + 64 * q] = make_ulonglong2(kEmptyKey, kEmptyKey);
#pragma unroll
  for (int q = 0; q < SLOTS / 256; ++q) {
    reinterpret_cast<int4*>(L.hs)[lane + 64 * q] = make_int4(kNoSlot, kNoSlot, kNoSlot, kNoSlot);
    reinterpret_cast<uint32_t*>(L.used)[lane + 64 * q] = 0u;
  }
#pragma unroll
  for (int q = 0; q < kWinCells / 256; ++q) {
    reinterpret_cast<int4*>(L.grid)[lane + 64 * q] = make_int4(kNoSlot, kNoSlot, kNoSlot, kNoSlot);
    reinterpret_cast<uint32_t*>(L.gused)[lane + 64 * q] = 0u;
  }
  // the window's origin (entry 0)
  int org[3];
  unpack_key(((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(e[0].key >> 32)) << 32) |
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)e[0].key),
             org[0], org[1], org[2]);
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (cnt == 0) org[d] = kFarOrigin;
  if (lane == 0) {
    L.miss = 0;
    L.cnt = cnt;
    L.nref = L.cells[0] = L.cells[1] = 0u;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      L.org[d] = org[d];
      L.lo[d] = INT_MAX;
      L.hi[d] = INT_MIN;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const TileCache<SLOTS> wc = L.cache(org[0], org[1], org[2]);
#pragma unroll
  for (int q = 0; q < kLoads; ++q) {
    const int i = lane + 64 * q;
    if (!(i >= 1 && i <= cnt && e[q].key != kEmptyKey && (e[q].slot >= 0 || e[q].epoch == epoch))) continue;
    int p[3];
    unpack_key(e[q].key, p[0], p[1], p[2]);
    const int cl = wc.cell(p[0], p[1], p[2]);
    if (cl >= 0) L.grid[cl] = e[q].slot;
    else wc.insert(p[0], p[1], p[2], e[q].key, e[q].slot, false);
  }
}

// The pairs used in this launch become the tile's cache for the next one, and
// the centre of their bounding box its window's.  Called by the whole workgroup
// after a lookup missed; otherwise the cache stays as it is, which spares most
// launches the pass over the window, and every launch the search for the
// window's place that used to come before the pairs were placed.
template <int SLOTS>
__device__ __forceinline__ void write_tile_cache(BlockRef* tab, uint32_t* tcount, int nrefs, uint32_t epoch,
                                                 CacheLds<SLOTS>& L) {
  constexpr int kWin = CacheLds<SLOTS>::kWin, kWinCells = CacheLds<SLOTS>::kWinCells;
  const int lane = threadIdx.x & 63;
  // one position counter atomic per wavefront
  auto keep = [&](bool yes, unsigned long long key, int slot) {
    const unsigned long long bal = __ballot(yes);
    if (bal == 0ull) return;  // uniform
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&L.nref, (uint32_t)__popcll(bal));
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + 1u;
    const uint32_t pos =
        base + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
    if (yes && pos < (uint32_t)nrefs) tab[pos] = BlockRef{key, slot, epoch};
  };
  // Pairs not used in this launch stay too while the tile has few: the steps of
  // a registration come by the same blocks in the next one.  Those in the
  // window stay below half of the room; those outside are costlier to place
  // (the LDS hash), and a tile of the coarsest level at 0.5 cm has up to 230, so
  // they stay below a quarter.  640x480 at 1 cm / 0.5 cm, whole frame: none kept
  // 954 / 1216 us, all below half 929 / 1280, window only 948 / 1205, this rule
  // 933 / 1202.
  const bool all = 2 * L.cnt < nrefs, few = 4 * L.cnt < nrefs;
  static_assert(kWinCells % kTrackBlock == 0, "the walk over the window ends with it");
  // the window's cells in use, a bit per x, y and z
  uint32_t cells[2] = {0u, 0u};
#pragma unroll
  for (int q = 0; q < kWinCells / kTrackBlock; ++q) {
    const int h = threadIdx.x + q * kTrackBlock;
    const int ss = L.grid[h], x = h % kWin, y = (h / kWin) % kWin, z = h / (kWin * kWin);
    const bool yes = ss != kNoSlot && L.gused[h];
    keep(yes || (all && ss != kNoSlot), pack_key(L.org[0] + x, L.org[1] + y, L.org[2] + z), ss);
    if (yes) {
      cells[0] |= 1u << x | 65536u << y;
      cells[1] |= 1u << z;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    cells[0] |= (uint32_t)__shfl_xor((int)cells[0], o);
    cells[1] |= (uint32_t)__shfl_xor((int)cells[1], o);
  }
  if (lane == 0 && cells[1]) {
    atomicOr(&L.cells[0], cells[0]);
    atomicOr(&L.cells[1], cells[1]);
  }
  for (int h0 = 0; h0 < SLOTS; h0 += kTrackBlock) {
    // every lane takes part in keep(); with more threads than slots those
    // beyond the hash have nothing
    const bool in = SLOTS % kTrackBlock == 0 || h0 + (int)threadIdx.x < SLOTS;
    const int h = in ? h0 + threadIdx.x : 0;
    const unsigned long long kk = L.hk[h];
    const int ss = L.hs[h];
    const bool known = in && kk != kEmptyKey && ss != kNoSlot, yes = known && L.used[h];
    keep(yes || (few && known), kk, ss);
    const unsigned long long bal = __ballot(yes);
    if (bal == 0ull) continue;  // uniform
    // their bounding box, relative to one of them (16 bits are plenty: it only
    // centres a window): the minimum of d and of -d together
    typedef short short2v __attribute__((ext_vector_type(2)));
    const int first = __ffsll((long long)bal) - 1;
    int p[3];
    unpack_key(kk, p[0], p[1], p[2]);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int ref = __builtin_amdgcn_readlane(p[d], first);
      const int off = yes ? max(-32767, min(32767, p[d] - ref)) : 0;
      short2v v = {(short)off, (short)-off};
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const int w = __shfl_xor(__builtin_bit_cast(int, v), o);
        v = __builtin_elementwise_min(v, __builtin_bit_cast(short2v, w));
      }
      if (lane == 0) {
        atomicMin(&L.lo[d], ref + v.x);
        atomicMax(&L.hi[d], ref - v.y);
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t n = min(L.nref, (uint32_t)(nrefs - 1));
    *tcount = n;
    int org[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const uint32_t c = (L.cells[d >> 1] >> (d == 1 ? 16 : 0)) & 0xFFFFu;
      const int lo = min(L.lo[d], c ? L.org[d] + __ffs((int)c) - 1 : INT_MAX);
      const int hi = max(L.hi[d], c ? L.org[d] + 31 - __clz((int)c) : INT_MIN);
      org[d] = n ? ((lo + hi) >> 1) - (kWin / 2 - 1) : 0;
    }
    tab[0] = BlockRef{pack_key(org[0], org[1], org[2]), 0, epoch};
  }
}

// Normal-equation sums of a wavefront.  Each lane forms the 28 products of its
// pixel in FP64 (products of FP32 factors are exact; the 29th term, the count,
// is a ballot), and the wavefront adds them up by exchanging halves: a step
// over lane bit b gives half of the terms to the lanes with the bit set and
// half to the others, adding the partner's, so 28 terms take 14 + 7 + 4 + 2 + 1
// additions (and one plain one) instead of 28 x 6.  The last lane bit is
// summed plainly, so pairs of lanes end with the same term.  Parking the
// factors in LDS for 232 threads to sum took 116 LDS reads a pixel and a second
// barrier: registration of 160x120 229 -> 212 us, 640x480 454 -> 432 us, eight
// mixed sessions a step 3145 -> 3069 us.
__device__ __forceinline__ void f64_words(double v, uint32_t& lo, uint32_t& hi) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  lo = (uint32_t)b;
  hi = (uint32_t)(b >> 32);
}
__device__ __forceinline__ double f64_of(uint32_t lo, uint32_t hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// a in the lower 32 lanes plus a in the upper ones (lower lanes), likewise b
// (upper lanes); ROWS: the same between the even and odd rows of 16 lanes.
template <bool ROWS>
__device__ __forceinline__ double swap_add(double a, double b) {
  uint32_t al, ah, bl, bh;
  f64_words(a, al, ah);
  f64_words(b, bl, bh);
  if constexpr (ROWS) {
    const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return f64_of(l[0], h[0]) + f64_of(l[1], h[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return f64_of(l[0], h[0]) + f64_of(l[1], h[1]);
  }
}
// The value of the lane that DPP control CTRL pairs with this one.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  uint32_t lo, hi;
  f64_words(v, lo, hi);
  lo = __builtin_amdgcn_update_dpp(0u, lo, CTRL, 0xF, 0xF, false);
  hi = __builtin_amdgcn_update_dpp(0u, hi, CTRL, 0xF, 0xF, false);
  return f64_of(lo, hi);
}
// a over both lanes of a pair for the lanes with bit clear, b for the others;
// CTRL pairs every lane with one whose bit differs.
template <int CTRL>
__device__ __forceinline__ double pair_add(double a, double b, bool bit) {
  const double keep = bit ? b : a, send = bit ? a : b;
  return keep + dpp_f64<CTRL>(send);
}
constexpr int kRowMirror = 0x140, kHalfMirror = 0x141, kQuadHalves = 0x4E, kQuadPairs = 0xB1;

// Packed upper triangle: row and column of H's term k < 21.
__host__ __device__ constexpr int ne_row(int k) { return k < 6 ? 0 : (k < 11 ? 1 : (k < 15 ? 2 : (k < 18 ? 3 : (k < 20 ? 4 : 5)))); }
__host__ __device__ constexpr int ne_col(int k) {
  return k - (6 * ne_row(k) - (ne_row(k) * (ne_row(k) - 1)) / 2) + ne_row(k);
}

// The wavefront's sum of one term for every lane: term index in *k (28 and
// over: none).  t: J_d(6) J_c(6) r_d r_c of the lane's pixel, zeros without one.
__device__ __forceinline__ double wave_sums(const float t[14], double w_c, int lane, int* k) {
  double d[7], c[7];  // J and the residual
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    d[i] = (double)t[i < 6 ? i : 12];
    c[i] = (double)t[i < 6 ? 6 + i : 13];
  }
  // term q: H (21), g (6), cost; row by row, so that few values are live at once
  auto term = [&](int q) {
    const int r = q < 21 ? ne_row(q) : (q < 27 ? q - 21 : 6), l = q < 21 ? ne_col(q) : 6;
    return fma(w_c * c[r], c[l], d[r] * d[l]);
  };
  double b[8];
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    const double a0 = swap_add<false>(term(4 * i), term(4 * i + 1)), a1 = swap_add<false>(term(4 * i + 2), term(4 * i + 3));
    b[i] = swap_add<true>(a0, a1);
  }
  b[7] = 0.0;
  const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
  double e[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) e[i] = pair_add<kRowMirror>(b[2 * i], b[2 * i + 1], b3);
  const double g0 = pair_add<kHalfMirror>(e[0], e[1], b2), g1 = pair_add<kHalfMirror>(e[2], e[3], b2);
  double v = pair_add<kQuadHalves>(g0, g1, b1);
  v += dpp_f64<kQuadPairs>(v);
  // undo the halvings: bit 5 picked the lowest bit of the index, then 4, 3, 2, 1
  *k = ((lane >> 5) & 1) | ((lane >> 4) & 1) << 1 | ((lane >> 3) & 1) << 2 | ((lane >> 2) & 1) << 3 | ((lane >> 1) & 1) << 4;
  return v;
}

// SLOTS: pairs the tile cache holds in LDS (256 at levels 0-1, 512 at the
// coarser levels, whose few tiles each touch more blocks; more LDS and
// registers there cost nothing, since those launches have few workgroups).
// SOLVE: the launch solves the previous evaluation's system at its start if asked
// to (kSeparateSolveTiles); one that never does keeps 6 wavefronts a SIMD.
// ONE: a batch of one job, whose arguments are then asked for at once instead
// of after the search for the workgroup's job.
//
// What bounds a launch of few workgroups is its chain: arguments, totals, solve,
// corner slots, corner records, sums, atomics.  With the totals asked for
// before the pixels, the solve by every lane and single-job arguments a
// registration of 160x120 (20 launches) takes 152 us instead of 184, of 640x480
// (30) 330 instead of 383.
template <int DF, int STORAGE, bool LM, int SLOTS, bool SOLVE, bool ONE>
__global__ __launch_bounds__(kTrackBlock, SOLVE ? 5 : 6) void track_kernel(Batch b, TrackArgs a) {
  __shared__ double s_g[kTrackBlock / 64][kNE];  // per wavefront: its sums of the terms
  __shared__ double s_ne[kNE];
  __shared__ double s_nc[kLmWords];
  __shared__ double s_st[kLmWords];
  __shared__ double s_T[16];
  __shared__ alignas(16) float s_Tf[12];  // the pose as the pixels use it
  __shared__ int s_state;
  __shared__ uint16_t s_mark[kTrackBlock];       // per thread: its lookup's window cells
  __shared__ CacheLds<SLOTS> s_cache;
  const int jb = ONE ? 0 : batch_job(b, blockIdx.x);
  const Job& J = b.job[jb];
  const MapDev& m = J.m;
  const FrameDev& f = J.f;
  const uint8_t* mask = J.mask;
  double* user_pose = J.pose;
  rf_track_stats* stats = J.stats;
  const int g0 = ONE ? (int)blockIdx.x : (int)blockIdx.x - b.base[jb];  // tile index within the job
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // the solving wavefront (and the cache builder after it) rotate with the
  // tile index, so the solves of the workgroups sharing a CU spread over its
  // SIMDs
  const int sw = g0 & 3, cw = (sw + 1) & 3;
  SolveLoads<LM> solve_in;
  if (SOLVE && wave == sw && a.solve) solve_loads<LM>(m, user_pose, a, stats, lane, solve_in);
  // Set only by earlier launches.  Read here but acted on after the pixel
  // loads and the solve are under way: only publishing waits for it.
  const uint32_t stopped = m.st->track_stop;
  const uint32_t epoch = m.st->epoch;

  // pose-independent loads first, so their latency overlaps the solve
  // workgroup = kTileW x 16 tile of the level's pixel grid, wavefront = 8x8 sub-tile
  const int lv = a.level;
  const int wl = (f.W + (1 << lv) - 1) >> lv;
  const int hl = (f.H + (1 << lv) - 1) >> lv;
  const int tiles_x = (wl + kTileW - 1) / kTileW;
  const int ul = (g0 % tiles_x) * kTileW + (wave % (kTileW / 8)) * 8 + (lane & 7);
  const int vl = (g0 / tiles_x) * 16 + (wave / (kTileW / 8)) * 8 + (lane >> 3);
  // Depth, mask and colour are loaded without a branch (pixels outside the
  // level read pixel 0; a missing mask reads the colour plane) so the loads
  // share one round trip and are first used after the solve.
  const bool inside = ul < wl && vl < hl;
  const int u = inside ? ul << lv : 0, v = inside ? vl << lv : 0;
  const int pix = v * f.W + u;
  const float D = load_depth<DF>(f, pix);
  const uint8_t mk_raw = (mask ? mask : f.rgb)[pix];
  const uint8_t* px = f.rgb + 3 * pix;
  const uint8_t c0 = px[0], c1 = px[1], c2 = px[2];
  if (a.acc_clear >= 0) {
    // the workgroups of the job share the clearing of the used chunk pairs
    const int q = g0 + (int)threadIdx.x * (b.base[jb + 1] - b.base[jb]);
    if (q < kUsedPairs) *used_pair(acc_buf(m, a.acc_clear), q) = make_ulonglong2(0ull, 0ull);
  }
  // the tile's cached block pairs (the wavefront after the solving one,
  // while it solves); tiles without a cache entry start from an empty table
  const bool cached = a.level < kCacheLevels && g0 < (int)m.tc_tiles;
  BlockRef* tab = m.tcache + (size_t)m.tc_tiles * tile_refs_before(cached ? a.level : 0) +
                  (size_t)(cached ? g0 : 0) * tile_refs(cached ? a.level : 0);
  uint32_t* tcount = m.tc_count + (size_t)(cached ? a.level : 0) * m.tc_tiles + (cached ? g0 : 0);
  const int nrefs = tile_refs(a.level);
  if (wave == cw) build_tile_cache<SLOTS>(tab, tcount, cached, nrefs, epoch, lane, s_cache);
  if (wave == sw) {
    if (SOLVE && a.solve) {
      solve_step<LM>(m, user_pose, a, stats, solve_in, s_ne, s_T, s_Tf, &s_state, g0 == 0, stopped != 0, false, s_nc, s_st);
    } else {
      const double* Tin = pose_buf(m, user_pose, a.pose_read);
      if (lane < 16) {
        if (lane < 12) s_Tf[lane] = (float)Tin[lane];
        if (g0 == 0 && !stopped && a.pose_write >= 0) pose_buf(m, user_pose, a.pose_write)[lane] = Tin[lane];
      }
      if (LM && g0 == 0 && !stopped && a.state_write >= 0) {
        // the starting pose is the accepted one until the first decision
        double* S = lm_state(m, a.state_write);
        if (lane < 16) S[lane] = Tin[lane];
        if (lane == 0) S[45] = a.lm_lambda;
      }
      if (lane == 0) s_state = 0;
    }
  }
  __syncthreads();
  if (stopped || s_state != 0) return;  // stopped or degenerate: pose kept, the pass stops
  const TileCache<SLOTS> cache = s_cache.cache(s_cache.org[0], s_cache.org[1], s_cache.org[2]);

  float term[kTerms];  // J_d(6) J_c(6) r_d r_c
  bool counts = false;
  int mark = -1;
#pragma unroll
  for (int k = 0; k < kTerms; ++k) term[k] = 0.0f;
  if (inside && depth_ok(D, m.dmax) && !(mask && mk_raw)) {
    const float Ipix = luminance((float)c0, (float)c1, (float)c2);
    float R[9], t[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
      for (int c = 0; c < 3; ++c) R[3 * r + c] = s_Tf[4 * r + c];
      t[r] = s_Tf[4 * r + 3];
    }
    const float x[3] = {(((float)u - f.cx) * f.ifx) * D, (((float)v - f.cy) * f.ify) * D, D};
    float y[3];
    xform(R, t, x, y);
    float S, gS[3], Iv, gI[3];
    if (sample_map<STORAGE, true, true>(m, y, S, gS, Iv, gI, CachedSlots<SLOTS>{cache, &mark}) && fabsf(S) < m.tau) {
      term[0] = gS[0];
      term[1] = gS[1];
      term[2] = gS[2];
      term[3] = y[1] * gS[2] - y[2] * gS[1];
      term[4] = y[2] * gS[0] - y[0] * gS[2];
      term[5] = y[0] * gS[1] - y[1] * gS[0];
      term[6] = gI[0];
      term[7] = gI[1];
      term[8] = gI[2];
      term[9] = y[1] * gI[2] - y[2] * gI[1];
      term[10] = y[2] * gI[0] - y[0] * gI[2];
      term[11] = y[0] * gI[1] - y[1] * gI[0];
      term[12] = S;
      term[13] = Iv - Ipix;
      counts = true;
    }
  }
  s_mark[threadIdx.x] = (uint16_t)mark;
  {
    int k;
    const double v = wave_sums(term, (double)a.w_c, lane, &k);
    const unsigned long long cb = __ballot(counts);
    if (!(lane & 1) && k < 28) s_g[wave][k] = v;
    if (lane == 0) s_g[wave][28] = (double)__popcll(cb);
  }
  __syncthreads();
  if (threadIdx.x < kNE) {
    double tot = 0.0;
#pragma unroll
    for (int w = 0; w < kTrackBlock / 64; ++w) tot += s_g[w][threadIdx.x];
    if (!fixed_add(acc_buf(m, a.acc_write) + (g0 % kAccCopies) * kCopyWords + threadIdx.x * kTermWords, tot)) {
      atomicOr(&m.st->flags, (uint32_t)RF_FLAG_TRACK_RANGE);
      if (stats) atomicOr(&stats->flags, (uint32_t)RF_FLAG_TRACK_RANGE);
    }
  }
  if (cached && s_cache.miss) {  // uniform
    mark_used<win_of(SLOTS)>(s_cache.gused, (int16_t)s_mark[threadIdx.x]);
    __syncthreads();
    write_tile_cache<SLOTS>(tab, tcount, nrefs, epoch, s_cache);
  }
}

// Residual of the dynamic mask (Sec. III-C): r = S(T x)^2 of every valid
// pixel at full resolution and the raw decision r > gamma tau^2, with the
// pixels in the 16x16 tiles of the finest tracking level so that the corner
// blocks resolve through that level's tile cache (the pairs the last
// registration at this level used; a tile without them starts empty).  The
// cache only replaces hash-table probes, so the result is that of plain
// lookups.
template <int DF, int STORAGE, int SLOTS>
__global__ __launch_bounds__(kTrackBlock) void residual_kernel(Batch b, float gamma) {
  __shared__ CacheLds<SLOTS> s_cache;
  const int jb = batch_job(b, blockIdx.x);
  const Job& J = b.job[jb];
  const MapDev& m = J.m;
  const FrameDev& f = J.f;
  const int g0 = blockIdx.x - b.base[jb];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int tiles_x = (f.W + kTileW - 1) / kTileW;
  const int u = (g0 % tiles_x) * kTileW + (wave % (kTileW / 8)) * 8 + (lane & 7);
  const int v = (g0 / tiles_x) * 16 + (wave / (kTileW / 8)) * 8 + (lane >> 3);
  const bool inside = u < f.W && v < f.H;
  const int pix = inside ? v * f.W + u : 0;
  const float D = load_depth<DF>(f, pix);
  const bool cached = g0 < (int)m.tc_tiles;
  const BlockRef* tab = m.tcache + (size_t)(cached ? g0 : 0) * tile_refs(0);
  const uint32_t* tcount = m.tc_count + (cached ? g0 : 0);
  if (wave == 1)
    build_tile_cache<SLOTS>(tab, tcount, cached, tile_refs(0), m.st->epoch, lane, s_cache);
  __syncthreads();
  const TileCache<SLOTS> cache = s_cache.cache(s_cache.org[0], s_cache.org[1], s_cache.org[2]);
  uint8_t out = 0;
  float r = -1.0f;
  if (inside && depth_ok(D, m.dmax)) {
    float R[9], t[3];
    load_pose_f(J.pose, R, t);
    const float x[3] = {(((float)u - f.cx) * f.ifx) * D, (((float)v - f.cy) * f.ify) * D, D};
    float y[3];
    xform(R, t, x, y);
    float S, Iv, g3[3], h3[3];
    int mark;  // nothing is written back
    // a tile without pairs (a map that has not tracked at this level; never in a
    // frame, whose mask follows a registration) has nothing to gain from filling
    // a cache that is not kept: 640x480 18.0 us through it, 12.9 without;
    // 1280x720 31 and 22.8; with its pairs 8.8
    const bool defined = s_cache.cnt != 0 ? sample_map<STORAGE, false, false>(m, y, S, g3, Iv, h3,
                                                                            CachedSlots<SLOTS>{cache, &mark})
                                          : sample_map<STORAGE, false, false>(m, y, S, g3, Iv, h3);
    if (defined) {
      r = S * S;
      out = (r > gamma * (m.tau * m.tau)) ? 1 : 0;
    }
  }
  if (inside) {
    (J.raw ? J.raw : J.mask_out)[pix] = out;
    if (J.residual) J.residual[pix] = r;
  }
}

// Solve of the last evaluation of a pass (mode 0), the raw totals (mode 1),
// or, for launches with many workgroups, the solve a tracking launch would
// otherwise run at its start (mode 2): one workgroup per job.
__global__ __launch_bounds__(64) void track_finalize_kernel(Batch b, TrackArgs a, double* out29) {
  __shared__ double s_ne[kNE];
  __shared__ double s_nc[kLmWords];
  __shared__ double s_st[kLmWords];
  __shared__ double s_T[16];
  __shared__ int s_state;
  const Job& J = b.job[blockIdx.x];
  const MapDev& m = J.m;
  double* user_pose = J.pose;
  if (a.mode == 1) {
    TermLoads L;
    load_terms(acc_buf(m, a.acc_read), threadIdx.x, L);
    const double tot = fixed_total(L);
    if (threadIdx.x < kNE) out29[threadIdx.x] = tot;
    return;
  }
  if (m.st->track_stop) {
    // stopped earlier: both scratch poses hold the last good pose
    if (a.mode == 0 && threadIdx.x < 16) user_pose[threadIdx.x] = pose_buf(m, user_pose, a.pose_read)[threadIdx.x];
    return;
  }
  // mode 2: the solve a tracking launch would run at its start, once per job
  const bool final_only = a.mode != 2;
  auto solve = [&](auto lm) {
    constexpr bool LM = decltype(lm)::value;
    SolveLoads<LM> L;
    solve_loads<LM>(m, user_pose, a, J.stats, threadIdx.x, L);
    solve_step<LM>(m, user_pose, a, J.stats, L, s_ne, s_T, nullptr, &s_state, true, false, LM && final_only, s_nc, s_st);
  };
  if (a.adaptive) solve(std::true_type{});
  else solve(std::false_type{});
}

__global__ void track_reset_kernel(Batch b) {
  const Job& J = b.job[blockIdx.x];
  for (int bi = 0; bi < 3; ++bi) {
    unsigned long long* acc = acc_buf(J.m, bi);
    for (int q = threadIdx.x; q < kUsedPairs; q += blockDim.x) *used_pair(acc, q) = make_ulonglong2(0ull, 0ull);
  }
  if (threadIdx.x == 0) {
    J.m.st->track_stop = 0;
    J.m.st->track_counter = 0;
    rf_track_stats* stats = J.stats;
    if (stats) {
      stats->cost = 0.0;
      stats->count = 0.0;
      stats->iters = 0;
      stats->flags = 0;
      for (int l = 0; l < 8; ++l) stats->level_count[l] = 0.0;
    }
  }
}

// Tracking levels whose launches have more workgroups than this (all jobs
// together; two resident rounds of the chip) solve in a launch of their own,
// once per job, instead of redundantly at the start of every workgroup: with
// many workgroups the redundant solves and the reads of the accumulator
// copies they share cost more than the extra launch.  Both schedules run the
// same solve on the same totals, so the poses are identical.
// Eight mixed sessions, a whole step: 2575 us with this line, 2636 at 1280 (one
// resident round).  The evaluation that then never solves is compiled without
// the solve: 80 registers, 6 wavefronts a SIMD.
constexpr int kSeparateSolveTiles = 3072;

static int track_tiles(const FrameDev& f, int level) {
  const int wl = (f.W + (1 << level) - 1) >> level;
  const int hl = (f.H + (1 << level) - 1) >> level;
  return ((wl + kTileW - 1) / kTileW) * ((hl + 15) >> 4);
}

static void track_dispatch(Batch& b, int df, int st, const TrackArgs& a, hipStream_t s) {
  int total = 0;
  for (int j = 0; j < b.n; ++j) {
    b.base[j] = total;
    total += track_tiles(b.job[j].f, a.level);
  }
  b.base[b.n] = total;
  const dim3 g(total), blk(kTrackBlock);
  auto run = [&](auto lm, auto slots, auto solve, auto one) {
    constexpr bool L = decltype(lm)::value;
    constexpr int S = decltype(slots)::value;
    constexpr bool V = decltype(solve)::value;
    constexpr bool O = decltype(one)::value;
    if (df == RF_DEPTH_U16) {
      if (st == RF_STORAGE_FP32) track_kernel<RF_DEPTH_U16, RF_STORAGE_FP32, L, S, V, O><<<g, blk, 0, s>>>(b, a);
      else track_kernel<RF_DEPTH_U16, RF_STORAGE_FP16_U8, L, S, V, O><<<g, blk, 0, s>>>(b, a);
    } else {
      if (st == RF_STORAGE_FP32) track_kernel<RF_DEPTH_F32, RF_STORAGE_FP32, L, S, V, O><<<g, blk, 0, s>>>(b, a);
      else track_kernel<RF_DEPTH_F32, RF_STORAGE_FP16_U8, L, S, V, O><<<g, blk, 0, s>>>(b, a);
    }
  };
  using Small = std::integral_constant<int, tile_refs(1) * 2>;
  using Large = std::integral_constant<int, kTileRefs>;
  using Solve = std::true_type;
  using Apart = std::false_type;
  static_assert(tile_refs(0) <= Small::value && tile_refs(1) <= Small::value, "level 0-1 pairs fit the small cache");
  auto pick = [&](auto lm) {
    using One = std::true_type;
    using Many = std::false_type;
    if (a.level >= 2) b.n == 1 ? run(lm, Large{}, Solve{}, One{}) : run(lm, Large{}, Solve{}, Many{});
    else if (!a.solve) run(lm, Small{}, Apart{}, Many{});
    else b.n == 1 ? run(lm, Small{}, Solve{}, One{}) : run(lm, Small{}, Solve{}, Many{});
  };
  if (a.adaptive) pick(std::true_type{});
  else pick(std::false_type{});
}

void launch_track(Batch& b, int df, int st, const rf_track_params& tp, hipStream_t s) {
  track_reset_kernel<<<b.n, 256, 0, s>>>(b);
  int j = 0, prev_level = -1, prev_first = 0;
  for (int l = tp.levels - 1; l >= 0; --l) {
    int tiles = 0;
    for (int q = 0; q < b.n; ++q) tiles += track_tiles(b.job[q].f, l);
    const bool separate = tiles > kSeparateSolveTiles;
    for (int it = 0; it < tp.iters_per_level; ++it, ++j) {
      TrackArgs a{};
      a.level = l;
      a.w_c = tp.w_c;
      a.min_valid = tp.min_valid;
      a.lm_lambda = tp.lm_lambda;
      a.solve = j > 0;
      a.prev_level = prev_level;
      a.prev_first = prev_first;
      a.acc_read = j > 0 ? (j - 1) % 3 : -1;
      a.acc_write = j % 3;
      a.acc_clear = j > 0 ? (j + 1) % 3 : -1;
      a.pose_read = j > 0 ? (j - 1) % 2 : 2;
      a.pose_write = j % 2;
      a.mode = 0;
      a.adaptive = tp.adaptive;
      a.state_read = j > 0 ? (j - 1) % 2 : -1;
      a.state_write = j % 2;
      if (separate && a.solve) {
        // the solve once per job, then the evaluation at the pose it wrote
        TrackArgs c = a;
        c.mode = 2;
        track_finalize_kernel<<<b.n, 64, 0, s>>>(b, c, nullptr);
        a.solve = 0;
        a.pose_read = j % 2;
        a.pose_write = -1;
        a.state_write = -1;
      }
      track_dispatch(b, df, st, a, s);
      prev_level = l;
      prev_first = it == 0;
    }
  }
  if (j == 0) return;
  TrackArgs a{};
  a.level = -1;
  a.min_valid = tp.min_valid;
  a.lm_lambda = tp.lm_lambda;
  a.solve = 1;
  a.prev_level = prev_level;
  a.prev_first = prev_first;
  a.acc_read = (j - 1) % 3;
  a.acc_write = -1;
  a.acc_clear = -1;
  a.pose_read = (j - 1) % 2;
  a.pose_write = 2;
  a.adaptive = tp.adaptive;
  a.state_read = (j - 1) % 2;
  a.state_write = -1;
  track_finalize_kernel<<<b.n, 64, 0, s>>>(b, a, nullptr);
}

void launch_residual(Batch& b, int df, int st, float gamma, hipStream_t s) {
  int total = 0;
  for (int j = 0; j < b.n; ++j) {
    b.base[j] = total;
    total += track_tiles(b.job[j].f, 0);
  }
  b.base[b.n] = total;
  constexpr int S = tile_refs(1) * 2;  // the finest level's cache size, as in tracking
  static_assert(tile_refs(0) <= S, "level-0 pairs fit the cache");
  const dim3 g(total), blk(kTrackBlock);
  if (df == RF_DEPTH_U16) {
    if (st == RF_STORAGE_FP32) residual_kernel<RF_DEPTH_U16, RF_STORAGE_FP32, S><<<g, blk, 0, s>>>(b, gamma);
    else residual_kernel<RF_DEPTH_U16, RF_STORAGE_FP16_U8, S><<<g, blk, 0, s>>>(b, gamma);
  } else {
    if (st == RF_STORAGE_FP32) residual_kernel<RF_DEPTH_F32, RF_STORAGE_FP32, S><<<g, blk, 0, s>>>(b, gamma);
    else residual_kernel<RF_DEPTH_F32, RF_STORAGE_FP16_U8, S><<<g, blk, 0, s>>>(b, gamma);
  }
}

void launch_normal_equations(Batch& b, int df, int st, int level, float w_c, double* out29, hipStream_t s) {
  for (int j = 0; j < b.n; ++j) b.job[j].stats = nullptr;
  track_reset_kernel<<<b.n, 256, 0, s>>>(b);
  TrackArgs a{};
  a.level = level;
  a.w_c = w_c;
  a.solve = 0;
  a.acc_read = -1;
  a.acc_write = 0;
  a.acc_clear = -1;
  a.pose_read = 2;
  a.pose_write = 0;
  track_dispatch(b, df, st, a, s);
  TrackArgs c{};
  c.mode = 1;
  c.acc_read = 0;
  track_finalize_kernel<<<b.n, 64, 0, s>>>(b, c, out29);
}

}  // namespace rf
