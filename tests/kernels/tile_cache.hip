// The tracking tile cache of a build with 512-thread workgroups
// (RF_TRACK_BLOCK=512, set by build.py here), one workgroup: pairs put into an
// empty LDS cache, written back to the tile's pairs, loaded from there into a
// second one and written back again.
#include "rf_track.hip"

static_assert(rf::kTrackBlock == 512, "built with RF_TRACK_BLOCK=512");

namespace {

template <int SLOTS>
__global__ __launch_bounds__(rf::kTrackBlock) void round_trip(rf::BlockRef* tab, uint32_t* count, int nrefs,
                                                              const int* blocks, int n, int again) {
  __shared__ rf::CacheLds<SLOTS> L;
  const int t = threadIdx.x;
  if (t < 64) rf::build_tile_cache<SLOTS>(tab, count, true, nrefs, 1u, t, L);
  __syncthreads();
  if (!again && t < n) {
    const int* b = blocks + 3 * t;
    L.cache(L.org[0], L.org[1], L.org[2]).insert(b[0], b[1], b[2], rf::pack_key(b[0], b[1], b[2]), t, true);
  }
  __syncthreads();
  rf::write_tile_cache<SLOTS>(tab, count, nrefs, 1u, L);
}

}  // namespace

// tab: nrefs pairs of 16 bytes, count: a word, both device memory and zero;
// blocks: n <= 64 block coordinates (device).  Returns the HIP error.
extern "C" __attribute__((visibility("default"))) int tile_cache_round_trip(void* tab, uint32_t* count, int nrefs,
                                                                            int slots, const int* blocks, int n,
                                                                            int again, void* stream) {
  if (n > 64 || n >= nrefs || (slots != 256 && slots != 512) || nrefs > slots) return (int)hipErrorInvalidValue;
  rf::BlockRef* r = static_cast<rf::BlockRef*>(tab);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (slots == 256) round_trip<256><<<1, rf::kTrackBlock, 0, s>>>(r, count, nrefs, blocks, n, again);
  else round_trip<512><<<1, rf::kTrackBlock, 0, s>>>(r, count, nrefs, blocks, n, again);
  return (int)hipGetLastError();
}
