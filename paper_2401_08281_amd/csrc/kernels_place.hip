// Placement of newly added vectors into the inverted lists (Sec. 5.1 "Inverted files": the vectors
// of a cluster are stored contiguously), entirely on the device.
// Input: the list of every new vector, list_of [n].  Output: for every new vector its slot in the
// grown store, dest [n] -- behind the entries its list already holds and behind the new vectors of
// the same list that come earlier in the batch (add order is kept inside a list) -- and the grown
// lists' offsets new_off [nlist + 1].
// The order inside a list needs a STABLE sort of the batch by list.  It is a radix sort by list
// number, least significant digit first, 12 bits per pass (one pass up to 4096 lists, two up to
// 16.7M); every pass is a counting sort that keeps equal digits in input order:
//   place_hist_kernel     per chunk of consecutive positions, the count of every digit   mat [nchunk][4096]
//   place_colscan_kernel  per digit, exclusive running sum down the chunks (in place) and its total
//   place_digit_offsets_kernel  exclusive sum of the totals: first slot of every digit
//   place_scatter_kernel  one wavefront per chunk walks over its positions in order, 64 at a
//                         time; lanes with the same digit are ranked by lane number (ballots)
// then the grown offsets from the places where the list changes in the sorted batch, and dest from
// each vector's rank in it.
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"

namespace {

constexpr int kDigitBits = 12;
constexpr int kBuckets = 1 << kDigitBits;
constexpr int kMaxChunks = 1024;

__device__ __forceinline__ int digit_of(int32_t key, int shift) { return (key >> shift) & (kBuckets - 1); }

// position p of the pass holds vector perm[p] (or p itself when perm is null)
__global__ __launch_bounds__(256) void place_hist_kernel(const int32_t* __restrict__ keys,
                                                         const int32_t* __restrict__ perm, int64_t n, int nlist,
                                                         int shift, int64_t chunk, int32_t* __restrict__ mat,
                                                         int* __restrict__ bad) {
  __shared__ int h[kBuckets];
  for (int j = threadIdx.x; j < kBuckets; j += 256) h[j] = 0;
  __syncthreads();
  const int64_t p0 = blockIdx.x * chunk, p1 = min(n, p0 + chunk);
  for (int64_t p = p0 + threadIdx.x; p < p1; p += 256) {
    const int32_t key = keys[perm ? perm[p] : p];
    if (key < 0 || key >= nlist) *bad = 1;
    else atomicAdd(&h[digit_of(key, shift)], 1);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < kBuckets; j += 256) mat[(int64_t)blockIdx.x * kBuckets + j] = h[j];
}

// 64 digits per workgroup; wavefront s of 16 first sums, then rewrites its sixteenth of the chunks
// (1024 chunks x 4096 digits with one thread per digit: 256 us, all of it latency)
__global__ __launch_bounds__(1024) void place_colscan_kernel(int32_t* __restrict__ mat, int nchunk,
                                                             int64_t* __restrict__ cnt) {
  __shared__ int32_t part[16][64];
  const int s = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = blockIdx.x * 64 + lane, per = (nchunk + 15) / 16;
  const int c0 = min(nchunk, s * per), c1 = min(nchunk, c0 + per);
  int32_t sum = 0;
#pragma unroll 16
  for (int c = c0; c < c1; ++c) sum += mat[(int64_t)c * kBuckets + j];
  part[s][lane] = sum;
  __syncthreads();
  int32_t run = 0;
  for (int u = 0; u < s; ++u) run += part[u][lane];
#pragma unroll 16
  for (int c = c0; c < c1; ++c) {
    const int32_t v = mat[(int64_t)c * kBuckets + j];
    mat[(int64_t)c * kBuckets + j] = run;
    run += v;
  }
  if (s == 15) cnt[j] = run;
}

// one workgroup of 256: thread t owns digits [16 t, 16 t + 16)
__global__ __launch_bounds__(256) void place_digit_offsets_kernel(const int64_t* __restrict__ cnt,
                                                                  int64_t* __restrict__ off) {
  __shared__ int64_t part[256];
  constexpr int per = kBuckets / 256;
  const int t = threadIdx.x;
  int64_t sum = 0;
  for (int j = t * per; j < (t + 1) * per; ++j) sum += cnt[j];
  part[t] = sum;
  __syncthreads();
  int64_t base = 0;
  for (int u = 0; u < t; ++u) base += part[u];
  for (int j = t * per; j < (t + 1) * per; ++j) { off[j] = base; base += cnt[j]; }
}

__global__ __launch_bounds__(64) void place_scatter_kernel(const int32_t* __restrict__ keys,
                                                           const int32_t* __restrict__ perm, int64_t n, int nlist,
                                                           int shift, int64_t chunk, const int32_t* __restrict__ mat,
                                                           const int64_t* __restrict__ off,
                                                           int32_t* __restrict__ out) {
  __shared__ int next[kBuckets];                        // next slot of every digit for this chunk
  const int lane = lane_id();
  for (int j = lane; j < kBuckets; j += VS_WAVE) next[j] = (int)(off[j] + mat[(int64_t)blockIdx.x * kBuckets + j]);
  wave_lds_sync();
  const int64_t p0 = blockIdx.x * chunk, p1 = min(n, p0 + chunk);
  for (int64_t g = p0; g < p1; g += VS_WAVE) {
    const int64_t p = g + lane;
    int32_t i = -1, dg = -1;
    if (p < p1) {
      i = perm ? perm[p] : (int32_t)p;
      const int32_t key = keys[i];
      if (key >= 0 && key < nlist) dg = digit_of(key, shift);   // (others were flagged by the histogram pass)
    }
    const WaveRank r = wave_rank(dg >= 0, (u32)dg, kDigitBits);
    int slot = 0;
    if (dg >= 0) slot = next[dg] + r.rank;
    wave_lds_sync();                                    // everyone has read the counters before they move
    if (dg >= 0 && r.rank == 0) next[dg] = slot + r.count;
    if (dg >= 0) out[slot] = i;
    wave_lds_sync();
  }
}

// With first_new(l) = the rank of list l's first new vector in the sorted batch (what an empty list
// would have), known from the places where the list changes, the grown lists begin at
//   new_off[l] = old_off[l] + first_new(l):   old sizes and new counts of the lists before l.
// Thread p looks at ranks p - 1 and p and fills the lists in between (p = n: the rest).  Where many
// lists get nothing (a few vectors added to many lists, or all of them to a few) the gaps are long:
// those of more than kGap lists are filled by the whole workgroup, one after the other.  Adding one
// vector to 65536 lists: 6802 us with a thread per gap, 18 us like this (100 vectors: 565 and 53).
constexpr int kGap = 32;
__global__ __launch_bounds__(1024) void place_first_kernel(const int32_t* __restrict__ order,
                                                           const int32_t* __restrict__ keys, int64_t n, int nlist,
                                                           const int64_t* __restrict__ old_off,
                                                           int64_t* __restrict__ new_off, const int* __restrict__ bad) {
  __shared__ int long_gaps, gap_first[1024], gap_last[1024], gap_p[1024];
  if (*bad) return;
  if (threadIdx.x == 0) long_gaps = 0;
  __syncthreads();
  const int64_t p = blockIdx.x * 1024ll + threadIdx.x;
  if (p <= n) {
    const int first = (p > 0 ? keys[order[p - 1]] : -1) + 1, last = p < n ? keys[order[p]] : nlist;
    if (last - first >= kGap) {
      const int at = atomicAdd(&long_gaps, 1);
      gap_first[at] = first; gap_last[at] = last; gap_p[at] = (int)p;
    } else {
      for (int l = first; l <= last; ++l) new_off[l] = old_off[l] + p;
    }
  }
  __syncthreads();
  for (int g = 0; g < long_gaps; ++g)
#pragma unroll 4
    for (int l = gap_first[g] + threadIdx.x; l <= gap_last[g]; l += 1024) new_off[l] = old_off[l] + gap_p[g];
}

// the vector at rank p of the sorted batch goes behind its list's old entries and the p -
// first_new(l) new ones before it: new_off[l] + old size + p - first_new(l) = old_off[l + 1] + p
__global__ __launch_bounds__(256) void place_dest_kernel(const int32_t* __restrict__ order,
                                                         const int32_t* __restrict__ keys, int64_t n, int nlist,
                                                         const int64_t* __restrict__ old_off,
                                                         const int* __restrict__ bad,
                                                         int64_t* __restrict__ dest) {
  const int64_t p = blockIdx.x * 256ll + threadIdx.x;
  if (p >= n || *bad) return;
  const int32_t i = order[p];
  const int32_t l = keys[i];
  if (l < 0 || l >= nlist) return;
  dest[i] = old_off[l + 1] + p;   // = new_off[l] + old size + (p - first_new[l])
}

struct PlaceWork {
  int32_t *order_a, *order_b, *mat;
  int64_t *digit_cnt, *digit_off;
  int* bad;
  size_t bytes;
};
PlaceWork carve(char* base, int64_t n) {
  PlaceWork w;
  size_t o = 0;
  auto take = [&](size_t b) { const size_t at = o; o += (b + 255) & ~(size_t)255; return base ? base + at : nullptr; };
  w.order_a = reinterpret_cast<int32_t*>(take((size_t)n * sizeof(int32_t)));
  w.order_b = reinterpret_cast<int32_t*>(take((size_t)n * sizeof(int32_t)));
  w.mat = reinterpret_cast<int32_t*>(take((size_t)kMaxChunks * kBuckets * sizeof(int32_t)));
  w.digit_cnt = reinterpret_cast<int64_t*>(take((size_t)kBuckets * sizeof(int64_t)));
  w.digit_off = reinterpret_cast<int64_t*>(take((size_t)kBuckets * sizeof(int64_t)));
  w.bad = reinterpret_cast<int*>(take(sizeof(int64_t)));
  w.bytes = o;
  return w;
}

}  // namespace

size_t ivf_place_work_bytes(int64_t n) { return carve(nullptr, n).bytes; }

int* launch_ivf_place(const int32_t* list_of, int64_t n, int nlist, const int64_t* old_off, char* work,
                      int64_t* dest, int64_t* new_off, hipStream_t st) {
  const PlaceWork w = carve(work, n);
  launch_fill_u64(reinterpret_cast<u64*>(w.bad), 1, 0ull, st);
  const int64_t chunk = std::max<int64_t>(1024, ((n + kMaxChunks - 1) / kMaxChunks + 63) / 64 * 64);
  const int nchunk = (int)((n + chunk - 1) / chunk);
  const int32_t* perm = nullptr;
  int32_t* out = w.order_a;
  for (int shift = 0; shift == 0 || (nlist - 1) >> shift != 0; shift += kDigitBits) {
    hipLaunchKernelGGL(place_hist_kernel, dim3((unsigned)nchunk), dim3(256), 0, st, list_of, perm, n, nlist, shift,
                       chunk, w.mat, w.bad);
    hipLaunchKernelGGL(place_colscan_kernel, dim3(kBuckets / 64), dim3(1024), 0, st, w.mat, nchunk, w.digit_cnt);
    hipLaunchKernelGGL(place_digit_offsets_kernel, dim3(1), dim3(256), 0, st, w.digit_cnt, w.digit_off);
    hipLaunchKernelGGL(place_scatter_kernel, dim3((unsigned)nchunk), dim3(64), 0, st, list_of, perm, n, nlist, shift,
                       chunk, w.mat, w.digit_off, out);
    perm = out;
    out = out == w.order_a ? w.order_b : w.order_a;
  }
  hipLaunchKernelGGL(place_first_kernel, dim3((unsigned)((n + 1024) / 1024)), dim3(1024), 0, st, perm, list_of, n, nlist,
                     old_off, new_off, w.bad);
  hipLaunchKernelGGL(place_dest_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, perm, list_of, n, nlist,
                     old_off, w.bad, dest);
  return w.bad;
}
