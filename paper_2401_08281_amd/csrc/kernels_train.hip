// Training kernels (Sec. 4.1 "The k-means vector quantizer"; Sec. 5.1 "Encoding
// residuals"): the update step of Lloyd's iteration and the residual sub-vectors the
// sub-quantizers are trained on.  The assignment step is the library's k-nearest-rows
// routine with k = 1.
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"

namespace {

constexpr int64_t kBlock = 4096;   // vectors per summation block (a multiple of every batch below)

// Block bk of centroid j has the number off[j] / kBlock + j + bk: the numbers of different centroids
// never overlap, there are n / kBlock + K of them whatever the clusters' sizes, and they leave out at
// most one per centroid.  So workgroups can be launched for all blocks of the largest cluster at once
// without knowing on the host which one that is.
// Four rounds of 262144 x 8 into 256 centroids of which one holds 90 %, with four times the blocks of
// equal clusters side by side instead: 7.9 ms, and 1.3 like this; x 128 into 1024: 9.2 and 2.2.
__device__ __forceinline__ int64_t first_block(const int64_t* __restrict__ off, int j) { return off[j] / kBlock + j; }

// The centroid whose blocks number s belongs to: the last j with first_block(j) <= s.  Every group of W
// lanes looks for an s of its own, W centroids at a time.
template <int W>
__device__ __forceinline__ int block_owner(const int64_t* __restrict__ off, int K, int64_t s) {
  const int lane = lane_id(), t = lane % W, g0 = lane - t;
  const u64 mask = W == 64 ? ~0ull : ((1ull << (W & 63)) - 1ull) << g0;
  int lo = 0, len = K;
  while (__builtin_amdgcn_ballot_w64(len > 1) != 0) {
    const int step = (len + W - 1) / W;
    const int j = t * step;
    const bool before = j < len && first_block(off, lo + j) <= s;     // (t = 0: always)
    const int last = __popcll(__builtin_amdgcn_ballot_w64(before) & mask) - 1;
    lo += last * step;
    len = min(step, len - last * step);
  }
  return lo;
}

// One wavefront per (centroid j, block of kBlock vectors).  order[off[j] .. off[j + 1])
// lists the vectors assigned to centroid j in ascending order; they are summed in float64 in
// blocks of kBlock: a block from 0 in the list's order, the block sums in block order -- a
// fixed order, so the sum has one value however the kernels are scheduled, and the blocks of
// a large cluster run side by side (sixteen centroids over millions of sub-vectors would
// otherwise be sixteen chains).  A centroid of one block stores sum / count rounded to fp32
// directly; the others store their block sums to `partial`, by number, and
// segmented_mean_finish_kernel adds them up.  A centroid without vectors is left as it is.
// A wavefront takes 64 of the dimensions (grid y), one per lane.
// The chain of a large cluster is long (it sets the kernel's time), so the memory latency is taken
// off it: 32 vectors at a time, their numbers come in with one load and their rows are all
// requested a batch ahead of the additions, which run in the list's order.  262144 x 128 into 1024
// centroids, clusters of up to some thousand: 710 us with one batch in flight and two dimensions
// per lane, 63 us like this.
__global__ __launch_bounds__(256) void segmented_mean_kernel(const float* __restrict__ x, int d,
                                                             const int32_t* __restrict__ order,
                                                             const int64_t* __restrict__ off, int K,
                                                             float* __restrict__ centroids,
                                                             double* __restrict__ partial) {
  constexpr int NB = 32;
  const int wave = threadIdx.x >> 6, lane = lane_id();
  const int64_t s = blockIdx.x * 4ll + wave;
  const int j = block_owner<64>(off, K, s);
  const int64_t b0 = off[j], e0 = off[j + 1];
  const double count = (double)(e0 - b0);
  const int64_t nblk = (e0 - b0 + kBlock - 1) / kBlock, bk = s - first_block(off, j);
  if (bk >= nblk) return;
  const int64_t b = b0 + bk * kBlock, e = min(e0, b + kBlock);
  for (int64_t t0 = blockIdx.y * 64ll; t0 < d; t0 += gridDim.y * 64ll) {
    const int t = (int)t0 + lane;
    const int tc = min(t, d - 1);                                // (lanes past d load what they drop)
    double acc = 0.0;
    float v0[NB], v1[NB];
    auto fetch = [&](int64_t i, float (&v)[NB]) {
      const int32_t mine = order[min(i + (lane & (NB - 1)), e - 1)];
#pragma unroll
      for (int u = 0; u < NB; ++u) v[u] = x[(int64_t)__builtin_amdgcn_readlane(mine, u) * d + tc];
    };
    auto add = [&](int64_t i, const float (&v)[NB]) {
      if (i + NB <= e) {
#pragma unroll
        for (int u = 0; u < NB; ++u) acc += (double)v[u];
      } else {
#pragma unroll
        for (int u = 0; u < NB; ++u) if (i + u < e) acc += (double)v[u];
      }
    };
    fetch(b, v0);
    for (int64_t i = b; i < e; i += 2 * NB) {
      if (i + NB < e) fetch(i + NB, v1);
      add(i, v0);
      if (i + NB >= e) break;
      if (i + 2 * NB < e) fetch(i + 2 * NB, v0);
      add(i + NB, v1);
    }
    if (t < d) {
      if (nblk == 1) centroids[j * d + t] = (float)(acc / count);
      else partial[s * d + t] = acc;
    }
  }
}

// The same for rows of at most 32 floats (the sub-vectors of a product quantizer), where one
// row per load instruction would leave most lanes idle: lane (c, t) = (lane / DP, lane % DP) adds up
// dimension t of the c-th of 64 / DP centroids, so every lane runs one chain of its own and a load
// instruction fetches 64 / DP rows.  Rows are requested 32 vectors ahead of the additions and their
// numbers 64 ahead, so that waiting for a number never waits for the rows just requested.  16
// problems of 262144 x 8 descriptors' residuals into 256 centroids: 209 us with one batch of 64 in
// flight, 183 us like this with four times the workgroups and a loop over blocks, 135 us with one
// block per group of lanes.  The largest clusters' chains set the time: keeping a problem on one XCD and
// 32-bit offsets changed nothing.
// DP: d rounded up to 8, 16 or 32.  Grid z: independent problems of the same shape (the
// sub-quantizers of a product quantizer), their arrays one after the other.
template <int DP>
__global__ __launch_bounds__(256) void segmented_mean_small_kernel(const float* __restrict__ x, int d,
                                                                   const int32_t* __restrict__ order,
                                                                   const int64_t* __restrict__ off, int K,
                                                                   float* __restrict__ centroids,
                                                                   double* __restrict__ partial) {
  constexpr int CPW = 64 / DP, NB = 32, NO = NB / DP;            // centroids per wavefront, vectors per batch
  const int lane = lane_id(), c = lane / DP, t = lane % DP;
  const int64_t s = (blockIdx.x * 4ll + (threadIdx.x >> 6)) * CPW + c;
  off += (int64_t)blockIdx.z * (K + 1);
  const int64_t n = off[K];
  x += (int64_t)blockIdx.z * n * d;
  order += (int64_t)blockIdx.z * n;
  centroids += (int64_t)blockIdx.z * K * d;
  partial += (int64_t)blockIdx.z * (n / kBlock + K + 1) * d;
  const int j = block_owner<DP>(off, K, s);
  const int64_t b0 = off[j], e0 = off[j + 1];
  const double count = (double)(e0 - b0);
  const int64_t nblk = (e0 - b0 + kBlock - 1) / kBlock, bk = s - first_block(off, j);
  const int tc = min(t, d - 1);                                  // (lanes past d load what they drop)
  const bool mine_too = bk < nblk;
  const int64_t b = mine_too ? b0 + bk * kBlock : 0, e = mine_too ? min(e0, b + kBlock) : 0;
  if (__builtin_amdgcn_ballot_w64(mine_too) == 0) return;
  double acc = 0.0;
  int32_t n0[NO], n1[NO];
  float v0[NB], v1[NB];
  auto numbers = [&](int64_t i, int32_t (&num)[NO]) {          // (a group without vectors reads slot 0 and drops it)
#pragma unroll
    for (int o = 0; o < NO; ++o) num[o] = order[max(min(i + o * DP + t, e - 1), (int64_t)0)];
  };
  auto request = [&](const int32_t (&num)[NO], float (&v)[NB]) {
#pragma unroll
    for (int u = 0; u < NB; ++u)
      v[u] = x[(int64_t)__shfl(num[u / DP], c * DP + u % DP) * d + tc];
  };
  auto add = [&](int64_t i, const float (&v)[NB]) {
#pragma unroll
    for (int u = 0; u < NB; ++u) acc += i + u < e ? (double)v[u] : 0.0;
  };
  numbers(b, n0);
  numbers(b + NB, n1);
  request(n0, v0);
  for (int64_t i = b; __builtin_amdgcn_ballot_w64(i < e) != 0; i += 2 * NB) {
    numbers(i + 2 * NB, n0);
    request(n1, v1);
    add(i, v0);
    if (__builtin_amdgcn_ballot_w64(i + NB < e) == 0) break;
    numbers(i + 3 * NB, n1);
    request(n0, v0);
    add(i + NB, v1);
  }
  if (mine_too && t < d) {
    if (nblk == 1) centroids[j * d + t] = (float)(acc / count);
    else partial[s * d + t] = acc;
  }
}

// Centroids of more than one block: the block sums in block order, then the mean.
__global__ __launch_bounds__(256) void segmented_mean_finish_kernel(const double* __restrict__ partial,
                                                                    int d,
                                                                    const int64_t* __restrict__ off, int K,
                                                                    float* __restrict__ centroids) {
  const int wave = threadIdx.x >> 6, lane = lane_id();
  const int64_t j = blockIdx.x * 4ll + wave;
  if (j >= K) return;
  off += (int64_t)blockIdx.z * (K + 1);
  const int64_t b0 = off[j], e0 = off[j + 1];
  const int64_t nblk = (e0 - b0 + kBlock - 1) / kBlock;
  if (nblk <= 1) return;
  partial += (int64_t)blockIdx.z * (off[K] / kBlock + K + 1) * d;
  centroids += (int64_t)blockIdx.z * K * d;
  const double count = (double)(e0 - b0);
  const double* __restrict__ src = partial + (b0 / kBlock + j) * d;
  for (int t = lane; t < d; t += VS_WAVE) {
    double total = 0.0;
    for (int64_t bk = 0; bk < nblk; ++bk) total += src[bk * d + t];
    centroids[j * d + t] = (float)(total / count);
  }
}

// ---- bookkeeping of a k-means round on the device -----------------------------------
// The update needs, for every centroid, the numbers of its vectors in ascending order: a
// stable counting sort of the assignment idx [n] by centroid.  The vectors are cut into at
// most 256 chunks of consecutive vectors:
//   km_hist_kernel     per chunk, how many vectors go to each centroid        mat [nchunk][K]
//   km_colscan_kernel  per centroid, exclusive running sum down the chunks (in place) and the total
//   km_offsets_kernel  exclusive sum of the totals = first slot of each centroid, off [K + 1]
//   km_scatter_kernel  one wavefront per chunk walks over its vectors in order, 64 at a time:
//                      every vector gets slot off[j] + (vectors of j in earlier chunks) +
//                      (earlier vectors of j in this chunk): the stable order.
// K <= 16384 (one counter per centroid in LDS); the host does the same sort otherwise.
// Grid y: independent problems of the same shape, their arrays one after the other.
template <typename T>
__global__ __launch_bounds__(256) void km_hist_kernel(const T* __restrict__ idx, int64_t n, int K,
                                                      int64_t chunk, int32_t* __restrict__ mat,
                                                      int* __restrict__ bad) {
  extern __shared__ int km_lds[];
  idx += (int64_t)blockIdx.y * n;
  mat += (int64_t)blockIdx.y * gridDim.x * K;
  for (int j = threadIdx.x; j < K; j += 256) km_lds[j] = 0;
  __syncthreads();
  const int64_t i0 = blockIdx.x * chunk, i1 = min(n, i0 + chunk);
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
    const int32_t j = (int32_t)idx[i];
    if (j < 0 || j >= K) *bad = 1;
    else atomicAdd(&km_lds[j], 1);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < K; j += 256) mat[(int64_t)blockIdx.x * K + j] = km_lds[j];
}

// 64 centroids per workgroup; wavefront s first sums, then rewrites its quarter of the chunks
__global__ __launch_bounds__(256) void km_colscan_kernel(int32_t* __restrict__ mat, int nchunk, int K,
                                                         int64_t* __restrict__ cnt) {
  __shared__ int32_t part[4][64];
  mat += (int64_t)blockIdx.y * nchunk * K;
  cnt += (int64_t)blockIdx.y * K;
  const int s = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = blockIdx.x * 64 + lane, per = (nchunk + 3) / 4;
  const int c0 = min(nchunk, s * per), c1 = min(nchunk, c0 + per);
  const bool ok = j < K;
  int32_t sum = 0;
#pragma unroll 8
  for (int c = c0; c < c1; ++c) sum += ok ? mat[(int64_t)c * K + j] : 0;
  part[s][lane] = sum;
  __syncthreads();
  if (!ok) return;
  int32_t run = 0;
  for (int u = 0; u < s; ++u) run += part[u][lane];
#pragma unroll 8
  for (int c = c0; c < c1; ++c) {
    const int32_t v = mat[(int64_t)c * K + j];
    mat[(int64_t)c * K + j] = run;
    run += v;
  }
  if (s == 3) cnt[j] = run;
}

// one workgroup per problem: lane t owns centroids [t * per, (t + 1) * per)
__global__ __launch_bounds__(256) void km_offsets_kernel(const int64_t* __restrict__ cnt, int K,
                                                         int64_t* __restrict__ off) {
  __shared__ int64_t wsum[4];
  cnt += (int64_t)blockIdx.y * K;
  off += (int64_t)blockIdx.y * (K + 1);
  const int t = threadIdx.x, per = (K + 255) / 256;
  const int j0 = min(K, t * per), j1 = min(K, j0 + per);
  int64_t sum = 0;
  for (int j = j0; j < j1; ++j) sum += cnt[j];
  int64_t inc = sum;                                    // inclusive over the wavefront, then the workgroup
  for (int o = 1; o < 64; o <<= 1) { const int64_t v = __shfl_up(inc, o); if ((t & 63) >= o) inc += v; }
  if ((t & 63) == 63) wsum[t >> 6] = inc;
  __syncthreads();
  int64_t base = inc - sum;
  for (int w = 0; w < (t >> 6); ++w) base += wsum[w];
  for (int j = j0; j < j1; ++j) { off[j] = base; base += cnt[j]; }
  if (t == 255) off[K] = base;
}

template <typename T>
__global__ __launch_bounds__(64) void km_scatter_kernel(const T* __restrict__ idx, int64_t n, int K, int bits,
                                                        int64_t chunk, const int32_t* __restrict__ mat,
                                                        const int64_t* __restrict__ off,
                                                        int32_t* __restrict__ order) {
  extern __shared__ int km_lds[];                       // next slot of every centroid for this chunk
  const int lane = lane_id();
  idx += (int64_t)blockIdx.y * n;
  order += (int64_t)blockIdx.y * n;
  mat += (int64_t)blockIdx.y * gridDim.x * K;
  off += (int64_t)blockIdx.y * (K + 1);
  for (int j = lane; j < K; j += VS_WAVE) km_lds[j] = (int)(off[j] + mat[(int64_t)blockIdx.x * K + j]);
  wave_lds_sync();
  const int64_t i0 = blockIdx.x * chunk, i1 = min(n, i0 + chunk);
  int32_t next = i0 + lane < i1 ? (int32_t)idx[i0 + lane] : -1;
  for (int64_t g = i0; g < i1; g += VS_WAVE) {
    const int64_t i = g + lane;
    const int32_t key = next;
    next = i + VS_WAVE < i1 ? (int32_t)idx[i + VS_WAVE] : -1;
    const bool valid = key >= 0 && key < K;             // (others were flagged by km_hist_kernel; never stored)
    const WaveRank r = wave_rank(valid, (u32)key, bits);
    int slot = 0;
    if (valid) slot = km_lds[key] + r.rank;
    wave_lds_sync();                                    // everyone has read the counters before they move
    if (valid && r.rank == 0) km_lds[key] = slot + r.count;
    if (valid) order[slot] = (int32_t)i;
    wave_lds_sync();
  }
}

// Sum of val [n] in float64 in a fixed order: workgroup w sums a contiguous slice (lane-strided,
// then a fixed tree), the host adds the 256 partial sums in order.
__global__ __launch_bounds__(256) void km_objective_kernel(const float* __restrict__ val, int64_t n,
                                                           double* __restrict__ partial) {
  __shared__ double red[256];
  val += (int64_t)blockIdx.y * n;
  partial += (int64_t)blockIdx.y * gridDim.x;
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t i0 = blockIdx.x * per, i1 = min(n, i0 + per);
  double acc = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) acc += (double)val[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// out[m][i][u] = x[i][m * dsub + u] - centroids[list_of[i]][m * dsub + u]: the residual of
// every vector (one fp32 subtraction per component), regrouped into M contiguous matrices
// of sub-vectors.
__global__ __launch_bounds__(256) void residual_slices_kernel(const float* __restrict__ x, int64_t n,
                                                              int d, int dsub,
                                                              const float* __restrict__ centroids,
                                                              const int32_t* __restrict__ list_of,
                                                              float* __restrict__ out) {
  const int64_t total = n * d, stride = (int64_t)gridDim.x * 256;   // grid-stride: n * d may exceed 2^32
  for (int64_t e = blockIdx.x * 256ll + threadIdx.x; e < total; e += stride) {
    const int64_t i = e / d;
    const int t = (int)(e - i * d);
    const int m = t / dsub, u = t - m * dsub;
    out[((int64_t)m * n + i) * dsub + u] = x[e] - centroids[(int64_t)list_of[i] * d + t];
  }
}

}  // namespace

size_t segmented_mean_partial_bytes(int64_t n, int d, int K, int problems) {
  if (n <= kBlock) return 0;
  return (size_t)(n / kBlock + K + 1) * d * sizeof(double) * problems;
}

void launch_segmented_mean(const float* x, int64_t n, int d, const int32_t* order, const int64_t* off, int K,
                           int problems, float* centroids, double* partial, hipStream_t st) {
  if (K <= 0 || n <= 0) return;
  const int64_t most = (n + kBlock - 1) / kBlock;
  const int64_t blocks = n / kBlock + K;                         // block numbers, see first_block
  const unsigned P = (unsigned)problems, gk = (unsigned)((K + 3) / 4);
  const int per_wave = d <= 8 ? 8 : (d <= 16 ? 4 : (d <= 32 ? 2 : 1));
  const unsigned gx = (unsigned)((blocks + 4 * per_wave - 1) / (4 * per_wave));
  const dim3 block(256);
  if (d <= 8) hipLaunchKernelGGL((segmented_mean_small_kernel<8>), dim3(gx, 1, P), block, 0, st, x, d, order, off, K, centroids, partial);
  else if (d <= 16) hipLaunchKernelGGL((segmented_mean_small_kernel<16>), dim3(gx, 1, P), block, 0, st, x, d, order, off, K, centroids, partial);
  else if (d <= 32) hipLaunchKernelGGL((segmented_mean_small_kernel<32>), dim3(gx, 1, P), block, 0, st, x, d, order, off, K, centroids, partial);
  else   // (problems == 1)
    hipLaunchKernelGGL(segmented_mean_kernel, dim3(gx, (unsigned)std::min((d + 63) / 64, 65535)), block, 0, st, x, d, order, off, K, centroids, partial);
  if (most > 1)
    hipLaunchKernelGGL(segmented_mean_finish_kernel, dim3(gk, 1, P), block, 0, st, partial, d, off, K,
                       centroids);
}

size_t kmeans_sort_bytes(int K, int problems) {
  return ((size_t)256 * K * sizeof(int32_t) + (size_t)K * sizeof(int64_t)) * problems;
}

template <typename T>
static void kmeans_sort(const T* idx, const float* val, int64_t n, int K, int problems, char* work, int32_t* order,
                        int64_t* off, int* bad, double* partial, hipStream_t st) {
  const int64_t chunk = std::max<int64_t>(1024, ((n + 255) / 256 + 63) / 64 * 64);
  const unsigned nchunk = (unsigned)((n + chunk - 1) / chunk), P = (unsigned)problems;
  int64_t* cnt = reinterpret_cast<int64_t*>(work);
  int32_t* mat = reinterpret_cast<int32_t*>(cnt + (size_t)K * problems);
  const size_t lds = (size_t)K * sizeof(int);
  if (lds > 48 * 1024) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&km_hist_kernel<T>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&km_scatter_kernel<T>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  }
  int bits = 1;
  while ((1 << bits) < K) ++bits;
  hipLaunchKernelGGL((km_hist_kernel<T>), dim3(nchunk, P), dim3(256), lds, st, idx, n, K, chunk, mat, bad);
  hipLaunchKernelGGL(km_colscan_kernel, dim3((unsigned)((K + 63) / 64), P), dim3(256), 0, st, mat, (int)nchunk, K, cnt);
  hipLaunchKernelGGL(km_offsets_kernel, dim3(1, P), dim3(256), 0, st, cnt, K, off);
  hipLaunchKernelGGL((km_scatter_kernel<T>), dim3(nchunk, P), dim3(64), lds, st, idx, n, K, bits, chunk, mat, off, order);
  hipLaunchKernelGGL(km_objective_kernel, dim3(256, P), dim3(256), 0, st, val, n, partial);
}
void launch_kmeans_sort(const int32_t* idx, const float* val, int64_t n, int K, char* work, int32_t* order,
                        int64_t* off, int* bad, double* partial, hipStream_t st) {
  kmeans_sort(idx, val, n, K, 1, work, order, off, bad, partial, st);
}
void launch_kmeans_sort_bytes(const uint8_t* idx, const float* val, int64_t n, int K, int problems, char* work,
                              int32_t* order, int64_t* off, int* bad, double* partial, hipStream_t st) {
  kmeans_sort(idx, val, n, K, problems, work, order, off, bad, partial, st);
}

void launch_residual_slices(const float* x, int64_t n, int d, int dsub, const float* centroids,
                            const int32_t* list_of, float* out, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(residual_slices_kernel,
                     dim3((unsigned)std::min<int64_t>(1 << 22, (n * d + 255) / 256)), dim3(256), 0, st,
                     x, n, d, dsub, centroids, list_of, out);
}
