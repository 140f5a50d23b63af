// Matrix-core scan of inverted lists for batches of queries (Sec. 5.1 inverted files; Sec. 4.3
// compressed-domain search; App. A.3 "GPU Faiss").
//
// In a batch a list is probed by several queries, and the distances between the queries that probe a
// list and the vectors stored in it are a matrix product.  The scan computes them list by list on the
// matrix cores, in fp16 with fp32 sums, from vectors that are decoded straight into matrix fragments
// -- PQ codes by one look-up of a whole sub-vector in an fp16 copy of the codebook in LDS, 8-bit
// scalar codes and raw vectors by a conversion -- and uses the products only to decide WHICH stored
// vectors can be among a query's k best: those whose approximate distance is within the proven error
// bound of the query's threshold are kept, evaluated again with the arithmetic of the query-major
// scans (the same instructions in the same order: the same bits) and selected from.
//
//   ms_count / ms_offsets / ms_scatter   the (query, probe) pairs grouped by list, the work items of the
//                                        sweeps, the queries laid out in fragment order
//   ms_sweep, MODE 0 (bound)             upper bounds of the distances to the vectors of every query's first
//                                        lists, the smallest of every four vectors kept
//   ms_bound                             their k-th smallest: at least k stored vectors are that close, so it
//                                        bounds the k-th best of the whole search from above
//   ms_sweep, MODE 1 (collect)           all probed lists: vectors whose lower bound does not exceed the query's
//                                        threshold go to the query's candidate buffer
//   ms_rerank_*                          exact evaluation of the candidates, k best; queries whose buffer
//                                        overflowed are listed for the query-major scan
//
// Error bound.  u = 2^-11 (fp16 rounding), a = the query's side, b = the stored vector's side (L2: both
// relative to the list's centroid, so that errors are relative to residuals, not to the vectors), a^, b^
// their fp16 images, both scaled by a power of two (sigma) that puts the data in the middle of fp16's
// range, D = |a - b|^2, D^ = |a^ - b^|^2:
//   sqrt(D^) and sqrt(D) differ by at most u (|a| + |b|) + 2 s sqrt(d), s = 2^-25 the half spacing of fp16
//   subnormals, hence |D^ - D| <= 3u D + u (|a|^2 + |b|^2) + small terms; fp32 sums of either evaluation
//   differ from the real sums by at most phi (|a|^2 + |b|^2) with phi = 2^-22 per addition in a chain.
//   Inner products: |<a, b> - <a^, b^>| <= (2u + u^2) |a| |b| + s sqrt(d) (|a| + |b|) + d s^2.
//   4-bit inner products of long sub-vectors (see ms_onehot_sweep_kernel) have a bound of their own: every table entry
//   is rounded to a whole number of steps, and the largest error of each sub-quantizer is added up.
// The kernels use kappa = 1.02 u + phi, 4 u for 3 u, and absolute terms of 2^-26 d in scaled units (which also
// cover subnormal squares that the dot product instruction may drop).  Where a value has no finite fp16
// image (overflow, NaN), the vector or the query passes every test and is decided exactly.
//   The exact evaluation knows no scale: it must not leave fp32's range where the scaled bounds stay inside theirs,
// or it ties what they tell apart (an infinite or vanishing distance, a NaN).  The scan therefore serves indexes whose
// scale is within 2^-40 .. 2^40 (mscan_scale_fits): components with an fp16 image are then below 2^56, sums of 512
// of their squares below 2^121, and what underflows is below 2^-149 512 2^80 in scaled units, far below the absolute
// terms.  Terms that are not such sums (|c|^2, <q, c>, the cells of scalar codes) have a limit each in the sweep.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "survivors.hpp"

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kQueue = 128;          // candidates a wavefront keeps before it writes them out
// words of LDS a wavefront's queue takes: three per candidate, four per query of the item
constexpr __host__ __device__ int queue_words(int nt) { return 3 * kQueue + 32 * nt; }
constexpr int kSweepThreads = 512;

// sum over the four 16-lane rows of a wavefront, in every lane
__device__ __forceinline__ float sum_rows(float v) {
  u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  v = __uint_as_float(r.x) + __uint_as_float(r.y);
  r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  return __uint_as_float(r.x) + __uint_as_float(r.y);
}

__device__ __forceinline__ float dot8(f16x8 a, f16x8 b, float c) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f16x2 x = {a[2 * i], a[2 * i + 1]}, y = {b[2 * i], b[2 * i + 1]};
    c = __builtin_amdgcn_fdot2(x, y, c, false);
  }
  return c;
}

// lanes with a candidate of this lane's query (of an item's 64)
__device__ __forceinline__ u64 same_lanes(bool on, u32 lp) {
  u64 same = __builtin_amdgcn_ballot_w64(on);
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    const bool bit = (lp >> b) & 1u;
    const u64 m = __builtin_amdgcn_ballot_w64(bit);
    same &= bit ? m : ~m;
  }
  return same;
}

// ---- the order of a vector's components in matrix fragments -----------------------------------
// Slot e of a vector: step e / 32 of the product (32 dimensions), lane row (e / 8) mod 4, element e mod 8
// of the lane's eight.  Any order serves as long as both sides use it; each kind takes the one in
// which its stored side is cheapest to produce.
struct SlotMap {
  int kind;                    // kMsPq, kMsFlat, kMsSq8
  int d, dsub, mg, parts, gh;  // PQ: sub-quantizers per lane row, granules per sub-vector, halfs per granule
};
__device__ __forceinline__ int slot_dim(const SlotMap& m, int e) {
  const int s = e >> 5, g = (e >> 3) & 3, t = e & 7;
  if (m.kind == kMsPq) {
    const int j = s * (8 / m.gh) + t / m.gh;
    if (j >= m.mg * m.parts) return -1;
    const int dd = (j % m.parts) * m.gh + t % m.gh;
    return dd < m.dsub ? (g * m.mg + j / m.parts) * m.dsub + dd : -1;
  }
  const int dim = m.kind == kMsFlat ? 32 * s + (t < 4 ? 4 * g + t : 16 + 4 * g + t - 4) : 32 * s + 8 * g + t;
  return dim < m.d ? dim : -1;
}

// ---- grouping ----------------------------------------------------------------------------------
// One wavefront per query.  Its first lists, as far as they fill `slots` groups of four codes, give its
// threshold: pair_slot = first slot | groups << 16 of such a pair, 0 for the others.  Pairs per list (the
// former apart from the others) and every pair's place among them.  The blocks behind them lay the
// queries out in fragment order, zeros where a slot holds no dimension.
__global__ __launch_bounds__(256) void ms_count_kernel(const int32_t* __restrict__ probes, int64_t nq, int npr, int slots, int capcodes,
                                                       const int64_t* __restrict__ list_off, u32* __restrict__ lfirst,
                                                       u32* __restrict__ lrest, u32* __restrict__ rank,
                                                       u32* __restrict__ pair_slot, u32* __restrict__ qslots,
                                                       unsigned pair_blocks, const float* __restrict__ q, int kp,
                                                       SlotMap map, float* __restrict__ qperm) {
  if (blockIdx.x < pair_blocks) {
    const int64_t qi = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (qi >= nq) return;
    const int lane = lane_id();
    int used = 0;
    for (int p0 = 0; p0 < npr; p0 += VS_WAVE) {
      const int p = p0 + lane;
      const int l = p < npr ? probes[qi * npr + p] : -1;
      int64_t len = 0;
      if (l >= 0) len = list_off[l + 1] - list_off[l];
      const int g = (int)min((int64_t)slots, 16 * ((min(len, (int64_t)capcodes) + 63) >> 6));
      int incl = g;
      for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(incl, o, 64); if (lane >= o) incl += t; }
      const int base = used + incl - g;
      const int ng = max(0, min(slots - base, g));
      if (p < npr) {
        u32 r = 0xFFFFFFFFu;
        if (len > 0) r = atomicAdd(ng > 0 ? &lfirst[l] : &lrest[l], 1u);
        rank[qi * npr + p] = r;
        pair_slot[qi * npr + p] = ng > 0 ? (u32)base | ((u32)ng << 16) : 0u;
      }
      used = min(slots, used + __shfl(incl, 63, 64));
    }
    if (lane == 0) qslots[qi] = (u32)used;
    return;
  }
  const int64_t e = ((int64_t)blockIdx.x - pair_blocks) * 256 + threadIdx.x;
  if (e >= nq * kp) return;
  const int64_t qi = e / kp;
  const int dim = slot_dim(map, (int)(e - qi * kp));
  qperm[e] = dim >= 0 ? q[qi * map.d + dim] : 0.f;
}

// segments a list is cut into, and work items of n pairs of it
__device__ __forceinline__ u32 ceil_div(u32 a, u32 b) { return (a + b - 1) / b; }

// off[l] = exclusive prefix sums of the lists' pairs (x) and of their work items in the bound (y) and the collect
// sweep (z): one for every group of at most `group` pairs and every segment of `seg` codes (bound: of the first
// `capcodes` codes).  A workgroup takes 1024 lists and adds up the lists before them by itself, so that no second
// launch is needed.
__global__ __launch_bounds__(1024) void ms_offsets_kernel(const u32* __restrict__ lfirst, const u32* __restrict__ lrest,
                                                          const int64_t* __restrict__ list_off, int nlist, u32 group,
                                                          u32 seg, u32 capcodes, uint4* __restrict__ off, u32 max_a,
                                                          u32 max_b, u32* __restrict__ nitems) {
  __shared__ u32 wsum[3][16];
  __shared__ u32 base_s[3];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int l0 = blockIdx.x * 1024;
  u32 b0 = 0, b1 = 0, b2 = 0;
  auto of = [&](int l, u32& n, u32& f, u32& na, u32& nb) {
    f = lfirst[l];
    n = f + lrest[l];
    const u32 len = (u32)(list_off[l + 1] - list_off[l]);
    na = n ? ceil_div(f, group) * ceil_div(min(len, capcodes), seg) : 0u;
    nb = n ? ceil_div(n, group) * ceil_div(len, seg) : 0u;
  };
  for (int l = tid; l < l0; l += 1024) {
    u32 n, f, na, nb;
    of(l, n, f, na, nb);
    b0 += n; b1 += na; b2 += nb;
  }
  for (int o = 32; o > 0; o >>= 1) { b0 += __shfl_down(b0, o, 64); b1 += __shfl_down(b1, o, 64); b2 += __shfl_down(b2, o, 64); }
  if (lane == 0) { wsum[0][wave] = b0; wsum[1][wave] = b1; wsum[2][wave] = b2; }
  __syncthreads();
  if (tid < 3) {
    u32 t = 0;
    for (int w = 0; w < 16; ++w) t += wsum[tid][w];
    base_s[tid] = t;
  }
  __syncthreads();
  const int l = l0 + tid;
  u32 n = 0, f = 0, na = 0, nb = 0;
  if (l < nlist) of(l, n, f, na, nb);
  u32 s0 = n, s1 = na, s2 = nb;      // inclusive scans
  for (int o = 1; o < 64; o <<= 1) {
    const u32 t0 = __shfl_up(s0, o, 64), t1 = __shfl_up(s1, o, 64), t2 = __shfl_up(s2, o, 64);
    if (lane >= o) { s0 += t0; s1 += t1; s2 += t2; }
  }
  if (lane == 63) { wsum[0][wave] = s0; wsum[1][wave] = s1; wsum[2][wave] = s2; }
  __syncthreads();
  u32 p0 = base_s[0], p1 = base_s[1], p2 = base_s[2];
  for (int w = 0; w < wave; ++w) { p0 += wsum[0][w]; p1 += wsum[1][w]; p2 += wsum[2][w]; }
  const u32 e0 = p0 + s0, e1 = p1 + s1, e2 = p2 + s2;     // one past this list's
  if (l < nlist) {
    off[l] = make_uint4(e0 - n, e1 - na, e2 - nb, 0u);
    if (l == nlist - 1) { nitems[0] = min(e1, max_a); nitems[1] = min(e2, max_b); }
  }
}

// The pairs grouped by list, the first ones of their queries in front, and the work items {list, first pair, pairs,
// segment}: the pairs of a group write one segment's item each, in turn.
__global__ __launch_bounds__(256) void ms_scatter_kernel(const int32_t* __restrict__ probes, int64_t npairs,
                                                         const u32* __restrict__ pair_slot, const u32* __restrict__ rank,
                                                         const u32* __restrict__ lfirst, const u32* __restrict__ lrest,
                                                         const uint4* __restrict__ off, const int64_t* __restrict__ list_off,
                                                         u32 group, u32 seg, u32 capcodes, uint4* __restrict__ items_a,
                                                         u32 max_a, uint4* __restrict__ items_b, u32 max_b,
                                                         u32* __restrict__ pairs) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= npairs) return;
  const u32 r = rank[i];
  if (r == 0xFFFFFFFFu) return;
  const u32 l = (u32)probes[i], f = lfirst[l], n = f + lrest[l];
  const bool first = pair_slot[i] != 0u;
  const uint4 o = off[l];
  const u32 at = first ? r : f + r, len = (u32)(list_off[l + 1] - list_off[l]);
  pairs[o.x + at] = (u32)i;
  auto items = [&](uint4* dst, u32 base, u32 most, u32 pos, u32 count, u32 nseg) {
    const u32 ng = ceil_div(count, group), g = pos / group, size = min(group, count - g * group);
    for (u32 s = pos - g * group; s < nseg; s += size) {
      const u32 w = base + s * ng + g;
      if (w < most) dst[w] = make_uint4(l, o.x + g * group, size, s);
    }
  };
  if (first) items(items_a, o.y, max_a, r, f, ceil_div(min(len, capcodes), seg));
  items(items_b, o.z, max_b, at, n, ceil_div(len, seg));
}

// ---- the sweeps ----------------------------------------------------------------------------------
struct SweepArgs {
  const float* qperm;           // [nq][kp] queries in fragment order
  int kp, npr, slots;           // slots: groups of four codes kept per query
  const void* cperm;            // [nlist][kp] centroids in fragment order: fp32 (PQ) or fp16 (the others)
  const uint4* items;
  const u32* nitems;
  const u32* pairs;
  const u32* pair_slot;
  const int64_t* list_off;
  const void* codes;            // rows / scalar codes, list-contiguous
  const uint8_t* units;         // PQ codes in units of 32 (see PqSide)
  const f16x2* cb16;            // PQ: fp16 codebook in granules
  int cb16_bytes;
  const float* vmin;            // SQ8
  const float* step;
  const u32* sigma_src;         // bits of the value that gives the scale (scale_of)
  int sigma_exp, sigma_sqrt;
  int form;                     // PQ: 0 residual tables, 1 inner product, 2 stored norms, 3 precomputed tables
  const float* cdist;           // [nq][npr] coarse values
  const float* cnorm;           // [nlist], forms 2 and 3
  const float* qbound;          // [nq] thresholds, scaled
  float* gmin;                  // [nq][slots]
  u32* cand_count;              // [nq]
  uint4* cand;                  // [nq][cap]: storage position, probe rank, bits of the lower and the upper bound
  int cap;
  u32 seg, capcodes;
  SlotMap map;
  float kappa, c4u, phi, phi2, abs_err, u2, sd;   // see sweep_args
  float norm_lo, norm_hi;       // PqSide::NORM: what the stored half norm is multiplied by, below and above 1
  const u32x4* tables;          // one-hot: [nq][M] entries of a sub-quantizer in steps, 16 signed bytes
  const float4* tinfo;          // one-hot: [nq] step, sum of the tables' middles, error bound
  float phi_c;                  // one-hot: rounding of the exact sum by the size of <q, c>
};

// The next item of this workgroup for this wavefront.  Items differ by the lengths of lists and the queries that probe
// them: dealt out to the wavefronts in turn as well, a few items each left half of them idle at the end of a sweep (eight
// wavefronts of a workgroup even out what one cannot: collect sweeps of 16 x 8 at 16 probes 91 -> 85 us, at 64 probes 159 ->
// 147, of 100 million 32 x 8 1190 -> 1142, of scalar codes 243 -> 229).  A counter in memory for all is no way: one address
// serves some 50 requests a microsecond, and the first requests of all wavefronts alone took 30 us with eight counters.
__device__ __forceinline__ u32 take_item(u32* taken) {
  constexpr u32 kWaves = kSweepThreads / VS_WAVE;
  u32 n = 0;
  if (lane_id() == 0) n = __hip_atomic_fetch_add((__attribute__((address_space(3))) u32*)taken, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  n = (u32)__builtin_amdgcn_readfirstlane((int)n);
  return (n / kWaves * gridDim.x + (u32)blockIdx.x) * kWaves + n % kWaves;
}

// power of two that scales the data: a vector of the norm (or a component of the size) `v` becomes 2^exp
// (nothing but zeros: as it is)
__device__ __forceinline__ float scale_of(u32 bits, int exp, int is_square) {
  const float v = __uint_as_float(bits);
  if (!(v > 0.f)) return 1.f;
  int e;
  (void)frexpf(is_square ? sqrtf(v) : v, &e);
  return ldexpf(1.f, exp - e);
}

// -- PQ codes.  A lane row g of the wavefront holds sub-quantizers g * MG .. g * MG + MG - 1 of its code: MG (or
// MG / 2) consecutive code bytes.  The codebook lies in LDS as granules of GB bytes (2, 4 or 8 halfs),
// [m][part][entry], so that a fragment of eight halfs is one, two or four look-ups.  Random look-ups of 8
// bytes by 64 lanes cost about twice the LDS cycles of conflict-free ones; per code there are M of them whatever
// the number of queries, which is what makes this cheaper than a table per query from two queries on.
//
// The codes are read from a copy in which a lane's bytes of two blocks of 16 codes lie next to each other and a
// unit of two blocks is consecutive memory: 1 instruction of 512 or 1024 consecutive bytes per unit.  Read from the
// lists themselves the bytes of a code, rotated by its position, took three 4-byte loads per lane and block, 27
// cycles of the address unit each -- two thirds of the sweep's time at 100M codes of 32 bytes.
constexpr __host__ __device__ int pq_lane_bytes(int cby) { return cby <= 2 ? 2 : (cby <= 4 ? 4 : (cby <= 8 ? 8 : 16)); }
template <int MG, int PARTS, int GB, int NBITS, bool ROT>
struct PqSide {
  static constexpr int KIND = kMsPq;
  static constexpr int GH = GB / 2, GPF = 8 / GH;               // halfs per granule, granules per fragment
  static constexpr int NGR = MG * PARTS;                        // granules per lane
  static constexpr int KS = (NGR + GPF - 1) / GPF;
  static constexpr int K = 1 << NBITS, M = 4 * MG;
  static constexpr int CBY = MG * NBITS / 8;                    // code bytes of a lane row
  static constexpr int CBP = pq_lane_bytes(CBY);                // ... as the blocked copy holds them
  static constexpr int NW = (2 * CBP + 3) / 4;                  // words per lane of a unit (two blocks of 16 codes)
  static constexpr bool NEED_C = false;                         // the stored side does not involve the centroid
  static constexpr bool UNITS = true;                           // codes come in units of two blocks
  // d / M = 3: the fourth half of a granule holds -|t|^2 / 2 and meets a constant on the query's side, so that the
  // product contains the stored vector's norm
  static constexpr bool NORM = ROT && MG == 8;
  static constexpr bool CHECK = false;                          // every codeword has a finite image (mscan_scale_fits)
  struct Raw { u32 w[NW]; };
  const uint8_t* units;                                         // this lane's bytes of unit 0
  const unsigned char* lut;                                     // this lane row's granules in LDS
  __device__ __forceinline__ static void stage(const SweepArgs& A, unsigned char* smem) {
    const u32x4* src = reinterpret_cast<const u32x4*>(A.cb16);
    u32x4* dst = reinterpret_cast<u32x4*>(smem);
    for (int i = threadIdx.x; i < A.cb16_bytes / 16; i += kSweepThreads) dst[i] = src[i];
  }
  __device__ __forceinline__ static int lds_bytes(const SweepArgs& A) { return A.cb16_bytes; }
  __device__ __forceinline__ void init(const SweepArgs& A, unsigned char* smem, int col, int g) {
    units = A.units;
    lane_at = (u32)(16 * g + col) * (2 * CBP);
    lut = smem + g * (NGR * K * GB);
  }
  u32 lane_at;
  __device__ __forceinline__ void begin_list(const SweepArgs&, int64_t, float, float&, float&) {}
  __device__ __forceinline__ Raw load(u64 unit) const {         // (wave-uniform)
    Raw r;
    const uint8_t* p = units + unit * (64 * 2 * CBP) + lane_at;
    if constexpr (NW == 1) r.w[0] = *reinterpret_cast<const u32*>(p);
    else if constexpr (NW == 2) { const u32x2 v = *reinterpret_cast<const u32x2*>(p); r.w[0] = v[0]; r.w[1] = v[1]; }
    else {
#pragma unroll
      for (int i = 0; i < NW / 4; ++i) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(p + 16 * i);
#pragma unroll
        for (int t = 0; t < 4; ++t) r.w[4 * i + t] = v[t];
      }
    }
    return r;
  }
  // block BLOCK (0 or 1) of a unit
  template <int BLOCK>
  __device__ __forceinline__ void decode(const Raw& r, float, f16x8 (&f)[KS]) const {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int h = 0; h < GPF; ++h) {
        const int j = s * GPF + h;
        if (j < NGR) {
          const int m = j / PARTS, part = j % PARTS;
          u32 c;
          if constexpr (NBITS == 8) c = (r.w[(BLOCK * CBP + m) >> 2] >> (8 * ((BLOCK * CBP + m) & 3))) & 0xFFu;
          else c = (r.w[(2 * BLOCK * CBP + m) >> 3] >> (4 * ((2 * BLOCK * CBP + m) & 7))) & 0xFu;
          const unsigned char* e = lut + (m * PARTS + part) * (K * GB) + c * GB;
          if constexpr (GB == 16) f[s] = *reinterpret_cast<const f16x8*>(e);
          else if constexpr (GB == 8) {
            const f16x4 v = *reinterpret_cast<const f16x4*>(e);
#pragma unroll
            for (int t = 0; t < 4; ++t) f[s][4 * h + t] = v[t];
          } else {
            const f16x2 v = *reinterpret_cast<const f16x2*>(e);
            f[s][2 * h] = v[0]; f[s][2 * h + 1] = v[1];
          }
        } else {
#pragma unroll
          for (int t = 0; t < GH; ++t) f[s][GH * h + t] = (_Float16)0.f;
        }
      }
    }
  }
};

// -- raw vectors, relative to the fp16 image of the list's centroid
template <int KSTEPS>
struct FlatSide {
  static constexpr int KIND = kMsFlat;
  static constexpr int KS = KSTEPS;
  static constexpr bool NEED_C = true, NORM = false, CHECK = true;
  static constexpr bool UNITS = false;
  struct Raw { f32x4 v[2 * KS]; };
  const float* rows;
  int d, g, col;
  f16x8 c16[KS];
  __device__ __forceinline__ static void stage(const SweepArgs&, unsigned char*) {}
  __device__ __forceinline__ static int lds_bytes(const SweepArgs&) { return 0; }
  __device__ __forceinline__ void init(const SweepArgs& A, unsigned char*, int col_, int g_) {
    rows = static_cast<const float*>(A.codes);
    d = A.map.d;
    g = g_;
    col = col_;
  }
  // c2: this lane's share of |c~|^2 (scaled); extra: nothing
  __device__ __forceinline__ void begin_list(const SweepArgs& A, int64_t l, float, float& c2, float&) {
    const f16x8* c = reinterpret_cast<const f16x8*>(static_cast<const _Float16*>(A.cperm) + l * A.kp) + g;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      c16[s] = c[4 * s];
#pragma unroll
      for (int t = 0; t < 8; ++t) c2 = __builtin_fmaf((float)c16[s][t], (float)c16[s][t], c2);
    }
  }
  __device__ __forceinline__ Raw load(u64 first, bool vec) const {
    Raw r;
    const unsigned char* p = reinterpret_cast<const unsigned char*>(rows + first * (u32)d);
    const u32 o = ((u32)col * (u32)d + 4u * (u32)g) * 4u;
    if (vec) {
#pragma unroll
      for (int h = 0; h < 2 * KS; ++h) {
        r.v[h] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (16 * h + 4 * g < d) r.v[h] = *reinterpret_cast<const f32x4*>(p + o + 64 * h);
      }
    } else {
#pragma unroll
      for (int h = 0; h < 2 * KS; ++h)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          r.v[h][t] = 0.f;
          if (16 * h + 4 * g + t < d) r.v[h][t] = *reinterpret_cast<const float*>(p + o + 64 * h + 4 * t);
        }
    }
    return r;
  }
  __device__ __forceinline__ void decode(const Raw& r, float sigma, f16x8 (&f)[KS]) const {
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int t = 0; t < 8; ++t)
        f[s][t] = (_Float16)((r.v[2 * s + (t >> 2)][t & 3] - (float)c16[s][t]) * sigma);
  }
};

// -- 8-bit scalar codes: reconstruction relative to the fp16 image of the list's centroid
template <int KSTEPS>
struct Sq8Side {
  static constexpr int KIND = kMsSq8;
  static constexpr int KS = KSTEPS;
  static constexpr bool NEED_C = true, NORM = false, CHECK = true;
  static constexpr bool UNITS = false;
  struct Raw { u32x2 v[KS]; };
  const uint8_t* codes;
  const float *step, *middle;    // LDS, [32 KS] each, scaled: cell width, middle of cell 0
  int d, g, col;
  f16x8 c16[KS];
  float off[8 * KS];             // scaled cell middle of code 0 minus centroid
  __device__ __forceinline__ static void stage(const SweepArgs& A, unsigned char* smem) {
    const float sigma = scale_of(*A.sigma_src, A.sigma_exp, A.sigma_sqrt);
    float* s = reinterpret_cast<float*>(smem);
    for (int t = threadIdx.x; t < 32 * KS; t += kSweepThreads) {
      s[t] = t < A.map.d ? A.step[t] * sigma : 0.f;
      s[32 * KS + t] = t < A.map.d ? __builtin_fmaf(0.5f, A.step[t], A.vmin[t]) * sigma : 0.f;
    }
  }
  __device__ __forceinline__ static int lds_bytes(const SweepArgs&) { return 64 * KS * (int)sizeof(float); }
  __device__ __forceinline__ void init(const SweepArgs& A, unsigned char* smem, int col_, int g_) {
    codes = static_cast<const uint8_t*>(A.codes);
    step = reinterpret_cast<const float*>(smem) + 8 * g_;
    middle = step + 32 * KS;
    d = A.map.d;
    g = g_;
    col = col_;
  }
  // extra: this lane's share of |middle|^2 + |255 step|^2 (scaled), the size of what the evaluations round
  __device__ __forceinline__ void begin_list(const SweepArgs& A, int64_t l, float sigma, float& c2, float& extra) {
    const f16x8* c = reinterpret_cast<const f16x8*>(static_cast<const _Float16*>(A.cperm) + l * A.kp) + g;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      c16[s] = c[4 * s];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float st = step[32 * s + t], mid = middle[32 * s + t];   // (scaled)
        const float cc = (float)c16[s][t];
        off[8 * s + t] = __builtin_fmaf(-cc, sigma, mid);
        c2 = __builtin_fmaf(cc, cc, c2);
        const float w = 255.f * st;
        extra = __builtin_fmaf(w, w, __builtin_fmaf(mid, mid, extra));
      }
    }
  }
  __device__ __forceinline__ Raw load(u64 first, bool vec) const {
    Raw r;
    const uint8_t* p = codes + first * (u32)d + (u32)col * (u32)d;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int dim = 32 * s + 8 * g;
      r.v[s] = u32x2{0u, 0u};
      if (vec) {                                                // d a multiple of 8
        if (dim < d) r.v[s] = *reinterpret_cast<const u32x2*>(p + dim);
      } else {
#pragma unroll
        for (int t = 0; t < 8; ++t)
          if (dim + t < d) r.v[s][t >> 2] |= (u32)p[dim + t] << (8 * (t & 3));
      }
    }
    return r;
  }
  __device__ __forceinline__ void decode(const Raw& r, float, f16x8 (&f)[KS]) const {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      // (read in every block: kept in registers the cell widths would cost eight of them per step)
      int at = 32 * s;
      asm volatile("" : "+s"(at));
      const f32x4 s0 = *reinterpret_cast<const f32x4*>(step + at), s1 = *reinterpret_cast<const f32x4*>(step + at + 4);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float code = (float)((r.v[s][t >> 2] >> (8 * (t & 3))) & 0xFFu);
        f[s][t] = (_Float16)__builtin_fmaf(code, t < 4 ? s0[t & 3] : s1[t & 3], off[8 * s + t]);
      }
    }
  }
};

// One wavefront per work item, nothing shared between wavefronts but the codebook in LDS: the item's
// queries (at most 16 NT) are converted into fragments that stay in registers, the segment's codes
// pass by in blocks of 16.  The product has the queries as rows and the codes as columns, so that lane l
// holds the products of code l mod 16 with queries 4 (l / 16) + i: the queries' terms start the
// accumulators, the code's term is one number per lane, and a block without a candidate costs one
// compare per four products.
template <class S, int METRIC, int MODE, int NT>
__global__ __launch_bounds__(kSweepThreads) __attribute__((amdgpu_waves_per_eu(S::KIND == kMsPq && S::KS <= 4 ? 4 : 2)))
void ms_sweep_kernel(const SweepArgs A) {
  constexpr int KS = S::KS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  S::stage(A, smem);
  u32* taken = reinterpret_cast<u32*>(smem + S::lds_bytes(A)) + (kSweepThreads / VS_WAVE) * queue_words(NT);
  if (threadIdx.x == 0) *taken = kSweepThreads / VS_WAVE;
  __syncthreads();
  const int lane = lane_id(), col = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
  typedef __attribute__((address_space(3))) volatile u32* lds_u32_ptr;
  // this wavefront's queue: (query of the item << 26 | code of the segment), margin, code's term; and the
  // terms of the item's queries that the bounds are formed from
  u32* qmem = reinterpret_cast<u32*>(smem + S::lds_bytes(A)) + wave * queue_words(NT);
  const lds_u32_ptr queue = (lds_u32_ptr)qmem, qrow = (lds_u32_ptr)(qmem + 3 * kQueue);
  S side;
  side.init(A, smem, col, g);
  const bool vec = S::KIND == kMsFlat ? (A.map.d & 3) == 0 : (A.map.d & 7) == 0;
  const float sigma = scale_of(*A.sigma_src, A.sigma_exp, A.sigma_sqrt), sigma2 = sigma * sigma;
  const u32 nitems = *A.nitems;
  const float inf = __builtin_inff();

  // Items are dealt out to workgroups in turn, neighbours (groups of one list, segments of one list) to the same one,
  // and its wavefronts take the next one when they are through with theirs (take_item).  The next item's list and
  // pairs are fetched during this one's codes.
  u32 item = (u32)blockIdx.x * (kSweepThreads / VS_WAVE) + (u32)__builtin_amdgcn_readfirstlane(wave);
  if (item >= nitems) return;
  uint4 it = A.items[item];
  u32 lb = (u32)A.list_off[it.x], len = (u32)A.list_off[it.x + 1] - lb;
  u32 pr[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) pr[t] = A.pairs[it.y + min((u32)(t * 16 + col), it.z - 1)];
  for (;;) {
    const u32 l = it.x, sg = it.w;
    const int np = (int)it.z;
    const u32 next = take_item(taken);
    if (MODE == 0) len = min(len, A.capcodes);
    const u32 cb = lb + sg * A.seg, cn = min(len - sg * A.seg, A.seg);   // the segment: cn codes from cb on
    const int nb = (int)((cn + 15) >> 4), nt = (np + 15) >> 4;
    const uint4 nit = A.items[min(next, nitems - 1)];

    // (lanes past the end read what follows -- the store is that much longer -- and are masked)
    const u64 unit0 = (u64)(lb >> 5) + l + (sg * A.seg >> 5);
    auto fetch = [&](int i) {                                   // UNITS: unit i of the segment, else: block i
      if constexpr (S::UNITS) return side.load(unit0 + (u32)i);
      else return side.load((u64)cb + 16u * (u32)i, vec);
    };
    typename S::Raw raw0 = fetch(0), raw1;
    const int nu = (nb + 1) >> 1;
    if constexpr (S::UNITS) raw1 = fetch(nu > 1 ? 1 : 0);

    // -- the queries
    float c2 = 0.f, extra = 0.f;
    side.begin_list(A, (int64_t)l, sigma, c2, extra);
    c2 = sum_rows(c2) * sigma2;
    extra = sum_rows(extra);
    f16x8 qa[NT][KS];
    float a2[NT], cd[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) a2[t] = cd[t] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      float cf[8];
      if constexpr (S::NEED_C) {
#pragma unroll
        for (int t = 0; t < 8; ++t) cf[t] = (float)side.c16[s][t];
      } else if constexpr (METRIC == 0) {
        const float* src = static_cast<const float*>(A.cperm) + (u64)l * (u32)A.kp + 32 * s + 8 * g;
        const f32x4 v0 = *reinterpret_cast<const f32x4*>(src), v1 = *reinterpret_cast<const f32x4*>(src + 4);
#pragma unroll
        for (int t = 0; t < 8; ++t) cf[t] = t < 4 ? v0[t & 3] : v1[t & 3];
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t >= nt) continue;
        const float* src = A.qperm + (u64)(pr[t] / (u32)A.npr) * (u32)A.kp + 32 * s + 8 * g;
        const f32x4 v0 = *reinterpret_cast<const f32x4*>(src), v1 = *reinterpret_cast<const f32x4*>(src + 4);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          float v = i < 4 ? v0[i & 3] : v1[i & 3];
          if (METRIC == 0) v -= cf[i];
          else if (S::NEED_C) cd[t] = __builtin_fmaf(v, cf[i], cd[t]);
          qa[t][s][i] = (_Float16)(v * sigma);
        }
        a2[t] = dot8(qa[t][s], qa[t][s], a2[t]);
        if (S::NORM && METRIC == 0) qa[t][s][3] = qa[t][s][7] = (_Float16)(MODE == 0 ? A.norm_hi : A.norm_lo);
      }
    }
    // terms of a row (lane: query col of the tile), then of the rows 4 g + i that the lane's products belong to
    f32x4 ai[NT], bi[NT];
    wave_lds_sync();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t >= nt) continue;
      a2[t] = sum_rows(a2[t]);
      float arow, brow = 0.f;
      const u32 qi = pr[t] / (u32)A.npr;
      float ex = A.abs_err;
      bool bad = !(a2[t] < 1.0e30f);
      if (S::KIND == kMsSq8) bad = bad || !(extra < 0x1p40f);   // (cells far beyond what they code: middle and width below 2^60)
      if (METRIC == 0) {
        if (S::KIND == kMsPq && A.form >= 2) {
          ex += A.phi2 * (6.f * A.cnorm[l] + 4.f * A.cdist[pr[t]]) * sigma2;
          bad = bad || !(A.cnorm[l] < 0x1p119f);                // (|x'|^2 and the sums it enters stay finite)
        }
        if (S::KIND == kMsSq8) ex += 0x1p-31f * extra;
        bad = bad || !(ex < 1.0e30f);
        if (MODE == 0) arow = __builtin_fmaf(1.f + A.c4u + A.kappa, a2[t], ex);
        else arow = 0.5f * (A.qbound[qi] * (1.f + A.c4u) + ex - (1.f - A.kappa) * a2[t]);
        ex = __builtin_fmaf(A.kappa, a2[t], ex);
      } else {
        const float an = sqrtf(a2[t] + A.abs_err);
        float c;
        if constexpr (S::NEED_C) {
          c = sum_rows(cd[t]) * sigma2;
          ex += 2.f * A.phi * an * sqrtf(c2);
          if (S::KIND == kMsSq8) ex += 2.f * A.phi * an * sqrtf(extra);
        } else {
          c = A.cdist[pr[t]];
          bad = bad || !(fabsf(c) < 0x1p119f);
          c *= sigma2;
        }
        ex += A.phi * fabsf(c);
        bad = bad || !(fabsf(c) < 1.0e30f) || !(ex < 1.0e30f);
        brow = an + A.sd / A.u2;
        if (MODE == 0) arow = ex - c;
        else { const float U = A.qbound[qi]; arow = c + ex + U + A.phi * fabsf(U); }
      }
      if (bad) {
        arow = inf; brow = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
          for (int i = 0; i < 8; ++i) qa[t][s][i] = (_Float16)0.f;
      }
      // (the four lanes of a row agree on `bad`: a2, c and ex are the same numbers in all of them)
      if (MODE == 0) {
        if (g == 0) {   // where the row's values go, how many, and what is added to them
          const u32 sl = t * 16 + col < np ? A.pair_slot[pr[t]] : 0u;
          queue[3 * (t * 16 + col)] = qi * (u32)A.slots + (sl & 0xFFFFu);
          queue[3 * (t * 16 + col) + 1] = sl >> 16;
          queue[3 * (t * 16 + col) + 2] = __float_as_uint(arow);
        }
      } else {
        if (t * 16 + col >= np) arow = -inf;
        if (g == 0) {   // what a candidate's record is formed from (an infinite term: no bounds)
          qrow[2 * (t * 16 + col)] = __float_as_uint(bad ? inf : ex);
          qrow[2 * (t * 16 + col) + 1] = __float_as_uint(brow);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (MODE == 1) ai[t][i] = __shfl(arow, 4 * g + i, 64);
        if (METRIC == 1) bi[t][i] = __shfl(brow, 4 * g + i, 64);
      }
    }
    wave_lds_sync();
    // the next item's list and pairs
    const u32 nlb = (u32)A.list_off[nit.x], nlen = (u32)A.list_off[nit.x + 1] - nlb;
#pragma unroll
    for (int t = 0; t < NT; ++t) pr[t] = A.pairs[nit.y + min((u32)(t * 16 + col), nit.z - 1)];

    // -- the codes
    int queued = 0;                                             // MODE 1
    f32x4 best[NT];                                             // MODE 0
#pragma unroll
    for (int t = 0; t < NT; ++t) best[t] = f32x4{inf, inf, inf, inf};
    // queued candidates to their queries' buffers, with a lower and an upper bound of their exact value: one atomic per
    // query of up to 64 candidates
    auto flush = [&]() {
      wave_lds_sync();
      for (int e0 = 0; e0 < queued; e0 += VS_WAVE) {
        const bool on = e0 + lane < queued;
        const u32 e = on ? queue[3 * (e0 + lane)] : 0u;
        const float z = on ? __uint_as_float(queue[3 * (e0 + lane) + 1]) : 0.f;
        const float w = on ? __uint_as_float(queue[3 * (e0 + lane) + 2]) : 0.f;
        const u32 lp = e >> 26;
        const float ra = __uint_as_float(qrow[2 * lp]), rb = __uint_as_float(qrow[2 * lp + 1]);
        const u32 prn = A.pairs[it.y + lp];
        const u32 qi = prn / (u32)A.npr, p = prn - qi * (u32)A.npr;
        const u64 same = same_lanes(on, lp);
        const int first = on ? (int)__builtin_ctzll(same) : 0;
        u32 at = 0;
        if (on && lane == first) at = atomicAdd(&A.cand_count[qi], (u32)__popcll(same));
        const float U = A.qbound[qi];
        float lo, hi;
        if (METRIC == 0) {
          lo = U - 2.f * z;                                     // (z >= 0 over 1 + 4 u would be exact)
          const float dh = lo + A.c4u * fabsf(U);
          // (the norm inside the product: 1 - norm_lo too small, and rounded)
          hi = __builtin_fmaf(dh, 1.f + A.c4u, 2.02f * (ra + (S::NORM ? A.kappa + A.norm_hi - A.norm_lo : A.kappa) * w));
        } else {
          lo = U - z;
          hi = lo + 2.02f * (ra + rb * w) + 2.f * A.phi * fabsf(U);
        }
        if (!(fabsf(lo) < 1.0e30f) || !(fabsf(hi) < 1.0e30f)) { lo = -inf; hi = inf; }
        at = __shfl(at, first, 64) + (u32)__popcll(same & ((1ull << lane) - 1ull));
        if (on && at < (u32)A.cap)
          A.cand[(u64)qi * (u32)A.cap + at] = make_uint4(cb + (e & 0x3FFFFFFu), p, __float_as_uint(lo), __float_as_uint(hi));
      }
      queued = 0;
      wave_lds_sync();
    };
    auto block = [&](int b, f16x8 (&f)[KS]) {
      f32x4 acc[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = MODE == 1 ? ai[t] : f32x4{0.f, 0.f, 0.f, 0.f};
      float b2 = 0.f;
      bool badcode = false;
      u64 anybad = 0;
      if constexpr (!(S::NORM && METRIC == 0)) {
#pragma unroll
        for (int s = 0; s < KS; ++s) b2 = dot8(f[s], f[s], b2);
        b2 = sum_rows(b2);
      }
      if constexpr (S::CHECK) {
        badcode = !(b2 < 1.0e30f);
        anybad = __builtin_amdgcn_ballot_w64(badcode);
        if (anybad != 0 && badcode) {
#pragma unroll
          for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int i = 0; i < 8; ++i) f[s][i] = (_Float16)0.f;
          b2 = 0.f;
        }
      }
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          if (t < nt) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[t][s], f[s], acc[t], 0, 0, 0);
      if (MODE == 0) {
        const float w = METRIC == 0 ? (1.f + A.c4u + A.kappa) * b2 : __builtin_fmaf(A.u2, sqrtf(b2 + A.abs_err), A.sd);
        const float kill = 16u * (u32)b + (u32)col < cn && !badcode ? 0.f : inf;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t >= nt) continue;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float v;
            if (METRIC == 0) v = __builtin_fmaf(-2.f * (1.f + A.c4u), acc[t][i], w);
            else v = __builtin_fmaf(bi[t][i], w, -acc[t][i]);
            best[t][i] = fminf(best[t][i], v + kill);
          }
        }
        if ((b & 3) == 3 || b + 1 == nb) {
          const u32 at = (sg * A.seg >> 6) * 16u + (u32)(b >> 2) * 16u + (u32)col;
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            if (t >= nt) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int row = 3 * (t * 16 + 4 * g + i);
              const float v = best[t][i] + __uint_as_float(queue[row + 2]);
              if (at < queue[row + 1]) A.gmin[queue[row] + at] = v < inf ? v : inf;
              best[t][i] = inf;
            }
          }
        }
      } else {
        const float w = METRIC == 0 ? 0.5f * (1.f - A.kappa) * b2 : __builtin_fmaf(A.u2, sqrtf(b2 + A.abs_err), A.sd);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t >= nt) continue;
          float z[4];
          u64 m = anybad;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            z[i] = METRIC == 0 ? acc[t][i] : __builtin_fmaf(bi[t][i], w, acc[t][i]);
            m |= __builtin_amdgcn_ballot_w64(z[i] >= (METRIC == 0 ? w : 0.f));
          }
          if (m == 0) continue;
          const u32 rel = 16u * (u32)b + (u32)col;
          const bool valid = rel < cn;
          float bq = METRIC == 0 ? b2 : w;
          if constexpr (S::NORM && METRIC == 0) {               // |b^|^2 without the norm's own halves
#pragma unroll
            for (int s = 0; s < KS; ++s) {
              const f16x2 minus2 = {(_Float16)0.f, (_Float16)-2.f}, n0 = {f[s][2], f[s][3]}, n1 = {f[s][6], f[s][7]};
              bq = __builtin_amdgcn_fdot2(n0, minus2, bq, false);
              bq = __builtin_amdgcn_fdot2(n1, minus2, bq, false);
            }
            bq = sum_rows(bq);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int lp = t * 16 + 4 * g + i;
            if (METRIC == 0) z[i] -= w;
            const bool pass = (z[i] >= 0.f || badcode) && valid && lp < np;
            const u64 mask = __builtin_amdgcn_ballot_w64(pass);
            if (mask == 0) continue;
            if (queued + VS_WAVE > kQueue) flush();
            if (pass) {
              const int at = 3 * (queued + (int)__popcll(mask & ((1ull << lane) - 1ull)));
              queue[at] = ((u32)lp << 26) | rel;
              queue[at + 1] = __float_as_uint(badcode ? inf : z[i]);
              queue[at + 2] = __float_as_uint(bq);
            }
            queued += (int)__popcll(mask);
          }
        }
      }
    };
    if constexpr (S::UNITS) {                                   // codes two units ahead
      // (Left to itself the compiler does not inline a block of a single step: its operands then pass through scratch,
      // 454 us for 59.  Inlined as early as that the larger ones get a worse schedule: 172 -> 262 us at rows of 128.)
      auto unit = [&](const typename S::Raw& raw, int u) {
        {
          f16x8 f[KS];
          side.template decode<0>(raw, sigma, f);
          if constexpr (KS == 1) [[clang::always_inline]] block(2 * u, f);
          else block(2 * u, f);
        }
        if (2 * u + 1 < nb) {
          f16x8 f[KS];
          side.template decode<1>(raw, sigma, f);
          if constexpr (KS == 1) [[clang::always_inline]] block(2 * u + 1, f);
          else block(2 * u + 1, f);
        }
      };
      for (int u = 0; u < nu; u += 2) {
        unit(raw0, u);
        if (u + 2 < nu) raw0 = fetch(u + 2);
        if (u + 1 < nu) {
          unit(raw1, u + 1);
          if (u + 3 < nu) raw1 = fetch(u + 3);
        }
      }
    } else {                                                    // one block: a row's floats fill as many registers as its fragments twice
      for (int b = 0; b < nb; ++b) {
        f16x8 f[KS];
        side.decode(raw0, sigma, f);
        if (b + 1 < nb) raw0 = fetch(b + 1);
        block(b, f);
      }
    }
    if (MODE == 1 && queued > 0) flush();
    if (next >= nitems) break;
    item = next;
    it = nit;
    lb = nlb;
    len = nlen;
  }
}

// ---- 4-bit codes, inner product, long sub-vectors -------------------------------------------------------
// A stored vector's score is a sum of one table entry per sub-quantizer, that is the product of the query's M x 16 table
// and a vector with a one in each of its M blocks of 16.  Decoding sub-vectors of 12 dimensions costs three look-ups per
// sub-quantizer and 24 matrix steps for 64 of them; one-hot rows cost one conflict-free look-up of 16 bytes (an entry is
// its own set of banks) and 16 steps of the 8-bit matrix product, which run at twice the rate, and need neither the
// centroid nor a copy of the codes.  The table is rounded to steps of 1 / 127 of its largest deviation from the
// sub-quantizers' middles; what that loses, at most half a step per sub-quantizer, is some tenth of the scores' spread.
// One lane per (query, sub-quantizer) and two such pairs at a time: the sixteen entries by the canon chain (the exact
// evaluation's bits, kept for it), rounded, and written as one piece.  The codebook lies in LDS, a sub-quantizer's
// codewords consecutive; V: dsub is a multiple of four and they are read 16 bytes at a time.
// (10,000 queries of 64 x 12: 36 us; a lane per entry, every extremum over 16 lanes, 75.)
__host__ __device__ constexpr int onehot_row(int dsub) { return 16 * dsub + (dsub % 4 == 0 ? 4 : 1); }   // floats; spreads the lanes over the banks
template <int MG, bool V>
__global__ __launch_bounds__(256) void ms_onehot_tables_kernel(const float* __restrict__ q, int64_t nq, int d, int dsub,
                                                               const float* __restrict__ codebooks, float eps_scale,
                                                               int passes, u32x4* __restrict__ tables,
                                                               float* __restrict__ exact, float4* __restrict__ tinfo) {
  constexpr int M = 4 * MG, QW = 64 / M, Q = 2;                  // queries of a wavefront side by side; in turn
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* T = reinterpret_cast<float*>(smem);
  const int row = onehot_row(dsub), wave = threadIdx.x >> 6, lane = lane_id(), m = lane % M;
  for (int r = wave; r < M; r += 4) {
    if constexpr (V) {
#pragma unroll 4
      for (int e = lane; e < 4 * dsub; e += VS_WAVE)
        reinterpret_cast<f32x4*>(T + r * row)[e] = reinterpret_cast<const f32x4*>(codebooks + r * 16 * dsub)[e];
    } else {
      for (int e = lane; e < 16 * dsub; e += VS_WAVE) T[r * row + e] = codebooks[r * 16 * dsub + e];
    }
  }
  __syncthreads();
  const float* Tm = T + m * row;
  auto over_m = [](float v, auto op) {                           // over the M lanes of a query
    for (int o = 1; o < M; o <<= 1) v = op(v, __shfl_xor(v, o));
    return v;
  };
  auto sum = [](float x, float y) { return x + y; };
  auto larger = [](float x, float y) { return fmaxf(x, y); };
  for (int pass = 0; pass < passes; ++pass) {
    const int64_t q0 = (((int64_t)blockIdx.x * 4 + wave) * passes + pass) * (Q * QW) + lane / M * Q;
    const float* qp[Q];
#pragma unroll
    for (int r = 0; r < Q; ++r) qp[r] = q + min(q0 + r, nq - 1) * d + m * dsub;
    float e[Q][16];
#pragma unroll
    for (int r = 0; r < Q; ++r)
#pragma unroll
      for (int j = 0; j < 16; ++j) e[r][j] = 0.f;
    for (int u = 0; u < dsub; u += V ? 4 : 1) {
      float x[Q][V ? 4 : 1];
#pragma unroll
      for (int r = 0; r < Q; ++r)
#pragma unroll
        for (int w = 0; w < (V ? 4 : 1); ++w) x[r][w] = qp[r][u + w];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        if constexpr (V) {
          const float4 t = *reinterpret_cast<const float4*>(Tm + j * dsub + u);
#pragma unroll
          for (int r = 0; r < Q; ++r)
            e[r][j] = __builtin_fmaf(x[r][3], t.w, __builtin_fmaf(x[r][2], t.z, __builtin_fmaf(x[r][1], t.y, __builtin_fmaf(x[r][0], t.x, e[r][j]))));
        } else {
          const float t = Tm[j * dsub + u];
#pragma unroll
          for (int r = 0; r < Q; ++r) e[r][j] = __builtin_fmaf(x[r][0], t, e[r][j]);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < Q; ++r) {
      const int64_t qi = q0 + r;
      float hi = e[r][0], lo = hi;
      bool fine = true;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        hi = fmaxf(hi, e[r][j]);
        lo = fminf(lo, e[r][j]);
        fine = fine && __builtin_fabsf(e[r][j]) < 1.0e30f;
      }
      const float mid = 0.5f * (lo + hi);
      const float step = fmaxf(over_m(fmaxf(hi - mid, mid - lo), larger) * (1.f / 127.f), 1.0e-36f), inv = 1.f / step;
      u32x4 out = {0u, 0u, 0u, 0u};
      float err = 0.f;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float off = e[r][j] - mid, v = fine ? fminf(fmaxf(rintf(off * inv), -127.f), 127.f) : 0.f;
        err = fmaxf(err, __builtin_fabsf(off - v * step));
        out[j >> 2] |= ((u32)(int)v & 0xFFu) << (8 * (j & 3));
      }
      const float size = over_m(fmaxf(__builtin_fabsf(lo), __builtin_fabsf(hi)), sum), base = over_m(mid, sum);
      const float bad = over_m(fine ? 0.f : 1.f, larger);
      // (the middles, their sum, an entry's deviation and the M additions of the exact sum each round by 2^-24 of `size`)
      err = eps_scale * (over_m(err, sum) * 1.0001f + (2 * M + 16) * 0x1p-23f * size);
      if (qi >= nq) continue;
      tables[qi * M + m] = out;
      f32x4* to = reinterpret_cast<f32x4*>(exact + (qi * M + m) * 16);
#pragma unroll
      for (int j = 0; j < 16; j += 4) to[j >> 2] = f32x4{e[r][j], e[r][j + 1], e[r][j + 2], e[r][j + 3]};
      if (m == 0) tinfo[qi] = bad != 0.f || !(size < 1.0e30f) ? make_float4(step, 0.f, __builtin_inff(), 0.f) : make_float4(step, base, err, 0.f);
    }
  }
}

// What those tables lose, before any query is there: sampled centroids in their place, a wavefront each, a lane per
// sub-quantizer.  The error is set against the spread that the sums would have if every sub-quantizer were like the middle
// one: those that set the step stand out, and codes that agree in them are what the bounds have to tell apart.
__global__ __launch_bounds__(256) void ms_onehot_slack_kernel(const float* __restrict__ centroids, int64_t nlist, int d, int M,
                                                              int dsub, const float* __restrict__ codebooks,
                                                              float* __restrict__ out) {
  const int lane = lane_id(), m = lane & (M - 1), s = (int)blockIdx.x * 4 + (threadIdx.x >> 6);
  const float* __restrict__ q = centroids + s * nlist / kOnehotSamples * d + m * dsub;
  const float* __restrict__ t = codebooks + m * 16 * dsub;
  float e[16] = {};
  for (int u = 0; u < dsub; ++u) {
    const float x = q[u];
#pragma unroll
    for (int j = 0; j < 16; ++j) e[j] = __builtin_fmaf(x, t[j * dsub + u], e[j]);
  }
  float hi = e[0], lo = e[0];
  bool fine = true;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    hi = fmaxf(hi, e[j]);
    lo = fminf(lo, e[j]);
    fine = fine && __builtin_fabsf(e[j]) < 1.0e30f;
  }
  const float dev = 0.5f * (hi - lo);
  float most = dev;                                              // (lanes from M on repeat the others)
  for (int o = 1; o < VS_WAVE; o <<= 1) most = fmaxf(most, __shfl_xor(most, o));
  const float inv = 1.f / most;                                  // (everything in units of it: squares stay in range)
  float mean = 0.f, var = 0.f, err = fminf(dev * inv, 0.5f / 127.f);
#pragma unroll
  for (int j = 0; j < 16; ++j) mean += (e[j] - lo) * inv;
  mean *= 1.f / 16.f;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const float off = (e[j] - lo) * inv - mean;
    var += off * off;
  }
  var *= 1.f / 16.f;
  for (int o = 1; o < M; o <<= 1) err += __shfl_xor(err, o);
  int smaller = 0;
  for (int o = 0; o < M; ++o) {
    const float other = __shfl(var, o);
    smaller += other < var || (other == var && o < m);
  }
  const u64 middle = __builtin_amdgcn_ballot_w64(smaller == M / 2);
  const float typical = __shfl(var, middle ? (int)__builtin_ctzll(middle) : 0);
  const float share = err / sqrtf((float)M * typical);
  if (lane == 0) out[s] = __builtin_amdgcn_ballot_w64(!fine) == 0 && share < 1.0e30f ? share : __builtin_inff();
}

// The sweeps, like ms_sweep_kernel: queries as rows, codes as columns.  A lane's MG sub-quantizers g * MG .. are read
// from the codes themselves, 16 of which are consecutive memory.
// 16384 lists of 610 codes of 64 x 4 bits, 10,000 queries x 32 probes: the query-major scan, a table per query in LDS and 64
// look-ups per pair, takes 1240 us; this one 90 for its bounds and 320 for the candidates (one look-up in flight: 420),
// and 60 for their exact evaluation.  Matrix cores and LDS are busy 40 % of the time each; 44 % of the wavefronts' time
// is the wait for an item's 32 KB of tables, which nothing but the SIMD's other wavefront hides.
template <int MG, int MODE, int NT>
__global__ __launch_bounds__(kSweepThreads) __attribute__((amdgpu_waves_per_eu(2)))
void ms_onehot_sweep_kernel(const SweepArgs A) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  constexpr int M = 4 * MG, CB = MG / 2, NW = (CB + 3) / 4, AHEAD = 3;
  constexpr int kNone = -(1 << 30);
  // (an array of its own: its address is a constant that the look-ups carry as their offset)
  __shared__ __attribute__((aligned(256))) u32 hot[64];
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if (threadIdx.x < 64)
    hot[threadIdx.x] = (threadIdx.x >> 4) == (threadIdx.x & 3) ? 1u << (8 * ((threadIdx.x >> 2) & 3)) : 0u;
  u32* taken = reinterpret_cast<u32*>(smem) + (kSweepThreads / VS_WAVE) * (2 * kQueue + 64 * NT);
  if (threadIdx.x == 0) *taken = kSweepThreads / VS_WAVE;
  __syncthreads();
  const int lane = lane_id(), col = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
  typedef __attribute__((address_space(3))) volatile u32* lds_u32_ptr;
  u32* qmem = reinterpret_cast<u32*>(smem) + wave * (2 * kQueue + 64 * NT);
  // candidates: (query of the item << 26 | code of the segment), sum; and per query of the item what a bound is formed
  // from (MODE 0: place, groups, ...): centre, step, error, threshold
  const lds_u32_ptr queue = (lds_u32_ptr)qmem, qrow = (lds_u32_ptr)(qmem + 2 * kQueue);
  const u32 nitems = *A.nitems;
  const float inf = __builtin_inff();
  const uint8_t* codes = static_cast<const uint8_t*>(A.codes);
  const u32 lane_at = (u32)col * (2 * MG) + (u32)g * CB;
  struct Raw { u32 w[NW]; };
  auto load = [&](u64 first) {
    Raw r;
    const uint8_t* p = codes + first * (2 * MG) + lane_at;
    if constexpr (CB == 8) { const u32x2 v = *reinterpret_cast<const u32x2*>(p); r.w[0] = v[0]; r.w[1] = v[1]; }
    else if constexpr (CB == 4) r.w[0] = *reinterpret_cast<const u32*>(p);
    else r.w[0] = *reinterpret_cast<const unsigned short*>(p);
    return r;
  };

  u32 item = (u32)blockIdx.x * (kSweepThreads / VS_WAVE) + (u32)__builtin_amdgcn_readfirstlane(wave);
  if (item >= nitems) return;
  uint4 it = A.items[item];
  u32 lb = (u32)A.list_off[it.x], len = (u32)A.list_off[it.x + 1] - lb;
  u32 pr[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) pr[t] = A.pairs[it.y + min((u32)(t * 16 + col), it.z - 1)];
  for (;;) {
    const u32 sg = it.w;
    const int np = (int)it.z;
    const u32 next = take_item(taken);
    if (MODE == 0) len = min(len, A.capcodes);
    const u32 cb = lb + sg * A.seg, cn = min(len - sg * A.seg, A.seg);   // the segment: cn codes from cb on
    const int nb = (int)((cn + 15) >> 4), nt = (np + 15) >> 4;
    const uint4 nit = A.items[min(next, nitems - 1)];
    // (lanes past the end read what follows -- the store is 16 codes longer -- and are masked)
    Raw raw[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) raw[i] = load((u64)cb + 16u * (u32)min(i, nb - 1));

    // -- the queries' tables, and their terms (lane: query col of the tile)
    i32x4 qa[NT][MG];
    i32x4 start[NT];
    wave_lds_sync();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t >= nt) continue;
      const u32 qi = pr[t] / (u32)A.npr;
#pragma unroll
      for (int s = 0; s < MG; ++s) qa[t][s] = __builtin_bit_cast(i32x4, A.tables[(u64)qi * M + g * MG + s]);
      const float4 ti = A.tinfo[qi];
      const float c = A.cdist[pr[t]], centre = c + ti.y;
      float ex = ti.z + A.phi_c * __builtin_fabsf(c) + 0x1p-20f * (__builtin_fabsf(c) + __builtin_fabsf(ti.y)) + 1.0e-36f;
      if (!(__builtin_fabsf(centre) < 1.0e30f) || !(ex < 1.0e30f)) ex = inf;
      const int at = t * 16 + col;
      int from = kNone;                                           // sums from here on are candidates
      if (MODE == 1) {
        const float U = A.qbound[qi];
        const float x = -(centre + U + ex + 0x1p-20f * __builtin_fabsf(U)) / ti.x;
        // (an infinite bound, a NaN: everything)
        if (x > -20000.f && ex < inf) from = (int)fminf(floorf(x) - 1.f, 20000.f);
        if (at >= np) from = 1 << 20;
      }
      if (g == 0) {
        if (MODE == 0) {
          const u32 sl = at < np ? A.pair_slot[pr[t]] : 0u;
          qrow[4 * at] = qi * (u32)A.slots + (sl & 0xFFFFu);
          qrow[4 * at + 1] = sl >> 16;
          qrow[4 * at + 2] = __float_as_uint(ex - centre);
          qrow[4 * at + 3] = __float_as_uint(ti.x);
        } else {
          qrow[4 * at] = __float_as_uint(centre);
          qrow[4 * at + 1] = __float_as_uint(ti.x);
          qrow[4 * at + 2] = __float_as_uint(ex);
          qrow[4 * at + 3] = (u32)from;
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) start[t][i] = MODE == 1 ? -__shfl(from, 4 * g + i, 64) : 0;
    }
    wave_lds_sync();
    const u32 nlb = (u32)A.list_off[nit.x], nlen = (u32)A.list_off[nit.x + 1] - nlb;
#pragma unroll
    for (int t = 0; t < NT; ++t) pr[t] = A.pairs[nit.y + min((u32)(t * 16 + col), nit.z - 1)];

    int queued = 0;
    i32x4 best[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) best[t] = i32x4{kNone, kNone, kNone, kNone};
    auto flush = [&]() {
      wave_lds_sync();
      for (int e0 = 0; e0 < queued; e0 += VS_WAVE) {
        const bool on = e0 + lane < queued;
        const u32 e = on ? queue[2 * (e0 + lane)] : 0u;
        const int sum = on ? (int)queue[2 * (e0 + lane) + 1] : 0;
        const u32 lp = e >> 26;
        const float centre = __uint_as_float(qrow[4 * lp]), step = __uint_as_float(qrow[4 * lp + 1]), ex = __uint_as_float(qrow[4 * lp + 2]);
        const u32 prn = A.pairs[it.y + lp];
        const u32 qi = prn / (u32)A.npr, p = prn - qi * (u32)A.npr;
        const u64 same = same_lanes(on, lp);
        const int first = on ? (int)__builtin_ctzll(same) : 0;
        u32 at = 0;
        if (on && lane == first) at = atomicAdd(&A.cand_count[qi], (u32)__popcll(same));
        const float dev = step * (float)(sum + (int)qrow[4 * lp + 3]), v = -(centre + dev), sl = ex + 0x1p-20f * __builtin_fabsf(dev);
        float lo = v - sl, hi = v + sl;
        if (!(fabsf(lo) < 1.0e30f) || !(fabsf(hi) < 1.0e30f)) { lo = -inf; hi = inf; }
        at = __shfl(at, first, 64) + (u32)__popcll(same & ((1ull << lane) - 1ull));
        if (on && at < (u32)A.cap)
          A.cand[(u64)qi * (u32)A.cap + at] = make_uint4(cb + (e & 0x3FFFFFFu), p, __float_as_uint(lo), __float_as_uint(hi));
      }
      queued = 0;
      wave_lds_sync();
    };
    // all blocks of the segment against `count` tiles of queries
    auto sweep = [&](auto count) {
      constexpr int N = decltype(count)::value;
      // Rows of a block are looked up PF steps ahead of their products, into the next block's: with the one or two in
      // flight that the compiler leaves, every step waited for the LDS.
      constexpr int PF = MG >= 8 ? 6 : 4;
      static_assert(AHEAD * MG % PF == 0, "the ring begins anew with raw[0]");
      i32x4 ring[PF];
      auto look_up = [&](const Raw& r, int s) {
        const u32 w = r.w[s >> 3], at = ((s & 7) == 0 ? w << 4 : w >> (4 * ((s & 7) - 1))) & 0xF0u;
        return *reinterpret_cast<const i32x4*>(reinterpret_cast<const unsigned char*>(hot) + at);
      };
      // (block i of AHEAD: rows of block b lie in the ring from i * MG on)
      auto block = [&](int b, int i, const Raw& r, const Raw& after) {
        i32x4 acc[N];
#pragma unroll
        for (int t = 0; t < N; ++t) acc[t] = start[t];
#pragma unroll
        for (int s = 0; s < MG; ++s) {
          const int at = (i * MG + s) % PF;
#pragma unroll
          for (int t = 0; t < N; ++t) acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(qa[t][s], ring[at], acc[t], 0, 0, 0);
          ring[at] = s + PF < MG ? look_up(r, s + PF) : look_up(after, s + PF - MG);
          __builtin_amdgcn_sched_barrier(0);
        }
        const u32 rel = 16u * (u32)b + (u32)col;
        const bool valid = rel < cn;
        if (MODE == 0) {
#pragma unroll
          for (int t = 0; t < N; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) best[t][i] = max(best[t][i], valid ? acc[t][i] : kNone);
          if ((b & 3) == 3 || b + 1 == nb) {
            const u32 at = (sg * A.seg >> 6) * 16u + (u32)(b >> 2) * 16u + (u32)col;
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int rw = 4 * (t * 16 + 4 * g + i);
                const float dev = __uint_as_float(qrow[rw + 3]) * (float)best[t][i];
                const float v = __uint_as_float(qrow[rw + 2]) - dev + 0x1p-20f * __builtin_fabsf(dev);
                if (at < qrow[rw + 1]) A.gmin[qrow[rw] + at] = best[t][i] != kNone && v < inf ? v : inf;
                best[t][i] = kNone;
              }
          }
        } else {
#pragma unroll
          for (int t = 0; t < N; ++t) {
            const int most = max(max(max(acc[t][0], acc[t][1]), acc[t][2]), acc[t][3]);
            if (__builtin_amdgcn_ballot_w64(most >= 0 && valid) == 0) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const bool pass = acc[t][i] >= 0 && valid;
              const u64 mask = __builtin_amdgcn_ballot_w64(pass);
              if (mask == 0) continue;
              if (queued + VS_WAVE > kQueue) flush();
              if (pass) {
                const int at = 2 * (queued + (int)__popcll(mask & ((1ull << lane) - 1ull)));
                queue[at] = ((u32)(t * 16 + 4 * g + i) << 26) | rel;
                queue[at + 1] = (u32)acc[t][i];
              }
              queued += (int)__popcll(mask);
            }
          }
        }
      };
#pragma unroll
      for (int s = 0; s < PF; ++s) ring[s] = look_up(raw[0], s);
      for (int b = 0; b < nb; b += AHEAD) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
          if (b + i >= nb) break;
          const Raw now = raw[i];
          raw[i] = load((u64)cb + 16u * (u32)min(b + i + AHEAD, nb - 1));
          block(b + i, i, now, raw[(i + 1) % AHEAD]);
        }
      }
    };
    if constexpr (NT == 1) sweep(std::integral_constant<int, 1>{});
    else if (nt == 1) sweep(std::integral_constant<int, 1>{});
    else sweep(std::integral_constant<int, NT>{});
    if (MODE == 1 && queued > 0) flush();
    if (next >= nitems) break;
    item = next;
    it = nit;
    lb = nlb;
    len = nlen;
  }
}

// ---- thresholds -----------------------------------------------------------------------------------
// The k-th smallest of the keys a wavefront holds in its first `used` registers, by bisection on the bits, the lowest
// eight rounded up (2^-15 of a value's magnitude).
template <int R>
__device__ __forceinline__ u32 kth_smallest(const u32 (&key)[R], int used, int k) {
  u32 t = 0;
  for (int b = 31; b >= 8; --b) {
    const u32 upto = t | ((1u << b) - 1u);
    int c = 0;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < used) c += (int)__popcll(__builtin_amdgcn_ballot_w64(key[r] <= upto));
    if (c < k) t |= 1u << b;
  }
  return t | 0xFFu;
}

// One wavefront per query: the k-th smallest of its groups' smallest upper bounds (values of different stored
// vectors: the exact k-th best of the search is not above it).  R registers per lane hold the values.
template <int R>
__global__ __launch_bounds__(256) void ms_bound_kernel(const float* __restrict__ gmin, const u32* __restrict__ qslots,
                                                       int64_t nq, int slots, int k, float* __restrict__ qbound) {
  const int64_t qi = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (qi >= nq) return;
  const int lane = lane_id(), n = (int)qslots[qi];
  u32 key[R];
  int have = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int s = r * 64 + lane;
    key[r] = 0xFFFFFFFFu;
    if (s < n) key[r] = order_f32(gmin[qi * slots + s]);
    have += (int)__popcll(__builtin_amdgcn_ballot_w64(key[r] < 0xFF800000u));   // (the image of +inf)
  }
  const u32 t = kth_smallest<R>(key, R, k);
  if (lane == 0) qbound[qi] = have >= k ? unorder_f32(t) : __builtin_inff();
}

// ---- exact evaluation of the candidates --------------------------------------------------------------
struct RerankArgs {
  const float* q;
  int64_t nq;
  int d, npr, cap, k, tot, force;                 // force: every query goes to the query-major scan
  const int32_t* probes;
  const int64_t* list_off;
  const u32* cand_count;
  const uint4* cand;
  u32* rescan_list;
  u32* rescan_count;
  uint4* surv;                                    // PQ: see ms_list_kernel
  u32 *surv_count, *surv_unwritten, *surv_first, *surv_number;
  u32 surv_cap;
  float* surv_value;
  const void* codes;
  KeySink sink;
  // PQ
  int M, dsub, form, batch;                       // batch: candidates whose entries are in LDS together (8, 16 or 32)
  const float *centroids, *codebooks, *cdist, *cnorm, *norms, *list_tables;
  // SQ8
  const float *vmin, *step;
};

// LDS of the exact evaluation
__host__ __device__ constexpr size_t pq_eval_cb_bytes(int M, int K, int dsub) { return ((size_t)M * K * dsub + 3) / 4 * 16; }
inline size_t pq_eval_bytes(int M, int K, int dsub, int lanes, int batch) {
  return pq_eval_cb_bytes(M, K, dsub) + (size_t)(kSweepThreads / VS_WAVE) * batch * (lanes + 1) * 4;
}
__host__ __device__ constexpr size_t rows_rerank_wave_bytes(int tot, int d, bool tiled) {
  return (size_t)tot * 8 + 1024 + VS_WAVE * 8 + (size_t)((d + 3) & ~3) * 4 + (tiled ? VS_WAVE * 36 * 4 : 0);
}
__host__ __device__ constexpr size_t onehot_rerank_wave_bytes(int M, int tot) { return (size_t)M * 64 + 1024 + (size_t)tot * 8; }
__host__ __device__ constexpr size_t sq8_rerank_wave_bytes(int tot, int d) {
  return ((size_t)tot * 8 + 1024 + (size_t)2 * d * 4 + 15) / 16 * 16;
}

// true if the query is left to the query-major scan (and listed for it)
__device__ __forceinline__ bool ms_overflowed(const RerankArgs& A, int64_t qi, u32 n) {
  if (n <= (u32)A.cap && !A.force) return false;
  if (lane_id() == 0) A.rescan_list[atomicAdd(A.rescan_count, 1u)] = (u32)qi;
  return true;
}

// Image of the k-th smallest upper bound among a query's candidates (the first 1024 of them: the k-th smallest of any
// part bounds the k-th smallest of the whole).
__device__ __forceinline__ u32 ms_limit(const RerankArgs& A, int64_t qi, u32 n) {
  constexpr int R = 16;
  if (n <= (u32)A.k) return 0xFFFFFFFFu;
  const int lane = lane_id();
  const uint4* __restrict__ src = A.cand + (u64)qi * (u32)A.cap;
  u32 key[R];
  const int used = (int)min((n + 63) >> 6, (u32)R);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    key[r] = 0xFFFFFFFFu;
    if (r < used && (u32)(r * 64 + lane) < n) key[r] = order_f32(__uint_as_float(src[r * 64 + lane].w));
  }
  return kth_smallest<R>(key, used, A.k);
}

// The candidates that can be among the k best, 64 at a time: those whose lower bound is not above `limit`.  Calls
// batch(number, lane's storage position, lane's probe rank) with every lane of the wavefront; lanes past
// `number` repeat a candidate.  keep: 256 words of LDS.
template <class F>
__device__ __forceinline__ void ms_survivors(const RerankArgs& A, int64_t qi, u32 n, u32 limit, u32* keep_, F&& batch) {
  typedef __attribute__((address_space(3))) volatile u32* lds_u32_ptr;
  const lds_u32_ptr keep = (lds_u32_ptr)keep_;
  const int lane = lane_id();
  const uint4* __restrict__ src = A.cand + (u64)qi * (u32)A.cap;
  int have = 0;
  for (u32 c0 = 0; c0 < n; c0 += VS_WAVE) {
    uint4 e = make_uint4(0u, 0u, 0u, 0u);
    if (c0 + (u32)lane < n) e = src[c0 + (u32)lane];
    const bool on = c0 + (u32)lane < n && order_f32(__uint_as_float(e.z)) <= limit;
    const u64 mask = __builtin_amdgcn_ballot_w64(on);
    if (on) {
      const int at = 2 * (have + (int)__popcll(mask & ((1ull << lane) - 1ull)));
      keep[at] = e.x;
      keep[at + 1] = e.y;
    }
    have += (int)__popcll(mask);
    wave_lds_sync();
    const bool last = c0 + VS_WAVE >= n;
    while (have >= VS_WAVE || (last && have > 0)) {
      const int m = min(have, VS_WAVE), from = have - m + min(lane, m - 1);
      const u32 pos = keep[2 * from], p = keep[2 * from + 1];
      wave_lds_sync();
      batch(m, pos, p);
      have -= m;
    }
  }
}

// PQ, in three launches.  (1) One wavefront per query: the survivors of all queries in one list {storage position,
// pair, list, position in the list}, a query's next to each other; 16 wavefronts share one addition to the list's
// length.  A query whose survivors do not all fit writes none of them and is scanned again; what it leaves empty of the
// list goes to *surv_unwritten, so that nobody reads it.
__global__ __launch_bounds__(1024) void ms_list_kernel(const RerankArgs A) {
  __shared__ u32 keep_s[16][256];
  __shared__ u32 count_s[16], base_s;
  const int wave = threadIdx.x >> 6, lane = lane_id();
  const int64_t qi = (int64_t)blockIdx.x * 16 + wave;
  const u32 n = qi < A.nq ? A.cand_count[qi] : 0u;
  const bool left = qi < A.nq && ms_overflowed(A, qi, n);
  u32 limit = 0u, mine = 0;
  // Up to 256 candidates (nearly all queries of a few results) stay in registers: read once instead of three times, and
  // the survivors' lists are asked for before the wait for a place.  Every step of this kernel is a round trip to memory;
  // 10,000 queries, k = 10, 32.2 -> 31.2 us; 333 queries, k = 100, 16.7 -> 14.1.
  constexpr int RC = 4;
  const bool few = !left && n > 0 && n <= 64u * RC;
  uint4 e[RC];
  u32 list[RC], rel[RC];
  if (few) {
    const uint4* __restrict__ src = A.cand + (u64)qi * (u32)A.cap;
    u32 key[RC];
#pragma unroll
    for (int r = 0; r < RC; ++r) e[r] = src[min((u32)(r * 64 + lane), n - 1)];
#pragma unroll
    for (int r = 0; r < RC; ++r) key[r] = (u32)(r * 64 + lane) < n ? order_f32(__uint_as_float(e[r].w)) : 0xFFFFFFFFu;
    limit = n <= (u32)A.k ? 0xFFFFFFFFu : kth_smallest<RC>(key, (int)((n + 63) >> 6), A.k);
#pragma unroll
    for (int r = 0; r < RC; ++r) {
      const bool on = (u32)(r * 64 + lane) < n && order_f32(__uint_as_float(e[r].z)) <= limit;
      e[r].w = on;
      mine += (u32)__popcll(__builtin_amdgcn_ballot_w64(on));
      list[r] = on ? (u32)A.probes[(u32)qi * (u32)A.npr + e[r].y] : 0u;
    }
#pragma unroll
    for (int r = 0; r < RC; ++r) rel[r] = e[r].x - (u32)A.list_off[list[r]];
  } else if (!left && n > 0) {
    limit = ms_limit(A, qi, n);
    const uint4* __restrict__ src = A.cand + (u64)qi * (u32)A.cap;
    for (u32 c0 = 0; c0 < n; c0 += VS_WAVE)
      mine += (u32)__popcll(__builtin_amdgcn_ballot_w64(c0 + (u32)lane < n && order_f32(__uint_as_float(src[min(c0 + (u32)lane, n - 1)].z)) <= limit));
  }
  if (lane == 0) count_s[wave] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    u32 t = 0;
    for (int w = 0; w < 16; ++w) { const u32 c = count_s[w]; count_s[w] = t; t += c; }
    base_s = t ? atomicAdd(A.surv_count, t) : 0u;
  }
  __syncthreads();
  if (qi >= A.nq) return;
  u32 at = base_s + count_s[wave];
  const SurvivorPlace place = survivor_place(at, mine, A.surv_cap);
  if (lane == 0) {
    A.surv_first[qi] = at;
    A.surv_number[qi] = left || place.full ? 0xFFFFFFFFu : mine;
    if (place.full) A.rescan_list[atomicAdd(A.rescan_count, 1u)] = (u32)qi;
    if (place.unwritten) *A.surv_unwritten = place.unwritten;   // (one query at most)
  }
  if (mine == 0 || place.full) return;
  if (few) {
#pragma unroll
    for (int r = 0; r < RC; ++r) {
      const u64 mask = __builtin_amdgcn_ballot_w64(e[r].w != 0u);
      if (e[r].w) A.surv[at + (u32)__popcll(mask & ((1ull << lane) - 1ull))] = make_uint4(e[r].x, (u32)qi * (u32)A.npr + e[r].y, list[r], rel[r]);
      at += (u32)__popcll(mask);
    }
    return;
  }
  ms_survivors(A, qi, n, limit, keep_s[wave], [&](int num, u32 pos, u32 p) {
    const u32 pr = (u32)qi * (u32)A.npr + p;
    const int l = A.probes[pr];
    if (lane < num) A.surv[at + (u32)lane] = make_uint4(pos, pr, (u32)l, pos - (u32)A.list_off[l]);
    at += (u32)num;
  });
}

// (2) LPC lanes per survivor, one sub-quantizer each: the table entry that the query-major scan would have looked up is
// computed by itself (codebook in LDS, query and centroid slices from memory) and goes to LDS; then one lane
// per survivor adds its M entries in the scan's order.  DS: d / M where known at compile time.
template <int LPC, int DS, int NBITS, bool ROT>
__global__ __launch_bounds__(kSweepThreads) void ms_eval_pq_kernel(const RerankArgs A) {
  constexpr int K = 1 << NBITS, CPI = VS_WAVE / LPC;            // survivors per iteration
  constexpr int LE = LPC + 1;                                   // row of entries of a survivor
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int U = DS == 3 ? 8 : 4;                            // iterations in flight: 16 to 32 survivors
  const int dsub = DS > 0 ? DS : A.dsub, M = ROT ? LPC : A.M, d = A.d, B = A.batch;   // (rotated codes: M = LPC)
  float* cbs = reinterpret_cast<float*>(smem);                  // [M][K][dsub]
  const int wave = threadIdx.x >> 6, lane = lane_id(), nw = kSweepThreads / VS_WAVE;
  float* ent = reinterpret_cast<float*>(smem + pq_eval_cb_bytes(M, K, dsub)) + (size_t)wave * B * LE;
  const u32 total = survivors_written(*A.surv_count, A.surv_cap, *A.surv_unwritten);
  if (blockIdx.x * (u32)(nw * B) >= total) return;              // (uniform)
  for (int i = threadIdx.x; i < M * K * dsub / 4; i += kSweepThreads)
    reinterpret_cast<f32x4*>(cbs)[i] = reinterpret_cast<const f32x4*>(A.codebooks)[i];
  __syncthreads();
  const uint8_t* codes = static_cast<const uint8_t*>(A.codes);
  const int b = lane % LPC, bm = min(b, M - 1), cs = M * NBITS / 8;
  for (u32 s0 = (blockIdx.x * (u32)nw + (u32)wave) * (u32)B; s0 < total; s0 += gridDim.x * (u32)(nw * B)) {
    const int cnt = (int)min((u32)B, total - s0);
    const uint4 own = A.surv[s0 + (u32)min(lane, cnt - 1)];     // lane i: survivor i of the batch
    float dist = 0.f;
    if (ROT || A.form != 0) dist = A.cdist[own.y];
    if (A.form == 2) dist = (dist - A.cnorm[own.z]) + A.norms[own.x];
    // (all of a step's bytes and slices are requested before the first entry is formed: with one survivor per LPC
    // lanes at a time a workgroup, alone on its CU with its codebook, mostly waits for its codes.  PQ32x8 of 100 million
    // vectors, 10,000 queries, k = 100: 276 -> 130 us; PQ16x8 of a million, k = 10: 23.4 -> 16.8)
    for (int c0 = 0; c0 < cnt; c0 += U * CPI) {
      u32 code[U];
      float qv[U][DS > 0 ? DS : 1], cv[U][DS > 0 ? DS : 1];
#pragma unroll
      for (int v = 0; v < U; ++v) {
        const int ci = min(c0 + v * CPI + lane / LPC, cnt - 1);
        const u32 cpos = __shfl(own.x, ci, 64), cpr = __shfl(own.y, ci, 64), cl = __shfl(own.z, ci, 64);
        const int m = ROT ? (b + (int)__shfl(own.w, ci, 64)) & (M - 1) : bm;
        code[v] = codes[(u64)cpos * (u32)cs + (NBITS == 8 ? bm : bm >> 1)];
        if constexpr (DS > 0) {
          const float* qr = A.q + (u64)(cpr / (u32)A.npr) * (u32)d + m * DS;
#pragma unroll
          for (int u = 0; u < DS; ++u) qv[v][u] = qr[u];
          if (A.form == 0) {
            const float* c = A.centroids + (u64)cl * (u32)d + m * DS;
#pragma unroll
            for (int u = 0; u < DS; ++u) cv[v][u] = c[u];
          }
        }
      }
#pragma unroll
      for (int v = 0; v < U; ++v) {
        const int ci = min(c0 + v * CPI + lane / LPC, cnt - 1);
        const u32 cpr = __shfl(own.y, ci, 64), cl = __shfl(own.z, ci, 64);
        const u32 crel = ROT ? __shfl(own.w, ci, 64) : 0u;
        const int m = ROT ? (b + (int)crel) & (M - 1) : bm;
        const u32 j = NBITS == 8 ? code[v] : (code[v] >> (4 * (bm & 1))) & 15u;
        const float* T = cbs + (m * K + (int)j) * dsub;
        const float* qr = A.q + (u64)(cpr / (u32)A.npr) * (u32)d + m * dsub;
        const float* c = A.centroids + (u64)cl * (u32)d + m * dsub;
        auto qu = [&](int u) { if constexpr (DS > 0) return qv[v][u]; else return qr[u]; };
        auto cu = [&](int u) { if constexpr (DS > 0) return cv[v][u]; else return c[u]; };
        float e = 0.f;
        if (A.form == 0) {
          if constexpr (ROT) {      // |t|^2 - 2 <r, t>, as the bank-private tables hold it
            float tn = 0.f;
#pragma unroll
            for (int u = 0; u < dsub; ++u) tn = __builtin_fmaf(T[u], T[u], tn);
            e = tn;
#pragma unroll
            for (int u = 0; u < dsub; ++u) e = __builtin_fmaf(qu(u) - cu(u), T[u] * -2.f, e);
          } else {
            for (int u = 0; u < dsub; ++u) {
              const float diff = (qu(u) - cu(u)) - T[u];
              e = __builtin_fmaf(diff, diff, e);
            }
          }
        } else {
          float acc = 0.f;
          for (int u = 0; u < dsub; ++u) acc = __builtin_fmaf(qu(u), T[u], acc);
          e = A.form == 1 ? acc : -2.f * acc;
          if (ROT && A.form == 3) e = e + A.list_tables[((u64)cl * K + j) * (u32)M + m];
        }
        // (lanes without a sub-quantizer, and past the batch's end, hold what others write)
        if (b < M && c0 + v * CPI + lane / LPC < cnt) ent[ci * LE + b] = e;
      }
    }
    wave_lds_sync();
    if (lane < cnt) {
      const float* row = ent + lane * LE;
#pragma unroll 16
      for (int t = 0; t < M; ++t) dist += row[t];
      if (ROT ? A.form != 1 : A.form == 2) dist = fmaxf(dist, 0.f);
      A.surv_value[s0 + (u32)lane] = dist;
    }
    wave_lds_sync();
  }
}

// (3) One wavefront per query: the k best of its survivors.
template <int R>
__global__ __launch_bounds__(256) void ms_select_kernel(const RerankArgs A) {
  __shared__ __attribute__((aligned(16))) u64 slots[4][64 * R];
  const int wave = threadIdx.x >> 6, lane = lane_id();
  const int64_t qi = (int64_t)blockIdx.x * 4 + wave;
  if (qi >= A.nq) return;
  const u32 n = A.surv_number[qi], first = A.surv_first[qi];
  if (n == 0xFFFFFFFFu) return;
  WaveSelect<R> ws;
  ws.init(slots[wave], A.tot, A.k);
  ws.set_metric(A.sink.metric);
  for (u32 c0 = 0; c0 < n; c0 += VS_WAVE) {
    const bool on = c0 + (u32)lane < n;
    const u32 at = first + (on ? c0 + (u32)lane : 0u);
    ws.push_value(on, A.surv_value[at], A.surv[at].x);
  }
  ws.finish();
  for (int j = lane; j < A.k; j += VS_WAVE) A.sink.put(qi * A.k + j, ws.s[j]);
}

// 4-bit inner products: one wavefront per query, its table in LDS, one candidate per lane; the entries are added in the
// query-major scan's order.
template <int MG, int R>
__global__ __launch_bounds__(256) void ms_rerank_onehot_kernel(const RerankArgs A, const float* __restrict__ exact) {
  constexpr int M = 4 * MG, W = MG / 2;                          // words of a code
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int wave = threadIdx.x >> 6, lane = lane_id();
  unsigned char* mine = smem + (size_t)wave * onehot_rerank_wave_bytes(M, A.tot);
  float* T = reinterpret_cast<float*>(mine);
  u32* keep = reinterpret_cast<u32*>(T + M * 16);
  u64* slots = reinterpret_cast<u64*>(keep + 256);
  const int64_t qi = (int64_t)blockIdx.x * 4 + wave;
  if (qi >= A.nq) return;
  const u32 n = A.cand_count[qi];
  if (ms_overflowed(A, qi, n)) return;
#pragma unroll
  for (int i = lane; i < M * 4; i += VS_WAVE)
    reinterpret_cast<f32x4*>(T)[i] = reinterpret_cast<const f32x4*>(exact + qi * M * 16)[i];
  WaveSelect<R> ws;
  ws.init(slots, A.tot, A.k);
  ws.set_metric(1);
  const u32* codes = static_cast<const u32*>(A.codes);
  const u32 limit = ms_limit(A, qi, n);
  wave_lds_sync();
  ms_survivors(A, qi, n, limit, keep, [&](int num, u32 pos, u32 p) {
    u32 w[W];
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = codes[(u64)pos * W + i];
    float dist = A.cdist[qi * A.npr + p];
#pragma unroll
    for (int m = 0; m < M; ++m) dist += T[m * 16 + (int)((w[m >> 3] >> (4 * (m & 7))) & 15u)];
    ws.push_value(lane < num, dist, pos);
  });
  ws.finish();
  for (int j = lane; j < A.k; j += VS_WAVE) A.sink.put(qi * A.k + j, ws.s[j]);
}

// raw vectors: the canon distance of every candidate row
template <int METRIC, bool TILED, int R>
__global__ __launch_bounds__(256) void ms_rerank_flat_kernel(const RerankArgs A) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int wave = threadIdx.x >> 6, lane = lane_id(), d = A.d, dp = (d + 3) & ~3;
  unsigned char* mine = smem + (size_t)wave * rows_rerank_wave_bytes(A.tot, d, TILED);
  u64* slots = reinterpret_cast<u64*>(mine);
  u32* keep = reinterpret_cast<u32*>(mine + (size_t)A.tot * 8);
  int64_t* rows_s = reinterpret_cast<int64_t*>(keep + 256);
  float* qs = reinterpret_cast<float*>(rows_s + VS_WAVE);
  float* tile = qs + dp;
  const int64_t qi = (int64_t)blockIdx.x * 4 + wave;
  if (qi >= A.nq) return;
  const u32 n = A.cand_count[qi];
  if (ms_overflowed(A, qi, n)) return;
  for (int t = lane; t < d; t += VS_WAVE) qs[t] = A.q[qi * d + t];
  WaveSelect<R> ws;
  ws.init(slots, A.tot, A.k);
  ws.set_metric(METRIC);
  const float* rows = static_cast<const float*>(A.codes);
  ms_survivors(A, qi, n, ms_limit(A, qi, n), keep, [&](int num, u32 pos, u32) {
    float v;
    if constexpr (TILED) v = wave_canon_rows_tiled<METRIC>(qs, rows, d, (int64_t)pos, rows_s, tile);
    else v = canon_row<METRIC>(qs, rows + (int64_t)pos * d, d, (d & 3) == 0);
    ws.push_value(lane < num, v, pos);
  });
  ws.finish();
  for (int j = lane; j < A.k; j += VS_WAVE) A.sink.put(qi * A.k + j, ws.s[j]);
}

// 8-bit scalar codes: the chain of the query-major scan over a candidate's bytes, one candidate per lane
template <int METRIC, int R>
__global__ __launch_bounds__(256) void ms_rerank_sq8_kernel(const RerankArgs A) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int wave = threadIdx.x >> 6, lane = lane_id(), d = A.d;
  unsigned char* mine = smem + (size_t)wave * sq8_rerank_wave_bytes(A.tot, d);
  u64* slots = reinterpret_cast<u64*>(mine);
  u32* keep = reinterpret_cast<u32*>(mine + (size_t)A.tot * 8);
  float* qs = reinterpret_cast<float*>(keep + 256);
  const int64_t qi = (int64_t)blockIdx.x * 4 + wave;
  if (qi >= A.nq) return;
  const u32 n = A.cand_count[qi];
  if (ms_overflowed(A, qi, n)) return;
  for (int t = lane; t < d; t += VS_WAVE) {
    const float mid = __builtin_fmaf(0.5f, A.step[t], A.vmin[t]), qv = A.q[qi * d + t];
    if (METRIC == 0) { qs[t] = qv - mid; qs[d + t] = A.step[t]; }
    else { qs[t] = qv * A.step[t]; qs[d + t] = qv * mid; }
  }
  wave_lds_sync();
  float acc0 = 0.f;
  if (METRIC == 1) for (int t = 0; t < d; ++t) acc0 += qs[d + t];
  WaveSelect<R> ws;
  ws.init(slots, A.tot, A.k);
  ws.set_metric(METRIC);
  const uint8_t* codes = static_cast<const uint8_t*>(A.codes);
  auto step1 = [&](float acc, int t, u32 byte) {
    const float code = (float)byte;
    if (METRIC == 0) { const float diff = __builtin_fmaf(-code, qs[d + t], qs[t]); return __builtin_fmaf(diff, diff, acc); }
    return __builtin_fmaf(code, qs[t], acc);
  };
  ms_survivors(A, qi, n, ms_limit(A, qi, n), keep, [&](int num, u32 pos, u32) {
    const uint8_t* c = codes + (u64)pos * (u32)d;
    float acc = acc0;
    if ((d & 15) == 0) {
      for (int t = 0; t < d; t += 16) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(c + t);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc = step1(acc, t + i, (w[i >> 2] >> (8 * (i & 3))) & 0xFFu);
      }
    } else {
      for (int t = 0; t < d; ++t) acc = step1(acc, t, c[t]);
    }
    ws.push_value(lane < num, acc, pos);
  });
  ws.finish();
  for (int j = lane; j < A.k; j += VS_WAVE) A.sink.put(qi * A.k + j, ws.s[j]);
}

// ---- what an index keeps for the scan --------------------------------------------------------------------
// The fp16 codebook as granules [m][part][entry] of gh halfs, scaled by the power of two that puts the largest
// component (its bits go to *maxbits; a NaN is larger than any) at 2^exp -- every workgroup finds the largest for itself --, and the
// centroids in fragment order.
__global__ __launch_bounds__(512) void ms_codebook_kernel(const float* __restrict__ codebooks, int M, int K, int dsub,
                                                          int parts, int gh, int exp, u32* __restrict__ maxbits,
                                                          _Float16* __restrict__ out, const float* __restrict__ centroids,
                                                          int64_t nlist, int kp, SlotMap map, int norm_slot,
                                                          float* __restrict__ cperm) {
  __shared__ u32 part_max[8];
  const int total = M * K * dsub;
  u32 mx = 0;
  // (four at a time, M is a multiple of four; 4096 lists of 128 dimensions, 16 x 8: 9.1 -> 8.0 us)
#pragma unroll 8
  for (int i = threadIdx.x; i < total / 4; i += 512) {
    const u32x4 v = reinterpret_cast<const u32x4*>(codebooks)[i];
#pragma unroll
    for (int t = 0; t < 4; ++t) mx = max(mx, v[t] & 0x7FFFFFFFu);
  }
  for (int o = 32; o > 0; o >>= 1) mx = max(mx, (u32)__shfl_xor((int)mx, o, 64));
  if ((threadIdx.x & 63) == 0) part_max[threadIdx.x >> 6] = mx;
  __syncthreads();
  for (int w = 0; w < 8; ++w) mx = max(mx, part_max[w]);
  if (blockIdx.x == 0 && threadIdx.x == 0) *maxbits = mx;
  const float sigma = scale_of(mx, exp, 0);
  const int halfs = M * parts * K * gh;
  for (int e = blockIdx.x * 512 + threadIdx.x; e < halfs; e += gridDim.x * 512) {
    const int t = e % gh, j = (e / gh) % K, part = (e / (gh * K)) % parts, m = e / (gh * K * parts);
    const int dd = part * gh + t;
    const float* cw = codebooks + ((int64_t)m * K + j) * dsub;
    float v = 0.f;
    if (dd < dsub) {
      v = cw[dd] * sigma;
    } else if (norm_slot && t == gh - 1) {      // -|t^|^2 / 2 of the fp16 image
      for (int u = 0; u < dsub; ++u) { const float c = (float)(_Float16)(cw[u] * sigma); v = __builtin_fmaf(-0.5f * c, c, v); }
    }
    out[e] = (_Float16)v;
  }
  for (int64_t e = (int64_t)blockIdx.x * 512 + threadIdx.x; e < nlist * kp; e += (int64_t)gridDim.x * 512) {
    const int64_t l = e / kp;
    const int dim = slot_dim(map, (int)(e - l * kp));
    cperm[e] = dim >= 0 ? centroids[l * map.d + dim] : 0.f;
  }
}

// Codes of the list-contiguous store into units (see PqSide): a wavefront per eight units, a lane per (code, lane row).
// The first unit's list is found by steps of 64 candidates at a time; a list has at least one unit number of its own, so
// that the other units' lists are among the 64 from there on, whose offsets one load brings.  The eight units then wait
// for memory together (one by one, a million codes of 16 bytes: 13.9 us, now 11.7).  Entries past a list's end repeat the
// store's first code.
constexpr int kUnitsPerWave = 8;
template <int CBP>
__global__ __launch_bounds__(256) void ms_units_kernel(const uint8_t* __restrict__ codes, const int64_t* __restrict__ list_off,
                                                       int nlist, int cs, int cby, int rot_m, int64_t units,
                                                       uint8_t* __restrict__ out) {
  constexpr int NW = CBP >= 4 ? CBP / 4 : 1;                    // words of a code in a lane
  constexpr int UNROLL = CBP <= 4 ? kUnitsPerWave : 2;
  const int lane = lane_id(), col = lane & 15, g = lane >> 4;
  const int64_t unit0 = ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * kUnitsPerWave;
  if (unit0 >= units) return;
  int lo = 0, hi = nlist;                                       // first unit of lo <= unit0 < first unit of hi (nlist: the end)
  while (hi - lo > 1) {
    const int step = (hi - lo + VS_WAVE - 1) / VS_WAVE, at = lo + lane * step;
    const bool before = at < hi && (list_off[min(at, nlist)] >> 5) + at <= unit0;
    lo += ((int)__popcll(__builtin_amdgcn_ballot_w64(before)) - 1) * step;
    hi = min(hi, lo + step);
  }
  const u32 off = (u32)list_off[min(lo + lane, nlist)];         // lane i: where list lo + i begins
  const int64_t first = lo + lane < nlist ? (int64_t)(off >> 5) + lo + lane : units;   // ... and its first unit
  const int words = cs / 4;
#pragma unroll UNROLL
  for (int u = 0; u < kUnitsPerWave; ++u) {
    const int64_t unit = unit0 + u;
    if (unit >= units) return;
    const int l = (int)__popcll(__builtin_amdgcn_ballot_w64(first <= unit)) - 1;       // (below 8, and lo + l below nlist)
    const u32 lb = (u32)__builtin_amdgcn_readlane((int)off, l), le = (u32)__builtin_amdgcn_readlane((int)off, l + 1);
    u32 v[2][NW];
#pragma unroll
    for (int block = 0; block < 2; ++block) {
      const int64_t rel = (unit - (lb >> 5) - lo - l) * 32 + 16 * block + col;
      const u32* src = reinterpret_cast<const u32*>(codes + (lb + rel < le ? lb + rel : 0) * cs);
      // stored byte b of the code at list position p is c_{(b + p) mod M} where the codes are rotated
      const int o = rot_m ? (int)(((int64_t)g * cby - rel) & (rot_m - 1)) : g * cby;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        int i0 = (o >> 2) + w, i1 = i0 + 1;
        if (rot_m) { i0 &= words - 1; i1 &= words - 1; }
        else { i0 = min(i0, words - 1); i1 = min(i1, words - 1); }   // (bytes past the code's end are not used)
        v[block][w] = __builtin_amdgcn_alignbyte(src[i1], src[i0], (u32)(o & 3));
      }
    }
    uint8_t* dst = out + (unit * 64 + lane) * (2 * CBP);
    if constexpr (CBP == 2) *reinterpret_cast<u32*>(dst) = (v[0][0] & 0xFFFFu) | (v[1][0] << 16);
    else if constexpr (CBP == 4) *reinterpret_cast<u32x2*>(dst) = u32x2{v[0][0], v[1][0]};
    else {
#pragma unroll
      for (int w = 0; w < 2 * NW; w += 4)
        *reinterpret_cast<u32x4*>(dst + 4 * w) = u32x4{v[w / NW][w % NW], v[(w + 1) / NW][(w + 1) % NW],
                                                       v[(w + 2) / NW][(w + 2) % NW], v[(w + 3) / NW][(w + 3) % NW]};
    }
  }
}

__global__ __launch_bounds__(256) void ms_centroids16_kernel(const float* __restrict__ centroids, int64_t nlist, int kp,
                                                             SlotMap map, _Float16* __restrict__ cperm) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nlist * kp; e += (int64_t)gridDim.x * 256) {
    const int64_t l = e / kp;
    const int dim = slot_dim(map, (int)(e - l * kp));
    cperm[e] = (_Float16)(dim >= 0 ? centroids[l * map.d + dim] : 0.f);
  }
}

// ---- launchers -------------------------------------------------------------------------------------------

// granules of a sub-vector: of 8 halfs where that pads least or as little as 4, of 4, or of 2
void pq_granule(int dsub, int* gb, int* parts) {
  const int r = dsub % 8;
  *gb = r == 0 || r > 4 ? 16 : (dsub > 2 ? 8 : 4);
  *parts = (dsub + *gb / 2 - 1) / (*gb / 2);
}

size_t up256(size_t v) { return (v + 255) / 256 * 256; }
int flat_ksteps(int d) { return (d + 31) / 32; }
constexpr int pq_tiles(int ks) { return ks <= 5 ? 2 : 1; }
constexpr int rows_tiles(int ks) { return ks <= 4 ? 4 : (ks <= 6 ? 2 : 1); }

// LDS of the one-hot tables' kernel
size_t onehot_tables_bytes(const IvfpqDims& g) { return (size_t)g.M * onehot_row(g.dsub) * sizeof(float); }

struct MsShape { int ks, nt; SlotMap map; int cb16 = 0; bool onehot = false; };
// queries per work item: 16 per tile, as many tiles as the registers hold
MsShape fragment_shape(int kind, const IvfpqDims& g) {
  MsShape s;
  s.map = SlotMap{kind, g.d, g.dsub, 0, 1, 8};
  if (kind == kMsPq) {
    int gb = 0, parts = 0;
    pq_granule(g.dsub, &gb, &parts);
    s.map.mg = g.M / 4;
    s.map.parts = parts;
    s.map.gh = gb / 2;
    const int gpf = 8 / (gb / 2);
    s.ks = (s.map.mg * parts + gpf - 1) / gpf;
    s.nt = pq_tiles(s.ks);
    s.cb16 = g.M * parts * g.K * gb;
  } else {
    s.ks = flat_ksteps(g.d);
    s.nt = rows_tiles(s.ks);
  }
  return s;
}

MsShape ms_shape(int kind, const IvfpqDims& g) {
  if (!mscan_onehot(kind, g)) return fragment_shape(kind, g);
  MsShape s;
  s.map = SlotMap{kind, g.d, g.dsub, 0, 1, 8};
  s.ks = 0;
  s.nt = 2;
  s.onehot = true;
  return s;
}

// L2 with d / M = 3: see PqSide::NORM
int norm_slot(const IvfpqDims& g) { return g.metric == 0 && ivfpq_codes_rotated(g) && g.M == 32 ? 1 : 0; }

// lanes per candidate of the exact evaluation
int pq_lanes(int M) { return M <= 8 ? 8 : (M <= 16 ? 16 : (M <= 32 ? 32 : 64)); }

}  // namespace

// 4-bit inner-product codes without a form below: the one-hot sweeps, where the tables' kernel has the LDS (sub-vectors of up
// to 159, 79 or 39 dimensions for 16, 32 or 64 sub-quantizers).  (Where there is such a form its matrix steps are fewer: 64
// dimensions of 32 x 4 bits take 2, one-hot 8.)
bool mscan_onehot(int kind, const IvfpqDims& g) {
  return kind == kMsPq && g.metric == 1 && g.nbits == 4 && (g.M == 16 || g.M == 32 || g.M == 64) &&
         mscan_index_bytes(kind, g) == 0 && onehot_tables_bytes(g) <= 160 * 1024;
}

void launch_mscan_onehot_slack(const IvfpqDims& g, const float* centroids, const float* codebooks, float* out, hipStream_t st) {
  hipLaunchKernelGGL(ms_onehot_slack_kernel, dim3(kOnehotSamples / 4), dim3(256), 0, st, centroids, (int64_t)g.nlist, g.d, g.M, g.dsub,
                     codebooks, out);
}

// The (sub-quantizers per lane row, granules per sub-vector, granule bytes, bits, rotated) forms with kernels: up to
// eight matrix steps per vector.  (64 sub-quantizers of 12 dimensions, 24 steps, are slower this way than by
// tables: 48 look-ups per code and lane for 16, 2590 us for 2000 at 262k queries x lists of 1526 codes; their inner
// products go one-hot.)
#define VS_MS_PQ_FORMS(X)                                                                                   \
  X(2, 1, 8, 8, true) X(4, 1, 16, 8, true) X(8, 1, 8, 8, true)                                              \
  X(2, 1, 16, 8, false) X(4, 1, 16, 8, false) X(5, 1, 16, 8, false)                                         \
  X(4, 1, 8, 8, false) X(8, 1, 8, 8, false)                                                                 \
  X(8, 1, 4, 4, false) X(16, 1, 4, 4, false) X(4, 1, 8, 4, false) X(8, 1, 8, 4, false) X(16, 1, 8, 4, false)

// Whether the data that an index's scale is taken from -- bits of the codebooks' largest magnitude (PQ) or of the
// centroids' largest squared norm -- lies where the scan's bounds hold (see the head of this file).  A codeword or a
// centroid that is not finite does not.
constexpr int kPqExp = 6, kRowsExp = 4, kScaleRange = 40;
bool mscan_scale_fits(int kind, u32 bits) {
  float v;
  static_assert(sizeof(v) == sizeof(bits), "");
  std::memcpy(&v, &bits, sizeof(v));
  if (v == 0.f) return true;
  if (!(v > 0.f) || !std::isfinite(v)) return false;
  int e;
  (void)std::frexp(kind == kMsPq ? v : std::sqrt(v), &e);
  return std::abs((kind == kMsPq ? kPqExp : kRowsExp) - e) <= kScaleRange;
}

// What an index keeps: PQ: fp16 codebook | centroids [nlist][kp] fp32 in fragment order; raw vectors and scalar
// codes: centroids [nlist][kp] fp16
size_t mscan_index_bytes(int kind, const IvfpqDims& g) {
  if (kind != kMsPq) {
    if (flat_ksteps(g.d) > 8) return 0;
    return up256((size_t)g.nlist * flat_ksteps(g.d) * 32 * 2);
  }
  if (g.M % 4 != 0 || g.M > 64 || (g.code_size & 3) != 0) return 0;
  const MsShape s = fragment_shape(kind, g);
  const bool rot = ivfpq_codes_rotated(g);
  bool found = false;
#define X(MG, PARTS, GB, NB, ROT) \
  found = found || (g.M == 4 * MG && s.map.parts == PARTS && 2 * s.map.gh == GB && g.nbits == NB && rot == ROT);
  VS_MS_PQ_FORMS(X)
#undef X
  if (!found || s.cb16 > 128 * 1024 || pq_eval_bytes(g.M, g.K, g.dsub, pq_lanes(g.M), 8) > 160 * 1024) return 0;
  return up256(s.cb16) + up256((size_t)g.nlist * s.ks * 32 * 4);
}

// The codes once more, in units of 32 (PQ): bytes, and their preparation from the list-contiguous store
size_t mscan_units_bytes(const IvfpqDims& g, int64_t ntotal) {
  return (size_t)((ntotal >> 5) + g.nlist + 2) * 64 * 2 * pq_lane_bytes(g.code_size / 4);
}
void launch_mscan_units(const IvfpqDims& g, const uint8_t* codes, const int64_t* list_off, int64_t ntotal, void* out,
                        hipStream_t st) {
  const int64_t units = (ntotal >> 5) + g.nlist + 1;
  const int cby = g.code_size / 4, rot = ivfpq_codes_rotated(g) ? g.M : 0;
  const dim3 grid((unsigned)((units + 4 * kUnitsPerWave - 1) / (4 * kUnitsPerWave)));
#define UNITS(CBP) hipLaunchKernelGGL((ms_units_kernel<CBP>), grid, dim3(256), 0, st, codes, list_off, g.nlist, g.code_size, cby, \
                                      rot, units, static_cast<uint8_t*>(out))
  switch (pq_lane_bytes(cby)) { case 2: UNITS(2); break; case 4: UNITS(4); break; case 8: UNITS(8); break; default: UNITS(16); }
#undef UNITS
}

void launch_mscan_index(int kind, const IvfpqDims& g, const float* centroids, const float* codebooks, PrepInfo* info,
                        void* out, hipStream_t st) {
  const MsShape s = ms_shape(kind, g);
  const int kp = 32 * s.ks;
  const unsigned grid = (unsigned)std::min<int64_t>(1024, ((int64_t)g.nlist * kp + 2047) / 2048 + 16);
  char* o = static_cast<char*>(out);
  if (kind == kMsPq)
    hipLaunchKernelGGL(ms_codebook_kernel, dim3(grid), dim3(512), 0, st, codebooks, g.M, g.K, g.dsub, s.map.parts,
                       s.map.gh, kPqExp, &info->codebook_max_bits, reinterpret_cast<_Float16*>(o), centroids,
                       (int64_t)g.nlist, kp, s.map, norm_slot(g), reinterpret_cast<float*>(o + up256(s.cb16)));
  else
    hipLaunchKernelGGL(ms_centroids16_kernel, dim3(grid), dim3(256), 0, st, centroids, (int64_t)g.nlist, kp, s.map,
                       reinterpret_cast<_Float16*>(o));
}

namespace {

struct MsLayout {
  size_t o_lfirst, o_lrest, o_count, o_ctr, zero_bytes;
  size_t o_poff, o_pairs, o_rank, o_pslot, o_qslots, o_items_a, o_items_b, o_qperm, o_tinfo, o_exact, o_bound, o_gmin, o_cand, o_rlist;
  size_t o_surv, o_sfirst, o_snum, o_sval, bytes;
};
MsLayout ms_layout(const MscanIndex& ix, const MscanPlan& p) {
  const MsShape s = ms_shape(ix.kind, ix.g);
  MsLayout L;
  size_t o = 0;
  auto take = [&](size_t b) { const size_t at = o; o += up256(b); return at; };
  const size_t np = (size_t)p.nq * p.npr;
  L.o_lfirst = take((size_t)ix.g.nlist * 4);
  L.o_lrest = take((size_t)ix.g.nlist * 4);
  L.o_count = take((size_t)p.nq * 4);
  L.o_ctr = take(64);
  L.zero_bytes = o;
  L.o_poff = take((size_t)ix.g.nlist * 16);
  L.o_pairs = take(np * 4);
  L.o_rank = take(np * 4);
  L.o_pslot = take(np * 4);
  L.o_qslots = take((size_t)p.nq * 4);
  L.o_items_a = take((size_t)p.max_a * 16);
  L.o_items_b = take((size_t)p.max_b * 16);
  L.o_qperm = take(s.onehot ? (size_t)p.nq * ix.g.M * 16 : (size_t)p.nq * s.ks * 32 * 4);   // (one-hot: tables)
  L.o_tinfo = take(s.onehot ? (size_t)p.nq * sizeof(float4) : 0);
  L.o_exact = take(s.onehot ? (size_t)p.nq * ix.g.M * 16 * sizeof(float) : 0);
  L.o_bound = take((size_t)p.nq * 4);
  L.o_gmin = take((size_t)p.nq * p.slots * 4);
  L.o_cand = take((size_t)p.nq * p.cap * 16);
  L.o_rlist = take((size_t)p.nq * 4);
  const size_t most = ix.kind == kMsPq && !s.onehot ? p.surv : 0;
  L.o_surv = take(most * 16);
  L.o_sval = take(most * 4);
  L.o_sfirst = take((size_t)p.nq * 4);
  L.o_snum = take((size_t)p.nq * 4);
  L.bytes = o;
  return L;
}

}  // namespace

bool mscan_supported(const MscanIndex& ix, int k) {
  if (k < 1 || k > 128) return false;
  if (mscan_onehot(ix.kind, ix.g)) return ix.codes != nullptr;
  return ix.mem != nullptr && (ix.kind != kMsPq || ix.units != nullptr);
}

// Sizes of a search.  slots: groups of four codes that give a query's threshold; seg: codes of a list per work item.
bool mscan_plan(const MscanIndex& ix, int64_t nq, int npr, int k, int asked, MscanPlan* out) {
  MscanPlan& p = *out;
  if (!mscan_supported(ix, k) || ix.ntotal < 1 || nq < 1 || nq * (int64_t)std::max(npr, 1024) >= (1ll << 32) || ix.max_list < 1)
    return false;
  const MsShape s = ms_shape(ix.kind, ix.g);
  p.nq = nq; p.npr = npr;
  const int64_t np = nq * npr;
  p.slots = k <= 16 ? 128 : (k <= 32 ? 256 : (k <= 64 ? 512 : 1024));
  p.capcodes = (u32)p.slots * 4u;
  // Candidates per query: four times what the list-major scan keeps (it only sees those behind the first lists), less
  // beyond 16,384 queries so that they stay near 1 GiB.  A query whose buffer overflows is scanned again, and
  // where nothing tells the probed lists apart -- unstructured data -- the threshold lets k of `capcodes` vectors
  // pass, `likely` of all that a query visits, and the error bounds two or three times that: four times it is kept as
  // far as 1 GiB goes, and eight times what it is for lists of the longest one's length as far as 128 MB go.
  // (12 million Gaussian vectors, 64 lists of 1465, 32 x 4 bits, k = 100: 40 queries 2123 us with 4096 candidates each,
  // 574 with room for them, 431 query-major; 256 queries 2455, 714, 818.)  Not where fewer than the default are asked
  // for.  No query has more candidates than its lists have vectors.
  const int64_t mean = (ix.ntotal + ix.g.nlist - 1) / ix.g.nlist, likely = k * npr * mean / p.capcodes;
  int64_t cap = std::max<int64_t>(256, std::min<int64_t>(4ll * asked, (1ll << 26) / nq));
  if (asked >= 1024) {
    cap = std::max(cap, std::min<int64_t>(4 * likely, (1ll << 26) / nq));
    cap = std::max(cap, std::min<int64_t>(8 * k * npr * ix.max_list / p.capcodes, (1ll << 23) / nq));
  }
  p.cap = (int)std::max<int64_t>(256, std::min<int64_t>(cap, (npr * ix.max_list + 63) / 64 * 64));
  // (short segments where there would be few work items for 2048 and more wavefronts, long ones to spread an item's
  // set-up)
  int64_t seg = std::min<int64_t>(np, ix.g.nlist) * ((mean + 511) / 512) < 32768 ? 256 : (s.onehot ? 512 : 1024);
  const int64_t group = 16 * s.nt, lists = std::min<int64_t>(np, ix.g.nlist);
  const int64_t first = std::min<int64_t>(npr, p.slots / 16);    // pairs of a query in the bound sweep, at most
  int64_t max_a, max_b;
  for (;; seg *= 2) {   // (at most four million items, 64 MB, however uneven the lists are)
    const int64_t maxseg = (ix.max_list + seg - 1) / seg, maxseg_a = std::min<int64_t>(maxseg, (p.capcodes + seg - 1) / seg);
    max_a = lists * maxseg_a + (nq * first / group) * maxseg_a;
    max_b = std::min<int64_t>(ix.ntotal / seg + ix.g.nlist, lists * maxseg) + (np / group) * maxseg;
    if (std::max(max_a, max_b) <= (1 << 22) || seg >= (1 << 25)) break;
  }
  if (std::max(max_a, max_b) >= (1ll << 28)) return false;
  p.seg = (u32)seg;
  p.max_a = (u32)max_a;
  p.max_b = (u32)max_b;
  // survivors of all queries: 4 k + 128 of each, and half a million (10 MB) at least
  p.surv = (u32)std::min<int64_t>(std::min<int64_t>(nq * p.cap, std::max<int64_t>(nq * (4 * k + 128), 1 << 19)), 1ll << 30);
  p.bytes = ms_layout(ix, p).bytes;
  return true;
}

const unsigned* mscan_rescan_count(const MscanIndex& ix, const MscanPlan& p, const char* ws) {
  return reinterpret_cast<const unsigned*>(ws + ms_layout(ix, p).o_ctr) + 4;
}
Rescan mscan_rescan(const MscanIndex& ix, const MscanPlan& p, const char* ws, u64* partial) {
  Rescan rs;
  rs.list = reinterpret_cast<const u32*>(ws + ms_layout(ix, p).o_rlist);
  rs.count = mscan_rescan_count(ix, p, ws);
  rs.cursor = reinterpret_cast<unsigned long long*>(const_cast<unsigned*>(rs.count) + 4);   // (cleared by part 0)
  rs.partial = partial;
  rs.pieces = (u32)std::min(p.npr, 16);
  rs.limit = (u32)std::min<int64_t>(p.nq, 65536);
  return rs;
}

namespace {

// As many workgroups as the chip holds at a time; each takes several items.  (One-hot rows of 16 sub-quantizers leave room for
// two per compute unit, of 32 and 64 for one: 10,000 queries of 16 x 1, 16 probes 525 -> 449 us, 64 probes, k = 100 1108 -> 915;
// of 16 x 9 350 -> 331 and 789 -> 702.)
void launch_persistent(void (*kern)(const SweepArgs), const SweepArgs& A, size_t lds, u32 max_items, hipStream_t st) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kSweepThreads, lds) != hipSuccess || per_cu < 1) per_cu = 1;
  const int64_t grid = std::min<int64_t>(256ll * per_cu, ((int64_t)max_items + 7) / 8);
  hipLaunchKernelGGL(kern, dim3((unsigned)std::max<int64_t>(1, grid)), dim3(kSweepThreads), lds, st, A);
}

template <class S, int METRIC, int MODE, int NT>
void launch_sweep(const SweepArgs& A, size_t lds, u32 max_items, hipStream_t st) {
  auto kern = &ms_sweep_kernel<S, METRIC, MODE, NT>;
  if (lds > 48 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  launch_persistent(kern, A, lds, max_items, st);
}

template <int MG, int MODE>
void launch_onehot_sweep(const SweepArgs& A, u32 max_items, hipStream_t st) {
  constexpr int NT = 2;
  auto kern = &ms_onehot_sweep_kernel<MG, MODE, NT>;
  const size_t lds = (size_t)(kSweepThreads / VS_WAVE) * (2 * kQueue + 64 * NT) * 4 + 16;
  launch_persistent(kern, A, lds, max_items, st);
}

template <int MODE>
void launch_sweep_any(const MscanIndex& ix, const MsShape& s, const SweepArgs& A, u32 max_items, hipStream_t st) {
  if (s.onehot) {
    if (ix.g.M == 16) launch_onehot_sweep<4, MODE>(A, max_items, st);
    else if (ix.g.M == 32) launch_onehot_sweep<8, MODE>(A, max_items, st);
    else launch_onehot_sweep<16, MODE>(A, max_items, st);
    return;
  }
  const size_t q = (size_t)(kSweepThreads / 64) * queue_words(s.nt) * 4 + 16;
  const bool rot = ix.kind == kMsPq && ivfpq_codes_rotated(ix.g);
  const int gb = 2 * s.map.gh;
  if (ix.kind == kMsPq) {
#define X(MG, PARTS, GB, NB, ROT)                                                                              \
    if (ix.g.M == 4 * MG && s.map.parts == PARTS && gb == GB && ix.g.nbits == NB && rot == ROT) {              \
      using P = PqSide<MG, PARTS, GB, NB, ROT>;                                                                \
      constexpr int NT = pq_tiles(P::KS);                                                                   \
      if (ix.g.metric == 0) launch_sweep<P, 0, MODE, NT>(A, s.cb16 + q, max_items, st);                        \
      else launch_sweep<P, 1, MODE, NT>(A, s.cb16 + q, max_items, st);                                         \
      return;                                                                                                  \
    }
    VS_MS_PQ_FORMS(X)
#undef X
    return;
  }
#define Y(KS_)                                                                                                 \
  case KS_: {                                                                                                  \
    constexpr int NT = rows_tiles(KS_);                                                                         \
    if (ix.kind == kMsFlat) {                                                                                  \
      if (ix.g.metric == 0) launch_sweep<FlatSide<KS_>, 0, MODE, NT>(A, q, max_items, st);                     \
      else launch_sweep<FlatSide<KS_>, 1, MODE, NT>(A, q, max_items, st);                                      \
    } else {                                                                                                   \
      if (ix.g.metric == 0) launch_sweep<Sq8Side<KS_>, 0, MODE, NT>(A, q + 256 * KS_, max_items, st);          \
      else launch_sweep<Sq8Side<KS_>, 1, MODE, NT>(A, q + 256 * KS_, max_items, st);                           \
    }                                                                                                          \
    return;                                                                                                    \
  }
  switch (s.ks) { Y(1) Y(2) Y(3) Y(4) Y(5) Y(6) Y(7) Y(8) }
#undef Y
}

SweepArgs sweep_args(const MscanIndex& ix, const MscanPlan& p, const MsShape& s, const MsLayout& L, const float* cdist,
                     int form, float eps_scale, char* ws) {
  SweepArgs A;
  A.qperm = reinterpret_cast<float*>(ws + L.o_qperm);
  A.kp = 32 * s.ks; A.npr = p.npr; A.slots = p.slots;
  A.pairs = reinterpret_cast<u32*>(ws + L.o_pairs);
  A.pair_slot = reinterpret_cast<u32*>(ws + L.o_pslot);
  A.list_off = ix.list_off;
  A.codes = ix.codes; A.units = static_cast<const uint8_t*>(ix.units);
  const char* mem = static_cast<const char*>(ix.mem);
  A.cb16 = reinterpret_cast<const f16x2*>(mem); A.cb16_bytes = s.cb16;
  A.cperm = ix.kind == kMsPq ? mem + up256((size_t)s.cb16) : mem;
  A.vmin = ix.vmin; A.step = ix.step;
  A.sigma_src = ix.sigma_src;
  A.sigma_exp = ix.kind == kMsPq ? kPqExp : kRowsExp; A.sigma_sqrt = ix.kind != kMsPq;
  A.form = form; A.cdist = cdist; A.cnorm = ix.cnorm;
  A.qbound = reinterpret_cast<float*>(ws + L.o_bound);
  A.gmin = reinterpret_cast<float*>(ws + L.o_gmin);
  A.cand_count = reinterpret_cast<u32*>(ws + L.o_count);
  A.cand = reinterpret_cast<uint4*>(ws + L.o_cand);
  A.cap = p.cap; A.seg = p.seg; A.capcodes = p.capcodes;
  A.map = s.map;
  // error bounds (see the head of this file); eps_scale scales them
  const double u = 0x1p-11, chain = 2.0 * ix.g.d + ix.g.M + 64.0, es = std::max(0.f, eps_scale);
  const double phi = chain * 0x1p-22;
  const double phi2 = ix.kind == kMsPq && form >= 2 ? chain * 0x1p-23 : 0.0;
  A.phi = (float)std::max(1e-30, phi * es);   // (not zero: it meets infinite thresholds)
  A.phi2 = (float)(phi2 * es);
  A.kappa = (float)((1.02 * u + phi + 4.0 * phi2) * es);
  A.c4u = (float)(4.0 * u * es);
  A.abs_err = (float)(32.0 * s.ks * 0x1p-26 * es);
  A.u2 = (float)std::max(1e-30, (2.02 * u + phi) * es);
  A.sd = (float)(std::sqrt(32.0 * s.ks) * 0x1p-25 * es);
  // (the norm inside the product is rounded to fp16: one u more; both factors are exact in fp16)
  const double off = A.kappa + 1.01 * u * es;
  A.tables = reinterpret_cast<const u32x4*>(ws + L.o_qperm);
  A.tinfo = reinterpret_cast<const float4*>(ws + L.o_tinfo);
  A.phi_c = (float)((ix.g.M + 4) * 0x1p-23 * es);
  A.norm_lo = (float)(1.0 - std::ceil(off * 0x1p11) * 0x1p-11);
  A.norm_hi = (float)(1.0 + std::ceil(off * 0x1p10) * 0x1p-10);
  return A;
}

}  // namespace

// Grouping, bound sweep and thresholds (part 0), collect sweep (part 1), exact evaluation (part 2; the queries that
// it leaves to the query-major scan are listed: mscan_rescan).
void launch_mscan(int part, const MscanIndex& ix, const MscanPlan& p, const float* q, const int32_t* probes,
                  const float* cdist, int form, int k, float eps_scale, char* ws, const int64_t* ids, float* out_dist,
                  int64_t* out_ids, hipStream_t st) {
  const MsShape s = ms_shape(ix.kind, ix.g);
  const MsLayout L = ms_layout(ix, p);
  SweepArgs A = sweep_args(ix, p, s, L, cdist, form, eps_scale, ws);
  u32* ctr = reinterpret_cast<u32*>(ws + L.o_ctr);   // items of both sweeps; from 4 on: queries to scan again, survivors, ...
  const int64_t np = p.nq * p.npr;
  if (part == 0) {
    launch_fill_u64(reinterpret_cast<u64*>(ws + L.o_lfirst), (int64_t)(L.zero_bytes / 8), 0ull, st);
    u32* lfirst = reinterpret_cast<u32*>(ws + L.o_lfirst);
    u32* lrest = reinterpret_cast<u32*>(ws + L.o_lrest);
    u32* rank = reinterpret_cast<u32*>(ws + L.o_rank);
    uint4* off = reinterpret_cast<uint4*>(ws + L.o_poff);
    uint4* items_a = reinterpret_cast<uint4*>(ws + L.o_items_a);
    uint4* items_b = reinterpret_cast<uint4*>(ws + L.o_items_b);
    u32* pslot = reinterpret_cast<u32*>(ws + L.o_pslot);
    u32* qslots = reinterpret_cast<u32*>(ws + L.o_qslots);
    const unsigned pb = (unsigned)((p.nq + 3) / 4), qb = (unsigned)((p.nq * 32 * s.ks + 255) / 256);
    hipLaunchKernelGGL(ms_count_kernel, dim3(pb + qb), dim3(256), 0, st, probes, p.nq, p.npr, p.slots, (int)p.capcodes, ix.list_off, lfirst,
                       lrest, rank, pslot, qslots, pb, q, 32 * s.ks, s.map, reinterpret_cast<float*>(ws + L.o_qperm));
    hipLaunchKernelGGL(ms_offsets_kernel, dim3((unsigned)((ix.g.nlist + 1023) / 1024)), dim3(1024), 0, st, lfirst, lrest,
                       ix.list_off, ix.g.nlist, (u32)(16 * s.nt), p.seg, p.capcodes, off, p.max_a, p.max_b, ctr);
    hipLaunchKernelGGL(ms_scatter_kernel, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, probes, np, pslot, rank,
                       lfirst, lrest, off, ix.list_off, (u32)(16 * s.nt), p.seg, p.capcodes, items_a, p.max_a, items_b, p.max_b,
                       reinterpret_cast<u32*>(ws + L.o_pairs));
    if (s.onehot) {
      // (passes of a wavefront: enough that staging the codebook is not what it does)
      const int per = 8 * (64 / ix.g.M), passes = (int)std::max<int64_t>(1, std::min<int64_t>(8, p.nq / (256 * per)));
      const size_t lds = onehot_tables_bytes(ix.g);
      const dim3 tg((unsigned)((p.nq + per * passes - 1) / (per * passes)));
#define OT(MG, V)                                                                                                     \
      do {                                                                                                            \
        auto kern = &ms_onehot_tables_kernel<MG, V>;                                                                  \
        if (lds > 48 * 1024)                                                                                          \
          (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
        hipLaunchKernelGGL(kern, tg, dim3(256), lds, st, q, p.nq, ix.g.d, ix.g.dsub, ix.codebooks,                    \
                           std::max(0.f, eps_scale), passes, reinterpret_cast<u32x4*>(ws + L.o_qperm),                \
                           reinterpret_cast<float*>(ws + L.o_exact), reinterpret_cast<float4*>(ws + L.o_tinfo));      \
      } while (0)
#define OT2(MG) do { if (ix.g.dsub % 4 == 0) OT(MG, true); else OT(MG, false); } while (0)
      if (ix.g.M == 16) OT2(4); else if (ix.g.M == 32) OT2(8); else OT2(16);
#undef OT2
#undef OT
    }
    A.items = items_a;
    A.nitems = ctr;
    launch_sweep_any<0>(ix, s, A, p.max_a, st);
    const dim3 grid((unsigned)((p.nq + 3) / 4)), block(256);
#define BOUND(RR) hipLaunchKernelGGL((ms_bound_kernel<RR>), grid, block, 0, st, A.gmin, qslots, p.nq, p.slots, k, \
                                     reinterpret_cast<float*>(ws + L.o_bound))
    if (p.slots <= 128) BOUND(2); else if (p.slots <= 256) BOUND(4); else if (p.slots <= 512) BOUND(8); else BOUND(16);
#undef BOUND
    return;
  }
  if (part == 1) {
    A.items = reinterpret_cast<const uint4*>(ws + L.o_items_b);
    A.nitems = ctr + 1;
    launch_sweep_any<1>(ix, s, A, p.max_b, st);
    return;
  }
  RerankArgs B;
  B.q = q; B.nq = p.nq; B.d = ix.g.d; B.npr = p.npr; B.cap = p.cap; B.k = k;
  B.tot = k <= 64 ? 128 : k + 64;
  B.force = eps_scale < 0.f;
  B.probes = probes; B.list_off = ix.list_off;
  B.cand_count = A.cand_count; B.cand = A.cand;
  B.rescan_list = reinterpret_cast<u32*>(ws + L.o_rlist); B.rescan_count = ctr + 4;
  B.surv = reinterpret_cast<uint4*>(ws + L.o_surv); B.surv_count = ctr + 5;
  B.surv_unwritten = ctr + 6;
  B.surv_first = reinterpret_cast<u32*>(ws + L.o_sfirst); B.surv_number = reinterpret_cast<u32*>(ws + L.o_snum);
  B.surv_cap = p.surv;
  B.surv_value = reinterpret_cast<float*>(ws + L.o_sval);
  B.codes = ix.codes;
  B.sink.keys = nullptr; B.sink.val = out_dist; B.sink.id64 = out_ids; B.sink.idx32 = nullptr; B.sink.idmap = ids;
  B.sink.metric = ix.g.metric;
  B.M = ix.g.M; B.dsub = ix.g.dsub; B.form = form;
  B.centroids = ix.centroids; B.codebooks = ix.codebooks; B.cdist = cdist; B.cnorm = ix.cnorm; B.norms = ix.norms;
  B.list_tables = ix.list_tables; B.vmin = ix.vmin; B.step = ix.step;
  const int r = B.tot <= 128 ? 2 : 4;
  if (s.onehot) {
    const size_t lds = 4 * onehot_rerank_wave_bytes(ix.g.M, B.tot);
    const float* exact = reinterpret_cast<const float*>(ws + L.o_exact);
    const dim3 grid((unsigned)((p.nq + 3) / 4));
#define RO(MG) do { if (r == 2) hipLaunchKernelGGL((ms_rerank_onehot_kernel<MG, 2>), grid, dim3(256), lds, st, B, exact); \
                    else hipLaunchKernelGGL((ms_rerank_onehot_kernel<MG, 4>), grid, dim3(256), lds, st, B, exact); } while (0)
    if (ix.g.M == 16) RO(4); else if (ix.g.M == 32) RO(8); else RO(16);
#undef RO
    return;
  }
  if (ix.kind == kMsPq) {
    hipLaunchKernelGGL(ms_list_kernel, dim3((unsigned)((p.nq + 15) / 16)), dim3(1024), 0, st, B);
    size_t lds = 0;
    for (B.batch = 32; B.batch >= 8; B.batch /= 2) {
      lds = pq_eval_bytes(ix.g.M, ix.g.K, ix.g.dsub, pq_lanes(ix.g.M), B.batch);
      if (lds <= 160 * 1024) break;
    }
    // (as many workgroups as the list could keep busy: those without a survivor leave before they stage the codebook)
    const int64_t most = std::min<int64_t>(((int64_t)p.surv + 8 * B.batch - 1) / (8 * B.batch), 256ll * (160 * 1024 / lds));
#define RK(LPC, DS, NB, ROT)                                                                                       \
    do {                                                                                                           \
      auto kern = &ms_eval_pq_kernel<LPC, DS, NB, ROT>;                                                            \
      if (lds > 48 * 1024)                                                                                         \
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
      hipLaunchKernelGGL(kern, dim3((unsigned)most), dim3(kSweepThreads), lds, st, B);                             \
    } while (0)
    if (ivfpq_codes_rotated(ix.g)) {
      if (ix.g.M == 8) RK(8, 4, 8, true);
      else if (ix.g.M == 16) RK(16, 8, 8, true);
      else RK(32, 3, 8, true);
    } else if (ix.g.nbits == 8) {
      if (ix.g.M == 8) RK(8, 0, 8, false);
      else if (ix.g.M <= 16) RK(16, 0, 8, false);
      else if (ix.g.M <= 32) RK(32, 0, 8, false);
      else RK(64, 0, 8, false);
    } else {
      if (ix.g.M <= 16) RK(16, 0, 4, false);
      else if (ix.g.M <= 32) RK(32, 0, 4, false);
      else RK(64, 0, 4, false);
    }
#undef RK
    const dim3 sgrid((unsigned)((p.nq + 3) / 4));
    if (r == 2) hipLaunchKernelGGL((ms_select_kernel<2>), sgrid, dim3(256), 0, st, B);
    else hipLaunchKernelGGL((ms_select_kernel<4>), sgrid, dim3(256), 0, st, B);
    return;
  }
  const dim3 grid((unsigned)((p.nq + 3) / 4)), block(256);
  if (ix.kind == kMsFlat) {
    const bool tiled = ix.g.d % 32 == 0;
    const size_t lds = 4 * rows_rerank_wave_bytes(B.tot, ix.g.d, tiled);
#define RF(MET, TL, RG)                                                                                            \
    do {                                                                                                           \
      auto kern = &ms_rerank_flat_kernel<MET, TL, RG>;                                                             \
      if (lds > 48 * 1024)                                                                                         \
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
      hipLaunchKernelGGL(kern, grid, block, lds, st, B);                                                           \
    } while (0)
#define RM(MET) do { if (tiled) { if (r == 2) RF(MET, true, 2); else RF(MET, true, 4); } \
                     else { if (r == 2) RF(MET, false, 2); else RF(MET, false, 4); } } while (0)
    if (ix.g.metric == 0) RM(0); else RM(1);
#undef RM
#undef RF
    return;
  }
  const size_t lds = 4 * sq8_rerank_wave_bytes(B.tot, ix.g.d);
#define RS(MET) do { if (r == 2) hipLaunchKernelGGL((ms_rerank_sq8_kernel<MET, 2>), grid, block, lds, st, B); \
                     else hipLaunchKernelGGL((ms_rerank_sq8_kernel<MET, 4>), grid, block, lds, st, B); } while (0)
  if (ix.g.metric == 0) RS(0); else RS(1);
#undef RS
}
