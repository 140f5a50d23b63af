// Nearest row of B for every row of A on the matrix cores, in ONE sweep: list assignment of
// vectors being added and the assignment step of k-means (Sec. 4.1), where only the best row
// is wanted, and the nearest codeword of every sub-vector (Sec. 4.1 product quantizer).
//
// The k-nearest-rows route (kernels_mfma.hip) needs two sweeps, a threshold and a re-rank
// because it selects k rows.  For one row a running maximum in registers is the selection:
// with the vectors on the COLUMN side of the 32 x 32 product every lane holds 16 scores of one
// vector, so best and runner-up cost three vector instructions per score (tag, median, maximum)
// and no exchange between lanes until the end.  The score of row b for vector a is
//     L2: <a, b> - |b|^2 / 2  (= (|a|^2 - distance) / 2; the accumulators start at -|b|^2 / 2)
//     IP: <a, b>
// A vector's answer is certain when best and runner-up are further apart than the error bound of
// the product.  The others go to a list; a second sweep over the listed vectors collects the rows
// within the bound of the best (two or three, usually) and the canon chain decides among them, so
// that every answer is the canon answer (ties to the smaller row).
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "internal.hpp"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr float kPadScore = -3.0e38f;   // finite: tagging an infinity would make it a NaN

// (round to nearest even; one instruction for two of them)
__device__ __forceinline__ unsigned short bf16_bits(float f) { return __builtin_bit_cast(unsigned short, (__bf16)f); }
__device__ __forceinline__ float bf16_value(unsigned short b) { return __uint_as_float(((u32)b) << 16); }

template <bool F16>
__device__ __forceinline__ floatx16 mfma16(u16x8 a, u16x8 b, floatx16 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The larger of two as their median with infinity: one instruction where fmaxf would first quiet its inputs, and one
// that the scheduler knows.  (The infinity sits in a scalar register the compiler knows nothing of, or it would be fmaxf
// again.)
struct Largest {
  float infinity;
  __device__ __forceinline__ void init() {
    infinity = __builtin_inff();
    asm volatile("" : "+s"(infinity));
  }
  __device__ __forceinline__ float operator()(float a, float b) const { return __builtin_amdgcn_fmed3f(a, b, infinity); }
};
// Best and runner-up of a stream of scores, the best tagged with a number below TAGS in its low bits (16: 2^-19 of its
// magnitude, part of the error bound): v_and_or and two v_med3.
template <int TAGS>
struct Top2 {
  float b1, b2;
  __device__ __forceinline__ void init() { b1 = b2 = -__builtin_inff(); }
  __device__ __forceinline__ void put(const Largest& largest, float s, int tag) {
    const float p = __uint_as_float((__float_as_uint(s) & ~(u32)(TAGS - 1)) | (u32)tag);
    b2 = __builtin_amdgcn_fmed3f(b1, b2, p);
    b1 = largest(b1, p);
  }
  __device__ __forceinline__ int tag() const { return (int)(__float_as_uint(b1) & (u32)(TAGS - 1)); }
};
// (a register at a time, not a half)
__device__ __forceinline__ u16x8 pick(int second, u16x8 a, u16x8 b) {
  const u32x4 x = __builtin_bit_cast(u32x4, a), y = __builtin_bit_cast(u32x4, b);
  u32x4 r;
#pragma unroll
  for (int u = 0; u < 4; ++u) r[u] = second ? y[u] : x[u];
  return __builtin_bit_cast(u16x8, r);
}
// row inside a 32-row block of accumulator register v in lane half h
__device__ __forceinline__ int block_row(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }

// what a sweep learns about a vector (one byte)
enum { VEC_INT = 1, VEC_EXACT = 2, VEC_NONNEG = 4, VEC_LARGE = 8 };

// ---------------------------------------------------------------------------
// One workgroup = 4 wavefronts x 64 (or 32) vectors; a wavefront converts its vectors straight from the
// fp32 rows (no prepared operand, no pass of its own over them) into fragments that stay in
// registers, and walks over a range of B in steps of 64 rows staged through LDS (double
// buffered, padded rows: conflict-free 128-bit reads), each tile read by all four wavefronts.
// BF == false: one product on the fp16 heads.  BF == true: bf16 heads, and the products with the
// tails of either side where that side is not exactly bf16.  A call launches both, one pass after the
// other, and NearestState says what each has to do (pass_vectors): where B's rows are in range and the
// heads have not failed too often they take all vectors, and the bf16 pass those that the heads left
// with too many candidates; else the bf16 pass takes all.
// COLLECT: the second sweep of a pass.  thr [e] = the score from which a row may still be the best;
// passing rows go to cand [e][kCandidates] and are counted in cnt [e].
// Per 32 x 32 block: KSTEPS products of 32 cycles against 16 x 3 selection instructions of 4.
// rows: the numbers of the vectors to do, where they are not all.
// Assignment of 1M integer vectors to 4096 rows at d = 128 (two sweeps, threshold, re-rank and
// operand preparation before): 6.1 -> 1.06 ms (first sweep 1.02, second 0.02).
// ---------------------------------------------------------------------------
// 32-vector blocks per wavefront: two, and one where heads and tails of two do not fit the registers
template <int KSTEPS, bool BF> constexpr int kNearestBlocks = BF && KSTEPS > 4 ? 1 : 2;

constexpr int kCandidates = 16;
// Threshold of a vector (or of a lane past the list) that collects nothing: no score compares with a
// NaN, while the scores of a vector beyond the fp16 range reach +infinity themselves.
__device__ __forceinline__ float collects_nothing() { return __builtin_nanf(""); }

// What a call's kernels tell each other (device memory).  listed: vectors whose best row a pass was
// not certain of; left: those that its candidates did not decide.
struct NearestState {
  int heads;                  // the fp16 heads take all vectors first
  int listed[2], left[2];     // of the fp16 pass and of the bf16 pass
};
// Few vectors that the heads left go straight to the canon chain, which spreads a single one over the
// chip; a bf16 sweep costs about what redoing one vector in 512 costs (the rule of the k-nearest-rows
// route's fallback).
__device__ __forceinline__ bool sweep_left(const NearestState* s, int64_t n) {
  return s->left[0] >= 8 && (int64_t)s->left[0] * 512 > n;
}
// vectors of the first sweep of a pass: all (null) or the ones left by the pass before
__device__ __forceinline__ int64_t pass_vectors(const NearestState* s, int64_t n, bool bf, const int*& rows) {
  if (!bf) { rows = nullptr; return s->heads ? n : 0; }
  if (!s->heads) { rows = nullptr; return n; }
  return sweep_left(s, n) ? min((int64_t)s->left[0], n) : 0;
}

template <int KSTEPS, int METRIC, bool BF, bool COLLECT>
__global__ __launch_bounds__(256, 2) void nearest_kernel(
    const float* __restrict__ x, int64_t n, int d, const unsigned short* __restrict__ Bh,
    const unsigned short* __restrict__ Bl, const float* __restrict__ Bnorm, const PrepInfo* __restrict__ Binfo,
    int64_t nb, int64_t tiles, int64_t cols_per_split, const int* rows,
    const NearestState* __restrict__ state, float* __restrict__ out_b1, float* __restrict__ out_b2,
    int* __restrict__ out_idx, float* __restrict__ out_norm, unsigned char* __restrict__ out_flags,
    const float* __restrict__ thr, int* __restrict__ cnt, int* __restrict__ cand) {
  constexpr int D = KSTEPS * 16, BN = 64, LDB = D + 8, NPL = BF ? 2 : 1, RB = kNearestBlocks<KSTEPS, BF>;
  constexpr int CPT = BN * (D / 8) / 256;                         // 16-byte chunks per lane, plane and step
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned short* bt = reinterpret_cast<unsigned short*>(smem);   // [2][NPL][BN][LDB]
  float* nrm_s = reinterpret_cast<float*>(bt + 2 * NPL * BN * LDB);   // [2][BN] starting values
  const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id(), half = lane >> 5;
  const int64_t total = COLLECT ? min((int64_t)state->listed[BF], n) : pass_vectors(state, n, BF, rows);
  // The second sweep cuts B by the vectors that are listed, which only the device knows: as many splits as two
  // workgroups per compute unit and the grid allow, of two steps or more (its results depend on no split).  Cut like
  // the first sweep, a few listed vectors of a million walked over all rows of B in one workgroup: 210 us at 4096 rows,
  // 24 like this; 262144 vectors against 1024 trained rows: 104 -> 40.
  if constexpr (COLLECT) {
    tiles = max((total + 128 * RB - 1) / (128 * RB), (int64_t)1);
    const int64_t steps = (nb + BN - 1) / BN, want = min((int64_t)gridDim.x, (int64_t)512) / tiles;
    const int64_t splits = max(min(want, steps / 2), (int64_t)1);
    cols_per_split = (steps + splits - 1) / splits * BN;
  }
  const int64_t split = blockIdx.x / tiles, tile = blockIdx.x - split * tiles;
  const int64_t e0 = tile * 128 * RB;
  if (e0 >= total) return;
  const int64_t c_begin = split * cols_per_split, c_end = min(nb, c_begin + cols_per_split);
  if (COLLECT && c_begin >= c_end) return;
  const bool use_bl = BF && Binfo->all_bf16 == 0u;
  const bool vec = (d & 3) == 0;

  u16x8 xh[RB][KSTEPS], xl[BF ? RB : 1][BF ? KSTEPS : 1];
  bool inexact = false;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int64_t e = e0 + wave * (32 * RB) + rb * 32 + (lane & 31);
    const int64_t ec = min(e, total - 1);
    const float* __restrict__ row = x + (rows ? (int64_t)rows[ec] : ec) * d;
    float ss = 0.f;
    bool is_int = true, exact = true, nonneg = true, large = false;
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
      float v[8];
      load_row8(row, kk * 16 + 8 * half, d, vec, v);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        float rem;
        if constexpr (BF) {
          const unsigned short h = bf16_bits(v[t]);
          rem = v[t] - bf16_value(h);
          xh[rb][kk][t] = h;
          xl[rb][kk][t] = bf16_bits(rem);
        } else {
          const _Float16 h = (_Float16)v[t];
          rem = v[t] - (float)h;
          xh[rb][kk][t] = __builtin_bit_cast(unsigned short, h);
        }
        exact = exact && rem == 0.f;
        is_int = is_int && v[t] == __builtin_rintf(v[t]);
        nonneg = nonneg && v[t] >= 0.f;
        large = large || !(__builtin_fabsf(v[t]) <= 32768.f);
        ss = __builtin_fmaf(v[t], v[t], ss);
      }
    }
    ss += __shfl_xor(ss, 32);
    int fl = (is_int ? VEC_INT : 0) | (exact ? VEC_EXACT : 0) | (nonneg ? VEC_NONNEG : 0);
    fl &= __shfl_xor(fl, 32);
    int lg = large ? VEC_LARGE : 0;
    lg |= __shfl_xor(lg, 32);
    inexact = inexact || !(fl & VEC_EXACT);
    if (!COLLECT && split == 0 && half == 0 && e < total) { out_norm[e] = ss; out_flags[e] = (unsigned char)(fl | lg); }
  }
  const bool use_al = BF && __builtin_amdgcn_ballot_w64(inexact) != 0;

  u32x4 stg[NPL][CPT];
  float stn = 0.f;
  auto fetch = [&](int64_t ct) {   // (planes are padded to a multiple of 64 rows)
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int64_t o = ct * D + (int64_t)(tid + 256 * i) * 8;
      stg[0][i] = *reinterpret_cast<const u32x4*>(Bh + o);
      if constexpr (BF) { if (use_bl) stg[1][i] = *reinterpret_cast<const u32x4*>(Bl + o); }
    }
    stn = Bnorm[ct + (tid & 63)];
  };
  auto stash = [&](int buf, int64_t ct) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int ch = tid + 256 * i;
      const int at = (ch / (D / 8)) * LDB + (ch % (D / 8)) * 8;
      *reinterpret_cast<u32x4*>(bt + (buf * NPL) * BN * LDB + at) = stg[0][i];
      if constexpr (BF) { if (use_bl) *reinterpret_cast<u32x4*>(bt + (buf * NPL + 1) * BN * LDB + at) = stg[1][i]; }
    }
    if (tid < BN) nrm_s[buf * BN + tid] = ct + tid < c_end ? (METRIC == 0 ? -0.5f * stn : 0.f) : kPadScore;
  };

  Top2<16> top[RB];
  int blk[RB] = {};
  Largest largest;
  largest.init();
  float th_e[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    top[rb].init();
    const int64_t e = e0 + wave * (32 * RB) + rb * 32 + (lane & 31);
    th_e[rb] = COLLECT && e < total ? thr[e] : collects_nothing();
  }
  if (c_begin < c_end) { fetch(c_begin); stash(0, c_begin); }
  wait_all_global_loads();
  block_sync_lds();
  int buf = 0;
  // The first sweep selects from the block of rows before while the products of the next one run: the matrix cores and
  // the vector units work side by side for one wavefront too, and not only where two of them happen to be out of step
  // (1M x 4096 x 128: 1092 -> 1015 us; the fragments' LDS reads are the next limit).
  floatx16 done[COLLECT ? 1 : RB];
  int done_block = 0;   // (what stands before the first block wins where no score compares, and has to name a row of B)
  float before[RB];
  auto select = [&](int rb, int v0, int v1) {
    if constexpr (!COLLECT) {
      if (v0 == 0) before[rb] = top[rb].b1;
#pragma unroll
      for (int v = v0; v < v1; ++v) top[rb].put(largest, done[rb][v], v);
      if (v1 == 16) blk[rb] = top[rb].b1 > before[rb] ? done_block : blk[rb];
    }
  };
  auto collect = [&](const floatx16 (&m)[RB], int64_t c0) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float mx = m[rb][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) mx = fmaxf(mx, m[rb][v]);
      if (__builtin_amdgcn_ballot_w64(mx >= th_e[rb]) == 0) continue;
      const int64_t e = e0 + wave * (32 * RB) + rb * 32 + (lane & 31);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (m[rb][v] >= th_e[rb]) {
          const int64_t c = c0 + block_row(v, half);
          if (c < c_end) {
            const int pos = atomicAdd(&cnt[e], 1);
            if ((u32)pos < (u32)kCandidates) cand[e * kCandidates + pos] = (int)c;
          }
        }
    }
  };
  if constexpr (!COLLECT) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int v = 0; v < 16; ++v) done[rb][v] = kPadScore;       // (no block before the first: loses to every row)
  }
  for (int64_t ct = c_begin; ct < c_end; ct += BN, buf ^= 1) {
    const bool more = ct + BN < c_end;
    if (more) fetch(ct + BN);                                     // in flight during the products
    const unsigned short* __restrict__ th = bt + (buf * NPL) * BN * LDB;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      floatx16 c0;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 t4 = *reinterpret_cast<const float4*>(nrm_s + buf * BN + cb * 32 + 8 * g + 4 * half);
        c0[4 * g] = t4.x; c0[4 * g + 1] = t4.y; c0[4 * g + 2] = t4.z; c0[4 * g + 3] = t4.w;
      }
      const unsigned short* __restrict__ fr = th + (cb * 32 + (lane & 31)) * LDB + 8 * half;
      floatx16 m[RB];
      constexpr int PF = KSTEPS < 3 ? KSTEPS : 3;                 // fragments requested ahead
      u16x8 frag[PF];
#pragma unroll
      for (int f = 0; f < PF; ++f) frag[f] = *reinterpret_cast<const u16x8*>(fr + f * 16);
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk) {
        const u16x8 b = frag[kk % PF];
        if (kk + PF < KSTEPS) frag[kk % PF] = *reinterpret_cast<const u16x8*>(fr + (kk + PF) * 16);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          m[rb] = mfma16<!BF>(b, xh[rb][kk], kk == 0 ? c0 : m[rb]);
          if constexpr (BF) {
            if (use_al) m[rb] = mfma16<false>(b, xl[rb][kk], m[rb]);
          }
          select(rb, 16 * kk / KSTEPS, 16 * (kk + 1) / KSTEPS);
          if constexpr (!COLLECT && !BF) {   // (keeps that order: a product, and 16 / KSTEPS selections beside it)
            asm volatile("" : "+v"(top[rb].b1), "+v"(top[rb].b2));
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      if constexpr (BF) {
        if (use_bl) {
#pragma unroll
          for (int kk = 0; kk < KSTEPS; ++kk) {
            const u16x8 b = *reinterpret_cast<const u16x8*>(fr + BN * LDB + kk * 16);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) m[rb] = mfma16<false>(b, xh[rb][kk], m[rb]);
          }
        }
      }
      if constexpr (COLLECT) {
        collect(m, ct + cb * 32);
      } else {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) done[rb] = m[rb];
        done_block = (int)((ct - c_begin) >> 5) + cb;
      }
    }
    if (more) stash(buf ^ 1, ct + BN);
    block_sync_lds();
  }
  if constexpr (!COLLECT) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) select(rb, 0, 16);
  }
  if constexpr (COLLECT) return;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {   // the two lanes of a vector
    const int64_t e = e0 + wave * (32 * RB) + rb * 32 + (lane & 31);
    int idx = blk[rb] * 32 + block_row(top[rb].tag(), half);
    const float o1 = __shfl_xor(top[rb].b1, 32), o2 = __shfl_xor(top[rb].b2, 32);
    const int oi = __shfl_xor(idx, 32);
    const float b1 = fmaxf(top[rb].b1, o1);
    const float b2 = fmaxf(fminf(top[rb].b1, o1), fmaxf(top[rb].b2, o2));
    if (o1 > top[rb].b1) idx = oi;
    if (half == 0 && e < total) {
      out_b1[split * n + e] = b1;
      out_b2[split * n + e] = b2;
      out_idx[split * n + e] = (int)min(c_begin + idx, nb - 1);   // (rows past the end never win; NaNs)
    }
  }
}

// Merges the splits, writes every vector's best row and puts those that are not certain on the
// list, each with the score down to which a row may still be the best.  left: the vectors that the
// fp16 pass left (for the bf16 pass).
template <int METRIC, bool BF>
__global__ __launch_bounds__(256) void nearest_finish_kernel(
    int64_t n, int d, int nsplit, const float* __restrict__ in_b1, const float* __restrict__ in_b2,
    const int* __restrict__ in_idx, const float* __restrict__ norm, const unsigned char* __restrict__ flags,
    const PrepInfo* __restrict__ Binfo, float eps_scale, int32_t* __restrict__ idx, const int* __restrict__ left,
    NearestState* __restrict__ state, int* __restrict__ list, float* __restrict__ thr, int* __restrict__ cnt) {
  const int64_t e = blockIdx.x * 256ll + threadIdx.x;
  constexpr bool bf = BF;
  const int* rows = left;
  const int64_t total = pass_vectors(state, n, BF, rows);
  if (BF && e == 0 && total == 0) state->left[1] = state->left[0];   // (no second pass: its list stands)
  if (blockIdx.x * 256ll >= total) return;
  bool unsure = false;
  float from = 0.f;
  int row = 0;
  if (e < total) {
    row = rows ? rows[e] : (int)e;
    float b1 = -__builtin_inff(), b2 = b1;
    int best = 0;
    for (int s = 0; s < nsplit; ++s) {
      const float o1 = in_b1[s * n + e], o2 = in_b2[s * n + e];
      const int oi = in_idx[s * n + e];
      b2 = fmaxf(fmaxf(b2, o2), fminf(b1, o1));
      if (o1 > b1) { b1 = o1; best = oi; }
    }
    // Bounds as in the re-rank of kernels_mfma.hip (on the distance; the score is half of it under
    // L2): fp16 heads 9.78e-4 (half of it where one side is exact), bf16 head and tail 6.2e-5 of
    // N = |a|^2 + max |b|^2, fp32 accumulation d 4.8e-7, and 4e-6 for the tags.  Integers that
    // the operands represent exactly leave the tags alone (and 1e-30: the tags tell scores of
    // zero apart, and products of tiny numbers vanish).
    const int fl = flags[e];
    const float nb2 = __uint_as_float(Binfo->max_norm_bits), nn = norm[e] + nb2;
    const bool b_exact = Binfo->all_bf16 != 0u && (bf || Binfo->all_int != 0u);   // (integers exact in bf16 and below 2^15 are exact in fp16)
    const bool a_exact = (fl & VEC_EXACT) != 0;
    const bool ints = a_exact && b_exact && (fl & VEC_INT) && Binfo->all_int != 0u &&
                      ((fl & VEC_NONNEG) && Binfo->all_nonneg ? nn < 8388608.f : nn < 5592405.f);
    float eps = 4e-6f * nn + 1e-30f;
    if (!ints) {
      const float split = a_exact && b_exact ? 0.f : (bf ? 6.2e-5f : (a_exact || b_exact ? 4.9e-4f : 9.78e-4f));
      const float sub = bf ? 0.f : 6.0e-8f * sqrtf(2.f * (float)d * nn) + 1.8e-15f * (float)d;   // fp16 subnormals
      const float rounding = ((float)d * 4.8e-7f + 2e-6f) * nn;
      eps += METRIC == 0 ? split * nn + sub + rounding : (bf ? 2.f : 1.f) * split * nn + sub + 2.f * rounding;
    }
    unsure = !(b1 - b2 > eps_scale * eps) || (!bf && (fl & VEC_LARGE)) || eps_scale < 0.f;
    // (a vector beyond the fp16 range or with a NaN, and every vector where a norm overflows -- their
    // scores are infinities and NaNs that say nothing -- collects nothing: it is left to the next pass
    // or the canon chain)
    from = (!bf && (fl & VEC_LARGE)) || eps_scale < 0.f || !(nn < __builtin_inff()) ? collects_nothing() : b1 - eps;
    idx[row] = best;
  }
  // one atomic per workgroup (per wavefront they were most of the kernel: 45 us for 4096 of them)
  __shared__ int wave_count[4], base_s;
  const u64 mask = __builtin_amdgcn_ballot_w64(unsure);
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  if (lane == 0) wave_count[wave] = __popcll(mask);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int all = wave_count[0] + wave_count[1] + wave_count[2] + wave_count[3];
    base_s = all > 0 ? atomicAdd(&state->listed[BF], all) : 0;
  }
  __syncthreads();
  if (unsure) {
    int at = base_s + __popcll(mask & ((1ull << lane) - 1ull));
    for (int w = 0; w < wave; ++w) at += wave_count[w];
    list[at] = row;
    thr[at] = from;
    cnt[at] = 0;
  }
}

// The canon best among a listed vector's candidates: 16 lanes per vector, one candidate each.
// Vectors whose candidates did not fit (or that have none) are left to the bf16 pass or, after it, to
// the canon chain over all rows.
// learn: this call's counts may clear B's heads_only (not where every vector is listed on request).
template <int METRIC, bool BF>
__global__ __launch_bounds__(256) void nearest_decide_kernel(
    const float* __restrict__ x, int64_t n, int d, const float* __restrict__ B, int64_t nb,
    PrepInfo* __restrict__ Binfo, const int* __restrict__ list, NearestState* __restrict__ state,
    const int* __restrict__ cnt, const int* __restrict__ cand, int32_t* __restrict__ idx,
    int* __restrict__ left, bool learn) {
  const int total = (int)min((int64_t)state->listed[BF], n);
  if (!BF && learn && blockIdx.x == 0 && threadIdx.x == 0 && total >= 64 && 2ll * total > n) {
    // the fp16 heads decided fewer than half of the vectors: later calls begin with bf16 (the heads
    // cost one product, the second sweep and three products for what they leave)
    atomicAnd(&Binfo->heads_only, ~PrepInfo::kHeadsSweep);
  }
  const bool vec = (d & 3) == 0;
  const int lane = lane_id(), sub = lane & 15;
  for (int e = blockIdx.x * 16 + (threadIdx.x >> 4); e - (int)(threadIdx.x >> 4) < total; e += gridDim.x * 16) {
    if (e >= total) continue;
    const int row = list[e], c = cnt[e];
    if (c < 1 || c > kCandidates) {
      if (sub == 0) left[atomicAdd(&state->left[BF], 1)] = row;
      continue;
    }
    u64 key = KEY_EMPTY;
    if (sub < c) {
      const int j = cand[(int64_t)e * kCandidates + sub];
      key = make_key(canon_row_padded<METRIC>(x + (int64_t)row * d, B + (int64_t)j * d, d, vec), (u32)j, METRIC);
    }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) { const u64 o = __shfl_xor(key, off); key = o < key ? o : key; }
    if (sub == 0) idx[row] = (int)min(key_index(key), (u32)(nb - 1));
  }
}

// val[i] = canon distance (L2) of vector i to row idx[i] of B.  One wavefront per 64 vectors: both
// rows are read in 128-byte runs (8 lanes per row), their differences go through LDS and lane r
// continues the chain of vector r in dimension order.
__global__ __launch_bounds__(64) void row_values_kernel(const float* __restrict__ x, int64_t n, int d,
                                                        const float* __restrict__ B,
                                                        const int32_t* __restrict__ idx, float* __restrict__ val) {
  constexpr int DC = 32, LD = 36;
  __shared__ __attribute__((aligned(16))) float tile[64 * LD];
  const int lane = lane_id(), r_ld = lane >> 3, c_ld = (lane & 7) * 4;
  const int64_t i0 = blockIdx.x * 64ll;
  const bool vec = (d & 3) == 0;
  int64_t ro[8], bo[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int64_t i = min(i0 + r_ld + 8 * j, n - 1);
    ro[j] = i * d;
    bo[j] = (int64_t)idx[i] * d;
  }
  float acc = 0.f;
  for (int c0 = 0; c0 < d; c0 += DC) {
    const int c = c0 + c_ld;
    float df[8][4];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (vec) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
        if (c < d) { a = *reinterpret_cast<const float4*>(x + ro[j] + c); b = *reinterpret_cast<const float4*>(B + bo[j] + c); }
        df[j][0] = a.x - b.x; df[j][1] = a.y - b.y; df[j][2] = a.z - b.z; df[j][3] = a.w - b.w;
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) df[j][u] = c + u < d ? x[ro[j] + c + u] - B[bo[j] + c + u] : 0.f;
      }
    }
    wave_lds_sync();                                  // the chunk before has been consumed
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u) tile[(r_ld + 8 * j) * LD + c_ld + u] = df[j][u];
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < DC; ++u) { const float t = tile[lane * LD + u]; acc = __builtin_fmaf(t, t, acc); }
  }
  if (i0 + lane < n) val[i0 + lane] = acc;
}

__global__ void nearest_state_kernel(const PrepInfo* __restrict__ Binfo, NearestState* __restrict__ s) {
  s->heads = (Binfo->heads_only & PrepInfo::kHeadsSweep) != 0u && Binfo->max_norm_bits <= 0x4E800000u;   // 2^30
  s->listed[0] = s->listed[1] = s->left[0] = s->left[1] = 0;
}

// ---------------------------------------------------------------------------
// Nearest codeword of every sub-vector (at most 16 dimensions, 256 or 16 codewords).
// Vectors again on the column side; the codewords of one sub-quantizer are the row side and stay
// in registers for the whole kernel.  A sub-vector has so few dimensions that the whole split
// product fits one or two matrix instructions: the 8-slot groups of the contraction hold
//     vector   [ head | head | tail | 1 1 1 0 ... ]
//     codeword [ head | tail | head | -|t|^2 / 2 in three bf16 pieces ]
// (NP groups of each kind for 8 NP dimensions), so the score <r, t> - |t|^2 / 2 comes out finished
// and costs only the selection.  A lane's four consecutive codewords of a product share one tag: their
// largest score is selected, 5 vector instructions for four scores (3 for every one of them before, which was most of
// the kernel), and the canon chain decides among the best four, two on either half of the wavefront.
// Sub-vectors whose best two fours are within the error bound are decided
// by the canon chain over all codewords, 64 codewords at a time (about one in a hundred;
// all of them where eps_scale, which scales the bound, is negative).
// RES: sub-vector m of x_i minus its list's centroid; else x is [M][n][dsub].
// Encoding 1M vectors of 16 x 8 dimensions: 688 -> 515 us; 16 x 262144 sub-vectors of 8 in training: 175 -> 117.  (Half
// the vector instructions; the second half of the gain is the padded codebook and the pieces of a row asked for together.)
// ---------------------------------------------------------------------------
// (four resp. two wavefronts per SIMD; a bound on the registers also keeps the products' results in
// vector registers, where the selection can read them without a copy)
// floats from one four of codewords to the next in LDS: 16-byte pieces stay aligned, and consecutive fours start in
// different banks
__host__ __device__ constexpr int pq_four_stride(int dsub, bool vec) { return 4 * dsub + (vec ? 4 : 1); }
template <int NP, int KB, bool RES, bool VEC>
__global__ __launch_bounds__(256, NP == 1 ? 4 : 2) void pq_nearest_kernel(
    const float* __restrict__ x, int64_t n, int d, int dsub, const float* __restrict__ centroids,
    const int32_t* __restrict__ list_of, const float* __restrict__ codebooks, int K, int M, int64_t chunks,
    int groups, float eps_scale, uint8_t* __restrict__ codes, int64_t stride_i, int64_t stride_m,
    float* __restrict__ val) {
  constexpr int NG = 3 * NP + 1, S = (NG + 1) / 2, DP = 8 * NP;
  // [K / 4][4][dsub] and padding: the gathers of a best four by every lane would otherwise fall into a few banks
  // (dsub = 8 without it: 676 cycles a product group waited for, and the whole kernel 35 % slower)
  extern __shared__ __attribute__((aligned(16))) float T[];
  const int fours = pq_four_stride(dsub, VEC);
  auto word = [&](int j) { return T + (j >> 2) * fours + (j & 3) * dsub; };
  const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id(), half = lane >> 5;
  // workgroup ids go round the eight XCDs: an XCD takes all sub-quantizers of a chunk of vectors in
  // a row, so that a chunk's rows come into its L2 once
  const int64_t seq = blockIdx.x >> 3;
  const int64_t chunk = seq / M * 8 + (blockIdx.x & 7);
  const int m = (int)(seq % M);
  if (chunk >= chunks) return;
  const float* __restrict__ Tm = codebooks + (int64_t)m * K * dsub;
  for (int e = tid; e < K * dsub; e += 256) T[e / (4 * dsub) * fours + e % (4 * dsub)] = Tm[e];
  __syncthreads();

  bool odd = false;   // a codeword with a NaN or a norm that overflows: its scores say nothing
  // codeword fragments: lane = codeword (row of the block), half = which group of a step
  u16x8 af[KB][S];
#pragma unroll
  for (int b = 0; b < KB; ++b) {
    const int j = b * 32 + (lane & 31);
    u16x8 th[NP], tl[NP], tn;
    float tt = 0.f;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = 8 * p + u;
        const float v = t < dsub && j < K ? word(j)[t] : 0.f;
        tt = __builtin_fmaf(v, v, tt);
        const unsigned short h = bf16_bits(v);
        th[p][u] = h;
        tl[p][u] = bf16_bits(v - bf16_value(h));
      }
    odd = odd || !(tt < __builtin_inff());
    const float hn = j < K ? -0.5f * tt : kPadScore;
    const unsigned short n1 = bf16_bits(hn);
    const float r1 = hn - bf16_value(n1);
    const unsigned short n2 = bf16_bits(r1);
    const unsigned short n3 = bf16_bits(r1 - bf16_value(n2));
#pragma unroll
    for (int u = 0; u < 8; ++u) tn[u] = 0;
    tn[0] = n1; tn[1] = j < K ? n2 : 0; tn[2] = j < K ? n3 : 0;
    const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < S; ++s) {
      auto group = [&](int g) { return g < NP ? th[g % NP] : (g < 2 * NP ? tl[g % NP] : (g < 3 * NP ? th[g % NP] : (g == 3 * NP ? tn : zero))); };
      af[b][s] = pick(half, group(2 * s), group(2 * s + 1));
    }
  }
  // (no difference of scores is larger than a NaN: every sub-vector goes through the canon branch)
  const float bound = __builtin_amdgcn_ballot_w64(odd) != 0 || eps_scale < 0.f ? __builtin_nanf("") : eps_scale * 4e-5f;
  const floatx16 fzero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  Largest largest;
  largest.init();
  const int64_t base = (chunk * 4 + wave) * 32ll * groups;
  // (a group's list numbers are there a group early, and all pieces of its rows are requested together)
  int next_list = RES ? list_of[min(base + (lane & 31), n - 1)] : 0;
  for (int g = 0; g < groups; ++g) {
    const int64_t i0 = base + g * 32;
    if (i0 >= n) break;
    const int64_t i = min(i0 + (lane & 31), n - 1);
    const int list = next_list;
    if (RES) next_list = list_of[min(i0 + 32 + (lane & 31), n - 1)];
    float r[DP];
    {
      const float* __restrict__ xi = RES ? x + i * d + m * dsub : x + ((int64_t)m * n + i) * dsub;
      const float* __restrict__ c = RES ? centroids + (int64_t)list * d + m * dsub : nullptr;
      if constexpr (VEC) {   // dsub % 4 == 0, rows of 16-byte pieces (those past the end: the first again, dropped)
        u32x4 a[DP / 4], cc[DP / 4];
#pragma unroll
        for (int t = 0; t < DP; t += 4) {
          const int at = t < dsub ? t : 0;
          a[t / 4] = *reinterpret_cast<const u32x4*>(xi + at);
          if (RES) cc[t / 4] = *reinterpret_cast<const u32x4*>(c + at);
        }
#pragma unroll
        for (int t = 0; t < DP; ++t) {
          const float v = __uint_as_float(a[t / 4][t & 3]);
          r[t] = RES ? v - __uint_as_float(cc[t / 4][t & 3]) : v;
          if (t >= dsub) r[t] = 0.f;
        }
      } else {
#pragma unroll
        for (int t = 0; t < DP; ++t) {
          r[t] = 0.f;
          if (t < dsub) { r[t] = xi[t]; if (RES) r[t] -= c[t]; }
        }
      }
    }
    float rr = 0.f;
    u16x8 rh[NP], rl[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float v = r[8 * p + u];
        rr = __builtin_fmaf(v, v, rr);
        const unsigned short h = bf16_bits(v);
        rh[p][u] = h;
        rl[p][u] = bf16_bits(v - bf16_value(h));
      }
    u16x8 xf[S];
    {
      const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
      const u16x8 ones = {0x3F80, 0x3F80, 0x3F80, 0, 0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < S; ++s) {
        auto group = [&](int q) { return q < 2 * NP ? rh[q % NP] : (q < 3 * NP ? rl[q % NP] : (q == 3 * NP ? ones : zero)); };
        xf[s] = pick(half, group(2 * s), group(2 * s + 1));
      }
    }
    // (16 codewords: half the selections saved are not worth the canon chain of four; 64 x 12 of 5 million vectors 3.09 ms
    // by fours, 2.77 by scores)
    constexpr bool FOURS = KB > 1;
    Top2<FOURS ? 4 * KB : 16> top;
    top.init();
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      floatx16 s = mfma16<false>(af[b][0], xf[0], fzero);
#pragma unroll
      for (int st = 1; st < S; ++st) s = mfma16<false>(af[b][st], xf[st], s);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (!FOURS) top.put(largest, s[v], v);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (FOURS) top.put(largest, fmaxf(fmaxf(largest(s[4 * q], s[4 * q + 1]), s[4 * q + 2]), s[4 * q + 3]), 4 * b + q);
    }
    int best = FOURS ? 8 * top.tag() + 4 * half : block_row(top.tag(), half);   // first codeword of the best four
    const float o1 = __shfl_xor(top.b1, 32), o2 = __shfl_xor(top.b2, 32);
    const int ob = __shfl_xor(best, 32);
    const float b1 = fmaxf(top.b1, o1), b2 = fmaxf(fminf(top.b1, o1), fmaxf(top.b2, o2));
    if (o1 > top.b1) best = ob;
    best = min(best, K - (FOURS ? 4 : 1));
    // the canon best of these four: two by either half of the wavefront
    float val_best = 0.f;
    if constexpr (FOURS) {
      const int j0 = best + 2 * half;
      const float* w0 = word(j0);
      float a0 = 0.f, a1 = 0.f;
      auto add = [&](int t, float t0, float t1) {
        const float d0 = r[t] - t0, d1 = r[t] - t1;
        a0 = __builtin_fmaf(d0, d0, a0);
        a1 = __builtin_fmaf(d1, d1, a1);
      };
#pragma unroll
      for (int t = 0; t < DP; t += VEC ? 4 : 1) {
        if (t >= dsub) continue;
        if constexpr (VEC) {
          const float4 t0 = *reinterpret_cast<const float4*>(w0 + t), t1 = *reinterpret_cast<const float4*>(w0 + dsub + t);
          add(t, t0.x, t1.x); add(t + 1, t0.y, t1.y); add(t + 2, t0.z, t1.z); add(t + 3, t0.w, t1.w);
        } else {
          add(t, w0[t], w0[dsub + t]);
        }
      }
      int j = a1 < a0 ? j0 + 1 : j0;
      float a = a1 < a0 ? a1 : a0;
      const float oa = __shfl_xor(a, 32);
      const int oj = __shfl_xor(j, 32);
      if (oa < a || (oa == a && oj < j)) { a = oa; j = oj; }
      best = j;
      val_best = a;
    }
    // Error of a score: 1.2e-5 |r||t| (dropped tails), 2e-6 (fp32, at most 48 terms, and the canon
    // chain), 3.9e-6 (tags) of N = |r|^2 + |t|^2, and any codeword that could be the nearest has
    // |t| <= |r| + its distance, whose square is at most |r|^2 - 2 b2 up to that error.
    const float dist = sqrtf(fmaxf(rr - 2.f * b2, 0.f)), tmax = sqrtf(rr) + 1.01f * dist;
    // (+ 1e-30: the tags alone tell scores of zero apart, and products of tiny numbers vanish)
    const bool unsure = !(b1 - b2 > bound * (rr + tmax * tmax) + 1e-30f);
    u32 todo = (u32)__builtin_amdgcn_ballot_w64(unsure);          // (both halves agree)
    const bool redone = !FOURS || todo != 0;
    while (todo != 0) {
      const int src = __builtin_ctz(todo);
      todo &= todo - 1;
      float rs[DP];
#pragma unroll
      for (int t = 0; t < DP; ++t) rs[t] = __uint_as_float((u32)__builtin_amdgcn_readlane((int)__float_as_uint(r[t]), src));
      u64 key = KEY_EMPTY;
      for (int j = lane; j < K; j += VS_WAVE) {
        const float* w = word(j);
        float acc = 0.f;
#pragma unroll
        for (int t = 0; t < DP; ++t)
          if (t < dsub) { const float diff = rs[t] - w[t]; acc = __builtin_fmaf(diff, diff, acc); }
        // (encoding never chose a codeword at a distance that is not finite; training orders a NaN's bits
        // like the keys of the nearest-row routes)
        const u64 kk = RES && !(acc < __builtin_inff()) ? KEY_EMPTY : make_key(acc, (u32)j, 0);
        key = kk < key ? kk : key;
      }
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) { const u64 o = __shfl_xor(key, off); key = o < key ? o : key; }
      if ((lane & 31) == src) best = RES && key == KEY_EMPTY ? 0 : (int)min(key_index(key), (u32)(K - 1));
    }
    if (half == 0 && i0 + lane < n) {
      codes[(i0 + lane) * stride_i + m * stride_m] = (uint8_t)best;
      if (val) {
        if (redone) {
          val_best = 0.f;
#pragma unroll
          for (int t = 0; t < DP; ++t)
            if (t < dsub) { const float diff = r[t] - word(best)[t]; val_best = __builtin_fmaf(diff, diff, val_best); }
        }
        val[(int64_t)m * n + i0 + lane] = val_best;
      }
    }
  }
}

struct NearestPlan { int nsplit; int64_t cols_per_split; size_t o_b2, o_idx, o_norm, o_flags, o_state, o_list, o_thr, o_cnt, o_cand, o_left, o_fb, bytes; };
NearestPlan nearest_plan(int64_t n, int64_t nb) {
  NearestPlan p;
  const int64_t tiles = (n + 255) / 256;
  const int64_t steps = std::max<int64_t>(1, (nb + 63) / 64);
  // two workgroups per compute unit; a short A splits B, by at least four steps each
  int64_t ns = std::max<int64_t>(1, 512 / std::max<int64_t>(1, tiles));
  ns = std::max<int64_t>(1, std::min(ns, steps / 4));
  const int64_t sps = (steps + ns - 1) / ns;
  p.nsplit = (int)((steps + sps - 1) / sps);
  p.cols_per_split = sps * 64;
  size_t o = 0;
  auto take = [&](size_t b) { const size_t at = o; o += (b + 255) / 256 * 256; return at; };
  take((size_t)p.nsplit * n * sizeof(float));
  p.o_b2 = take((size_t)p.nsplit * n * sizeof(float));
  p.o_idx = take((size_t)p.nsplit * n * sizeof(int));
  p.o_norm = take((size_t)n * sizeof(float));
  p.o_flags = take((size_t)n);
  p.o_state = take(sizeof(NearestState));
  p.o_list = take((size_t)n * sizeof(int));
  p.o_thr = take((size_t)n * sizeof(float));
  p.o_cnt = take((size_t)n * sizeof(int));
  p.o_cand = take((size_t)n * kCandidates * sizeof(int));
  p.o_left = take((size_t)n * sizeof(int));
  p.o_fb = take(mfma_knn_fallback_bytes(n, nb, 1));
  p.bytes = o;
  return p;
}

template <int KSTEPS, int METRIC, bool BF, bool COLLECT>
void launch_nearest_t(const NearestPlan& p, const float* x, int64_t n, int d, const MfmaOperand& B, char* w,
                      hipStream_t st) {
  constexpr size_t lds = (size_t)2 * (BF ? 2 : 1) * 64 * (KSTEPS * 16 + 8) * sizeof(unsigned short) + 2 * 64 * sizeof(float);
  auto kern = &nearest_kernel<KSTEPS, METRIC, BF, COLLECT>;
  if (lds > 48 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  constexpr int64_t per_tile = 128 * kNearestBlocks<KSTEPS, BF>;
  const int64_t tiles = (n + per_tile - 1) / per_tile;
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * p.nsplit)), dim3(256), lds, st, x, n, d, BF ? B.hi : B.h16, B.lo,
                     B.norm, B.info, B.n, tiles, p.cols_per_split,
                     reinterpret_cast<const int*>(w + (COLLECT ? p.o_list : p.o_left)),
                     reinterpret_cast<const NearestState*>(w + p.o_state),
                     reinterpret_cast<float*>(w), reinterpret_cast<float*>(w + p.o_b2),
                     reinterpret_cast<int*>(w + p.o_idx), reinterpret_cast<float*>(w + p.o_norm),
                     reinterpret_cast<unsigned char*>(w + p.o_flags), reinterpret_cast<const float*>(w + p.o_thr),
                     reinterpret_cast<int*>(w + p.o_cnt), reinterpret_cast<int*>(w + p.o_cand));
}
template <bool BF, bool COLLECT>
void launch_nearest_any(const NearestPlan& p, const float* x, int64_t n, int d, int metric, const MfmaOperand& B,
                        char* w, hipStream_t st) {
#define GO(KS) do { if (metric == 0) launch_nearest_t<KS, 0, BF, COLLECT>(p, x, n, d, B, w, st); \
                    else launch_nearest_t<KS, 1, BF, COLLECT>(p, x, n, d, B, w, st); } while (0)
  switch (mfma_padded_dim(d) / 16) {
    case 2: GO(2); break;
    case 4: GO(4); break;
    case 6: GO(6); break;
    default: GO(8); break;
  }
#undef GO
}

// One pass: sweep, list, second sweep over the listed vectors, decision.
template <int METRIC, bool BF>
void launch_nearest_pass(const NearestPlan& p, const float* x, int64_t n, int d, const MfmaOperand& B, float eps_scale,
                         int32_t* idx, char* w, hipStream_t st) {
  NearestState* state = reinterpret_cast<NearestState*>(w + p.o_state);
  int* list = reinterpret_cast<int*>(w + p.o_list);
  int* cnt = reinterpret_cast<int*>(w + p.o_cnt);
  int* left = reinterpret_cast<int*>(w + p.o_left);
  launch_nearest_any<BF, false>(p, x, n, d, METRIC, B, w, st);
  hipLaunchKernelGGL((nearest_finish_kernel<METRIC, BF>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, d,
                     p.nsplit, reinterpret_cast<const float*>(w), reinterpret_cast<const float*>(w + p.o_b2),
                     reinterpret_cast<const int*>(w + p.o_idx), reinterpret_cast<const float*>(w + p.o_norm),
                     reinterpret_cast<const unsigned char*>(w + p.o_flags), B.info, eps_scale, idx, left, state, list,
                     reinterpret_cast<float*>(w + p.o_thr), cnt);
  launch_nearest_any<BF, true>(p, x, n, d, METRIC, B, w, st);
  hipLaunchKernelGGL((nearest_decide_kernel<METRIC, BF>), dim3((unsigned)std::min<int64_t>((n + 15) / 16, 4096)),
                     dim3(256), 0, st, x, n, d, B.x, B.n, const_cast<PrepInfo*>(B.info), list, state, cnt,
                     reinterpret_cast<const int*>(w + p.o_cand), idx, left, eps_scale >= 0.f);
}

}  // namespace

// d up to 128: the fragments of 64 vectors stay in registers
bool nearest_supported(int d) { return d > 16 && d <= 128; }
size_t nearest_bytes(int64_t n, int64_t nb) { return nearest_plan(n, nb).bytes; }

void launch_nearest(const float* x, int64_t n, int d, int metric, const MfmaOperand& B, float eps_scale,
                    int32_t* idx, float* val, char* work, hipStream_t st) {
  if (n <= 0) return;
  const NearestPlan p = nearest_plan(n, B.n);
  NearestState* state = reinterpret_cast<NearestState*>(work + p.o_state);
  hipLaunchKernelGGL(nearest_state_kernel, dim3(1), dim3(1), 0, st, B.info, state);
  if (metric == 0) {
    launch_nearest_pass<0, false>(p, x, n, d, B, eps_scale, idx, work, st);
    launch_nearest_pass<0, true>(p, x, n, d, B, eps_scale, idx, work, st);
  } else {
    launch_nearest_pass<1, false>(p, x, n, d, B, eps_scale, idx, work, st);
    launch_nearest_pass<1, true>(p, x, n, d, B, eps_scale, idx, work, st);
  }
  SelectOut out;
  out.idx32 = idx;
  launch_canon_rows(x, n, B.x, B.n, d, metric, 1, out, &state->left[1], reinterpret_cast<const int*>(work + p.o_left),
                    reinterpret_cast<u64*>(work + p.o_fb), nullptr, st);
  if (val) hipLaunchKernelGGL(row_values_kernel, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, st, x, n, d, B.x, idx, val);
}

bool pq_nearest_supported(int dsub, int K) { return dsub >= 1 && dsub <= 16 && (K == 16 || K == 256); }

void launch_pq_nearest(const float* x, int64_t n, int d, int dsub, const float* centroids, const int32_t* list_of,
                       const float* codebooks, int K, int M, float eps_scale, uint8_t* codes, int64_t stride_i,
                       int64_t stride_m, float* val, hipStream_t st) {
  if (n <= 0) return;
  // groups of 32 vectors per wavefront: as many as leave about eight workgroups per compute unit
  // (the fragments of 256 codewords cost as much as one or two groups)
  int groups = (int)std::max<int64_t>(1, std::min<int64_t>(16, n * M / (128 * 2048)));
  const int64_t chunks = (n + 128ll * groups - 1) / (128ll * groups);
  const dim3 grid((unsigned)((chunks + 7) / 8 * 8 * M)), block(256);
  const bool vec = dsub % 4 == 0 && (centroids == nullptr || d % 4 == 0) &&
                   (reinterpret_cast<uintptr_t>(x) & 15) == 0;
  const size_t lds = (size_t)K / 4 * pq_four_stride(dsub, vec) * sizeof(float);
#define GO(NP, KB, RES, VEC) \
  hipLaunchKernelGGL((pq_nearest_kernel<NP, KB, RES, VEC>), grid, block, lds, st, x, n, d, dsub, centroids, list_of, \
                     codebooks, K, M, chunks, groups, eps_scale, codes, stride_i, stride_m, val)
#define GO2(NP, KB) do { if (centroids) { if (vec) GO(NP, KB, true, true); else GO(NP, KB, true, false); } \
                         else { if (vec) GO(NP, KB, false, true); else GO(NP, KB, false, false); } } while (0)
  if (dsub <= 8) { if (K == 256) GO2(1, 8); else GO2(1, 1); }
  else { if (K == 256) GO2(2, 8); else GO2(2, 1); }
#undef GO2
#undef GO
}
