// Host-side declarations shared by the translation units of libvs.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef unsigned long long u64;
typedef unsigned int u32;

// ---- canon distance tiles (kernels_dist.hip) --------------------------------
// out[a * ldo + b] = canon distance of A row a and B row b.
void launch_canon_matrix(const float* A, int64_t na, const float* B, int64_t nb, int d, int metric,
                         float* out, int64_t ldo, hipStream_t st);
// best[a] = min over b of key(canon(A_a, B_b), b); best must hold KEY_EMPTY on entry.
void launch_canon_argbest(const float* A, int64_t na, const float* B, int64_t nb, int d,
                          int metric, u64* best, hipStream_t st);

// ---- selection (kernels_select.hip) -----------------------------------------
void launch_fill_u64(u64* p, int64_t n, u64 v, hipStream_t st);
// Final outputs of a selection; any member may be null.
struct SelectOut {
  float* val = nullptr;       // [nrows, k] best values
  int64_t* id64 = nullptr;    // [nrows, k] indices as int64
  int32_t* idx32 = nullptr;   // [nrows, k] indices as int32
};
// keys[r][0..k) <- k best of (first ? {} : keys[r][0..k)) U {key(mat[r][c], col_base + c)}.
// When `last`, the result goes to `out` instead (already ordered best first) and keys is
// not written; keys may be null if first && last.
void launch_row_select(const float* mat, int64_t ld, int64_t nrows, int64_t ncols, u32 col_base,
                       int metric, int k, u64* keys, bool first, bool last, const SelectOut& out,
                       hipStream_t st);
// keys -> (value, int64 id); idmap == NULL: id = index, else id = idmap[index]; empty -> (-1, +-inf)
void launch_keys_to_results(const u64* keys, int64_t n, int metric, float* out_dist,
                            int64_t* out_ids, const int64_t* idmap, hipStream_t st);
// keys -> (int32 index, value); used for probes
void launch_keys_to_probes(const u64* keys, int64_t n, int metric, int32_t* out_idx,
                           float* out_val, hipStream_t st);
void launch_keys_to_index32(const u64* keys, int64_t n, int32_t* out_idx, hipStream_t st);

// ---- queries that a list-by-list scan leaves to the query-major one --------------------
// The listed queries (list and their number in device memory) are scanned query by query; while they are few, in
// `pieces` pieces each -- one query is a long scan for one workgroup -- whose k best keys go to `partial`
// [limit][k] and are merged by launch_rescan_merge.
struct Rescan {
  const u32* list = nullptr;
  const u32* count = nullptr;
  u64* partial = nullptr;
  u32 pieces = 1, limit = 0;
  unsigned long long* cursor = nullptr;   // a work counter that is zero when the scan starts, or null
  __device__ u32 split() const { return (u64)*count * pieces <= limit ? pieces : 1u; }
};
void launch_rescan_merge(const Rescan& rs, int k, int metric, const int64_t* ids, float* out_dist, int64_t* out_ids,
                         hipStream_t st);

// ---- IVF-PQ (kernels_ivfpq.hip) ----------------------------------------------
struct IvfpqDims {
  int d, metric, nlist, M, nbits, K, dsub, code_size;
};
// tmp_codes[i][m] = PQ code of sub-vector m of the residual of x_i (one byte per m)
void launch_pq_encode(const IvfpqDims& g, const float* x, int64_t n, const int32_t* list_of,
                      const float* centroids, const float* codebooks, bool matrix_cores, float eps_scale,
                      uint8_t* tmp_codes, hipStream_t st);
// move old entries to their new offsets and scatter the new ones
// norms / old_norms / tmp_norms: the stored norms of Sec. 4.3's decomposition, or all null
void launch_relayout(const IvfpqDims& g, const uint8_t* old_codes, const int64_t* old_ids,
                     const float* old_norms, int64_t old_total, const int64_t* old_off,
                     const int64_t* new_off, const uint8_t* tmp_codes,
                     const int64_t* new_ids_or_null, int64_t id_base, const float* tmp_norms,
                     const int64_t* dest, const int32_t* new_list_of, int64_t n_new, uint8_t* codes,
                     int64_t* ids, float* norms, hipStream_t st);
// Indexes of the shapes that the bank-private-table scan kernel serves keep the code at position
// p of its list rotated by p bytes (stored byte b = c_{(b + p) mod M}); launch_relayout writes
// that layout, launch_codes_canonical turns a copy back into byte m = c_m.
bool ivfpq_codes_rotated(const IvfpqDims& g);
void launch_codes_canonical(const IvfpqDims& g, const uint8_t* stored, const int64_t* off,
                            int64_t total, uint8_t* out, hipStream_t st);
// tmp_norms[i] = |c_list(i) + decoded code i|^2.  tmp_codes: one byte per (vector, m) as the encoder
// writes them; stored_form: code_size bytes per vector as the lists hold them (4-bit codes packed
// two per byte; byte order canonical, not rotated)
void launch_pq_norms(const IvfpqDims& g, const uint8_t* tmp_codes, int64_t n, const int32_t* list_of,
                     const float* centroids, const float* codebooks, float* tmp_norms,
                     hipStream_t st, bool stored_form = false);
// norms[i] = |row i|^2 (fma chain in dimension order)
void launch_row_norms(const float* x, int64_t n, int d, float* norms, hipStream_t st);
void launch_list_of_storage(const int64_t* off, int nlist, int64_t total, int32_t* list_of,
                            hipStream_t st);
void launch_list_sizes(const int64_t* off, int nlist, int64_t* sizes, hipStream_t st);
// nsplit > 1: partial[q][s][0..k) = k best keys (value, storage position) of the probes handled by
// split s.  nsplit == 1: final results go straight to out_dist / out_ids (ids[position]).
// counter: one 64-bit word of device memory the scan may use to hand out its work items.
int launch_ivfpq_scan(const IvfpqDims& g, const float* q, int64_t nq, const float* centroids,
                      const float* codebooks, const int32_t* probes, const float* cdist,
                      int nprobe, int nsplit, const int64_t* list_off, const uint8_t* codes,
                      const float* norms, const float* cnorm, const float* list_tables,
                      float* query_tables, int64_t ntotal, int k, u64* partial, u64* counter,
                      const int64_t* ids, float* out_dist, int64_t* out_ids, hipStream_t st,
                      const Rescan& rescan = Rescan());
// (rescan, nsplit == 1: only the listed queries are scanned)
// The wavefront-private scan (one wavefront per (query, probe split); every table form but the
// residual tables) is used while the mean list is at most this long; it needs query_tables:
// ivfpq_query_table_bytes() of device work space.
constexpr int kWaveScanMaxMeanList = 1024;
bool ivfpq_wave_scan_applies(const IvfpqDims& g, int64_t ntotal);
size_t ivfpq_query_table_bytes(const IvfpqDims& g, int64_t nq);
// Slots of n newly assigned vectors in the grown inverted lists, computed on the device:
// dest[i] = slot of vector i (behind its list's old entries, new vectors of a list in batch order),
// new_off [nlist + 1] = offsets of the grown lists.  list_of [n] (n < 2^31), old_off [nlist + 1],
// work: ivf_place_work_bytes(n) bytes, all device memory.  Returns the device address of a
// flag that is non-zero once the kernels have run if some list_of[i] is outside [0, nlist).
size_t ivf_place_work_bytes(int64_t n);
int* launch_ivf_place(const int32_t* list_of, int64_t n, int nlist, const int64_t* old_off, char* work,
                      int64_t* dest, int64_t* new_off, hipStream_t st);
// cdist[a][p] = <q_a, c_{probes[a][p]}> as one fp32 fused-multiply-add chain in dimension order
// (the value the coarse quantizer itself returns under the inner-product metric); probes < 0 are left alone
void launch_probe_inner_products(const float* q, int64_t nq, int d, const float* centroids,
                                 const int32_t* probes, int nprobe, float* cdist, hipStream_t st);
// stats[0] = sum over the n (query, probe) pairs of the probed list's size, stats[1] = pairs whose
// list is not empty, stats[2] = mfma_rows, stats[3] = *fallback_count (0 if null), stats[4] = p_first
// (probes per query that a list-major search scans query-major first; 0: the search is query-major),
// stats[5] = the part of stats[0] that falls on those probes, stats[6] = 0 (set after a list-major
// scan by launch_search_stats_rescan to the number of queries scanned again); device memory,
// written in stream order.
void launch_search_stats(const int32_t* probes, int64_t n, const int64_t* list_off, const int* fallback_count,
                         int64_t mfma_rows, int nprobe, int p_first, long long* stats, hipStream_t st);
void launch_search_stats_rescan(const unsigned* rescan_count, long long* stats, hipStream_t st);
// out [K][M][dsub] = codebooks [M][K][dsub] with the first two axes exchanged.  launch_ivfpq_scan
// expects it directly behind the codebooks it is given (codebooks + M * K * dsub).
void launch_pq_codebooks_by_entry(const IvfpqDims& g, const float* codebooks, float* out, hipStream_t st);
// out [nlist][K][M]: |T_m[j]|^2 + 2 <c_{l,m}, T_m[j]>, the per-list term of the split look-up tables
void launch_pq_list_tables(const IvfpqDims& g, const float* centroids, const float* codebooks, float* out,
                           hipStream_t st);
// List-major L2 scan with residual tables for large batches (shapes of the bank-private kernel).
bool ivfpq_listmajor_shape(const IvfpqDims& g);
size_t ivfpq_listmajor_bytes(const IvfpqDims& g, int64_t nq, int nprobe, int cap);
const unsigned* ivfpq_listmajor_rescan_count(const IvfpqDims& g, int64_t nq, int nprobe, int cap, const char* lm);
int launch_ivfpq_scan_listmajor(int part, const IvfpqDims& g, const float* q, int64_t nq, const float* centroids,
                                const float* codebooks, const int32_t* probes, const float* cdist, int nprobe,
                                int p_first, int cap, const int64_t* list_off, const uint8_t* codes,
                                int64_t ntotal, int k, u64* first, u64* counter, char* lm, const int64_t* ids,
                                float* out_dist, int64_t* out_ids, hipStream_t st);
// ---- matrix-core scan of inverted lists (kernels_mscan.hip) -----------------------
enum { kMsPq = 0, kMsFlat = 1, kMsSq8 = 2 };
// What the scan needs of an index (device pointers).
struct MscanIndex {
  int kind = kMsPq;
  IvfpqDims g{};                       // kMsFlat, kMsSq8: d, metric, nlist (code_size bytes per vector)
  int64_t ntotal = 0, max_list = 0;    // stored vectors, the longest list's
  const float* centroids = nullptr;
  const int64_t* list_off = nullptr;
  const void* codes = nullptr;
  const float* codebooks = nullptr;    // kMsPq
  const void* mem = nullptr;           // launch_mscan_index's output
  const void* units = nullptr;         // kMsPq: launch_mscan_units' output
  const float *cnorm = nullptr, *norms = nullptr, *list_tables = nullptr;
  const float *vmin = nullptr, *step = nullptr;   // kMsSq8
  const u32* sigma_src = nullptr;      // bits of the codebooks' largest magnitude (kMsPq), of the centroids' largest squared norm
  float slack = 0.f;                   // one-hot rows: see launch_mscan_onehot_slack
  double crowding = 0.0;               // length of a stored vector's list, on average, over the mean length of a list
};
struct MscanPlan {
  int64_t nq = 0;
  int npr = 0, cap = 0, slots = 0;
  u32 capcodes = 0, seg = 0, max_a = 0, max_b = 0, surv = 0;
  size_t bytes = 0;                    // work space
};
// bytes of what an index keeps for the scan (0 where the shape has none), and its preparation
size_t mscan_index_bytes(int kind, const IvfpqDims& g);
// (info: of the centroids' preparation, launched before; PQ: receives codebook_max_bits)
struct PrepInfo;
void launch_mscan_index(int kind, const IvfpqDims& g, const float* centroids, const float* codebooks, PrepInfo* info,
                        void* out, hipStream_t st);
// Whether the scan's bounds hold for an index: bits of the number that its scale is taken from (sigma_src)
bool mscan_scale_fits(int kind, u32 bits);
size_t mscan_units_bytes(const IvfpqDims& g, int64_t ntotal);
// indexes whose codes are swept as one-hot rows: the scan keeps nothing of them
bool mscan_onehot(int kind, const IvfpqDims& g);
// out [kOnehotSamples]: error bounds of one-hot sums, with centroids in the place of queries, over the spread of such sums
// (infinite where a table entry is not finite)
constexpr int kOnehotSamples = 256;
void launch_mscan_onehot_slack(const IvfpqDims& g, const float* centroids, const float* codebooks, float* out, hipStream_t st);
void launch_mscan_units(const IvfpqDims& g, const uint8_t* codes, const int64_t* list_off, int64_t ntotal, void* out,
                        hipStream_t st);
// plan of a search of npr probes per query and k results (asked: option "list_major_candidates"); false: not by this scan
bool mscan_plan(const MscanIndex& ix, int64_t nq, int npr, int k, int asked, MscanPlan* out);
// form: 0 residual tables (or no PQ), 1 inner product, 2 stored norms, 3 precomputed tables.  Parts 0, 1, 2 in
// turn; then the queries of mscan_rescan are the caller's to scan query by query.
void launch_mscan(int part, const MscanIndex& ix, const MscanPlan& p, const float* q, const int32_t* probes,
                  const float* cdist, int form, int k, float eps_scale, char* ws, const int64_t* ids, float* out_dist,
                  int64_t* out_ids, hipStream_t st);
const unsigned* mscan_rescan_count(const MscanIndex& ix, const MscanPlan& p, const char* ws);
// (partial: nq * k keys of work space)
Rescan mscan_rescan(const MscanIndex& ix, const MscanPlan& p, const char* ws, u64* partial);
void launch_ivfpq_merge(const u64* partial, int64_t nq, int nsplit, int k, int metric,
                        const int64_t* ids, float* out_dist, int64_t* out_ids, hipStream_t st);

// ---- MFMA shortlist + exact re-rank (kernels_mfma.hip) --------------------------
// What operand preparation learns about a matrix (device memory).
struct PrepInfo {
  u32 all_int;        // every value is an integer
  u32 all_bf16;       // every value is exactly representable in bf16
  u32 max_norm_bits;  // bits of the largest squared row norm (non-negative float)
  u32 all_nonneg;     // no value is negative
  // Of the column operand of a k-nearest-rows or one-sweep call only, and only where that operand
  // outlives the call (an index's centroids or vectors, the centroids of a k-means run): a bit for each
  // kind of call -- k = 1, k > 1, one sweep -- is set while the sweeps of such calls may use the fp16
  // heads alone on operands that are not exactly bf16 (one matrix product instead of three, with the
  // wider error bound that goes with it).  The bit is cleared for good by the exact fallback once more
  // than one row in 512 of a call failed the sufficiency test under that bound, and by the one-sweep
  // route (which takes the rows that fail through three products within the call) once more than half of
  // a call's vectors had to be swept again.
  static constexpr u32 kHeadsOne = 1u, kHeadsMany = 2u, kHeadsSweep = 4u, kHeadsAll = 7u;
  u32 heads_only;
  u32 codebook_max_bits;   // of an IVF-PQ index with a matrix-core scan: bits of the codebooks' largest magnitude
};
struct MfmaOperand {
  const float* x;             // [n, d] original fp32 rows
  const unsigned short* hi;   // [n, dp] bf16 heads, dp = mfma_padded_dim(d)
  const unsigned short* lo;   // [n, dp] bf16 tails
  const unsigned short* h16;  // [n, dp] fp16 heads (written by operand preparation right behind the tails)
  const float* norm;          // [n] squared norms
  const PrepInfo* info;
  int64_t n;
  int known_bf16;             // info->all_bf16 where the host has read it back (0 / 1), else -1
  bool try_heads_only;        // info->heads_only was set when the operand was prepared (it may have been cleared since)
};
bool mfma_knn_supported(int d, int k);
// operand planes hold this many rows (the tail is zero padding)
int64_t mfma_padded_rows(int64_t n);
int mfma_knn_kp(int k);
void launch_prep(const float* x, int64_t n, int d, unsigned short* hi, unsigned short* lo,
                 float* norm, PrepInfo* info, hipStream_t st, bool try_heads_only = false, bool write_f16 = true,
                 bool keep_heads = false);   // keep_heads: the operand is prepared again, what was learnt of heads_only stays
// operand planes hold this many dimensions per row (zeros past d)
int mfma_padded_dim(int d);
// bytes of the shortlist buffer [na, nsplit, kp] and the column split count to use
size_t mfma_knn_shortlist_bytes(int64_t na, int64_t nb, int d, int k, int* nsplit_out);
// (also clears *fb_count, the counter that launch_rerank of the same call adds to)
void launch_mfma_shortlist(const MfmaOperand& A, const MfmaOperand& B, int d, int metric, int k,
                           int nsplit, u64* shortlist, int* fb_count, hipStream_t st);
// exact k best per row of A from the shortlists; rows that cannot be proven exact are
// recomputed over all of B.  fb_count: 1 int, fb_rows: A.n ints, fb_partial:
// mfma_knn_fallback_bytes(...) bytes (device scratch; may be null when that is 0).
size_t mfma_knn_fallback_bytes(int64_t na, int64_t nb, int k);
void launch_rerank(const MfmaOperand& A, const MfmaOperand& B, int d, int metric, int k, int nsplit,
                   const u64* shortlist, float eps_scale, const SelectOut& out, int* fb_count,
                   int* fb_rows, u64* fb_partial, hipStream_t st);
// k best rows of B on the canon chain for the listed rows of A (count and list in device memory;
// fb_partial as in launch_rerank; adapt: the operand whose heads_only bit a large count clears, or null)
void launch_canon_rows(const float* A, int64_t na, const float* B, int64_t nb, int d, int metric, int k,
                       const SelectOut& out, const int* fb_count, const int* fb_rows, u64* fb_partial,
                       PrepInfo* adapt, hipStream_t st);
int read_fallback_total(unsigned long long* out);

// ---- nearest row in one sweep (kernels_nearest.hip) ------------------------------
// idx[i] = best row of B for row i of x under the canon chain (ties to the smaller row), and
// (L2 only) val[i] = its canon value where val is not null.  B: prepared with its fp16 heads.
// work: nearest_bytes(n, B.n) bytes.  d in (16, 128].
bool nearest_supported(int d);
size_t nearest_bytes(int64_t n, int64_t nb);
void launch_nearest(const float* x, int64_t n, int d, int metric, const MfmaOperand& B, float eps_scale,
                    int32_t* idx, float* val, char* work, hipStream_t st);
// codes[i * stride_i + m * stride_m] = nearest codeword (canon L2, ties to the smaller) of sub-vector
// m of vector i: of x [n, d] minus the centroid of its list, or (centroids null) of x [M][n][dsub];
// val [M][n] = its canon distance where not null.  dsub up to 16, K = 16 or 256.
bool pq_nearest_supported(int dsub, int K);
void launch_pq_nearest(const float* x, int64_t n, int d, int dsub, const float* centroids, const int32_t* list_of,
                       const float* codebooks, int K, int M, float eps_scale, uint8_t* codes, int64_t stride_i,
                       int64_t stride_m, float* val, hipStream_t st);

// ---- kernels_ivfflat.hip -------------------------------------------------------
void launch_ivfflat_relayout(int d, int nlist, const float* old_rows, const int64_t* old_ids,
                             int64_t old_total, const int64_t* old_off, const int64_t* new_off,
                             const float* x, const int64_t* new_ids_or_null, int64_t id_base,
                             const int64_t* dest, int64_t n_new, float* rows, int64_t* ids,
                             hipStream_t st);
size_t ivfflat_scan_lds_bytes(int d, int k);
// canon distance of every stored vector of the probed lists, k best per (query, probe split):
// results to out_dist / out_ids when nsplit == 1, else keys to partial [nq, nsplit, k]
void launch_ivfflat_scan(int d, int metric, const float* q, int64_t nq, const int32_t* probes,
                         int nprobe, int nsplit, const int64_t* list_off, const float* rows, int k,
                         u64* partial, const int64_t* ids, float* out_dist, int64_t* out_ids,
                         hipStream_t st, const Rescan& rescan = Rescan());

// IVF-SQ8 (same file): 8-bit scalar-quantizer codes [n, d]; scan = IVF-Flat over reconstructions
void launch_sq8_encode(const float* x, int64_t n, int d, const float* vmin, const float* step,
                       uint8_t* codes, hipStream_t st);
size_t ivfsq8_scan_lds_bytes(int d, int k);
void launch_ivfsq8_scan(int d, int metric, const float* q, int64_t nq, const float* vmin,
                        const float* step, const int32_t* probes, int nprobe, int nsplit,
                        const int64_t* list_off, const uint8_t* codes, int k, u64* partial,
                        const int64_t* ids, float* out_dist, int64_t* out_ids, hipStream_t st,
                        const Rescan& rescan = Rescan());

// ---- kernels_train.hip ---------------------------------------------------------
// centroids[j] <- mean of the rows x[order[off[j] .. off[j + 1])] (float64 sum in that order, in
// blocks of 4096 rows whose sums are added in block order); a centroid with an empty range keeps
// its value.  `problems` (d <= 32 where more than one) independent means of n rows each, arrays one
// after the other.  `partial` = work space of segmented_mean_partial_bytes (may be null when that is 0)
size_t segmented_mean_partial_bytes(int64_t n, int d, int K, int problems);
void launch_segmented_mean(const float* x, int64_t n, int d, const int32_t* order, const int64_t* off, int K,
                           int problems, float* centroids, double* partial, hipStream_t st);
// stable counting sort of the assignment idx [n] by centroid (K <= 16384) and the float64 sum
// of val [n]: order [n], off [K + 1]; *bad is set if an assignment was outside [0, K);
// partial [256] sums to the sum of val.  The second form: `problems` of them, idx as bytes.
size_t kmeans_sort_bytes(int K, int problems);
void launch_kmeans_sort(const int32_t* idx, const float* val, int64_t n, int K, char* work, int32_t* order,
                        int64_t* off, int* bad, double* partial, hipStream_t st);
void launch_kmeans_sort_bytes(const uint8_t* idx, const float* val, int64_t n, int K, int problems, char* work,
                              int32_t* order, int64_t* off, int* bad, double* partial, hipStream_t st);
// out[m][i][:] = (x[i] - centroids[list_of[i]])[m * dsub : (m + 1) * dsub], out is [d / dsub][n][dsub]
void launch_residual_slices(const float* x, int64_t n, int d, int dsub, const float* centroids,
                            const int32_t* list_of, float* out, hipStream_t st);

// ---- kernels_refine.hip --------------------------------------------------------
// k best of each query's kc candidates by canon distance to the candidates' rows of x
size_t refine_lds_bytes(int d, int k);   // LDS of one workgroup; the launch needs it to fit
void launch_refine(const float* x, int64_t nb, const float* q, int64_t nq, int d, int metric,
                   const int64_t* cand, int kc, int k, float* out_dist, int64_t* out_ids,
                   hipStream_t st);
