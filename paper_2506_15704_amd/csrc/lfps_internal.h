// Internal declarations shared by the translation units of liblfps (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lfps.h"
#include "range_rule.h"

namespace lfps {

constexpr int kD = 128;           // head_dim the kernels are written for
constexpr int kMaxSplits = 64;    // upper bound of split-K partials per head (full attention)
// What the memory-side cache holds (256 MB): rows of a pass that together take more are read past the caches, see the kernels.
constexpr int64_t kKeptBytes = 256 << 20;
// The same for rows that a pass reads whole and in order (dense scoring, full attention): most of a little more than the cache holds
// is found there still.  Kept -> past the caches, us: exact Top-k of 16 requests, 265 MB of bf16 keys 81.6 -> 84.5, 281 MB 87.0 ->
// 87.8, 289 MB 91.5 -> 88.8; FP8 265 MB 82.5 -> 85.9, 289 MB 89.8 -> 90.1, 305 MB 96.7 -> 93.5.  Full attention of 16 requests,
// bf16 265 MB 51.0 -> 52.3, 289 MB 56.4 -> 56.4, 305 MB 60.7 -> 58.6; FP8 265 MB 60.1 -> 65.7, 289 MB 70.3 -> 70.7, 305 MB 74.8 -> 73.7.
constexpr int64_t kKeptStreamBytes = 288 << 20;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Where the rows of a request live when the cache is paged (table != nullptr): a pool of blocks of
// 2^shift rows, table[b*table_stride + (i >> shift)] = block of row i of request b.
struct KvPage {
  const int32_t* table;
  int32_t table_stride, shift, n_blocks;
};

// Strided view of K or V in elements, resolved for one launch.
struct KvView {
  const void* k;
  const void* v;
  int64_t stride_b, stride_h, stride_n;
  const int32_t* seq_lens;
  KvPage page;
  bool k_fp8;   // K elements are one byte (OCP FP8 E4M3)
  bool v_fp8;   // V elements are one byte; otherwise V has the cache dtype
  bool f16;     // the cache dtype is fp16 (K and V)
  bool v_on_device;   // the values are known to be in device memory
};

// Row addressing of the two cache layouts, chosen at compile time.  A logical row i of request b
// is first turned into a "physical row" p (an int32: i itself, or block * block_size + i % block_size;
// the only step that reads memory, and only when paged), from which the element offset follows by
// arithmetic.  Kernels translate where a row id first lives in a register and keep p from there on.
template <bool kPaged>
struct RowMap {
  __device__ __forceinline__ static int phys(const KvPage& pg, int b, int i) {
    if constexpr (!kPaged) {
      return i;
    } else {
      return (kept_in_pool(pg, block(pg, b, i)) << pg.shift) | (i & ((1 << pg.shift) - 1));
    }
  }
  // A row's entry of the block table as it is there, and the offset that follows from it, for who asks for the entry long before it is
  // used (with phys the wait for the load comes right behind it).
  __device__ __forceinline__ static int block(const KvPage& pg, int b, int i) {
    return kPaged ? pg.table[(int64_t)b * pg.table_stride + (i >> pg.shift)] : 0;
  }
  __device__ __forceinline__ static int64_t offset_in(const KvPage& pg, int blk, int i, int64_t stride_b, int64_t stride_n) {
    return kPaged ? kept_in_pool(pg, blk) * stride_b + (i & ((1 << pg.shift) - 1)) * stride_n : i * stride_n;
  }
  __device__ __forceinline__ static int kept_in_pool(const KvPage& pg, int blk) {       // a bad entry reads a wrong block, never outside
    return blk < 0 ? 0 : (blk >= pg.n_blocks ? pg.n_blocks - 1 : blk);
  }
  // element offset of the start of (b, g)'s rows, to which offset(p) is added
  __device__ __forceinline__ static int64_t base(int b, int g, int64_t stride_b, int64_t stride_h) {
    return (kPaged ? (int64_t)0 : (int64_t)b * stride_b) + (int64_t)g * stride_h;
  }
  __device__ __forceinline__ static int64_t offset(const KvPage& pg, int p, int64_t stride_b, int64_t stride_n) {
    if constexpr (!kPaged) {
      return (int64_t)p * stride_n;
    } else {
      return (int64_t)(p >> pg.shift) * stride_b + (int64_t)(p & ((1 << pg.shift) - 1)) * stride_n;
    }
  }
};

// Shapes every kernel needs.
struct Shape {
  int32_t B, Hq, Hkv, G;
  int32_t Lcap, kmax, cand_cap;
  int32_t radius, n_recent, n_sink;
  int32_t score_stride;   // row length of the workspace score buffer [B, Hq, score_stride]
};

// ---- kernel launchers (each enqueues on `st` and returns the launch error) -------------
hipError_t configure_candidates(const Shape& s);
hipError_t configure_select(const Shape& s, int dtype, bool k_fp8, bool v_fp8);
// group_start [B,Hkv] / line_total [1] (or NULL): every group adds its candidate count to *line_total
// (zero on entry) and keeps the value before the addition as its place on the line of all candidate slots.
hipError_t launch_candidates(const Shape& s, const int32_t* prev_topk, const int32_t* k, const int32_t* seq_lens,
                             int32_t* cand, int32_t* cand_count, int32_t* flags, int64_t* group_start,
                             int64_t* line_total, hipStream_t st);

// Scores of candidate rows (cand != NULL) or of all rows 0..n_b-1 (cand == NULL) for the G heads
// of each KV group.  score is [B, Hq, score_stride].
// flags: the context's status word (LFPS_FLAG_Q_RANGE is raised there).  A candidate entry outside [0, n_b)
// scores -inf.  tops [B, Hq, score_stride / 16] (or NULL; all rows of 16-bit and FP8 keys only) receives the largest score of
// every 16 rows, made finite as the select does, of the requests whose select reads them (k: its budgets; select_takes_tops).
hipError_t launch_group_score(const Shape& s, int dtype, const float* q, const KvView& kv, const int32_t* cand,
                              const int32_t* cand_count, float* score, int64_t score_stride, int32_t* flags,
                              hipStream_t st, float* tops = nullptr, const int32_t* k = nullptr);

// S1 and S2 of a step over fp32 keys in one kernel, where step_fuses_f32: what launch_candidates (without a line) and
// launch_group_score leave.
bool step_fuses_f32(const Shape& s);
hipError_t launch_candidates_score_f32(const Shape& s, const float* q, const KvView& kv, const int32_t* prev_topk, const int32_t* k,
                                       int32_t* cand, int32_t* cand_count, float* score, int64_t score_stride, int32_t* flags,
                                       hipStream_t st);

// Filtered scoring (bf16, fp16 or FP8 keys; the kernel keeps its first name, k_filter_score_bf16): per
// head only rows with score >= thr_state[b,h] - margin (left in tau_out[b,h] where rows are kept: the select replaces thr_state) are kept, as
// (score, position) lists in at most filter_nseg(s) pieces per head.  The kernel runs with exactly
// n_blocks workgroups (filter_score_blocks: what the device holds at once) and cuts the candidate
// slots of all groups (placed on one line by the candidates kernel: group_start, line_total) into
// equal parts, one per wave; the part size of a step is written to *seg_rows_out by the scoring
// pass and read by the select, which also resets *line_total; see score.hip.
int filter_nseg(const Shape& s);
int filter_list_cap(const Shape& s);   // survivors per head the filtered select can hold
hipError_t filter_score_blocks(const Shape& s, int k_kind, int out[2]);
hipError_t launch_filter_score(const Shape& s, const float* q, const KvView& kv, const int32_t* cand,
                               const int32_t* cand_count, const int64_t* group_start, const int64_t* line_total,
                               const float* thr_state, float margin, float* tau_out, const int32_t* skip_if, float* score,
                               int32_t* slot_out, int64_t score_stride, int32_t* seg_count, int32_t* seg_rows_out,
                               int n_blocks, int32_t* flags, bool dense, int nseg, hipStream_t st);
// S1 + S2 of a chained step in one kernel (range_score.hip): candidates from the Top-k of the step before (prev_topk, k) or
// from the table scan's flags (f0, fm; prev_topk == NULL), scored and filtered as above.  seg_count[b, h, 4 i + w] =
// candidates << 16 | survivors of piece w of range i; bitmap [B, Hkv, bitmap_words] = the candidates.
struct RangeSource {
  const int32_t* prev_topk;          // [B, Hq, kmax]
  const int32_t* k;                  // [B]
  const uint32_t* f0;                // [B, Hq, flag_words]
  const uint32_t* fm;
  int flag_words;
};
int range_rows(const Shape& s, bool tables);   // see range_rows_for
hipError_t launch_range_score(const Shape& s, const float* q, const KvView& kv, const RangeSource& from,
                              const float* thr_state, float margin, float* tau_out, const int32_t* skip_if, float* score,
                              int32_t* slot_out, int64_t score_stride, int32_t* seg_count, int nseg, uint32_t* bitmap, int bitmap_words,
                              int range, int32_t* flags, hipStream_t st);
// The same from the Top-k for larger contexts (wide_score.hip), those with a wide_plan: a piece is a wave's part of a strip,
// and parts_of [B, Hkv] receives the workgroups of a group, with two strips each.
WidePlan wide_plan(const Shape& s);
hipError_t launch_wide_score(const Shape& s, const float* q, const KvView& kv, const int32_t* prev_topk, const int32_t* k,
                             const float* thr_state, float margin, float* tau_out, const int32_t* skip_if, float* score, int32_t* slot_out,
                             int64_t score_stride, int32_t* seg_count, int nseg, int32_t* parts_of, uint32_t* bitmap, int bitmap_words,
                             int32_t* flags, hipStream_t st);

// S3 + S4 of the chained steps in one kernel (select_attend.hip).  From the survivor lists of the filtered scoring
// pass: every head gets its Top-k rows (topk_idx, topk_score: both required) and its output row; a head whose list
// is short or overfull takes the unfiltered pass inside the kernel (counted in *rescored), which needs q, the K rows
// and the group's candidate list (cand; NULL = all rows 0 .. cand_count-1) and overwrites the head's score row.
// range > 0: the lists are those of launch_range_score with that range, or with parts_of those of launch_wide_score (cand, seg_rows, group_start, line_total unused;
// the candidates are in bitmap), and cand_count is written.
// keep: a head with fewer than keep.ratio * k candidates, and no more than keep.most, leaves -inf in thr_state instead of its
// k-th best score; keep.fits [B, Hq] (or NULL) receives whether it had no more than keep.most, and a bypassed head (skip_if)
// leaves -inf unless it has a score and had more.  The launchers set most: half of filter_list_cap,
// or all of it where it holds the candidates of any step.
struct KeepAll {
  int ratio;
  int32_t* fits;
  int most;
};
hipError_t configure_select_attend(const Shape& s, int dtype, bool k_fp8, bool v_fp8);
hipError_t launch_filter_select_attend(const Shape& s, int dtype, float* score, int32_t* slot,
                                       int64_t score_stride, const int32_t* seg_count, const int32_t* seg_rows, int nseg,
                                       const int32_t* cand, int32_t* cand_count, const int64_t* group_start,
                                       int64_t* line_total, int range, const int32_t* parts_of, const uint32_t* bitmap, int bitmap_words,
                                       const int32_t* k, int32_t* topk_idx, float* topk_score,
                                       float* thr_state, const float* tau, KeepAll keep, const int32_t* skip_if, int32_t* rescored,
                                       const float* q, int32_t* flags, const KvView& kv, float* out,
                                       hipStream_t st);   // out == NULL: select only

// Exact Top-k baseline, the first step of its filtered form (exact_topk.hip): a strided sample of at most ns_max rows per group (or
// all; sized for the select's list capacity list_cap, see plan_sample) is scored (score [B, Hq, score_stride]; x_ns [B] its
// length), every group's rows 0..n_b-1 are laid on the line (x_cnt, x_start, x_start[B*Hkv] = the line's length), and x_rank [B] is
// the rank whose sample score is taken as the threshold.
hipError_t launch_sample_score(const Shape& s, const float* q, const KvView& kv, const int32_t* k, int ns_max, int list_cap,
                               int32_t* x_cnt, int64_t* x_start, int32_t* x_ns, int32_t* x_rank, float* score, int64_t score_stride,
                               int32_t* flags, hipStream_t st);
// From the full score rows [B, Hq, score_stride] over cand, every head.
hipError_t launch_select_attend(const Shape& s, int dtype, const float* score, int64_t score_stride, const int32_t* cand,
                                const int32_t* cand_count, const int32_t* k, int32_t* topk_idx, float* topk_score,
                                float* thr_state, KeepAll keep, const int32_t* skip_if, const KvView& kv, float* out,
                                hipStream_t st);

// Per (b, h): the k_b best of score[b,h,0:count]; count = cand_count[b, g(h)] when cand != NULL,
// else seq_lens[b].  Writes positions (ascending) and their scores.
// thr_state [B,Hq] (or NULL) receives
// each head's k-th best score.  skip_if [B,Hq] (or NULL): heads whose entry is not 0 are skipped (bypassed heads).
// seq_lens [B] (or NULL; with cand only): a selected candidate entry outside [0, n_b) is written as -1.
// tops (or NULL; without cand only): what launch_group_score has left there for these scores.
hipError_t launch_select(const Shape& s, const float* score, int64_t score_stride, const int32_t* cand,
                         const int32_t* count, const int32_t* k, int32_t* topk_idx, float* topk_score,
                         float* thr_state, const int32_t* skip_if, const int32_t* seq_lens, hipStream_t st,
                         const float* tops = nullptr);
bool select_wants_tops(const Shape& s);   // worth asking launch_group_score for?

// Is the select of n scores and a budget of kb made from the largest scores of 16 rows each?  Asked by the pass that writes
// them and by the select.  The select reads the blocks of the budget's best maxima, and what passes the cut has to fit its list
// beside the blocks' numbers: of independent scores 1 - (1 - p)^(1/16) pass, p the share of blocks chosen.  The line is the p at
// which the list is full up to five standard deviations; below 32769 rows, where the select from all scores is faster, that at
// which 4096 pass (a longer list makes the last step twice as long); never more than 31/32, where nearly all of the row passes.
// Exact Top-k of 32 heads, from all scores -> from the blocks, us: 9000 rows, p = 7/8 19.6 -> 19.1, 1 19.8 -> 29.9; 32768 rows, 1/2
// 38.1 -> 27.4, 27/32 38.3 -> 32.1, 7/8 38.4 -> 38.9, 1 39.6 -> 47.3; 65536 rows, 15/16 84.3 -> 61.3, 1 84 -> 100; 120000 rows, 3/4
// 148.7 -> 90.3, 7/8 (the list overflows) 148.9 -> 176.3.
constexpr int kTopsMinRows = 8192, kTopsMaxRows = 262144;
__host__ __device__ inline bool select_takes_tops(const Shape& s, int n, int kb) {
  kb = kb > s.kmax ? s.kmax : kb;
  kb = kb > n ? n : kb;
  const int share = n <= 19712 ? 124 : n <= 32768 ? 124 - (n - 19712) / 932                        // in 128ths
                    : n <= 65536 ? 124 : n <= 147456 ? 124 - (n - 65536) / 2926
                    : n <= 200704 ? 96 - (n - 147456) / 3132 : 79 - (n - 200704) / 4389;
  return n > kTopsMinRows && n <= kTopsMaxRows && 128 * kb <= share * ((n + 15) >> 4);
}

// Scores of idx[b,h,0:k_b] rows against q[b,h] (one head at a time, no group sharing).
hipError_t launch_head_score(const Shape& s, int dtype, const float* q, const KvView& kv, const int32_t* idx,
                             const int32_t* k, float* idx_score, hipStream_t st);

// Sparse attention: one workgroup per (b, h), output row written directly.
hipError_t launch_sparse_attn(const Shape& s, int dtype, const KvView& kv, const int32_t* idx, const float* idx_score,
                              const int32_t* k, float* out, const int32_t* skip_if, hipStream_t st);

// Full attention: split partials [B*Hkv, n_split, G, D+2] + merge.
int full_attn_splits(const Shape& s);
hipError_t launch_full_attn(const Shape& s, int dtype, const float* q, const KvView& kv, float* part, int n_split,
                            hipStream_t st);
hipError_t launch_full_merge(const Shape& s, const int32_t* seq_lens, const float* part, int n_split, float* out,
                             hipStream_t st);

// Score tables (Eq. 4, 7-10): see tables.hip.  tab_ver [B*Hq, Lcap], tab_sla [B*Hq, 2*Lcap] unscaled fp32
// entries; state [B*Hq, kTableStateDoubles]; f0 / fm [B*Hq, flag_words] bitmaps written by the scan.
constexpr int kTableStateDoubles = 16;
// head state (doubles): scale, update count, raw moments of both tables, and "the table was flat (every
// entry equal) when it was imported with N entries" marks.  The thresholds of Eq. 8 are derived from the
// moments at the start of every scan for the number of rows that scan sees, so a head whose update was
// skipped (a bypassed head) or a cache that grew by several rows needs no special case: new positions are zeros.
enum {
  TS_G = 0, TS_CNT = 1,
  TS_MV = 2,            // M1..M4 of the vertical table: [2..5]
  TS_MS = 6,            // M1..M4 of the slash table:    [6..9]
  TS_FLAT_V = 10, TS_FLAT_S = 11, TS_FLAT_N = 12,
};
hipError_t launch_table_flags(const Shape& s, const float* tab_ver, const float* tab_sla, const double* state,
                              const int32_t* seq_lens, uint32_t* f0, uint32_t* fm, int flag_words, double a,
                              const int32_t* gate, hipStream_t st);
hipError_t launch_table_candidates(const Shape& s, const uint32_t* f0, const uint32_t* fm, int flag_words,
                                   const int32_t* seq_lens, int32_t* cand, int32_t* cand_count, int32_t* flags,
                                   int64_t* group_start, int64_t* line_total, hipStream_t st);
hipError_t launch_table_update(const Shape& s, float* tab_ver, float* tab_sla, double* state, const int32_t* seq_lens,
                               const int32_t* idx, const float* sc, const int32_t* k, double gamma, const int32_t* gate,
                               int32_t* flags, bool distinct, hipStream_t st);   // distinct: no position twice in a head's list
hipError_t launch_table_import(const Shape& s, float* tab_ver, float* tab_sla, double* state, const int32_t* seq_lens,
                               const float* phi_ver, const float* phi_sla, hipStream_t st);
hipError_t launch_table_export(const Shape& s, const float* tab_ver, const float* tab_sla, const double* state,
                               const int32_t* seq_lens, double* phi_ver, double* phi_sla, hipStream_t st);
hipError_t launch_table_init(const Shape& s, float* tab_ver, float* tab_sla, const int32_t* seq_lens,
                             const float* score, int64_t score_stride, double gamma, int j, int n_queries,
                             hipStream_t st);
// Eq. 4 from n_queries prefill queries, kHistBatch of them per pass over K (prefill.hip; 16-bit and FP8 keys);
// q_hist[j - 1] = query j, the j-th most recent.  dots [B, Hq, dots_stride]: room for one query's dot products.
// scratch: table_init_scratch_bytes.  *moment_parts: how many partials per head of the tables' moments it has left there (0:
// none).
constexpr int kHistBatch = 32;
// How many workgroups share a KV group: in those kernels' first, by the form of its chunks, and in their second.  Made once per
// context (the search takes the host 2 us).
enum { kPartsShort = 0, kPartsFp8 = 1, kPartsOneUnit = 2 };
struct HistPlan {
  int parts[3], blocks;
};
HistPlan plan_table_history(const Shape& s);
int64_t table_init_scratch_bytes(const Shape& s, const HistPlan& plan);
hipError_t configure_table_history(const Shape& s, int k_kind);
hipError_t launch_table_history(const Shape& s, const HistPlan& plan, float* tab_ver, float* tab_sla, const float* q_hist, int n_queries,
                                double gamma, const KvView& kv, float* dots, int64_t dots_stride, void* scratch,
                                int32_t* flags, int* moment_parts, hipStream_t st);
// Statistics and head state of freshly written tables.
hipError_t launch_table_state(const Shape& s, const float* tab_ver, const float* tab_sla, double* state,
                              const int32_t* seq_lens, void* scratch, int moment_parts, hipStream_t st);
// Head sparsity (Eq. 5-6) and the prefill priors it needs; gate [B,Hq] marks bypassed heads, whose output
// row (vbar) and index row (-1) the kernel writes when out != NULL.
hipError_t launch_head_sparsity(const Shape& s, int dtype, const float* q, const KvView& kv, const float* kbar,
                                const float* sigma2_hat, int n_local, float eps, float* rho, int32_t* gate,
                                const float* vbar, int32_t* topk_idx, float* topk_score, float* out,
                                hipStream_t st);
// scratch: prior_scratch_bytes.
int64_t prior_scratch_bytes(const Shape& s);
hipError_t launch_priors(const Shape& s, int dtype, const float* q, const KvView& kv, float* kbar, float* vbar,
                         float* sigma2_hat, void* scratch, int32_t* flags, hipStream_t st);

// ---- small device helpers ------------------------------------------------------------
// A kernel's arguments come through the scalar cache, where none of them is when it starts, and the compiler asks for an argument where
// it is used: every further 64-byte line of them is a trip to memory that all waves wait for, 0.4 us, and the longest kernels here have
// six lines.  request_arguments, called first, asks for all lines at once: a launch of the step's kernels becomes 0.3 to 0.9 us shorter
// (four steps of 1 x 32K 86.5 -> 82.6 us, of 16 x 64K paged FP8 323.6 -> 318.5, exact Top-k of one request 33.2 -> 32.4, sixteen
// table steps of 8 x 32K 1069 -> 1050; the two passes of a table start from many queries did not gain).
template <typename Kernel>
struct KernelArguments;
template <typename... Args>
struct KernelArguments<void (*)(Args...)> {
  static constexpr int bytes() {
    int at = 0;
    ((at = (at + (int)alignof(Args) - 1) / (int)alignof(Args) * (int)alignof(Args) + (int)sizeof(Args)), ...);
    return at;
  }
};
template <typename Kernel>
__device__ __forceinline__ void request_arguments() {
  constexpr int kLines = (KernelArguments<Kernel>::bytes() + 63) / 64;
  static_assert(kLines <= 8, "more lines than are asked for");
  typedef const __attribute__((address_space(4))) uint32_t* Words;
  const Words p = (Words)__builtin_amdgcn_kernarg_segment_ptr();
  uint32_t x[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = p[i < kLines ? 16 * i : 0];
  asm volatile("" ::"s"(x[0]), "s"(x[1]), "s"(x[2]), "s"(x[3]), "s"(x[4]), "s"(x[5]), "s"(x[6]), "s"(x[7]));
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// OCP FP8 E4M3 ("FN": no infinities, one NaN pattern per sign, largest value 448) to fp32: four values of
// one dword, lowest byte first.  The hardware conversion is exact.
__device__ __forceinline__ void fp8x4_to_f32(uint32_t w, float x[4]) {
  const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false);
  const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
  x[0] = lo[0];
  x[1] = lo[1];
  x[2] = hi[0];
  x[3] = hi[1];
}
// Eight E4M3 values as eight bf16 (exact: 3 mantissa bits fit bf16's 7, the exponent range is inside fp32's):
// the upper halves of the fp32 conversions, packed two per dword.
__device__ __forceinline__ bf16x8 fp8x8_to_bf16x8(uint32_t w0, uint32_t w1) {
  float a[4], b[4];
  fp8x4_to_f32(w0, a);
  fp8x4_to_f32(w1, b);
  auto pack = [](float lo, float hi) { return (__float_as_uint(hi) & 0xFFFF0000u) | (__float_as_uint(lo) >> 16); };
  union {
    u32x4 u;
    bf16x8 v;
  } r;
  r.u[0] = pack(a[0], a[1]);
  r.u[1] = pack(a[2], a[3]);
  r.u[2] = pack(b[0], b[1]);
  r.u[3] = pack(b[2], b[3]);
  return r.v;
}

// Eight consecutive elements of a K or V row as they are loaded (T = float, uint16_t = bf16 bits, _Float16,
// uint8_t = E4M3), converted to fp32 when used: a row waiting in registers costs 8, 4 or 2 of them.  load_once: past the
// caches, for lines that one instruction reads whole and nobody reads again soon.
template <typename T>
struct Raw8;
template <>
struct Raw8<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = reinterpret_cast<const f32x4*>(p)[0];
    b = reinterpret_cast<const f32x4*>(p)[1];
  }
  __device__ __forceinline__ void load_once(const float* p) {
    a = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    b = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p) + 1);
  }
  __device__ __forceinline__ void get(float x[8]) const {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      x[c] = a[c];
      x[4 + c] = b[c];
    }
  }
};
template <>
struct Raw8<uint16_t> {
  u32x4 w;
  __device__ __forceinline__ void load(const uint16_t* p) { w = *reinterpret_cast<const u32x4*>(p); }
  __device__ __forceinline__ void load_once(const uint16_t* p) { w = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)); }
  __device__ __forceinline__ void get(float x[8]) const {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      x[2 * c] = bf16_lo(w[c]);
      x[2 * c + 1] = bf16_hi(w[c]);
    }
  }
};
template <>
struct Raw8<_Float16> {
  f16x8 w;
  __device__ __forceinline__ void load(const _Float16* p) { w = *reinterpret_cast<const f16x8*>(p); }
  __device__ __forceinline__ void load_once(const _Float16* p) { w = __builtin_nontemporal_load(reinterpret_cast<const f16x8*>(p)); }
  __device__ __forceinline__ void get(float x[8]) const {
#pragma unroll
    for (int c = 0; c < 8; ++c) x[c] = (float)w[c];
  }
};
template <>
struct Raw8<uint8_t> {
  u32x2 w;
  __device__ __forceinline__ void load(const uint8_t* p) { w = *reinterpret_cast<const u32x2*>(p); }
  __device__ __forceinline__ void load_once(const uint8_t* p) { w = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p)); }
  __device__ __forceinline__ void get(float x[8]) const {
    fp8x4_to_f32(w[0], x);
    fp8x4_to_f32(w[1], x + 4);
  }
};
template <typename T>
__device__ __forceinline__ void load8(const T* p, float x[8]) {
  Raw8<T> r;
  r.load(p);
  r.get(x);
}

// Inclusive prefix sum over the 64 lanes of a wave, on the vector ALU alone (DPP row shifts inside each row of
// 16 lanes, then two row broadcasts for the carries); a scan by lane shuffles costs six LDS-crossbar round trips.
__device__ __forceinline__ int wave_inclusive_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

// Maximum over the wave, in its last lane (DPP, no LDS; a NaN counts as absent).  In the select, against two lane exchanges
// through LDS behind the rows' maxima: four steps of 64 groups x 32K rows 240.0 -> 239.2 us, of 96 paged groups x 20000 198.8 ->
// 197.2, of 8 groups x 100K rows with FP8 keys 146.3 -> 145.1, exact Top-k of one request 34.2 -> 34.1.
__device__ __forceinline__ float wave_max_in_last(float x) {
  auto step = [&](float y) { x = fmaxf(x, y); };
#define LFPS_DPP_MAX(ctrl, rows) \
  step(__int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), ctrl, rows, 0xf, false)))
  LFPS_DPP_MAX(0x111, 0xf);
  LFPS_DPP_MAX(0x112, 0xf);
  LFPS_DPP_MAX(0x114, 0xf);
  LFPS_DPP_MAX(0x118, 0xf);
  LFPS_DPP_MAX(0x142, 0xa);
  LFPS_DPP_MAX(0x143, 0xc);
#undef LFPS_DPP_MAX
  return x;
}

// Between LDS writes of some lanes of a wave and reads of them by others: a wave's LDS operations complete in order, so this
// only keeps the compiler from moving or reusing them across (no instruction).
__device__ __forceinline__ void wave_lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); }

// The value of lane (lane - kBy) mod 16 of my 16 lanes.
template <int kBy>
__device__ __forceinline__ float row16_rotate(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + kBy, 0xf, 0xf, false));   // row_ror
}
template <int kBy>
__device__ __forceinline__ double row16_rotate(double x) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x120 + kBy, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x120 + kBy, 0xf, 0xf, false));
}
// Sum and maximum over the 16 lanes of a row of lanes, left in every one of them (DPP rotations, no LDS).
template <typename T>
__device__ __forceinline__ T row16_sum(T x) {
  x += row16_rotate<8>(x);
  x += row16_rotate<4>(x);
  x += row16_rotate<2>(x);
  x += row16_rotate<1>(x);
  return x;
}
__device__ __forceinline__ float row16_max(float x) {
  x = fmaxf(x, row16_rotate<8>(x));
  x = fmaxf(x, row16_rotate<4>(x));
  x = fmaxf(x, row16_rotate<2>(x));
  x = fmaxf(x, row16_rotate<1>(x));
  return x;
}
// The same sum in the order of a butterfly over lane distances 1, 2, 4, 8 (the bits of four xor shuffles), without LDS:
// lanes of a quad by permutation, then, all lanes of a quad (of a half) being equal, the other one by mirroring.
__device__ __forceinline__ float row16_butterfly_sum(float x) {
#define LFPS_DPP(v, ctrl) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, false))
  x += LFPS_DPP(x, 0xB1);     // quad_perm 1 0 3 2
  x += LFPS_DPP(x, 0x4E);     // quad_perm 2 3 0 1
  x += LFPS_DPP(x, 0x141);    // row_half_mirror
  x += LFPS_DPP(x, 0x140);    // row_mirror
#undef LFPS_DPP
  return x;
}
// Do the rows that the requests hold, row_bytes each in every KV head, take more than kept_bytes (the memory-side cache, or what a
// pass leaves of it)?  The same for the whole grid.  In two parts, so that other loads can be asked for in between: the rows that
// my lane counts, and their sum over the wave.  (In fp32: requests may share rows, and B * Lcap need not fit an int.)
__device__ __forceinline__ float held_rows(const Shape& s, const int32_t* seq_lens) {
  auto rows = [&](int b) {
    const int n = seq_lens[b < s.B ? b : 0];
    return b < s.B ? (float)(n < 0 ? 0 : (n > s.Lcap ? s.Lcap : n)) : 0.f;
  };
  const int lane = threadIdx.x & 63;
  float sum = rows(lane);
  for (int b0 = 64; b0 < s.B; b0 += 64) sum += rows(b0 + lane);
  return sum;
}
__device__ __forceinline__ bool outgrow_cache(const Shape& s, float rows, int row_bytes, float kept_bytes) {
  rows = row16_sum(rows);
  rows += __shfl_xor(rows, 16);
  rows += __shfl_xor(rows, 32);
  return __builtin_amdgcn_readfirstlane(rows * (float)s.Hkv * (float)row_bytes > kept_bytes);
}
// exp(y), or kScaled exp(y / sqrt(D)), for y <= 0 to about one unit in the last place: exp2 of the rounded product, corrected by the
// product's rounding error, which grows with |y| (seven instructions; without expf's handling of other ranges: results below
// 2^-126 are 0).  -inf gives 0, a NaN stays one.
template <bool kScaled>
__device__ __forceinline__ float exp_below(float y) {
  constexpr double c = (kScaled ? 0.08838834764831845 : 1.0) * 1.4426950408889634;
  constexpr float hi = (float)c, lo = (float)(c - (double)hi), ln2 = 0.6931471805599453f;
  y = __builtin_elementwise_maximum(y, -1e30f);             // (the correction needs a finite y)
  const float t = y * hi;
  const float r = fmaf(y, lo, fmaf(y, hi, -t));
  const float e = __builtin_amdgcn_exp2f(t);
  return fmaf(e * ln2, r, e);
}

// Order-preserving map fp32 -> uint32 (larger float <=> larger key).
__device__ __forceinline__ uint32_t f2key(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

}  // namespace lfps
