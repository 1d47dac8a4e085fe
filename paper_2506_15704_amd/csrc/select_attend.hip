// S3 + S4 in one kernel, the dispatch (kernels: select_attend.h; their instantiations: select_attend_*.hip).
#include "select_attend.h"

namespace lfps {

// V type and K format go together: bf16 V with bf16 or FP8 keys, FP8 V with FP8 keys, fp16 V with fp16 keys.
#define LFPS_DECLARE(T, KIND)                                                            \
  extern template hipError_t configure_filter_select<T, KIND>(const Shape& s);           \
  extern template hipError_t launch_filter_select<T, KIND>(const FilterSelectArgs& a, hipStream_t st);
LFPS_DECLARE(uint16_t, kKindBf16)
LFPS_DECLARE(uint16_t, kKindFp8)
LFPS_DECLARE(uint8_t, kKindFp8)
LFPS_DECLARE(_Float16, kKindF16)
#undef LFPS_DECLARE
#define LFPS_DECLARE(T)                                                                  \
  extern template hipError_t configure_select_only<T>(const Shape& s);                   \
  extern template hipError_t launch_select_only<T>(const SelectArgs& a, hipStream_t st);
LFPS_DECLARE(uint16_t)
LFPS_DECLARE(uint8_t)
LFPS_DECLARE(_Float16)
#undef LFPS_DECLARE

int filter_list_cap(const Shape& s) { return kRegElems * filter_select_threads(s); }

// Called once per context at creation.
hipError_t configure_select_attend(const Shape& s, int dtype, bool k_fp8, bool v_fp8) {
  if (dtype == LFPS_F32) return configure_select_only<float>(s);
  const hipError_t e = dtype == LFPS_F16 ? configure_select_only<_Float16>(s)
                       : v_fp8           ? configure_select_only<uint8_t>(s)
                                         : configure_select_only<uint16_t>(s);
  if (e != hipSuccess) return e;
  if (dtype == LFPS_F16) return configure_filter_select<_Float16, kKindF16>(s);
  if (v_fp8) return configure_filter_select<uint8_t, kKindFp8>(s);
  return k_fp8 ? configure_filter_select<uint16_t, kKindFp8>(s) : configure_filter_select<uint16_t, kKindBf16>(s);
}

hipError_t launch_filter_select_attend(const Shape& s, int dtype, float* score, int32_t* slot,
                                       int64_t score_stride, const int32_t* seg_count, const int32_t* seg_rows, int nseg,
                                       const int32_t* cand, int32_t* cand_count, const int64_t* group_start,
                                       int64_t* line_total, int range, const int32_t* parts_of, const uint32_t* bitmap, int bitmap_words,
                                       const int32_t* k, int32_t* topk_idx, float* topk_score,
                                       float* thr_state, const float* tau, KeepAll keep, const int32_t* skip_if, int32_t* rescored,
                                       const float* q, int32_t* flags, const KvView& kv, float* out, hipStream_t st) {
  const FilterSelectArgs a{s, score, slot, score_stride, seg_count, seg_rows, nseg, cand, cand_count, group_start, line_total, range, parts_of, bitmap,
                           bitmap_words, k, topk_idx, topk_score, thr_state, tau, keep, skip_if, rescored, q, flags, &kv, out};
  if (dtype == LFPS_F16) return launch_filter_select<_Float16, kKindF16>(a, st);
  if (dtype != LFPS_BF16) return hipErrorInvalidValue;          // the filtered pass exists for 16-bit and FP8 caches only
  if (kv.v_fp8) return kv.k_fp8 ? launch_filter_select<uint8_t, kKindFp8>(a, st) : hipErrorInvalidValue;   // FP8 values come with FP8 keys
  return kv.k_fp8 ? launch_filter_select<uint16_t, kKindFp8>(a, st) : launch_filter_select<uint16_t, kKindBf16>(a, st);
}

hipError_t launch_select_attend(const Shape& s, int dtype, const float* score, int64_t score_stride, const int32_t* cand,
                                const int32_t* cand_count, const int32_t* k, int32_t* topk_idx, float* topk_score,
                                float* thr_state, KeepAll keep, const int32_t* skip_if, const KvView& kv, float* out,
                                hipStream_t st) {
  const SelectArgs a{s, score, score_stride, cand, cand_count, k, topk_idx, topk_score, thr_state, keep, skip_if, &kv, out};
  if (dtype == LFPS_BF16 && kv.v_fp8) return launch_select_only<uint8_t>(a, st);
  if (dtype == LFPS_F16) return launch_select_only<_Float16>(a, st);
  if (dtype == LFPS_BF16) return launch_select_only<uint16_t>(a, st);
  return launch_select_only<float>(a, st);
}

}  // namespace lfps
