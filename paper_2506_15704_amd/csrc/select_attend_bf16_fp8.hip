// k_filter_select_attend for bf16 values beside FP8 keys.
#include "select_attend.h"

namespace lfps {

template hipError_t configure_filter_select<uint16_t, kKindFp8>(const Shape& s);
template hipError_t launch_filter_select<uint16_t, kKindFp8>(const FilterSelectArgs& a, hipStream_t st);

}  // namespace lfps
