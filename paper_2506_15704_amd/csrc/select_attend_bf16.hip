// k_filter_select_attend and k_select_attend for bf16 values.
#include "select_attend.h"

namespace lfps {

template hipError_t configure_filter_select<uint16_t, kKindBf16>(const Shape& s);
template hipError_t launch_filter_select<uint16_t, kKindBf16>(const FilterSelectArgs& a, hipStream_t st);
template hipError_t configure_select_only<uint16_t>(const Shape& s);
template hipError_t launch_select_only<uint16_t>(const SelectArgs& a, hipStream_t st);

}  // namespace lfps
