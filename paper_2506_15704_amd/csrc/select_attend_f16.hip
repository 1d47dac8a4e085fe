// k_filter_select_attend and k_select_attend for fp16 values.
#include "select_attend.h"

namespace lfps {

template hipError_t configure_filter_select<_Float16, kKindF16>(const Shape& s);
template hipError_t launch_filter_select<_Float16, kKindF16>(const FilterSelectArgs& a, hipStream_t st);
template hipError_t configure_select_only<_Float16>(const Shape& s);
template hipError_t launch_select_only<_Float16>(const SelectArgs& a, hipStream_t st);

}  // namespace lfps
