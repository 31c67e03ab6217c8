// D3Q19 step pairs (two steps in one launch).
#include "pair.hpp"

namespace lbrr {
template hipError_t step_pair_by_order<D3Q19, double>(int, const void*, void*, const StepArgs&, hipStream_t);
template hipError_t step_pair_by_order<D3Q19, float>(int, const void*, void*, const StepArgs&, hipStream_t);
template int pair_rows_of<D3Q19>(int, int, bool);
}  // namespace lbrr
