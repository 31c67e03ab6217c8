// D3Q27 step pairs (two steps in one launch).
#include "pair.hpp"

namespace lbrr {
template hipError_t step_pair_by_order<D3Q27, double>(int, const void*, void*, const StepArgs&, hipStream_t);
template hipError_t step_pair_by_order<D3Q27, float>(int, const void*, void*, const StepArgs&, hipStream_t);
template int pair_rows_of<D3Q27>(int, int, bool);
}  // namespace lbrr
