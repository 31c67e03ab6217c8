// D2Q9 step pairs (two steps in one launch).
#include "pair.hpp"

namespace lbrr {
template hipError_t step_pair_by_order<D2Q9, double>(int, const void*, void*, const StepArgs&, hipStream_t);
template hipError_t step_pair_by_order<D2Q9, float>(int, const void*, void*, const StepArgs&, hipStream_t);
template int pair_rows_of<D2Q9>(int, int, bool);
}  // namespace lbrr
