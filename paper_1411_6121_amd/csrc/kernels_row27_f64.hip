// kernels_row27_f64.hip -- instances of the 3-D step kernel (row3.hpp) for
// D3Q27 in FP64
#include "row3.hpp"

namespace dugks {
template int row_step<D3Q27, double>(dugks_ctx*, const Inst<double>&, const void*, void*, const void*, double, hipStream_t,
                                   int);
}  // namespace dugks
