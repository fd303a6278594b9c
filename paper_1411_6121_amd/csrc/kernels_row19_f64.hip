// kernels_row19_f64.hip -- instances of the 3-D step kernel (row3.hpp) for
// D3Q19 in FP64
#include "row3.hpp"

namespace dugks {
template int row_step<D3Q19, double>(dugks_ctx*, const Inst<double>&, const void*, void*, const void*, double, hipStream_t,
                                   int);
template long long row_batch_slots<D3Q19, double>(int);
template void row_batch_launch<D3Q19, double>(const void*, const long long*, const BatchGeom*, int, long long, const void*,
                                           const void*, void*, const long long*, int, hipStream_t);

// for the batch's launch geometry (the same for every precision)
int row_chunk_of(long long tiles, int nz, long long slots) { return row_chunk(tiles, nz, slots); }
void row_tile_shape(int* bx, int* by)
{
    *bx = ROW_X;
    *by = RowShape<D3Q19, double>::BY;
}
}  // namespace dugks
