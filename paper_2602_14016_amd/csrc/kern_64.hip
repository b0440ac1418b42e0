// Row and column passes for N = 64 (both FFT plan variants).
#include "kernels_impl.hpp"

namespace pa {
template struct Launch<64>;
// Nothing launches these two up to 64 points; they are built because the check of the code of
// global->LDS loads reads them here.
template __global__ void row_sq_pipe_kernel<64>(Dims, RowArgs, int);
template __global__ void row_mul_pipe_kernel<64>(Dims, RowArgs, int);
}  // namespace pa
