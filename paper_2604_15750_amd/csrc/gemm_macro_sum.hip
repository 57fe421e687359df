// The macro-tile GEMM's instantiations with the EPI_SUM epilogue (one source per epilogue: they compile in parallel).
#define GEMM_MACRO_INSTANTIATE
#include "gemm_macro_kernel.h"

template void launch_macro_epi<EPI_SUM>(const op_t*, const op_t*, int, int, int, const MacroPlan&, const GemmEpi&, hipStream_t);
