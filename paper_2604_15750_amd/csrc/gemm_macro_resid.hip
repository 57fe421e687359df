// The macro-tile GEMM's instantiations with the EPI_RESID epilogue (one source per epilogue: they compile in parallel).
#define GEMM_MACRO_INSTANTIATE
#include "gemm_macro_kernel.h"

template void launch_macro_epi<EPI_RESID>(const op_t*, const op_t*, int, int, int, const MacroPlan&, const GemmEpi&, hipStream_t);
