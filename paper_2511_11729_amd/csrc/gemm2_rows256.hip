// Weight GEMM of the finetune unit: tiles of 256 rows.
#include "gemm2_kernel.h"

namespace harli {
template harli_status gemm2_init<8>();
template harli_status gemm2_run<8>(const Gemm2Args&, const Gemm2Cut&, const Gemm2Plan&, bool, int, hipStream_t);
}
