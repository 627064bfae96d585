// Weight GEMM of the finetune unit: tiles of 192 rows.
#include "gemm2_kernel.h"

namespace harli {
template harli_status gemm2_init<6>();
template harli_status gemm2_run<6>(const Gemm2Args&, const Gemm2Cut&, const Gemm2Plan&, bool, int, hipStream_t);
}
