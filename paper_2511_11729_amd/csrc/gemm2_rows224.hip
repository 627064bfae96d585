// Weight GEMM of the finetune unit: tiles of 224 rows.
#include "gemm2_kernel.h"

namespace harli {
template harli_status gemm2_init<7>();
template harli_status gemm2_run<7>(const Gemm2Args&, const Gemm2Cut&, const Gemm2Plan&, bool, int, hipStream_t);
}
