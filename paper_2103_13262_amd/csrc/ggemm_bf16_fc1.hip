#include "ggemm_bf16_sk.h"

namespace moe::sk {
template void launch_kind<kRowsNN_GeLU>(const GemmArgs&, hipStream_t);
}
