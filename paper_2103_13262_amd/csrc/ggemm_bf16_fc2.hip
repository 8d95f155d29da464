#include "ggemm_bf16_sk.h"

namespace moe::sk {
template void launch_kind<kRowsNN>(const GemmArgs&, hipStream_t);
}
