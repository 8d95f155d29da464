#include "ggemm_bf16_sk.h"

namespace moe::sk {
template void launch_kind<kRowsNT>(const GemmArgs&, hipStream_t);
}
