#include "ggemm_bf16_sk.h"

namespace moe::sk {
template void launch_kind<kColsT>(const GemmArgs&, hipStream_t);
}
