#include "ggemm_bf16_sk.h"

namespace moe::sk {
template void launch_pair_kind<kRowsNT>(const GemmArgs&, const GemmArgs&, hipStream_t);
}
