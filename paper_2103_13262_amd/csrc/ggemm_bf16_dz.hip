#include "ggemm_bf16_sk.h"

namespace moe::sk {
template void launch_kind<kRowsNT_dGeLU>(const GemmArgs&, hipStream_t);
}
