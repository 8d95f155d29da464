// Grouped bf16 products: the host side that the kinds share.  The kernels are in ggemm_bf16_sk.h; every kind and pair is compiled
// in a file of its own (ggemm_bf16_*.hip).
#include <cstdlib>
#include <mutex>

#include "common.h"

namespace moe {
namespace sk {

constexpr int kSpinLimit = 1 << 20;             // bounded wait for a partial sum (on the order of a second)

template <int KIND> void launch_kind(const GemmArgs& a, hipStream_t st);
template <int KIND> void launch_pair_kind(const GemmArgs& rows, const GemmArgs& cols, hipStream_t st);

// Persistent workgroups of one launch: one per compute unit of the current device, a multiple of the 8 XCDs, at most
// kMaxPersistentWgs (the workspace holds one partial-sum buffer per workgroup and phase).  0 after fail_launch.
int persistent_wgs()
{
    static std::mutex mu;
    static int cached[kMaxDevices] = {};
    const int dev = current_device();
    if (dev < 0) return 0;
    std::lock_guard<std::mutex> lk(mu);
    if (!cached[dev]) {
        int cus = 0;
        const hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) { fail_launch("grouped GEMM: compute-unit count of device %d: %s", dev, hipGetErrorString(e)); return 0; }
        cus = cus / 8 * 8;
        if (cus < 8) { fail_launch("grouped GEMM: device %d has fewer than 8 compute units", dev); return 0; }
        cached[dev] = cus > kMaxPersistentWgs ? kMaxPersistentWgs : cus;
    }
    return cached[dev];
}

}  // namespace sk

// How often a workgroup polls for its predecessor's partial sum before it gives up and sets the workspace's status
// word.  MOE355_SPIN_LIMIT overrides the default (about a second); a negative value makes every wait give up at once,
// which is how the tests reach the status word without making anything hang.
static int spin_limit()
{
    const char* s = getenv("MOE355_SPIN_LIMIT");
    return s && *s ? atoi(s) : sk::kSpinLimit;
}

bool ggemm_pair_pays(const GemmArgs& rows)
{
    const int wgs = sk::persistent_wgs();
    return wgs >= 8 && pair_pays(rows, wgs);
}

void launch_ggemm_pair_bf16_sk(const GemmArgs& rows_, const GemmArgs& cols_, hipStream_t st)
{
    using namespace sk;
    GemmArgs rows = rows_, cols = cols_;
    rows.spin_limit = cols.spin_limit = spin_limit();
    if (rows.kind == kRowsNT_dGeLU) launch_pair_kind<kRowsNT_dGeLU>(rows, cols, st);
    else launch_pair_kind<kRowsNT>(rows, cols, st);
}

void launch_ggemm_bf16_sk(const GemmArgs& a_, hipStream_t st)
{
    using namespace sk;
    GemmArgs a = a_;
    a.spin_limit = spin_limit();
    switch (a.kind) {
        case kRowsNN_GeLU: launch_kind<kRowsNN_GeLU>(a, st); break;
        case kRowsNN: launch_kind<kRowsNN>(a, st); break;
        case kRowsNT_dGeLU: launch_kind<kRowsNT_dGeLU>(a, st); break;
        case kRowsNT: launch_kind<kRowsNT>(a, st); break;
        default: launch_kind<kColsT>(a, st); break;
    }
}

}  // namespace moe
