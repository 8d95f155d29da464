"""Every kernel that asks for more dynamic LDS than the default has its own limit raised, once per device: instances of one kernel
template have one type, and a limit raised for the first says nothing about the others.  (The header is compiled for the host,
with the HIP calls replaced by ones that keep a record.)"""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cassert>
#include <vector>
#include "dynamic_lds.h"

struct Raised { const void* kernel; int device, bytes; };
static std::vector<Raised> raised;
static int device = 0;
static bool refuse = false;
static int failures = 0;
extern "C" hipError_t hipFuncSetAttribute(const void* kernel, hipFuncAttribute, int bytes)
{
    if (refuse) return hipErrorInvalidValue;
    raised.push_back({kernel, device, bytes});
    return hipSuccess;
}
extern "C" const char* hipGetErrorString(hipError_t) { return "refused"; }
namespace moe {
int current_device() { return device; }
void fail_launch(const char*, ...) { ++failures; }
}
template <int I> void kernel(int* p) { *p = I; }

int main()
{
    using moe::allow_dynamic_lds;
    assert(allow_dynamic_lds<kernel<1>>(1000) && allow_dynamic_lds<kernel<2>>(2000));
    assert(raised.size() == 2 && raised[0].kernel == (const void*)kernel<1> && raised[1].kernel == (const void*)kernel<2>);
    assert(raised[0].bytes == 1000 && raised[1].bytes == 2000);
    assert(allow_dynamic_lds<kernel<1>>(1000) && raised.size() == 2);                 // once is enough
    assert(allow_dynamic_lds<kernel<1>>(1500) && raised.size() == 3);                 // more than it has
    device = 3;
    assert(allow_dynamic_lds<kernel<1>>(1000) && raised.size() == 4 && raised[3].device == 3);
    refuse = true;
    assert(!allow_dynamic_lds<kernel<3>>(1000) && failures == 1);
    refuse = false;
    assert(allow_dynamic_lds<kernel<3>>(1000) && raised.size() == 5);                 // a refusal is not remembered
    device = -1;
    assert(!allow_dynamic_lds<kernel<1>>(1000));
    return 0;
}
"""


def test_the_limit_is_raised_for_every_kernel(tmp_path):
    source, program = tmp_path / "limits.cpp", tmp_path / "limits"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++20", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "paper_2103_13262_amd", "csrc"),
                    str(source), "-o", str(program), "-pthread"], check=True)
    subprocess.run([str(program)], check=True)
