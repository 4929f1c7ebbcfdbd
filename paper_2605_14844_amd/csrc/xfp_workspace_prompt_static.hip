// The prompt kernel's copies of the activations for xfp_gemv_noalloc, beside its one static array; loaded with its first prompt.
#include "xfp_internal.h"

#include <atomic>

namespace xfp {

namespace {

__device__ __align__(256) unsigned char g_prompt_static[sizeof(PromptCopies)];
std::atomic<void *> g_base[kMaxDevices];           // its device address, per device

}  // namespace

hipError_t prompt_copies_static(PromptCopies **out)
{
    const int dev = current_device();
    if (dev < 0) return hipErrorInvalidDevice;
    void *p = g_base[dev].load(std::memory_order_acquire);
    if (!p) {
        hipError_t err = hipGetSymbolAddress(&p, HIP_SYMBOL(g_prompt_static));
        if (err != hipSuccess) return err;
        g_base[dev].store(p, std::memory_order_release);
    }
    *out = static_cast<PromptCopies *>(p);
    return hipSuccess;
}

}  // namespace xfp
