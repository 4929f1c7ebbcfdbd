// The prompt kernel's copies of the activations for the ring of workspaces: one pair per slot, so that calls that do not
// share a slot do not share copies either.  A file (a code object) of its own: a process that sends no prompts never loads it.
#include "xfp_internal.h"

#include <atomic>

namespace xfp {

namespace {

__device__ __align__(256) unsigned char g_prompt[kRingSlots][sizeof(PromptCopies)];
std::atomic<void *> g_base[kMaxDevices];           // its device address, per device

}  // namespace

hipError_t prompt_copies_ring(int slot, PromptCopies **out)
{
    const int dev = current_device();
    if (dev < 0) return hipErrorInvalidDevice;
    void *p = g_base[dev].load(std::memory_order_acquire);
    if (!p) {
        hipError_t err = hipGetSymbolAddress(&p, HIP_SYMBOL(g_prompt));
        if (err != hipSuccess) return err;
        g_base[dev].store(p, std::memory_order_release);
    }
    *out = static_cast<PromptCopies *>(p) + slot;
    return hipSuccess;
}

}  // namespace xfp
