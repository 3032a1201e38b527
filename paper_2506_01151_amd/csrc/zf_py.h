// What the two extension modules of the Python binding share: the calls that need to look into tensors, handed over by _native_torch.
#pragma once
#include <cstdint>

namespace zfpy {

struct TensorInfo {
    void *data;
    int64_t size[2], stride[2];
    int32_t dim, device;          // device: ordinal of the GPU, -1 = not on one
    int32_t dtype;                // 0 = fp32, 1 = bf16, 2 = int32, -1 = another
    int32_t contiguous;
};
struct TensorCalls {
    bool (*look)(void *obj, TensorInfo *out) noexcept;      // false: not a plain torch.Tensor, or one that cannot be looked at
    bool (*stream)(int32_t device, void **out) noexcept;    // torch's current stream there; false: torch has none to give
};
static const char *const TENSOR_CALLS_NAME = "paper_2506_01151_amd._native_torch.calls";

}  // namespace zfpy
