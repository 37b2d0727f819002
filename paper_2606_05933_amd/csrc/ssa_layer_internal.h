// What ssa_layer_forward uses of the dense kernels beyond include/ssa_layer.h.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace ssa {

// Split tickets at the start of a linear workspace.
constexpr size_t kLinearTicketBytes = 256;

// Two runs of words to set to zero (n[i] = 0: none).
struct ClearWords {
  uint32_t* at[2];
  int64_t n[2];
};

// ssa_rms_norm whose launch also clears words; the buffers must not overlap.
int rms_norm(int32_t m, int32_t n, const uint16_t* x, const uint16_t* weight, float eps,
             uint16_t* out, const ClearWords& clear, void* stream);

}  // namespace ssa
