// Batched GEMV on the matrix cores (batch.hip), called by the C ABI's entry
// point in kernels.hip.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "leech_internal.h"

namespace leech {

// Y[b] = W X[b], b < batch: the checked arguments of leech_gemv_batch.
struct BatchCall {
  const uint8_t* main;
  const DevClass* table;
  const uint16_t* scale;
  const uint16_t* x;      // activation b at x + b · ldx
  float* y;               // output b at y + b · ldy
  float cen0, cen1;
  uint64_t main_bytes;
  int64_t M, nb, ldx, ldy;
  int C, R, batch;
};

int launch_batch_mfma(const BatchCall& c, hipStream_t st);

}  // namespace leech
