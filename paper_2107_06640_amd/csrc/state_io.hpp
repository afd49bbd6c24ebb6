// DOFs between the caller's array [E][B][9] (FP64, the caller's element order)
// and the device's tiled state, for checkpoints and initial states.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace seis {

// Pinned staging of one handle, allocated at its first transfer and kept.
struct StateIO {
  const int32_t* at = nullptr;  // [E] device: position of the caller's element
  double* pin = nullptr;
  int64_t pin_values = 0;
};

void state_io_free(StateIO& io);

// B rows of nine quantities for E elements; synchronous. The caller's host threads share the copies.
template <typename T>
hipError_t state_write(StateIO& io, T* Q, const double* dofs, int64_t E, int B, hipStream_t s);
template <typename T>
hipError_t state_read(StateIO& io, const T* Q, double* dofs, int64_t E, int B, hipStream_t s);

}  // namespace seis
