// The order pass of the list evaluation as a kernel of its own (rows.h says what it does).
#include "rows.h"

namespace fpsched {

template <int VBITS, bool NO_W, bool SHARED>
__global__ __launch_bounds__(kCheckMaxThreads) __attribute__((amdgpu_waves_per_eu(kCheckWavesPerSimd, kCheckWavesPerSimd))) void check_rows_kernel(
    ListTables T, const uint16_t* __restrict__ ops, long long n_rows, int stride, int rows_per_wave, long long* __restrict__ out_info,
    int* __restrict__ out_peak, unsigned long long* __restrict__ counter, unsigned long long counter_value, int draw_blocks, int dynamic) {
  check_rows<VBITS, NO_W, SHARED>(T, ops, n_rows, stride, rows_per_wave, out_info, out_peak, counter, counter_value, draw_blocks, dynamic, (int)blockDim.x);
}

#define FPSCHED_INSTANTIATE(VBITS, NO_W, SHARED) \
  template __global__ void check_rows_kernel<VBITS, NO_W, SHARED>(ListTables, const uint16_t*, long long, int, int, long long*, int*, unsigned long long*, unsigned long long, int, int);
#define FPSCHED_INSTANTIATE_LOADS(SHARED) \
  FPSCHED_INSTANTIATE(0, false, SHARED)   \
  FPSCHED_INSTANTIATE(1, false, SHARED)   \
  FPSCHED_INSTANTIATE(2, false, SHARED)   \
  FPSCHED_INSTANTIATE(0, true, SHARED)    \
  FPSCHED_INSTANTIATE(1, true, SHARED)    \
  FPSCHED_INSTANTIATE(2, true, SHARED)
FPSCHED_INSTANTIATE_LOADS(false)
FPSCHED_INSTANTIATE_LOADS(true)
#undef FPSCHED_INSTANTIATE_LOADS
#undef FPSCHED_INSTANTIATE

}  // namespace fpsched
