// Internal interface of the on-chip segment transform (ltgw_fft.hip) for the
// data preparation.  Not part of the public boundary.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace ltgw {

// Whether segments of n_fft samples have an on-chip transform: the powers of two
// 4096 .. 32768, whose n_fft / 2 complex points a workgroup holds in registers.
// Shorter segments are too small a share of any run to carry a kernel each, longer
// ones don't fit a CU; both, and every other even length, go through hipFFT.
bool chip_fft_has(int32_t n_fft);
size_t chip_fft_table_bytes(int32_t n_fft);
hipError_t launch_chip_fft_tables(int32_t n_fft, float2 *tab, hipStream_t st);
// |windowed transform|^2 of bins k_first .. k_first + n_out - 1 (within 0 .. n_fft / 2)
// of n_seg consecutive segments, rows of n_out.
hipError_t launch_chip_fft(int32_t n_fft, const float *strain, int32_t n_seg, int64_t k_first, int32_t n_out,
                           const float2 *tab, float *power, hipStream_t st);

}  // namespace ltgw
