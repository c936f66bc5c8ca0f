// Fast transform path for period parameters M = n + 1 = 64, 128, 256 or 512:
// device tables and launchers (see xform_fft.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace h6 {

struct FftTables {
  int M = 0;                       // period parameter (a power of two)
  const double2* tw = nullptr;     // exp(-2 pi i t / M), t = 0..M-1
  const double2* hw = nullptr;     // exp(-pi i q / M), q = 0..M-1
  const float2* tw_f = nullptr;    // the same tables rounded to single precision (complex64 path)
  const float2* hw_f = nullptr;
};

inline bool fft_ok(int M) { return M == 64 || M == 128 || M == 256 || M == 512; }

// Same conventions as launch_rader_x / launch_rader_y (forward: W^{-1},
// inverse: W; accumulate: out += result, x lines with a complex128 output only).
template <typename R, typename Tin, typename Tout>
hipError_t launch_fft_x(bool neumann, bool inverse, const Tin* in, Tout* out, int nlines, int L,
                        const FftTables& tab, hipStream_t s, int accumulate, const int* skip = nullptr);
template <typename R, typename T>
hipError_t launch_fft_y(bool neumann, bool inverse, const T* in, T* out, int nx, int L, int nz,
                        const FftTables& tab, hipStream_t s, const int* skip = nullptr);

}  // namespace h6
