// Fast sine / cosine transforms of Section 3.3 for power-of-two period
// parameters M = n + 1 (the grids h = 1/64 .. 1/512 of Section 4's tables).
//
// A line's odd (sine) or even (cosine) extension to period 2 M has the transform as
// its DFT of length 2 M.  The first step of that DFT, with s_q = x_q + x_{M-q} and
// d_q = x_q - x_{M-q}, q = 1..M-1, leaves two DFTs of length M:
//   even outputs: of d (sine; S_2j = i/2 D_j), of s (cosine; C_2j = S_j / 2);
//   odd outputs: of s_q exp(-i pi q / M) and of d_q exp(-i pi q / M), the same way,
// with zeros at q = 0 in the sine basis and 2 (x_0 +- x_M) in the cosine basis.  Only
// j <= M / 2 of each is formed in the last stage.  One DFT of s_q sin(pi q / M) + d_q
// would do instead of two, but leaves the odd outputs as running sums over j, which
// gather the rounding errors of all values before: complex128, sine, M = 64 .. 512,
// white noise: 7.0e-16 .. 2.4e-15 relative that way, 1.7e-16 .. 2.1e-16 this way,
// 2.0e-16 .. 5.3e-16 the dense product (on a CPU; complex64 in proportion).
//
// DFT_M by Stockham's autosort algorithm in radix 8 (last stages radix 4 where
// 8 does not divide): M / 8 lanes per line, eight values of each sequence per lane,
// natural order in and out; a stage with Ns values already combined takes butterfly b's
// inputs from b + r M / R, times exp(-2 pi i (b mod Ns) r / (Ns R)), and puts its
// outputs at (b div Ns) Ns R + (b mod Ns) + r Ns.  A line's lanes sit in one
// wave, so the exchanges between stages (LDS, one pad value per eight, both sequences
// through the same buffer) need no workgroup barrier; only the loads and stores of y
// columns, which the whole workgroup shares, do.  Bound by memory, but for the y
// columns of M = 256 and 512, where the registers of two sequences leave four waves per
// SIMD.  Sine, averages of forward and inverse, dense product (slab kernels) -> this:
// 511 x 511 x 512 complex128 x 2773 -> 915 us (4.7 TB/s), y 2782 -> 1074, complex64 1428
// -> 653, 1488 -> 660; 255 x 255 x 256 204 -> 114, 229 -> 131, 135 -> 89, 132 -> 79;
// 127 x 127 x 128 22.7 -> 20.1, 24.1 -> 19.7, 17.5 -> 14.5, 18.5 -> 15.1.
#include "fft16.h"
#include "h6_internal.h"
#include "xform_fft.h"

namespace h6 {
namespace {

using namespace fftdev;

#define T2 typename V2<R>::T

template <typename R> __device__ __forceinline__ T2 tf_tw(const FftTables& t, int i) {
  if constexpr (sizeof(R) == 4) return t.tw_f[i]; else return t.tw[i];
}
template <typename R> __device__ __forceinline__ T2 tf_hw(const FftTables& t, int i) {
  if constexpr (sizeof(R) == 4) return t.hw_f[i]; else return t.hw[i];
}

// forward FFT of length 8 in registers (natural order in and out)
template <typename R> __device__ __forceinline__ void fft8(T2 (&v)[8]) {
  fft4<R, false>(v[0], v[2], v[4], v[6]);
  fft4<R, false>(v[1], v[3], v[5], v[7]);
  const R c = R(0.70710678118654752440);
  // odd half times w8^k: 1, (1 - i) c, -i, (-1 - i) c
  const T2 b0 = v[1], b1 = mk2<R>(c * (v[3].x + v[3].y), c * (v[3].y - v[3].x)), b2 = mk2<R>(v[5].y, -v[5].x),
           b3 = mk2<R>(c * (v[7].y - v[7].x), -c * (v[7].x + v[7].y));
  const T2 a0 = v[0], a1 = v[2], a2 = v[4], a3 = v[6];
  v[0] = add<R>(a0, b0);
  v[4] = sub<R>(a0, b0);
  v[1] = add<R>(a1, b1);
  v[5] = sub<R>(a1, b1);
  v[2] = add<R>(a2, b2);
  v[6] = sub<R>(a2, b2);
  v[3] = add<R>(a3, b3);
  v[7] = sub<R>(a3, b3);
}

__device__ __forceinline__ constexpr int padi(int i) { return i + (i >> 3); }

template <typename R, int M, int RAD, int NS>
__device__ __forceinline__ void stage_out(const T2 (&v)[8], T2* buf, int t) {
  constexpr int T = M / 8, NB = 8 / RAD;      // lanes per line, butterflies per lane
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int b = t + T * u;
    const int o = (b & (NS - 1)) + (b & ~(NS - 1)) * RAD;
#pragma unroll
    for (int r = 0; r < RAD; ++r) buf[padi(o + r * NS)] = v[u * RAD + r];
  }
}

template <typename R, int M, int RAD>
__device__ __forceinline__ void stage_in(T2 (&v)[8], const T2* buf, int t) {
  constexpr int T = M / 8, NB = 8 / RAD;
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int r = 0; r < RAD; ++r) v[u * RAD + r] = buf[padi(t + T * u + r * (M / RAD))];
}

// Keeps the compiler from spreading loads ahead over steps that hold both sequences, so
// that the kernels fit the registers of four waves per SIMD (complex128 sine: 511 x 511 x
// 128 y 324 -> 272 us, 255 x 255 x 256 y 153 -> 130, x 122 -> 111).  Not for complex64
// x lines (255 x 255 x 256 87 against 91).
template <bool TIGHT> __device__ __forceinline__ void in_order() {
  if constexpr (TIGHT) __builtin_amdgcn_sched_barrier(0);
}

// The two sequences from the outputs of a stage of radix RAD0, NS0 values combined before
// it, through the line's buffer (one after the other) to the outputs of the next, of radix
// RAD; they share its factors.
template <typename R, int M, int RAD0, int NS0, int RAD, bool TIGHT>
__device__ __forceinline__ void stage(T2 (&e)[8], T2 (&o)[8], T2* buf, int t, const FftTables& tab) {
  constexpr int T = M / 8, NB = 8 / RAD, NS = NS0 * RAD0;
  T2 w[8];
  auto factors = [&]() {
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
      for (int r = 1; r < RAD; ++r) w[u * RAD + r] = tf_tw<R>(tab, ((t + T * u) & (NS - 1)) * r * (M / (NS * RAD)));
  };
  auto pass = [&](T2 (&v)[8]) {
    wave_sync();
    stage_out<R, M, RAD0, NS0>(v, buf, t);
    wave_sync();
    stage_in<R, M, RAD>(v, buf, t);
  };
  auto combine = [&](T2 (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i % RAD > 0) v[i] = mul<R>(v[i], w[i]);
    if constexpr (RAD == 8) {
      fft8<R>(v);
    } else {
      fft4<R, false>(v[0], v[1], v[2], v[3]);
      fft4<R, false>(v[4], v[5], v[6], v[7]);
    }
  };
  if (!TIGHT) factors();
  pass(e);
  pass(o);
  in_order<TIGHT>();
  if (TIGHT) factors();
  combine(e);
  in_order<TIGHT>();
  combine(o);
}

template <typename R, int AXIS, bool NEU, bool INV, int M, int KL, typename Tin, typename Tout>
__global__ __launch_bounds__(KL * M / 8, sizeof(R) == 8 && AXIS == 1 ? 4 : 1) void fft_kernel(
    const Tin* __restrict__ in, Tout* __restrict__ out, int nlines, int nx, FftTables tab, int acc,
    const int* __restrict__ skip) {
  if (skip && *skip) return;
  constexpr int T = M / 8, L = NEU ? M + 1 : M - 1, OFF = NEU ? 0 : -1;   // array index of node q: q + OFF
  constexpr int NTH = KL * T;
  constexpr bool TIGHT = AXIS == 1 || sizeof(R) == 8;
  constexpr int STR = M + M / 8 + (AXIS == 1 ? 1 : 2);                    // LDS values per line (>= padi(M) + 1)
  __shared__ T2 buf[KL][STR];
  const int tid = threadIdx.x, g = tid / T, t = tid % T;
  T2* line = buf[g];
  int bx = blockIdx.x, by = 0, nl;
  size_t gbase;
  if (AXIS == 0) {
    nl = min(KL, nlines - bx * KL);
    gbase = size_t(bx) * KL * L;
  } else {
    // neighbouring column groups share 128-byte lines: kept on one XCD
    const int nsx = (nx + KL - 1) / KL;
    const int lid = xcd_remap(blockIdx.x, gridDim.x);
    bx = lid % nsx;
    by = lid / nsx;
    nl = min(KL, nx - bx * KL);
    gbase = size_t(by) * nx * L + bx * KL;
  }
  // ---- load: x lines by their own lanes, y columns by the whole workgroup; the sine
  // basis has zeros at the end nodes ----
  if (!NEU && t == 0) line[padi(0)] = line[padi(M)] = mk2<R>(0, 0);
  if (AXIS == 0) {
    constexpr int NP = (L + T - 1) / T;
    if (g < nl) {
      const Tin* src = in + gbase + size_t(g) * L;
      T2 r[NP];
#pragma unroll
      for (int k = 0; k < NP; ++k) r[k] = cv<T2>(src[min(t + k * T, L - 1)]);
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const int p = t + k * T;
        if (p < L) line[padi(p - OFF)] = r[k];
      }
    }
    wave_sync();
  } else {
    constexpr int NP = (KL * L + NTH - 1) / NTH;
    const int c = tid % KL, cc = min(c, nl - 1), q0 = tid / KL;
    T2 r[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) r[k] = cv<T2>(in[gbase + unsigned(min(q0 + k * T, L - 1)) * nx + cc]);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int p = q0 + k * T;
      if (p < L) buf[c][padi(p - OFF)] = r[k];
    }
    __syncthreads();
  }
  // ---- the two sequences at q = t + T r ----
  T2 ev[8], od[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int q = t + T * r;
    const T2 xq = line[padi(q)], xr = line[padi(M - q)];
    const T2 s = add<R>(xq, xr), d = sub<R>(xq, xr), w = tf_hw<R>(tab, q);
    ev[r] = NEU ? s : d;
    od[r] = mul<R>(NEU ? d : s, w);
    if (r == 3) in_order<TIGHT>();
  }
  if (NEU && INV && t == 0) {      // the end nodes enter twice (forward: with half their value)
    ev[0] = scl<R>(ev[0], R(2));
    od[0] = scl<R>(od[0], R(2));
  }
  in_order<TIGHT>();
  fft8<R>(ev);
  in_order<TIGHT>();
  fft8<R>(od);
  in_order<TIGHT>();
  if constexpr (M == 64) {
    stage<R, M, 8, 1, 8, TIGHT>(ev, od, line, t, tab);
  } else if constexpr (M == 128) {
    stage<R, M, 8, 1, 4, TIGHT>(ev, od, line, t, tab);
    stage<R, M, 4, 8, 4, TIGHT>(ev, od, line, t, tab);
  } else if constexpr (M == 256) {
    stage<R, M, 8, 1, 8, TIGHT>(ev, od, line, t, tab);
    stage<R, M, 8, 8, 4, TIGHT>(ev, od, line, t, tab);
  } else {
    stage<R, M, 8, 1, 8, TIGHT>(ev, od, line, t, tab);
    stage<R, M, 8, 8, 8, TIGHT>(ev, od, line, t, tab);
  }
  // ---- outputs m = 2j (ev) and 2j + 1 (od), j < M / 2, to the line in array order: value
  // u RAD + r of the last stage is j = t + T u + r M / RAD ----
  wave_sync();
  constexpr int RAD = M == 64 || M == 512 ? 8 : 4;
  const R fs = INV ? R(0.5) : R(1) / R(M);
#pragma unroll
  for (int u = 0; u < 8 / RAD; ++u)
#pragma unroll
    for (int r = 0; r < RAD / 2; ++r) {
      const int j = t + T * u + r * (M / RAD);
      const T2 a = ev[u * RAD + r], b = od[u * RAD + r];
      if (NEU) {
        line[padi(2 * j)] = scl<R>(a, (!INV && j == 0) ? R(0.5) * fs : fs);
        line[padi(2 * j + 1)] = scl<R>(b, fs);
      } else {                                            // i / 2 times the DFT's
        if (j > 0) line[padi(2 * j - 1)] = mk2<R>(-fs * a.y, fs * a.x);
        line[padi(2 * j)] = mk2<R>(-fs * b.y, fs * b.x);
      }
    }
  if (NEU && t == 0) line[padi(M)] = scl<R>(ev[RAD / 2], INV ? fs : R(0.5) * fs);      // j = M / 2
  // ---- store (coalesced); with acc, out += result ----
  if (AXIS == 0) {
    wave_sync();
    constexpr int NP = (L + T - 1) / T;
    if (g >= nl) return;
    Tout* dst = out + gbase + size_t(g) * L;
    Tout o[NP];
    if (acc) {
#pragma unroll
      for (int k = 0; k < NP; ++k) o[k] = dst[min(t + k * T, L - 1)];
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int p = t + k * T;
      if (p < L) {
        Tout w = cv<Tout>(line[padi(p)]);
        if (acc) {
          w.x += o[k].x;
          w.y += o[k].y;
        }
        dst[p] = w;
      }
    }
  } else {
    __syncthreads();
    constexpr int NP = (KL * L + NTH - 1) / NTH;
    const int c = tid % KL, q0 = tid / KL;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int p = q0 + k * T;
      if (p < L && c < nl) out[gbase + unsigned(p) * nx + c] = cv<Tout>(buf[c][padi(p)]);
    }
  }
}

#undef T2

template <typename R, int AXIS, int M, int KL, typename Tin, typename Tout>
void launch_f(bool neumann, bool inv, const Tin* in, Tout* out, int nlines, int nx, int nz, const FftTables& tab,
              hipStream_t s, int acc, const int* skip) {
  const dim3 grid = AXIS == 0 ? dim3((nlines + KL - 1) / KL) : dim3(unsigned((nx + KL - 1) / KL) * nz);
#define H6_FL(N, I)                                                                                              \
  if (neumann == N && inv == I) {                                                                                \
    hipLaunchKernelGGL((fft_kernel<R, AXIS, N, I, M, KL, Tin, Tout>), grid, dim3(KL * M / 8), 0, s, in, out,      \
                       nlines, nx, tab, acc, skip);                                                              \
    return;                                                                                                      \
  }
  H6_FL(true, true) H6_FL(true, false) H6_FL(false, true) H6_FL(false, false)
#undef H6_FL
}

}  // namespace

template <typename R, typename Tin, typename Tout>
hipError_t launch_fft_x(bool neumann, bool inverse, const Tin* in, Tout* out, int nlines, int L, const FftTables& tab,
                        hipStream_t s, int accumulate, const int* skip) {
  if (L != tab.M + (neumann ? 1 : -1)) return hipErrorInvalidValue;
  switch (tab.M) {
    case 64: launch_f<R, 0, 64, 32>(neumann, inverse, in, out, nlines, 0, 0, tab, s, accumulate, skip); break;
    case 128: launch_f<R, 0, 128, 16>(neumann, inverse, in, out, nlines, 0, 0, tab, s, accumulate, skip); break;
    case 256: launch_f<R, 0, 256, 8>(neumann, inverse, in, out, nlines, 0, 0, tab, s, accumulate, skip); break;
    case 512: launch_f<R, 0, 512, 4>(neumann, inverse, in, out, nlines, 0, 0, tab, s, accumulate, skip); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// columns per workgroup along y: 32 for M = 64, 16 for 128 and 256 (128- and 256-byte row
// segments), 8 for 512, where 16 leave a CU one workgroup (complex64 511 x 511 x 128, sine
// and cosine: 190 + 177 us with 16, 173 + 184 with 8)
template <typename R, typename T>
hipError_t launch_fft_y(bool neumann, bool inverse, const T* in, T* out, int nx, int L, int nz, const FftTables& tab,
                        hipStream_t s, const int* skip) {
  if (L != tab.M + (neumann ? 1 : -1)) return hipErrorInvalidValue;
  switch (tab.M) {
    case 64: launch_f<R, 1, 64, 32>(neumann, inverse, in, out, 0, nx, nz, tab, s, 0, skip); break;
    case 128: launch_f<R, 1, 128, 16>(neumann, inverse, in, out, 0, nx, nz, tab, s, 0, skip); break;
    case 256: launch_f<R, 1, 256, 16>(neumann, inverse, in, out, 0, nx, nz, tab, s, 0, skip); break;
    case 512: launch_f<R, 1, 512, 8>(neumann, inverse, in, out, 0, nx, nz, tab, s, 0, skip); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template hipError_t launch_fft_x<double, double2, double2>(bool, bool, const double2*, double2*, int, int,
                                                           const FftTables&, hipStream_t, int, const int*);
template hipError_t launch_fft_x<float, double2, float2>(bool, bool, const double2*, float2*, int, int,
                                                         const FftTables&, hipStream_t, int, const int*);
template hipError_t launch_fft_x<float, float2, double2>(bool, bool, const float2*, double2*, int, int,
                                                         const FftTables&, hipStream_t, int, const int*);
template hipError_t launch_fft_x<float, float2, float2>(bool, bool, const float2*, float2*, int, int,
                                                        const FftTables&, hipStream_t, int, const int*);
template hipError_t launch_fft_y<double, double2>(bool, bool, const double2*, double2*, int, int, int,
                                                  const FftTables&, hipStream_t, const int*);
template hipError_t launch_fft_y<float, float2>(bool, bool, const float2*, float2*, int, int, int, const FftTables&,
                                                hipStream_t, const int*);

}  // namespace h6
