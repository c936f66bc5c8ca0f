// Fast sine / cosine transforms of Section 3.3 for power-of-two period
// parameters M = n + 1 (the grids h = 1/64 .. 1/512 of Section 4's tables).
//
// The reduction to one complex DFT of length M per line is the one of
// xform_rader.hip (it holds for every M): with s_q = x_q + x_{M-q} and
// d_q = x_q - x_{M-q}, y_q = s_q sin(pi q / M) + d_q (sine basis) or
// y_q = s_q + d_q sin(pi q / M) (cosine basis), q = 1..M-1, y_0 = 0,
// Y = DFT_M(y), the even outputs from Y_j +- Y_{M-j} and the odd ones from a
// running sum of them.
//
// DFT_M by Stockham's autosort algorithm in radix 8 (last stages radix 4 where
// 8 does not divide): M / 8 lanes per line, eight values each, natural order in
// and out; a stage with Ns values already combined takes butterfly b's inputs
// from b + r M / R, times exp(-2 pi i (b mod Ns) r / (Ns R)), and puts its
// outputs at (b div Ns) Ns R + (b mod Ns) + r Ns.  A line's lanes sit in one
// wave, so the exchanges between stages (LDS, one pad value per eight) need no
// workgroup barrier; only the loads and stores of y columns, which the whole
// workgroup shares, do.  Eight values per lane keep the registers low enough
// for the loads of other waves to hide behind these: the passes are bound by
// memory.  Against the dense product of the slab kernels (averages of forward
// and inverse): 511 x 511 x 512 complex128 x 2785 -> 843 us (5.1 TB/s), y 2805 ->
// 1025; 255 x 255 x 256 complex128 x 199 -> 112, y 230 -> 129, complex64 131 -> 84,
// 132 -> 72; 127^3 complex64 17.8 -> 14.6, 18.8 -> 14.6; 63^3 9.6 -> 6.9, 9.7 -> 7.7.
// Errors against 64 bits are the dense product's within 2 %.
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
template <typename R> __device__ __forceinline__ R tf_sin(const FftTables& t, int i) {
  if constexpr (sizeof(R) == 4) return t.sin_f[i]; else return t.sin_q[i];
}
template <typename R> __device__ __forceinline__ R tf_cos(const FftTables& t, int i) {
  if constexpr (sizeof(R) == 4) return t.cos_f[i]; else return t.cos_q[i];
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
__device__ __forceinline__ void stage_in(T2 (&v)[8], const T2* buf, int t, const FftTables& tab) {
  constexpr int T = M / 8, NB = 8 / RAD;      // lanes per line, butterflies per lane
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int b = t + T * u, k = b & (NS - 1);
#pragma unroll
    for (int r = 0; r < RAD; ++r) {
      T2 x = buf[padi(b + r * (M / RAD))];
      if (r > 0) x = mul<R>(x, tf_tw<R>(tab, k * r * (M / (NS * RAD))));
      v[u * RAD + r] = x;
    }
  }
}
template <typename R, int M, int RAD, int NS>
__device__ __forceinline__ void stage_out(const T2 (&v)[8], T2* buf, int t) {
  constexpr int T = M / 8, NB = 8 / RAD;
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int b = t + T * u;
    const int o = (b & (NS - 1)) + (b & ~(NS - 1)) * RAD;
#pragma unroll
    for (int r = 0; r < RAD; ++r) buf[padi(o + r * NS)] = v[u * RAD + r];
  }
}
template <typename R, int M, int RAD, int NS>
__device__ __forceinline__ void stage(T2 (&v)[8], T2* buf, int t, const FftTables& tab) {
  stage_in<R, M, RAD, NS>(v, buf, t, tab);
  if constexpr (RAD == 8) {
    fft8<R>(v);
  } else {
    fft4<R, false>(v[0], v[1], v[2], v[3]);
    fft4<R, false>(v[4], v[5], v[6], v[7]);
  }
  wave_sync();
  stage_out<R, M, RAD, NS>(v, buf, t);
  wave_sync();
}

template <typename R, int AXIS, bool NEU, bool INV, int M, int KL, typename Tin, typename Tout>
__global__ __launch_bounds__(KL * M / 8) void fft_kernel(const Tin* __restrict__ in, Tout* __restrict__ out,
                                                         int nlines, int nx, FftTables tab, int acc,
                                                         const int* __restrict__ skip) {
  if (skip && *skip) return;
  constexpr int T = M / 8, L = NEU ? M + 1 : M - 1, OFF = NEU ? 0 : -1;   // array index of node q: q + OFF
  constexpr int NTH = KL * T;
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
  // ---- load: x lines by their own lanes, y columns by the whole workgroup ----
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
  // ---- y_q for q = t + T r, first stage in registers ----
  T2 v[8];
  T2 c1sum = mk2<R>(0, 0), xa = mk2<R>(0, 0), xb = mk2<R>(0, 0);
  if (NEU) {
    xa = line[padi(0)];
    xb = line[padi(M)];
    if (!INV) {
      xa = scl<R>(xa, R(0.5));
      xb = scl<R>(xb, R(0.5));
    }
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int q = t + T * r;
    const bool ok = r > 0 || t > 0;
    const T2 xq = line[padi(ok ? q : 1)], xr = line[padi(ok ? M - q : 1)];
    const T2 s = add<R>(xq, xr), d = sub<R>(xq, xr);
    const R sn = tf_sin<R>(tab, q);
    T2 y;
    if (NEU) {
      y = add<R>(s, scl<R>(d, sn));
      c1sum = add<R>(c1sum, scl<R>(d, R(0.5) * tf_cos<R>(tab, q)));      // q = 0: d = 0
    } else {
      y = add<R>(scl<R>(s, sn), d);
    }
    v[r] = ok ? y : mk2<R>(0, 0);
  }
  if (NEU) {
#pragma unroll
    for (int o = T / 2; o > 0; o >>= 1) {
      c1sum.x += __shfl_xor(c1sum.x, o, T);
      c1sum.y += __shfl_xor(c1sum.y, o, T);
    }
  }
  fft8<R>(v);
  wave_sync();
  stage_out<R, M, 8, 1>(v, line, t);
  wave_sync();
  if constexpr (M == 64) {
    stage<R, M, 8, 8>(v, line, t, tab);
  } else if constexpr (M == 128) {
    stage<R, M, 4, 8>(v, line, t, tab);
    stage<R, M, 4, 32>(v, line, t, tab);
  } else if constexpr (M == 256) {
    stage<R, M, 8, 8>(v, line, t, tab);
    stage<R, M, 4, 64>(v, line, t, tab);
  } else {
    stage<R, M, 8, 8>(v, line, t, tab);
    stage<R, M, 8, 64>(v, line, t, tab);
  }
  // ---- post-processing: lane t takes j = 4t .. 4t + 3 (and j = M / 2 for C_M);
  // the odd outputs need running sums over j ----
  T2 ev[4], od[4];
  const T2 Y0 = line[padi(0)];
  T2 loc = mk2<R>(0, 0);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = 4 * t + u;
    const T2 Yj = line[padi(j)], Ym = line[padi(j == 0 ? 0 : M - j)];
    T2 inc = NEU ? scl<R>(sub<R>(Yj, Ym), R(0.5)) : scl<R>(add<R>(Yj, Ym), R(0.5));
    if (j == 0) inc = mk2<R>(0, 0);
    loc = add<R>(loc, inc);
    od[u] = loc;
    if (NEU) {
      const T2 A = scl<R>(add<R>(Yj, Ym), R(0.25));
      ev[u] = add<R>(add<R>(xa, xb), A);                          // C_{2j}
    } else {
      const T2 D = sub<R>(Yj, Ym);
      ev[u] = mk2<R>(-R(0.25) * D.y, R(0.25) * D.x);              // S_{2j}
    }
  }
  T2 last = mk2<R>(0, 0);
  if (NEU) last = add<R>(add<R>(xa, xb), scl<R>(line[padi(M / 2)], R(0.5)));   // C_M
  T2 sc = loc;
#pragma unroll
  for (int o = 1; o < T; o <<= 1) {
    const R px = __shfl_up(sc.x, o, T), py = __shfl_up(sc.y, o, T);
    if (t >= o) {
      sc.x += px;
      sc.y += py;
    }
  }
  const T2 before = sub<R>(sc, loc);                              // sum over the lanes before t
  wave_sync();
  // scaled outputs in array order over the line
  const R fs = INV ? R(1) : R(2) / R(M);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = 4 * t + u;
    const T2 run = add<R>(before, od[u]);
    if (NEU) {
      const T2 o = add<R>(sub<R>(xa, xb), add<R>(c1sum, mk2<R>(run.y, -run.x)));      // C_{2j+1}
      line[padi(2 * j)] = scl<R>(ev[u], (!INV && j == 0) ? R(0.5) * fs : fs);
      line[padi(2 * j + 1)] = scl<R>(o, fs);
    } else {
      const T2 o = add<R>(scl<R>(Y0, R(0.5)), run);                                    // S_{2j+1}
      if (j > 0) line[padi(2 * j - 1)] = scl<R>(ev[u], fs);
      line[padi(2 * j)] = scl<R>(o, fs);
    }
  }
  if (NEU && t == 0) line[padi(M)] = scl<R>(last, INV ? fs : R(0.5) * fs);
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

// columns per workgroup along y: 16 (128- and 256-byte row segments), 32 for
// M = 64; at M = 512 complex128 columns take 8 (36 KB of LDS per 4 lines: 16
// would leave one workgroup per CU, 1230 against 1025 us at 511 x 511 x 512;
// complex64 573 against 613 us the other way round)
template <typename R, typename T>
hipError_t launch_fft_y(bool neumann, bool inverse, const T* in, T* out, int nx, int L, int nz, const FftTables& tab,
                        hipStream_t s, const int* skip) {
  if (L != tab.M + (neumann ? 1 : -1)) return hipErrorInvalidValue;
  switch (tab.M) {
    case 64: launch_f<R, 1, 64, 32>(neumann, inverse, in, out, 0, nx, nz, tab, s, 0, skip); break;
    case 128: launch_f<R, 1, 128, 16>(neumann, inverse, in, out, 0, nx, nz, tab, s, 0, skip); break;
    case 256: launch_f<R, 1, 256, 16>(neumann, inverse, in, out, 0, nx, nz, tab, s, 0, skip); break;
    case 512: launch_f<R, 1, 512, (sizeof(R) == 4 ? 16 : 8)>(neumann, inverse, in, out, 0, nx, nz, tab, s, 0, skip); break;
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
