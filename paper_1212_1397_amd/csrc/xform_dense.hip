// Sine / cosine transforms of Section 3.3 as dense products on the matrix
// cores, for the axes the FFT paths do not take.  Along an axis with L
// unknowns the transform of each line is out_m = sum_q W[m][q] in_q with the
// L x L basis matrix W of the plan (scale factors folded in).
//
// Every such W (inverse and forward, sine and cosine basis) is even or odd
// under the reflection of the nodes q -> M - q, i.e. of the array index
// q -> L - 1 - q: W[m][L-1-q] = (-1)^m W[m][q].  So with H = ceil(L / 2),
// h = floor(L / 2), u_p = x_p + x_{L-1-p}, v_p = x_p - x_{L-1-p} (p < h) and
// u_h = x_h for odd L (the middle node),
//   out_{2j}   = sum_{p < H} We[j][p] u_p,   We[j][p] = W[2j][p],
//   out_{2j+1} = sum_{p < h} Wo[j][p] v_p,   Wo[j][p] = W[2j+1][p]:
// two half-size products, half the matrix-core work of the L x L one.  A pass
// is one GEMM pair per z-plane (y) or per block of lines (x):
//   y: C[m][c] = sum_q W[m][q] X[q][c],   X = the plane as L x 2n'x reals
//      (row q = y index; real and imaginary parts of each x are columns);
//   x: C[r][m] = sum_q X[r][q] W[m][q],   rows r = (line, real or imaginary part).
// Complex data times a real matrix needs no extra flops.  One MFMA tile is
// 16 x 16 with K = 4 (v_mfma_f32_16x16x4f32 in complex64 plans,
// v_mfma_f64_16x16x4f64 in complex128 ones).  A workgroup of 4 waves owns the
// 64 consecutive outputs m = 64 b .. 64 b + 63 (32 even and 32 odd ones, j =
// 32 b .. 32 b + 31) of 32 lines (x) or 64 columns (y), folding the line
// halves into u and v as it stages K chunks in LDS.  We and Wo are stored
// zero-padded to [Hm][Hk] (Hm a multiple of 32, Hk of the K chunk), so
// operand reads of them need no bounds checks.  (These K-chunked kernels take the
// lines too long for the slab kernels below, long lines that are few and short x
// lines, see slab_shape.)
#include <algorithm>

#include "h6_internal.h"

namespace h6 {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// MFMA 16x16x4: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and
// receives D[row(l, e)][l % 16], e = 0..3 (layouts checked on gfx950).
template <typename R> struct Mma;
template <> struct Mma<float> {
  using V = f32x4;
  static __device__ __forceinline__ V mma(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int l, int e) { return 4 * (l >> 4) + e; }
  // x pass: row of (line li of the 16-row tile, part c) so that each lane's
  // four outputs are two whole complex values (lines 2g, 2g + 1)
  static __device__ __forceinline__ int xrow(int li, int c) { return 2 * li + c; }
};
template <> struct Mma<double> {
  using V = f64x4;
  static __device__ __forceinline__ V mma(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int l, int e) { return 4 * e + (l >> 4); }
  // lines g and g + 4 (re in rows 0..7, im in rows 8..15)
  static __device__ __forceinline__ int xrow(int li, int c) { return li + 8 * c; }
};

constexpr int kT = 64;       // output tile edge
constexpr int kKC = kDenseKChunk;                  // K chunk staged per step
constexpr int kXL = (kT / 2) * kKC / 256;          // (line, p) values of a chunk per thread (x)
constexpr int kWL = kT * kKC / 256;                // W values of a chunk per thread
constexpr int kYL = kKC * kT / 256;                // (p, column) values of a chunk per thread (y)
static_assert(kWL == kYL, "the y kernel stages W and data in one loop");
constexpr int kPad = kKC + 1;

template <typename R, typename Tin, typename Tout>
__global__ __launch_bounds__(256) void dense_x_kernel(const Tin* __restrict__ in, Tout* __restrict__ out,
                                                      const R* __restrict__ W, int Hm, int Hk, int L, int nlines,
                                                      int acc, const int* __restrict__ skip) {
  if (skip && *skip) return;
  using M = Mma<R>;
  __shared__ R Au[kT][kPad];   // rows (line, part) of 32 lines, K chunk of u
  __shared__ R Av[kT][kPad];   // the same rows, K chunk of v
  __shared__ R Ws[kT][kPad];   // rows j of We (0..31), then of Wo (32..63), K chunk
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int j0 = blockIdx.x * (kT / 2), line0 = blockIdx.y * (kT / 2);
  const int h = L >> 1, H = L - h;
  typename M::V acc4[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc4[t] = typename M::V{0, 0, 0, 0};
  // accumulator tile t: even outputs (t < 2) or odd ones, j = j0 + 16 (t & 1) ..;
  // tiles 1 and 3 idle when j0 + 16 is past the last j
  const bool upper = j0 + 16 < H;
  // staging of one K chunk in registers: 32 lines x 16 p of u and v (two
  // coalesced reads per value, one ascending and one descending along the
  // line) and 64 rows x 16 p of We / Wo (padded: always in bounds); the next
  // chunk's loads are issued before the current chunk's MFMAs
  R ure[kXL], uim[kXL], vre[kXL], vim[kXL], wv4[kWL];
  auto load = [&](int p0) {
#pragma unroll
    for (int j = 0; j < kXL; ++j) {
      const int i = tid + 256 * j;
      const int ll = i / kKC, pp = i % kKC;
      const int line = line0 + ll, p = p0 + pp;
      ure[j] = 0;
      uim[j] = 0;
      vre[j] = 0;
      vim[j] = 0;
      if (line < nlines && p < H) {
        const Tin a = in[size_t(line) * L + p];
        if (p < h) {
          const Tin b = in[size_t(line) * L + (L - 1 - p)];
          ure[j] = R(a.x) + R(b.x);
          uim[j] = R(a.y) + R(b.y);
          vre[j] = R(a.x) - R(b.x);
          vim[j] = R(a.y) - R(b.y);
        } else {
          ure[j] = R(a.x);
          uim[j] = R(a.y);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kWL; ++j) {
      const int i = tid + 256 * j;
      const int r = i / kKC;
      wv4[j] = W[(size_t(r >> 5) * Hm + j0 + (r & 31)) * Hk + p0 + i % kKC];
    }
  };
  load(0);
  for (int p0 = 0; p0 < H; p0 += kKC) {
#pragma unroll
    for (int j = 0; j < kXL; ++j) {
      const int i = tid + 256 * j;
      const int ll = i / kKC, pp = i % kKC;
      const int wv = ll >> 3, li = ll & 7;
      Au[16 * wv + M::xrow(li, 0)][pp] = ure[j];
      Au[16 * wv + M::xrow(li, 1)][pp] = uim[j];
      Av[16 * wv + M::xrow(li, 0)][pp] = vre[j];
      Av[16 * wv + M::xrow(li, 1)][pp] = vim[j];
    }
#pragma unroll
    for (int j = 0; j < kWL; ++j) {
      const int i = tid + 256 * j;
      Ws[i / kKC][i % kKC] = wv4[j];
    }
    __syncthreads();
    if (p0 + kKC < H) load(p0 + kKC);
    if (upper) {
#pragma unroll
      for (int kk = 0; kk < kKC / 4; ++kk) {
        const R au = Au[16 * w + (lane & 15)][4 * kk + (lane >> 4)];
        const R av = Av[16 * w + (lane & 15)][4 * kk + (lane >> 4)];
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc4[t] = M::mma(t < 2 ? au : av, Ws[16 * t + (lane & 15)][4 * kk + (lane >> 4)], acc4[t]);
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < kKC / 4; ++kk) {
        const R au = Au[16 * w + (lane & 15)][4 * kk + (lane >> 4)];
        const R av = Av[16 * w + (lane & 15)][4 * kk + (lane >> 4)];
        acc4[0] = M::mma(au, Ws[(lane & 15)][4 * kk + (lane >> 4)], acc4[0]);
        acc4[2] = M::mma(av, Ws[32 + (lane & 15)][4 * kk + (lane >> 4)], acc4[2]);
      }
    }
    __syncthreads();
  }
  // lane holds lines (la, lb) of its wave's 8, both parts, for output m
  const int g = lane >> 4;
  const int la = sizeof(R) == 4 ? 2 * g : g, lb = sizeof(R) == 4 ? 2 * g + 1 : g + 4;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int m = 2 * (j0 + 16 * (t & 1) + (lane & 15)) + (t >> 1);
    if (m >= L) continue;
    const typename M::V v = acc4[t];
    const R ra = v[0], ia = sizeof(R) == 4 ? v[1] : v[2];
    const R rb = sizeof(R) == 4 ? v[2] : v[1], ib = v[3];
    const int lines[2] = {line0 + 8 * w + la, line0 + 8 * w + lb};
    const R res[2][2] = {{ra, ia}, {rb, ib}};
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      if (lines[hh] >= nlines) continue;
      const size_t o = size_t(lines[hh]) * L + m;
      Tout u;
      if (acc) {
        u = out[o];
        u.x += res[hh][0];
        u.y += res[hh][1];
      } else {
        u.x = res[hh][0];
        u.y = res[hh][1];
      }
      out[o] = u;
    }
  }
}

template <typename R>
__global__ __launch_bounds__(256) void dense_y_kernel(const R* __restrict__ in, R* __restrict__ out,
                                                      const R* __restrict__ W, int Hm, int Hk, int L, int ncols,
                                                      const int* __restrict__ skip) {
  if (skip && *skip) return;
  using M = Mma<R>;
  __shared__ R Ws[kT][kPad];          // rows j of We (0..31), then of Wo (32..63), K chunk
  __shared__ R Us[kKC][kT + 1];       // K chunk of u, columns
  __shared__ R Vs[kKC][kT + 1];       // K chunk of v, columns
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int c0 = blockIdx.x * kT, j0 = blockIdx.y * (kT / 2);
  const int h = L >> 1, H = L - h;
  const size_t plane = size_t(L) * ncols;
  const R* __restrict__ X = in + blockIdx.z * plane;
  typename M::V acc4[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc4[t] = typename M::V{0, 0, 0, 0};
  // waves 0, 1: even outputs j0 + 16 w ..; waves 2, 3: odd outputs j0 + 16 (w - 2) ..
  const bool odd = w >= 2;
  const bool busy = j0 + 16 * (w & 1) < (odd ? h : H);
  // one K chunk in registers (64 rows x 16 p of We / Wo, 16 rows x 64 columns
  // of u and v from two coalesced plane rows each); the next chunk is loaded
  // during the MFMAs
  R wv4[kWL], uv4[kYL], vv4[kYL];
  auto load = [&](int p0) {
#pragma unroll
    for (int j = 0; j < kWL; ++j) {
      const int i = tid + 256 * j;
      const int r = i / kKC;
      wv4[j] = W[(size_t(r >> 5) * Hm + j0 + (r & 31)) * Hk + p0 + i % kKC];
      const int p = p0 + i / kT, c = c0 + i % kT;
      uv4[j] = 0;
      vv4[j] = 0;
      if (p < H && c < ncols) {
        const R a = X[size_t(p) * ncols + c];
        if (p < h) {
          const R b = X[size_t(L - 1 - p) * ncols + c];
          uv4[j] = a + b;
          vv4[j] = a - b;
        } else {
          uv4[j] = a;
        }
      }
    }
  };
  load(0);
  for (int p0 = 0; p0 < H; p0 += kKC) {
#pragma unroll
    for (int j = 0; j < kWL; ++j) {
      const int i = tid + 256 * j;
      Ws[i / kKC][i % kKC] = wv4[j];
      Us[i / kT][i % kT] = uv4[j];
      Vs[i / kT][i % kT] = vv4[j];
    }
    __syncthreads();
    if (p0 + kKC < H) load(p0 + kKC);
    if (busy) {
      const R(*B)[kT + 1] = odd ? Vs : Us;
#pragma unroll
      for (int kk = 0; kk < kKC / 4; ++kk) {
        const R a = Ws[16 * w + (lane & 15)][4 * kk + (lane >> 4)];
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc4[t] = M::mma(a, B[4 * kk + (lane >> 4)][16 * t + (lane & 15)], acc4[t]);
      }
    }
    __syncthreads();
  }
  if (!busy) return;
  R* __restrict__ Y = out + blockIdx.z * plane;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int c = c0 + 16 * t + (lane & 15);
    if (c >= ncols) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = 2 * (j0 + 16 * (w & 1) + M::row(lane, e)) + (odd ? 1 : 0);
      if (m < L) Y[size_t(m) * ncols + c] = acc4[t][e];
    }
  }
}

// ---- slab kernels -----------------------------------------------------------
// A workgroup holds a slab of whole lines in LDS, folded once into u and v, and
// forms every output of them, so each input is read from memory once and only
// the (L2-resident) basis matrices are read by every workgroup.  The K-chunked
// kernels above re-read the input once per 64 outputs and stop at two barriers
// per 16 values of K, which left them waiting on latency.
//
// The slab is 32 rows of K values (row = one real sequence: a column of the
// plane along y, one part of one line along x), K contiguous, so the data
// operand of four (complex64) or two (complex128) successive MFMAs is one
// 16-byte LDS read per lane, and the matrix operand one 16-byte global read:
// lane group g = lane / 16 takes k = 4 KV ch + KV g + e as its K index of step
// e of chunk ch (KV = 16 / sizeof(R); any assignment of k to slots is right as
// long as both operands agree).  The K remainder takes steps of four.  Rows are
// an odd number of 16-byte pieces apart: no bank conflicts.  A wave's unit is
// 16 outputs j of both parities for both 16-row tiles; 4 to 8 waves, as many as
// share the units evenly.  Where H = 16 a + 1 or + 2 (Neumann pairs of even n)
// the last one or two rows j are plain dot products on the vector units
// (border) instead of one more padded tile.
// 32 rows measured best of 16, 32 and 64 from 48^3 to 255^3 in both precisions
// (64 rows leave one or two workgroups per CU, 16 read the matrices twice as
// often).  Whole passes, average of forward and inverse, K-chunked kernels ->
// slab: 160^3 complex64 x 47.8 -> 30.9 us, y 51.6 -> 32.5; 200^3 complex64 115
// -> 67, 116 -> 63; 160 x 99 x 202 complex128 x 49.8 -> 42.9, y 48.5 -> 35.8;
// 257 columns complex64 y 274 -> 145.  Of that last figure 77 us are the
// products (54 at the matrix cores' rate) and the rest the loads and stores,
// which a workgroup does not overlap with its own products; co-resident
// workgroups run in step, so little of it is hidden.
template <typename R> struct Vec16;
template <> struct Vec16<float> { using T = float4; };
template <> struct Vec16<double> { using T = double2; };
template <typename R> struct alignas(2 * sizeof(R)) Cplx { R x, y; };

template <typename R> __device__ __forceinline__ R vget(const typename Vec16<R>::T& v, int e) {
  return reinterpret_cast<const R*>(&v)[e];
}

// stride between slab rows (values): H in whole groups of four, odd in 16-byte pieces
template <typename R> __host__ __device__ constexpr int slab_stride(int H) {
  constexpr int KV = 16 / int(sizeof(R));
  return ((H + 3) / 4 * 4 / KV | 1) * KV;
}
// rows of the matrix left to the vector units
__host__ __device__ constexpr int slab_border(int H) { return H > 16 && H % 16 <= 2 ? H % 16 : 0; }
// stride between output lines staged in LDS by the x pass (complex values): odd in 16-byte pieces
template <typename R> __host__ __device__ constexpr int slab_out_stride(int L) {
  return sizeof(R) == 4 ? 2 * ((L + 1) / 2 | 1) : (L | 1);
}

// D row r of a 16 x 16 tile -> position p so that lane group g's four D values
// sit at positions 4 g .. 4 g + 3 (rows 4 g + e in FP32, 4 e + g in FP64)
constexpr int kSlabTiles = 2, kSlabRows = 16 * kSlabTiles, kSlabLines = kSlabRows / 2;

template <typename R> __device__ __forceinline__ int tile_pos(int r) {
  return sizeof(R) == 4 ? r : 4 * (r & 3) + (r >> 2);
}

// ae / ao += products of one unit over all of K.  WA: the matrix is the A operand
// (D rows = outputs, x pass), else the B operand (D columns = outputs, y pass).
// du: this lane's row of each row tile (values from U); V = U + vofs.  Two chunks
// are in flight: the matrix values of chunk ch + 2 are requested as those of ch
// are used up, the slab values of ch + 1 before the products of ch.
template <typename R, bool WA, bool ODD>
__device__ __forceinline__ void slab_product(const R* __restrict__ We, const R* __restrict__ Wo, unsigned wofs,
                                             const R* U, int vofs, const int (&du)[kSlabTiles], int H, int g,
                                             typename Mma<R>::V (&ae)[kSlabTiles], typename Mma<R>::V (&ao)[kSlabTiles]) {
  using VT = typename Vec16<R>::T;
  constexpr int KV = 16 / int(sizeof(R)), KC = 4 * KV;
  auto mm = [](R w, R d, typename Mma<R>::V c) { return WA ? Mma<R>::mma(w, d, c) : Mma<R>::mma(d, w, c); };
  const int nch = H / KC;
  struct Buf {
    VT we, wo, u[kSlabTiles], v[kSlabTiles];
  };
  auto load_w = [&](Buf& b, int ch) {
    const unsigned k = wofs + unsigned(min(ch, nch - 1) * KC + KV * g);
    b.we = *reinterpret_cast<const VT*>(We + k);
    if (ODD) b.wo = *reinterpret_cast<const VT*>(Wo + k);
  };
  auto load_d = [&](Buf& b, int ch) {
    const int k = min(ch, nch - 1) * KC + KV * g;
#pragma unroll
    for (int t = 0; t < kSlabTiles; ++t) {
      b.u[t] = *reinterpret_cast<const VT*>(U + du[t] + k);
      if (ODD) b.v[t] = *reinterpret_cast<const VT*>(U + du[t] + vofs + k);
    }
  };
  auto mul = [&](const Buf& b) {
#pragma unroll
    for (int e = 0; e < KV; ++e)
#pragma unroll
      for (int t = 0; t < kSlabTiles; ++t) {
        ae[t] = mm(vget<R>(b.we, e), vget<R>(b.u[t], e), ae[t]);
        if (ODD) ao[t] = mm(vget<R>(b.wo, e), vget<R>(b.v[t], e), ao[t]);
      }
  };
  if (nch > 0) {
    Buf b0, b1;
    load_w(b0, 0);
    load_w(b1, 1);
    load_d(b0, 0);
    int ch = 0;
    for (; ch + 1 < nch; ch += 2) {
      load_d(b1, ch + 1);
      mul(b0);
      load_w(b0, ch + 2);
      load_d(b0, ch + 2);
      // (kept from sinking the loads of the next trip to their use)
      asm volatile("" ::: "memory");
      mul(b1);
      load_w(b1, ch + 3);
      asm volatile("" ::: "memory");
    }
    if (ch < nch) mul(b0);
  }
  for (int k = nch * KC; k < H; k += 4) {
    const R a = We[wofs + k + g], b = ODD ? Wo[wofs + k + g] : R(0);
#pragma unroll
    for (int t = 0; t < kSlabTiles; ++t) {
      ae[t] = mm(a, U[du[t] + k + g], ae[t]);
      if (ODD) ao[t] = mm(b, U[du[t] + vofs + k + g], ao[t]);
    }
  }
}

// border rows: bord[2 i + parity][row] = dot of matrix row jb + i with the slab row, eight lanes per row
template <typename R>
__device__ __forceinline__ void slab_border_rows(const R* __restrict__ We, const R* __restrict__ Wo, int Hk,
                                                 const R* U, int vofs, int Kp, int jb, int H, int h, R (*bord)[kSlabRows]) {
  using VT = typename Vec16<R>::T;
  constexpr int KV = 16 / int(sizeof(R));
  const int np = (H + KV - 1) / KV;
  for (int task = threadIdx.x; task < 8 * kSlabRows; task += blockDim.x) {
    const int row = task >> 3, s8 = task & 7;
    for (int j = jb; j < H; ++j) {
      R a = 0, b = 0;
      for (int pc = s8; pc < np; pc += 8) {
        const VT u = *reinterpret_cast<const VT*>(U + row * Kp + KV * pc);
        const VT v = *reinterpret_cast<const VT*>(U + row * Kp + vofs + KV * pc);
        const VT e = *reinterpret_cast<const VT*>(We + size_t(j) * Hk + KV * pc);
        const VT o = *reinterpret_cast<const VT*>(Wo + size_t(j) * Hk + KV * pc);
#pragma unroll
        for (int k = 0; k < KV; ++k) {
          a += vget<R>(e, k) * vget<R>(u, k);
          b += vget<R>(o, k) * vget<R>(v, k);
        }
      }
#pragma unroll
      for (int o = 4; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 8);
        b += __shfl_xor(b, o, 8);
      }
      if (s8 == 0) {
        bord[2 * (j - jb)][row] = a;
        bord[2 * (j - jb) + 1][row] = b;
      }
    }
  }
}

// x pass: 16 lines per workgroup.  The row tiles are their real and their
// imaginary parts, so a lane ends with eight consecutive complex
// outputs of one line; they go through LDS (over the slab, once every wave is
// done with it) so that the stores are whole lines.  Up to RND units per wave.
template <typename R, typename Tin, typename Tout, int RND>
__global__ __launch_bounds__(512) void slab_x_kernel(const Tin* __restrict__ in, Tout* __restrict__ out,
                                                     const R* __restrict__ W, int Hm, int Hk, int L, int nlines,
                                                     unsigned hmagic, unsigned lmagic, int acc,
                                                     const int* __restrict__ skip) {
  if (skip && *skip) return;
  using MV = typename Mma<R>::V;
  using CR = Cplx<R>;
  constexpr int NL = kSlabLines, C = kSlabRows;
  extern __shared__ __attribute__((aligned(16))) unsigned char slab_lds[];
  __shared__ R bord[4][C];
  const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63, g = lane >> 4, l16 = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = L >> 1, H = L - h, Kp = slab_stride<R>(H), nb = slab_border(H);
  R* U = reinterpret_cast<R*>(slab_lds);
  const int vofs = C * Kp;
  const int line0 = blockIdx.x * NL;
  const int nl = min(NL, nlines - line0);
  const Tin* __restrict__ src = in + size_t(line0) * L;
  // fold: (line, p) pairs flattened over the workgroup
  const int items = nl * H;
  for (int i0 = tid; i0 < items; i0 += 4 * nth) {
    Tin a[4], b[4];
    int ll[4], pp[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = min(i0 + k * nth, items - 1);
      ll[k] = hmagic ? int(__umulhi(unsigned(i), hmagic)) : i;      // i / H (H = 1: hmagic = 0)
      pp[k] = i - ll[k] * H;
      const unsigned o = unsigned(ll[k]) * L;
      a[k] = src[o + pp[k]];
      b[k] = src[o + L - 1 - pp[k]];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i0 + k * nth < items) {
        R* u = U + ll[k] * Kp + pp[k];
        const bool two = pp[k] < h;
        const R ax = R(a[k].x), ay = R(a[k].y), bx = two ? R(b[k].x) : R(0), by = two ? R(b[k].y) : R(0);
        u[0] = ax + bx;
        u[16 * Kp] = ay + by;
        u[vofs] = two ? ax - bx : R(0);
        u[vofs + 16 * Kp] = two ? ay - by : R(0);
      }
    }
  }
  const int pad = (H + 3) / 4 * 4 - H;
  for (int i = tid; i < C * pad; i += nth) {
    const int row = i % C, p = H + i / C;
    U[row * Kp + p] = R(0);
    U[row * Kp + vofs + p] = R(0);
  }
  __syncthreads();
  const R* __restrict__ Wo = W + size_t(Hm) * Hk;
  const int units = (H - nb + 15) / 16, nw = nth >> 6;
  MV ae[RND][kSlabTiles], ao[RND][kSlabTiles];
#pragma unroll
  for (int rd = 0; rd < RND; ++rd) {
    const int jt = w + rd * nw;
#pragma unroll
    for (int t = 0; t < kSlabTiles; ++t) ae[rd][t] = ao[rd][t] = MV{0, 0, 0, 0};
    if (jt < units) {
      int du[kSlabTiles];
#pragma unroll
      for (int t = 0; t < kSlabTiles; ++t) du[t] = (16 * t + l16) * Kp;
      const unsigned wofs = unsigned(16 * jt + tile_pos<R>(l16)) * Hk;
      if (16 * jt < h)
        slab_product<R, true, true>(W, Wo, wofs, U, vofs, du, H, g, ae[rd], ao[rd]);
      else
        slab_product<R, true, false>(W, Wo, wofs, U, vofs, du, H, g, ae[rd], ao[rd]);
    }
  }
  if (nb) slab_border_rows<R>(W, Wo, Hk, U, vofs, Kp, H - nb, H, h, bord);
  __syncthreads();
  // outputs in line order over the slab
  CR* O = reinterpret_cast<CR*>(slab_lds);
  const int so = slab_out_stride<R>(L);
#pragma unroll
  for (int rd = 0; rd < RND; ++rd) {
    const int jt = w + rd * nw;
    if (jt < units) {
      const int m0 = 2 * (16 * jt + 4 * g);
      CR* o = O + l16 * so + m0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const CR a{ae[rd][0][e], ae[rd][1][e]}, b{ao[rd][0][e], ao[rd][1][e]};
        if (sizeof(R) == 4 && m0 + 2 * e + 1 < L) {
          *reinterpret_cast<float4*>(o + 2 * e) = make_float4(float(a.x), float(a.y), float(b.x), float(b.y));
        } else {
          if (m0 + 2 * e < L) o[2 * e] = a;
          if (m0 + 2 * e + 1 < L) o[2 * e + 1] = b;
        }
      }
    }
  }
  for (int i = tid; i < 2 * nb * NL; i += nth) {
    const int r = i / NL, ll = i % NL;
    const int m = 2 * (H - nb + (r >> 1)) + (r & 1);
    if (m < L) O[ll * so + m] = CR{bord[r][ll], bord[r][ll + 16]};
  }
  __syncthreads();
  Tout* __restrict__ dst = out + size_t(line0) * L;
  const int outs = nl * L;
  for (int i0 = tid; i0 < outs; i0 += 4 * nth) {
    Tout old[4];
    if (acc) {
#pragma unroll
      for (int k = 0; k < 4; ++k) old[k] = dst[min(i0 + k * nth, outs - 1)];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = i0 + k * nth;
      if (i >= outs) break;
      const int ll = lmagic ? int(__umulhi(unsigned(i), lmagic)) : i;
      const CR v = O[ll * so + i - ll * L];
      Tout r;
      r.x = v.x;
      r.y = v.y;
      if (acc) {
        r.x += old[k].x;
        r.y += old[k].y;
      }
      dst[i] = r;
    }
  }
}

// y pass: 16 complex columns of one z plane per workgroup.
template <typename R>
__global__ __launch_bounds__(512) void slab_y_kernel(const R* __restrict__ in, R* __restrict__ out,
                                                     const R* __restrict__ W, int Hm, int Hk, int L, int nx,
                                                     const int* __restrict__ skip) {
  if (skip && *skip) return;
  using MV = typename Mma<R>::V;
  using VT = typename Vec16<R>::T;
  using CR = Cplx<R>;
  constexpr int KV = 16 / int(sizeof(R)), NC = kSlabLines, C = kSlabRows;
  extern __shared__ __attribute__((aligned(16))) unsigned char slab_lds[];
  __shared__ R bord[4][C];
  const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63, g = lane >> 4, l16 = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = L >> 1, H = L - h, Kp = slab_stride<R>(H), nb = slab_border(H);
  R* U = reinterpret_cast<R*>(slab_lds);
  const int vofs = C * Kp;
  // neighbouring slabs share 128-byte lines: keep them under one L2
  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  const int nsx = (nx + NC - 1) / NC;
  const int x0 = (lid % nsx) * NC;
  const size_t base = size_t(lid / nsx) * nx * L + x0;
  const int nc = min(NC, nx - x0);
  const CR* __restrict__ src = reinterpret_cast<const CR*>(in) + base;
  // fold: KV successive rows of one complex column per item (16-byte LDS writes)
  const int items = NC * ((H + 3) / 4 * 4 / KV);
  constexpr int UN = sizeof(R) == 4 ? 2 : 4;      // 16 loads in flight per thread
  const unsigned last = unsigned(L - 1) * nx;
  for (int i0 = tid; i0 < items; i0 += UN * nth) {
    CR a[UN][KV], b[UN][KV];
#pragma unroll
    for (int k = 0; k < UN; ++k) {
      const int i = min(i0 + k * nth, items - 1);
      const int c = min(i % NC, nc - 1), p = i / NC * KV;
      unsigned o = unsigned(p) * nx + c;
#pragma unroll
      for (int e = 0; e < KV; ++e) {
        if (p + e < H) {
          a[k][e] = src[o];
          b[k][e] = src[last - o + 2 * c];
        } else {
          a[k][e] = CR{0, 0};
        }
        o += nx;
      }
    }
#pragma unroll
    for (int k = 0; k < UN; ++k) {
      const int i = i0 + k * nth;
      if (i < items) {
        const int c = i % NC, p = i / NC * KV;
        VT ux, uy, vx, vy;
#pragma unroll
        for (int e = 0; e < KV; ++e) {
          const bool two = p + e < h;
          const R bx = two ? b[k][e].x : R(0), by = two ? b[k][e].y : R(0);
          reinterpret_cast<R*>(&ux)[e] = a[k][e].x + bx;
          reinterpret_cast<R*>(&uy)[e] = a[k][e].y + by;
          reinterpret_cast<R*>(&vx)[e] = two ? a[k][e].x - bx : R(0);
          reinterpret_cast<R*>(&vy)[e] = two ? a[k][e].y - by : R(0);
        }
        R* u = U + 2 * c * Kp + p;
        *reinterpret_cast<VT*>(u) = ux;
        *reinterpret_cast<VT*>(u + Kp) = uy;
        *reinterpret_cast<VT*>(u + vofs) = vx;
        *reinterpret_cast<VT*>(u + vofs + Kp) = vy;
      }
    }
  }
  __syncthreads();
  const R* __restrict__ Wo = W + size_t(Hm) * Hk;
  const int units = (H - nb + 15) / 16, nw = nth >> 6;
  CR* __restrict__ dst = reinterpret_cast<CR*>(out) + base;
  const bool pair16 = sizeof(R) == 4 && (nx & 1) == 0;    // two complex64 columns are 16-byte aligned
  for (int jt = w; jt < units; jt += nw) {
    int du[kSlabTiles];
    MV ae[kSlabTiles], ao[kSlabTiles];
#pragma unroll
    for (int t = 0; t < kSlabTiles; ++t) {
      du[t] = (16 * t + tile_pos<R>(l16)) * Kp;
      ae[t] = ao[t] = MV{0, 0, 0, 0};
    }
    const int j0 = 16 * jt;
    const unsigned wofs = unsigned(j0 + l16) * Hk;
    if (j0 < h)
      slab_product<R, false, true>(W, Wo, wofs, U, vofs, du, H, g, ae, ao);
    else
      slab_product<R, false, false>(W, Wo, wofs, U, vofs, du, H, g, ae, ao);
    // lane: output j0 + l16 of both parities, columns c, c + 1 of each row tile
#pragma unroll
    for (int par = 0; par < 2; ++par) {
      const int m = 2 * (j0 + l16) + par;
      if (m >= L) continue;
      CR* om = dst + unsigned(m) * nx;
#pragma unroll
      for (int t = 0; t < kSlabTiles; ++t) {
        const int c = 8 * t + 2 * g;
        const MV r = par ? ao[t] : ae[t];
        if (pair16 && c + 1 < nc) {
          if constexpr (sizeof(R) == 4) *reinterpret_cast<float4*>(om + c) = make_float4(r[0], r[1], r[2], r[3]);
        } else {
          if (c < nc) om[c] = CR{r[0], r[1]};
          if (c + 1 < nc) om[c + 1] = CR{r[2], r[3]};
        }
      }
    }
  }
  if (nb) {
    slab_border_rows<R>(W, Wo, Hk, U, vofs, Kp, H - nb, H, h, bord);
    __syncthreads();
    for (int i = tid; i < 2 * nb * NC; i += nth) {
      const int r = i / NC, c = i % NC, m = 2 * (H - nb + (r >> 1)) + (r & 1);
      if (m < L && c < nc) dst[unsigned(m) * nx + c] = CR{bord[r][2 * c], bord[r][2 * c + 1]};
    }
  }
}

}  // namespace

namespace {

// Launch of the slab kernels for lines of L values: LDS bytes (0: the slab does
// not fit, the K-chunked kernels take the pass), waves, and units per wave.
// 159 KB leave room for the border rows beside the slab in a CU's 160 KB; the
// slab is 2 x 32 rows of about L / 2 values, so complex64 lines fit up to
// L = 1264 and complex128 ones up to L = 632.  The x pass holds its units'
// results in registers until the slab may be overwritten: at most two units
// per wave, L <= 516.
struct SlabShape {
  size_t lds = 0;
  int waves = 0, rounds = 0;
};

// Few long lines: a workgroup forms a line's outputs 256 at a time (a round of its waves),
// the K-chunked kernels 64 each in workgroups of their own, so while CUs are idle the
// slab kernels lose from the second round on in complex128 and along complex64 x lines
// of a single slab, from the fourth along complex64 y.  Slab against K-chunked: complex128
// x, 516 values, 128 / 1024 / 4096 lines 43 / 50 / 58 us against 33 / 43 / 97; y, 632
// values, 128 / 1024 / 2048 / 4096 columns 71 / 72 / 75 / 82 against 49 / 58 / 71 / 126;
// complex64 y, 1264 values, 128 / 1024 / 2048 columns 121 / 120 / 124 against 81 / 94 / 169.
// Complex128 x lines also lose while the last CUs' second slabs are few (300 values, 275
// slabs 43 against 36; 375 slabs 46 against 54).
// Short lines: the K-chunked kernels read lines of up to 64 values once too, and up to 32
// values are one unit, so one wave of a slab's workgroup has products to form.  Slabs are
// no faster along x from 9 to 32 values, and slower from 10^4 lines on (20 values, 131072
// lines: complex128 26 against 23 us, complex64 22 against 19; 8 values 19 against 21);
// along complex128 y of 25 to 32 values from about 600 slabs on (32 x 32 x 500 10.5 against
// 9.0, and the x passes after it 9.1 against 7.8); along complex64 y from
// about 1536 slabs on (20 values, 32768 columns 8.6 against 7.0 us; 33 to 64 values only
// there, 48 values 14 against 12, 65536 columns 19 against 20); along longer complex128 y
// with very many (40 values, 262144 columns 114 against 103).
template <typename R> SlabShape slab_shape(int L, bool x, int workgroups) {
  const int H = L - L / 2, units = (H - slab_border(H) + 15) / 16;
  size_t lds = 2 * size_t(kSlabRows) * slab_stride<R>(H) * sizeof(R);
  if (x) lds = std::max(lds, size_t(kSlabLines) * slab_out_stride<R>(L) * 2 * sizeof(R));
  SlabShape s;
  s.rounds = (units + 7) / 8;
  s.waves = std::max((units + s.rounds - 1) / s.rounds, 4);
  const bool f64 = sizeof(R) == 8;
  const bool tail = x && f64 && workgroups > 256 && workgroups < 352;
  const bool few = (workgroups < (x ? (f64 ? 256 : 2) : 128) || tail) && s.rounds > (x || f64 ? 1 : 3);
  const bool brief = x     ? H > 4 && H <= 16
                     : f64 ? (H <= 32 && workgroups >= 12288) || (H > 12 && H <= 16 && workgroups >= 600)
                           : workgroups >= 1536 && H <= (workgroups < 3072 ? 32 : 16);
  s.lds = lds <= 159 * 1024 && !(x && s.rounds > 2) && !few && !brief ? lds : 0;
  return s;
}

// ceil(2^32 / d) for n / d = high word of n times it (n d < 2^32); 0 for d = 1
unsigned div_magic(int d) { return d > 1 ? unsigned(((1ull << 32) + d - 1) / d) : 0u; }

}  // namespace

// Matrices of one direction: We then Wo, [Hm][Hk] each; the inverse follows the forward.
template <typename R, typename Tin, typename Tout>
hipError_t launch_dense_x(const AxisXform& X, bool inverse, const Tin* in, Tout* out, int nlines, int acc,
                          hipStream_t s, const int* skip) {
  const R* W = static_cast<const R*>(X.wmat) + (inverse ? 2 * size_t(X.Hm) * X.Hk : 0);
  const int H = X.L - X.L / 2;
  const int slabs = (nlines + kSlabLines - 1) / kSlabLines;
  const SlabShape sh = slab_shape<R>(X.L, true, slabs);
  if (sh.lds) {
    const dim3 grid(slabs), block(64 * sh.waves);
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, block, sh.lds, s, in, out, W, X.Hm, X.Hk, X.L, nlines, div_magic(H),
                         div_magic(X.L), acc, skip);
    };
    if (sh.rounds == 1) go(slab_x_kernel<R, Tin, Tout, 1>);
    else go(slab_x_kernel<R, Tin, Tout, 2>);
    return hipGetLastError();
  }
  const dim3 grid((H + kT / 2 - 1) / (kT / 2), (nlines + kT / 2 - 1) / (kT / 2));
  hipLaunchKernelGGL((dense_x_kernel<R, Tin, Tout>), grid, dim3(256), 0, s, in, out, W, X.Hm, X.Hk, X.L, nlines,
                     acc, skip);
  return hipGetLastError();
}

template <typename R, typename T2>
hipError_t launch_dense_y(const AxisXform& Y, bool inverse, const T2* in, T2* out, int nx, int nz,
                          hipStream_t s, const int* skip) {
  const R* W = static_cast<const R*>(Y.wmat) + (inverse ? 2 * size_t(Y.Hm) * Y.Hk : 0);
  const int ncols = 2 * nx, H = Y.L - Y.L / 2;
  const int slabs = (nx + kSlabLines - 1) / kSlabLines * nz;
  const SlabShape sh = slab_shape<R>(Y.L, false, slabs);
  if (sh.lds) {
    const dim3 grid(slabs), block(64 * sh.waves);
    hipLaunchKernelGGL((slab_y_kernel<R>), grid, block, sh.lds, s, reinterpret_cast<const R*>(in),
                       reinterpret_cast<R*>(out), W, Y.Hm, Y.Hk, Y.L, nx, skip);
    return hipGetLastError();
  }
  const dim3 grid((ncols + kT - 1) / kT, (H + kT / 2 - 1) / (kT / 2), nz);
  hipLaunchKernelGGL((dense_y_kernel<R>), grid, dim3(256), 0, s, reinterpret_cast<const R*>(in),
                     reinterpret_cast<R*>(out), W, Y.Hm, Y.Hk, Y.L, ncols, skip);
  return hipGetLastError();
}

template hipError_t launch_dense_x<double, double2, double2>(const AxisXform&, bool, const double2*, double2*,
                                                             int, int, hipStream_t, const int*);
template hipError_t launch_dense_x<float, double2, float2>(const AxisXform&, bool, const double2*, float2*,
                                                           int, int, hipStream_t, const int*);
template hipError_t launch_dense_x<float, float2, double2>(const AxisXform&, bool, const float2*, double2*,
                                                           int, int, hipStream_t, const int*);
template hipError_t launch_dense_x<float, float2, float2>(const AxisXform&, bool, const float2*, float2*,
                                                          int, int, hipStream_t, const int*);
template hipError_t launch_dense_y<double, double2>(const AxisXform&, bool, const double2*, double2*, int, int,
                                                    hipStream_t, const int*);
template hipError_t launch_dense_y<float, float2>(const AxisXform&, bool, const float2*, float2*, int, int,
                                                  hipStream_t, const int*);

}  // namespace h6
