// Learned correction network (see include/h6net.h for the definition):
// BF16 activations and weights, FP32 accumulation on the matrix cores.
//
// Convolutions are implicit GEMMs on the matrix cores:
//   forward / input gradient (v_mfma_f32_16x16x32_bf16): rows = output
//     channels, columns = voxels, k = two taps x 16 channels of one input
//     chunk, the chunk's input block and weights staged in LDS;
//   weight gradient (v_mfma_f32_16x16x16bf16_1k): rows = output channels,
//     columns = input channels, k = voxels, all taps of a voxel block in one
//     workgroup, deterministic two-stage reduction.
// Operand lane layouts (lane l; K = 16: e = 0..3, K = 32: e = 0..7):
//   K = 16: A[l % 16][4 (l / 16) + e], B[4 (l / 16) + e][l % 16];
//   K = 32: A[l % 16][8 (l / 16) + e], B[8 (l / 16) + e][l % 16];
//   both:   D[4 (l / 16) + e][l % 16] (e = 0..3).
// Activations are channels-last: element (v, c) of a view at p[v * cs + coff + c],
// so the skip concatenations are two producers writing channel ranges of one
// buffer.  The input-gradient convolution is the forward kernel with the
// taps mirrored and the channel roles swapped (a repacked weight copy).
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "h6_internal.h"
#include "h6net.h"

namespace h6 {
namespace {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned short bf16;

__device__ __forceinline__ float bf2f(bf16 v) { return __uint_as_float(unsigned(v) << 16); }
// round to nearest even: the conversion instruction of gfx950 (v_cvt_pk_bf16_f32)
__device__ __forceinline__ bf16 f2bf(float f) { return __builtin_bit_cast(bf16, static_cast<__bf16>(f)); }

struct Grid3 {
  int X, Y, Z;
  __host__ __device__ long long P() const { return (long long)X * Y * Z; }
};
Grid3 half(Grid3 g) { return Grid3{(g.X + 1) / 2, (g.Y + 1) / 2, (g.Z + 1) / 2}; }

struct View {           // channels-last BF16 view
  bf16* p;
  int cs, coff;
};

// Convolution out[v][co] = act(b[co] + sum_{tap, ci} W[tap][co][ci] in[v + tap][ci])
// (zero outside the grid) as an implicit GEMM on v_mfma_f32_16x16x32_bf16: rows =
// output channels, columns = 16 voxels along x, k = two taps x 16 channels of one
// input chunk (lanes 0-31 the first tap, 32-63 the second; tap 27 is zero weights).
// A workgroup owns 16 x MT x 4 output voxels (wave w: z offset w, accumulator m: y
// offset m) and 16 output channels; the input block with its one-voxel halo, one
// 16-channel chunk at a time, and the chunk's weights sit in LDS.
//
// Three things were in the way, by counters: the vector memory path of the CU (76 %
// busy with the weights that every wave loaded for itself), LDS reads waited for one
// by one, and VALU work (900 instructions per wave).  So the input and the weights
// go straight to LDS, 1 KB per instruction, the weights once per workgroup in
// fragment order (pack_kernel); sched_products has the LDS reads ahead of their
// products; with channels as rows a lane ends up with four channels of one voxel,
// which it stores itself, no exchange through LDS.  128 x 130 x 130, us before and
// after: 16 -> 16 54 -> 49, 48 -> 16 135 -> 98, 96 -> 32 on the half grid 73 -> 54, 32 -> 32
// 43 -> 25, 64 -> 64 on the quarter grid 37 -> 19; the whole forward pass 563 -> 393
// (650 TFLOP/s).  What is left is the overlap of loads and products (42 of the 98 us
// are matrix-core time).  Slower were two input buffers at two workgroups per CU
// (through registers 135, straight to LDS 166 us for 48 -> 16) and workgroups that
// walk blocks with the weights in registers (129).  Taking a halo row for its three
// dy taps at once (half the LDS reads) gave no more and changes the order of the
// sums, so the rounding of stored values.
//
// MODE 1: the first cu chunks of the input are the nearest-neighbour upsampling
// of `up` (a grid of half the size, gu): voxel v reads up[v / 2], so the
// decoder's concatenated input is never materialised; the other chunks come from
// `in`.  MODE 2 (first layer, inference): the input is formed from the residual
// fr: channels r re / rms, r im / rms, kh (zero for r = 0) and zeros, with
// rms^2 = *fnrm / voxels (the features of h6net.h).
// MODE 3 (input gradients): the result is zeroed where the activation mask, whose
// gradient it is, is not positive, so no pass of its own does it.
constexpr int kTX = 16, kTY = 4, kTZ = 4;
constexpr int kHX = kTX + 2, kHY = kTY + 2, kHZ = kTZ + 2;
constexpr int kPairs = 14;       // the 27 taps (dx + 3 dy + 9 dz) two at a time

typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned int u4w __attribute__((ext_vector_type(4)));
typedef unsigned int u2w __attribute__((ext_vector_type(2)));

// ReLU gradient of two stored values: all ones where the activation a is positive
__device__ __forceinline__ unsigned relu_mask(unsigned a) {
  return (bf2f(bf16(a & 0xffffu)) > 0.f ? 0x0000ffffu : 0u) | (bf2f(bf16(a >> 16)) > 0.f ? 0xffff0000u : 0u);
}

// voxel offset of tap t from tap 0 inside an LDS input block of HY rows per plane
template <int HY>
__host__ __device__ constexpr int tap_off(int t) {
  return t % 3 + kHX * (t / 3 % 3) + kHX * HY * (t / 9);
}

// Instruction order of a chunk's products: every LDS row is read kAhead products
// ahead, a step's weights during the step before (left alone, the compiler waits
// for each read in turn).
constexpr int kAhead = 4;
template <int MT, int N>
__device__ __forceinline__ void sched_products() {
  constexpr int total = kPairs * MT;
  constexpr int reads = (N + kAhead < total ? 1 : 0) + (N % MT == 0 && N / MT + 1 < kPairs ? 1 : 0);
  if constexpr (N == 0) __builtin_amdgcn_sched_group_barrier(0x100, 1 + kAhead, 0);  // 0x100: LDS reads
  __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);                                   // 0x8: matrix products
  if constexpr (reads > 0) __builtin_amdgcn_sched_group_barrier(0x100, reads, 0);
  if constexpr (N + 1 < total) sched_products<MT, N + 1>();
}

typedef __attribute__((address_space(1))) const void gvoid;
typedef __attribute__((address_space(3))) void lvoid;

template <int MT, int MODE, bool MULTI>
__global__ __launch_bounds__(256, 3) void conv_kernel(View in, const bf16* __restrict__ W, const float* __restrict__ bias,
                                                      View out, float* __restrict__ out32, int nchunks, int ntall,
                                                      int relu, Grid3 g, int ntx, int nty, View up, Grid3 gu,
                                                      int cu, const double2* __restrict__ fr,
                                                      const double* __restrict__ fnrm, float fkh, View pout, Grid3 gp, View mask) {
  constexpr int HY = MT + 2, HV = kHX * HY * kHZ;
  constexpr int NPIECE = HV * 2, NPER = (NPIECE + 255) / 256;   // 16-byte pieces of an input block
  static_assert(4 * 16 * MT <= HV, "results to be pooled fit the input buffer");
  __shared__ __attribute__((aligned(16))) bf16 xs[HV][16];
  __shared__ u4w ws[kPairs][64];
  const int tid = threadIdx.x, l = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = l & 15, half = (l >> 4) & 1, second = l >> 5;
  // a block's channel groups and neighbouring blocks (shared halos) run under one L2
  const int lid = xcd_remap(blockIdx.x, gridDim.x), t0 = lid % ntall, blk = lid / ntall;
  struct Org { int x, y, z; };
  const Org o{blk % ntx * kTX, blk / ntx % nty * MT, blk / (ntx * nty) * kTZ};
  // staging: piece tid + 256 k (k < NPER) is channel octet tid & 1 of block voxel
  // tid / 2 + 128 k, walked instead of divided.  fn(k, gx, gy, gz, inside)
  const int q8 = 8 * (tid & 1);
  auto for_pieces = [&](auto&& fn) {
    const int hv0 = tid >> 1;
    int hx = hv0 % kHX, hy = (hv0 / kHX) % HY, hz = hv0 / (kHX * HY);
    static_assert(128 / kHX + 1 < 2 * HY, "at most two plane wraps per step");
#pragma unroll
    for (int k = 0; k < NPER; ++k) {
      const int gx = o.x - 1 + hx, gy = o.y - 1 + hy, gz = o.z - 1 + hz;
      const bool inside = hz < kHZ && unsigned(gx) < unsigned(g.X) && unsigned(gy) < unsigned(g.Y) &&
                          unsigned(gz) < unsigned(g.Z);
      fn(k, gx, gy, gz, inside);
      hx += 128 % kHX;
      const int cx = hx >= kHX ? 1 : 0;
      hx -= cx * kHX;
      hy += 128 / kHX + cx;
#pragma unroll
      for (int w2 = 0; w2 < 2; ++w2) {
        const int cy = hy >= HY ? 1 : 0;
        hy -= cy * HY;
        hz += cy;
      }
    }
  };
  // byte offsets of this thread's pieces in the source's first chunk (they fit 32
  // bits, see h6net_create), the same for every chunk of one source; a bit of
  // `outside` per piece out of the grid.  sh = 1: voxel v reads voxel v / 2
  unsigned goff[NPER], outside = 0;
  auto set_offsets = [&](const View& v, Grid3 gs, int sh) {
    for_pieces([&](int k, int gx, int gy, int gz, bool inside) {
      goff[k] = 2u * unsigned(((gx >> sh) + gs.X * ((gy >> sh) + gs.Y * (gz >> sh))) * v.cs + v.coff + q8);
      if (!inside) outside |= 1u << k;
    });
  };
  // chunk kc of the input (channels 16 kc .. 16 kc + 15) and its weights, straight to LDS
  const int nc = MULTI ? nchunks : 1;
  auto load = [&](int kc) {
    for (int n = wave; n < kPairs; n += 4)
      __builtin_amdgcn_global_load_lds((gvoid*)(reinterpret_cast<const u4w*>(W) + ((kc * kPairs + n) * ntall + t0) * 64 + l),
                                       (lvoid*)ws[n], 16, 0, 0);
    if (MODE == 2) return;
    const bool hi = MODE == 1 && kc < cu;
    const char* src = reinterpret_cast<const char*>((hi ? up.p : in.p) + 16 * (MODE == 1 && !hi ? kc - cu : kc));
#pragma unroll
    for (int k = 0; k < NPER; ++k)
      if (!(outside >> k & 1))
        __builtin_amdgcn_global_load_lds((gvoid*)(src + goff[k]), (lvoid*)(&xs[0][0] + (256 * k + 64 * wave) * 8), 16, 0,
                                         0);
  };
  if (MODE == 2) {      // features from the residual (channels 0..2 of octet 0, zeros elsewhere)
    load(0);
    const double ms = *fnrm / double(g.P());
    const double inv = ms > 0.0 ? 1.0 / sqrt(ms) : 0.0;
    const unsigned kb = f2bf(ms > 0.0 ? fkh : 0.f);
    double2 a[NPER];
    bool in_grid[NPER];
    for_pieces([&](int k, int gx, int gy, int gz, bool inside) {
      in_grid[k] = inside && q8 == 0;
      a[k] = fr[in_grid[k] ? gx + g.X * (gy + g.Y * gz) : 0];
    });
#pragma unroll
    for (int k = 0; k < NPER; ++k) {
      u4w v = {unsigned(f2bf(float(a[k].x * inv))) | (unsigned(f2bf(float(a[k].y * inv))) << 16), kb, 0u, 0u};
      if (!in_grid[k]) v = u4w{0u, 0u, 0u, 0u};
      if (tid + 256 * k < NPIECE) *reinterpret_cast<u4w*>(&xs[0][0] + (tid + 256 * k) * 8) = v;
    }
  } else {
    if (MODE == 1) set_offsets(up, gu, 1);
    else set_offsets(in, g, 0);
    load(0);
    // zeros outside the grid: no load writes there
    if (outside)
#pragma unroll
      for (int k = 0; k < NPER; ++k)
        if ((outside >> k & 1) && tid + 256 * k < NPIECE)
          *reinterpret_cast<u4w*>(&xs[0][0] + (tid + 256 * k) * 8) = u4w{0u, 0u, 0u, 0u};
  }
  {
    f4 acc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] = f4{0.f, 0.f, 0.f, 0.f};
    for (int kc = 0; kc < nc; ++kc) {
      __builtin_amdgcn_s_waitcnt(0x0070);      // vmcnt(0) lgkmcnt(0): this wave's rows are in LDS
      __syncthreads();
      u4w w[kPairs];
      w[0] = ws[0][l];
#pragma unroll
      for (int p = 0; p < kPairs; ++p) {
        if (p + 1 < kPairs) w[p + 1] = ws[p + 1][l];
        // the lane's voxel of row 0 at its tap (27: zero weights on tap 26's input)
        const int ta = 2 * p, tb = 2 * p + 1 < 27 ? 2 * p + 1 : 26;
        const int row0 = i + kHX * HY * wave + (second ? tap_off<HY>(tb) : tap_off<HY>(ta));
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const bf8v x = __builtin_bit_cast(bf8v, *reinterpret_cast<const u4w*>(&xs[row0 + kHX * m][8 * half]));
          acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, w[p]), x, acc[m], 0, 0, 0);
        }
      }
      sched_products<MT, 0>();
      if (MULTI && kc + 1 < nc) {
        __syncthreads();
        if (MODE == 1 && kc + 1 == cu) set_offsets(in, g, 0);      // the rest of the input comes from `in`
        load(kc + 1);
      }
    }
    const bool pool = pout.p != nullptr;
    if (pool) __syncthreads();         // every wave is done with the input block
    // lane: channels 16 t0 + 4 (l / 16) + e of voxel (x0 + i, y0 + m, z0 + wave)
    const int x = o.x + i, z = o.z + wave, q = l >> 4;
    const long long vz = x + (long long)g.X * (o.y + (long long)g.Y * z);
    if (out32) {                       // the last layer: two channels in FP32
      if (q == 0 && x < g.X && z < g.Z) {
        const float c0 = bias ? bias[0] : 0.f, c1 = bias ? bias[1] : 0.f;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          float v0 = acc[m][0] + c0, v1 = acc[m][1] + c1;
          if (relu) {
            v0 = fmaxf(v0, 0.f);
            v1 = fmaxf(v1, 0.f);
          }
          if (o.y + m < g.Y) *reinterpret_cast<float2*>(out32 + (vz + (long long)g.X * m) * 2) = make_float2(v0, v1);
        }
      }
      return;
    }
    bf16* res = &xs[0][0];             // [z][y][x][16] of the block, where it is pooled
    const int co = 16 * t0 + 4 * q;
    float b[4] = {0.f, 0.f, 0.f, 0.f};
    if (bias) {
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = bias[co + e];
    }
    bf16* dst = out.p + vz * out.cs + out.coff + co;
    const bf16* act = mask.p + vz * mask.cs + mask.coff + co;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = relu ? fmaxf(acc[m][e] + b[e], 0.f) : acc[m][e] + b[e];
      u2w w = {unsigned(f2bf(v[0])) | (unsigned(f2bf(v[1])) << 16),
               unsigned(f2bf(v[2])) | (unsigned(f2bf(v[3])) << 16)};
      if (pool) *reinterpret_cast<u2w*>(res + ((wave * MT + m) * 16 + i) * 16 + 4 * q) = w;
      if (x < g.X && z < g.Z && o.y + m < g.Y) {
        if (MODE == 3) {
          const u2w a = *reinterpret_cast<const u2w*>(act + (long long)g.X * m * mask.cs);
          w = u2w{w[0] & relu_mask(a[0]), w[1] & relu_mask(a[1])};
        }
        *reinterpret_cast<u2w*>(dst + (long long)g.X * m * out.cs) = w;
      }
    }
    // pout: the 2 x 2 x 2 average pool of the block's results on the half grid
    // gp (blocks are even-aligned; children outside the grid add nothing,
    // divisor 8, children summed z, y, x in FP32 as pool8_kernel does)
    if (!pool) return;
    __syncthreads();
    constexpr int PY = MT / 2, PV = 8 * PY * 2;
    for (int k = tid; k < PV * 2; k += 256) {
      const int pv = k / 2, c8 = k & 1;
      const int px = pv & 7, py = (pv >> 3) % PY, pz = pv / (8 * PY);
      const int qx = o.x / 2 + px, qy = o.y / 2 + py, qz = o.z / 2 + pz;
      if (qx >= gp.X || qy >= gp.Y || qz >= gp.Z) continue;
      float sacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
          for (int dx = 0; dx < 2; ++dx) {
            const int fx = 2 * px + dx, fy = 2 * py + dy, fz = 2 * pz + dz;
            if (o.x + fx >= g.X || o.y + fy >= g.Y || o.z + fz >= g.Z) continue;
            const u4w w = *reinterpret_cast<const u4w*>(res + ((fz * MT + fy) * 16 + fx) * 16 + 8 * c8);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
              sacc[2 * kk] += bf2f(bf16(w[kk] & 0xffffu));
              sacc[2 * kk + 1] += bf2f(bf16(w[kk] >> 16));
            }
          }
      u4w pk;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        pk[kk] = unsigned(f2bf(sacc[2 * kk] * 0.125f)) | (unsigned(f2bf(sacc[2 * kk + 1] * 0.125f)) << 16);
      *reinterpret_cast<u4w*>(pout.p + (qx + (long long)gp.X * (qy + (long long)gp.Y * qz)) * pout.cs + pout.coff +
                              16 * t0 + 8 * c8) = pk;
    }
  }
}

// Weight gradient: a workgroup walks 16 x 4 x 4 voxel blocks (grid-stride) for 16
// input and 16 NA output channels (blockIdx.y: which), stages the block's output
// gradient (dzs[v][co]) and its input with the one-voxel halo (xh[hv][ci]) in
// LDS and forms dW[tap][co][ci] += sum_v dz[v][co] x[v + tap][ci] for all 27 taps
// by v_mfma_f32_16x16x16_bf16 (rows co, columns ci, k = voxels).  Both operands
// need four voxels of one channel per lane, which gfx950's transposing LDS read
// (ds_read_b64_tr_b16) gives straight from the voxel-major tiles.  Wave w takes
// the nine taps of one x offset: it holds the block's 16 rows of dz in registers
// and reads each of the 36 halo rows of x once for up to nine products (one LDS
// read per 4 NA products; five reads per product, with two-byte reads and taps
// shared out over the waves, took 41 us per 16 -> 16 layer at 64 x 66 x 66).
// Partials per workgroup, summed in order by wgrad_reduce_kernel; bias partials
// sum dz over the same voxels.
constexpr int kWgThreads = 192;
constexpr int kWgRows = 768;      // workgroups aimed at: three per CU

typedef __attribute__((address_space(3))) s4 lds_s4;
__device__ __forceinline__ s4 lds_tr(const bf16* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p));
}

template <int NA>
__global__ __launch_bounds__(kWgThreads) void wgrad_kernel(View dz, View xin, float* __restrict__ part,
                                                           float* __restrict__ bpart, Grid3 g, int ntx, int nty,
                                                           int nblocks, int cinp, int coutp) {
  constexpr int HV = kHX * kHY * kHZ, NV = kTX * kTY * kTZ, CO = 16 * NA;
  __shared__ __attribute__((aligned(16))) bf16 dzs[NV * CO];
  __shared__ __attribute__((aligned(16))) bf16 xh[HV * 16];
  __shared__ float bred[kWgThreads];
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63, i = l & 15, kq = l >> 4;
  const int nci = cinp / 16, ci0 = 16 * (blockIdx.y % nci), co0 = CO * (blockIdx.y / nci);
  const bool bias = ci0 == 0;
  // transposing read: lane l of a 16-lane group addresses voxel (l & 15) / 4 of the
  // group's four, channels 4 (l & 3) ..; it receives channel l & 15 of the four
  const int tv = 4 * kq + (i >> 2), tc = 4 * (i & 3);
  f4 acc[9][NA];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int q = 0; q < NA; ++q) acc[t][q] = f4{0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f;
  for (int blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
    const int bx = blk % ntx, by = (blk / ntx) % nty, bz = blk / (ntx * nty);
    const int x0 = bx * kTX, y0 = by * kTY, z0 = bz * kTZ;
    __syncthreads();                                  // the previous block's reads are done
    for (int idx = tid; idx < NV * 2 * NA; idx += kWgThreads) {
      const int v = idx / (2 * NA), c8 = 8 * (idx % (2 * NA));
      const int gx = x0 + (v & 15), gy = y0 + ((v >> 4) & 3), gz = z0 + (v >> 6);
      u4w a = u4w{0u, 0u, 0u, 0u};
      if (gx < g.X && gy < g.Y && gz < g.Z)
        a = *reinterpret_cast<const u4w*>(dz.p + (gx + (long long)g.X * (gy + (long long)g.Y * gz)) * dz.cs + dz.coff +
                                          co0 + c8);
      *reinterpret_cast<u4w*>(&dzs[v * CO + c8]) = a;
    }
    for (int idx = tid; idx < HV * 2; idx += kWgThreads) {
      const int hv = idx >> 1, c8 = 8 * (idx & 1);
      const int hx = hv % kHX, hy = (hv / kHX) % kHY, hz = hv / (kHX * kHY);
      const int gx = x0 - 1 + hx, gy = y0 - 1 + hy, gz = z0 - 1 + hz;
      u4w a = u4w{0u, 0u, 0u, 0u};
      if (unsigned(gx) < unsigned(g.X) && unsigned(gy) < unsigned(g.Y) && unsigned(gz) < unsigned(g.Z))
        a = *reinterpret_cast<const u4w*>(xin.p + (gx + (long long)g.X * (gy + (long long)g.Y * gz)) * xin.cs +
                                          xin.coff + ci0 + c8);
      *reinterpret_cast<u4w*>(&xh[hv * 16 + c8]) = a;
    }
    __syncthreads();
    // bias partials: thread tid sums channel tid % CO over voxels tid / CO + k kWgThreads / CO
    if (bias)
      for (int v = tid / CO; v < NV; v += kWgThreads / CO) bsum += bf2f(dzs[v * CO + tid % CO]);
    s4 a[16][NA];                                     // x rows of dz: y = r & 3, z = r >> 2
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int q = 0; q < NA; ++q) a[r][q] = lds_tr(&dzs[(16 * r + tv) * CO + 16 * q + tc]);
#pragma unroll
    for (int hz = 0; hz < kHZ; ++hz)
#pragma unroll
      for (int hy = 0; hy < kHY; ++hy) {
        const s4 b = lds_tr(&xh[(kHX * (hy + kHY * hz) + wave + tv) * 16 + tc]);
#pragma unroll
        for (int z = 0; z < kTZ; ++z)
#pragma unroll
          for (int y = 0; y < kTY; ++y) {
            const int dy = hy - y, dz3 = hz - z;      // tap offsets + 1
            if (dy < 0 || dy > 2 || dz3 < 0 || dz3 > 2) continue;
#pragma unroll
            for (int q = 0; q < NA; ++q)
              acc[3 * dz3 + dy][q] =
                  __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[y + 4 * z][q], b, acc[3 * dz3 + dy][q], 0, 0, 0);
          }
      }
  }
  const int gi = blockIdx.x;
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    float* dst = part + (((size_t)gi * 27 + 3 * t + wave) * coutp + co0) * cinp + ci0;
#pragma unroll
    for (int q = 0; q < NA; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[(q * 16 + 4 * kq + e) * cinp + i] = acc[t][q][e];
  }
  if (bias) {          // the kWgThreads / CO bias partials of each channel, added in thread order
    bred[tid] = bsum;
    __syncthreads();
    if (tid < CO) {
      float t = 0.f;
      for (int k = tid; k < kWgThreads; k += CO) t += bred[k];
      bpart[(size_t)gi * coutp + co0 + tid] = t;
    }
  }
}

// Second stage of the weight gradients: gw = sum over the G partial rows, in
// the parameter layout.  A workgroup takes 32 consecutive entries of the
// partial layout [tap][co][ci] (128-byte reads) and splits the rows 16 ways
// (row q to slice q mod 16, each slice summed in row order, eight rows' loads in
// flight); the slice sums are added in slice order, so the result is
// deterministic.  Workgroups past the weights do the bias rows the same way.
constexpr int kWrW = 32, kWrS = 16;
__global__ __launch_bounds__(kWrW * kWrS) void wgrad_reduce_kernel(const float* __restrict__ part,
                                                                   const float* __restrict__ bpart, int G, int cin,
                                                                   int cout, int cinp, int coutp,
                                                                   float* __restrict__ gw, float* __restrict__ gb) {
  const int lane = threadIdx.x % kWrW, slice = threadIdx.x / kWrW;
  const int npad = 27 * coutp * cinp;
  const int nwb = (npad + kWrW - 1) / kWrW;
  const bool bias = int(blockIdx.x) >= nwb;
  const int e = (bias ? int(blockIdx.x) - nwb : int(blockIdx.x)) * kWrW + lane;
  const int n = bias ? coutp : npad;
  const size_t stride = bias ? size_t(coutp) : size_t(npad);
  const float* __restrict__ src = bias ? bpart : part;
  float a = 0.f;
  if (e < n) {
    constexpr int U = 8;
    for (int q0 = slice; q0 < G; q0 += U * kWrS) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u * kWrS;
        v[u] = src[size_t(q < G ? q : slice) * stride + e];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) a += q0 + u * kWrS < G ? v[u] : 0.f;
    }
  }
  __shared__ float red[kWrS][kWrW];
  red[slice][lane] = a;
  __syncthreads();
  if (slice != 0 || e >= n) return;
  float t = red[0][lane];
#pragma unroll
  for (int k = 1; k < kWrS; ++k) t += red[k][lane];
  if (bias) {
    if (e < cout) gb[e] = t;
    return;
  }
  const int ci = e % cinp, co = (e / cinp) % coutp, tap = e / (cinp * coutp);
  if (co < cout && ci < cin) gw[(size_t(co) * cin + ci) * 27 + tap] = t;
}

// BF16 weight copies of one layer from the FP32 master (parameter layout), in the
// order in which conv_kernel stages them: [chunk][pair][16 output channels][lane][8],
// lane l of pair p holding output channel l % 16, channels 8 (l / 16 % 2) .. + 7 of
// the chunk, tap 2 p + l / 32 (zero for tap 27 and for padded channels).  fwd: input
// ci, output co; bwd (input gradient): input co, output ci, the taps mirrored.
__host__ __device__ constexpr int packed_weights(int cinp, int coutp) { return 2 * kPairs * cinp * coutp; }
__global__ void pack_kernel(const float* __restrict__ w, int cin, int cout, int cinp, int coutp,
                            bf16* __restrict__ fwd, bf16* __restrict__ bwd) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= packed_weights(cinp, coutp)) return;
  const int lane = (idx >> 3) & 63, frag = idx >> 9;
  auto value = [&](int outp, bool back) {
    const int nt = outp / 16, t = frag % nt, p = frag / nt % kPairs, kc = frag / (nt * kPairs);
    const int o = 16 * t + (lane & 15), in = 16 * kc + 8 * ((lane >> 4) & 1) + (idx & 7), tap = 2 * p + (lane >> 5);
    const int co = back ? in : o, ci = back ? o : in;
    return tap < 27 && ci < cin && co < cout ? w[(size_t(co) * cin + ci) * 27 + (back ? 26 - tap : tap)] : 0.f;
  };
  fwd[idx] = f2bf(value(coutp, false));
  bwd[idx] = f2bf(value(cinp, true));
}

// network input: (Re r / s, Im r / s, kh, 0 ...) with s^2 = mean |r|^2 (16 channels)
__global__ void features_kernel(const double2* __restrict__ r, const double* __restrict__ nrm2,
                                long long P, float kh, bf16* __restrict__ x) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= P) return;
  const double ms = *nrm2 / double(P);
  const double inv = ms > 0.0 ? 1.0 / sqrt(ms) : 0.0;
  const double2 a = r[v];
  bf16* d = x + v * 16;
  d[0] = f2bf(float(a.x * inv));
  d[1] = f2bf(float(a.y * inv));
  d[2] = f2bf(ms > 0.0 ? kh : 0.f);
}

// forward 2x2x2 average pool (extent ceil(n/2), divisor 8) and nearest-
// neighbour upsampling (out[v] = in[v / 2]), 8 channels (16 bytes) per
// thread: the views' channel offsets and strides are multiples of 16
// channels, so every access is a 16-byte aligned load or store
typedef unsigned int u4v __attribute__((ext_vector_type(4)));

__global__ void pool8_kernel(View in, Grid3 gi, View out, Grid3 go, int C) {
  const long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int C8 = C / 8;
  if (idx >= go.P() * C8) return;
  const int c = 8 * int(idx % C8);
  const long long vo = idx / C8;
  const int x = int(vo % go.X), y = int((vo / go.X) % go.Y), z = int(vo / ((long long)go.X * go.Y));
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b)
      for (int d = 0; d < 2; ++d) {
        const int xi = 2 * x + d, yi = 2 * y + b, zi = 2 * z + a;
        if (xi < gi.X && yi < gi.Y && zi < gi.Z) {
          const u4v w = *reinterpret_cast<const u4v*>(
              in.p + (xi + (long long)gi.X * (yi + (long long)gi.Y * zi)) * in.cs + in.coff + c);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            s[2 * k] += bf2f(bf16(w[k] & 0xffffu));
            s[2 * k + 1] += bf2f(bf16(w[k] >> 16));
          }
        }
      }
  u4v o;
#pragma unroll
  for (int k = 0; k < 4; ++k) o[k] = unsigned(f2bf(s[2 * k] * 0.125f)) | (unsigned(f2bf(s[2 * k + 1] * 0.125f)) << 16);
  *reinterpret_cast<u4v*>(out.p + vo * out.cs + out.coff + c) = o;
}

__global__ void up8_kernel(View in, Grid3 gi, View out, Grid3 go, int C) {
  const long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int C8 = C / 8;
  if (idx >= go.P() * C8) return;
  const int c = 8 * int(idx % C8);
  const long long v = idx / C8;
  const int x = int(v % go.X), y = int((v / go.X) % go.Y), z = int(v / ((long long)go.X * go.Y));
  const long long vi = (x / 2) + (long long)gi.X * ((y / 2) + (long long)gi.Y * (z / 2));
  *reinterpret_cast<u4v*>(out.p + v * out.cs + out.coff + c) =
      *reinterpret_cast<const u4v*>(in.p + vi * in.cs + in.coff + c);
}

// backward element-wise steps, 8 channels (16 bytes) per thread like the
// forward pool and upsampling (channel counts are multiples of 8)
__device__ __forceinline__ void unpack8(u4v w, float (&f)[8]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    f[2 * k] = bf2f(bf16(w[k] & 0xffffu));
    f[2 * k + 1] = bf2f(bf16(w[k] >> 16));
  }
}
__device__ __forceinline__ u4v pack8(const float (&f)[8]) {
  u4v w;
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = unsigned(f2bf(f[2 * k])) | (unsigned(f2bf(f[2 * k + 1])) << 16);
  return w;
}

// g where the activation act (8 channels from c of voxel v) is positive, else zero
__device__ __forceinline__ u4v relu_mask8(View act, long long v, int c, u4v g) {
  const u4v a = *reinterpret_cast<const u4v*>(act.p + v * act.cs + act.coff + c);
#pragma unroll
  for (int k = 0; k < 4; ++k) g[k] &= relu_mask(a[k]);
  return g;
}

// gradient of the pool, added to din, and the ReLU gradient of the sum:
// din[v] = (act > 0) (din[v] + dout[v / 2] / 8)
__global__ void pool_back_kernel(View dout, Grid3 go, View din, Grid3 gi, int C, View act) {
  const long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int C8 = C / 8;
  if (idx >= gi.P() * C8) return;
  const int c = 8 * int(idx % C8);
  const long long v = idx / C8;
  const int x = int(v % gi.X), y = int((v / gi.X) % gi.Y), z = int(v / ((long long)gi.X * gi.Y));
  const long long vo = (x / 2) + (long long)go.X * ((y / 2) + (long long)go.Y * (z / 2));
  u4v* d = reinterpret_cast<u4v*>(din.p + v * din.cs + din.coff + c);
  float a[8], g[8];
  unpack8(*d, a);
  unpack8(*reinterpret_cast<const u4v*>(dout.p + vo * dout.cs + dout.coff + c), g);
#pragma unroll
  for (int k = 0; k < 8; ++k) a[k] = a[k] + 0.125f * g[k];
  *d = relu_mask8(act, v, c, pack8(a));
}

// gradient of the upsampling and of the ReLU before it: din[v] = (act > 0) sum of dout
// over the children of v
__global__ void up_back_kernel(View dout, Grid3 go, View din, Grid3 gi, int C, View act) {
  const long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int C8 = C / 8;
  if (idx >= gi.P() * C8) return;
  const int c = 8 * int(idx % C8);
  const long long v = idx / C8;
  const int x = int(v % gi.X), y = int((v / gi.X) % gi.Y), z = int(v / ((long long)gi.X * gi.Y));
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b)
      for (int d = 0; d < 2; ++d) {
        const int xo = 2 * x + d, yo = 2 * y + b, zo = 2 * z + a;
        if (xo < go.X && yo < go.Y && zo < go.Z) {
          float g[8];
          unpack8(*reinterpret_cast<const u4v*>(
                      dout.p + (xo + (long long)go.X * (yo + (long long)go.Y * zo)) * dout.cs + dout.coff + c),
                  g);
#pragma unroll
          for (int k = 0; k < 8; ++k) s[k] += g[k];
        }
      }
  *reinterpret_cast<u4v*>(din.p + v * din.cs + din.coff + c) = relu_mask8(act, v, c, pack8(s));
}

// correction c = s (y0 + i y1): mode 0 writes complex128, 1 adds to complex128,
// 2 adds to complex64
__global__ void output_kernel(const float* __restrict__ y, const double* __restrict__ nrm2, long long P,
                              void* dst, int mode) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= P) return;
  const double s = sqrt(*nrm2 / double(P));
  const double cx = s * y[2 * v], cy = s * y[2 * v + 1];
  if (mode == 0) {
    static_cast<double2*>(dst)[v] = make_double2(cx, cy);
  } else if (mode == 1) {
    double2* d = static_cast<double2*>(dst) + v;
    *d = make_double2(d->x + cx, d->y + cy);
  } else {
    float2* d = static_cast<float2*>(dst) + v;
    *d = make_float2(float(d->x + cx), float(d->y + cy));
  }
}

// loss numerator partials and the output gradient dY = 2 s (c - t) / den
// (BF16, channels 0, 1 of a 16-channel buffer)
__global__ __launch_bounds__(256) void loss_kernel(const float* __restrict__ y,
                                                   const double* __restrict__ nrm2,
                                                   const double* __restrict__ den,
                                                   const double2* __restrict__ t, long long P,
                                                   bf16* __restrict__ dy, double* __restrict__ partials) {
  __shared__ double red[4];
  double acc = 0.0;
  const double s = sqrt(*nrm2 / double(P));
  const double dn = *den;
  const double f = dn > 0.0 ? 2.0 * s / dn : 0.0;
  for (long long v = blockIdx.x * 256LL + threadIdx.x; v < P; v += (long long)gridDim.x * 256) {
    const double2 tv = t[v];
    const double ex = s * y[2 * v] - tv.x, ey = s * y[2 * v + 1] - tv.y;
    acc += ex * ex + ey * ey;
    dy[v * 16] = f2bf(float(f * ex));
    dy[v * 16 + 1] = f2bf(float(f * ey));
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// b = a - t (complex128)
__global__ void sub_kernel(const double2* __restrict__ a, const double2* __restrict__ t, double2* __restrict__ b,
                           long long P) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= P) return;
  const double2 x = a[v], y = t[v];
  b[v] = make_double2(x.x - y.x, x.y - y.y);
}

// training target t = (U* - U) - t, where t holds A_p^{-1} r on entry
__global__ void pair_target_kernel(const double2* __restrict__ us, const double2* __restrict__ u,
                                   double2* __restrict__ t, long long P) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= P) return;
  const double2 a = us[v], b = u[v], c = t[v];
  t[v] = make_double2((a.x - b.x) - c.x, (a.y - b.y) - c.y);
}

// b = conj(a)
__global__ void conj_kernel(const double2* __restrict__ a, double2* __restrict__ b, long long P) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= P) return;
  const double2 x = a[v];
  b[v] = make_double2(x.x, -x.y);
}

// operator-weighted loss: the output gradient from w = A conj(u), u = A (c - t):
// dL/dc = 2 conj(w) / den, dY = s dL/dc (BF16, channels 0, 1)
__global__ void op_grad_kernel(const double2* __restrict__ w, const double* __restrict__ nrm2,
                               const double* __restrict__ den, long long P, bf16* __restrict__ dy) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= P) return;
  const double s = sqrt(*nrm2 / double(P));
  const double dn = *den;
  const double f = dn > 0.0 ? 2.0 * s / dn : 0.0;
  const double2 x = w[v];
  dy[v * 16] = f2bf(float(f * x.x));
  dy[v * 16 + 1] = f2bf(float(-f * x.y));
}

__global__ void adam_kernel(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, long long n, float lr, float c1, float c2) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = 0.9f * m[i] + 0.1f * gi;
  const float vi = 0.999f * v[i] + 0.001f * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + 1e-8f);
}

struct LayerDef {
  int cin, cout, relu;
};
constexpr LayerDef kLayers[11] = {{3, 16, 1},  {16, 16, 1}, {16, 32, 1}, {32, 32, 1},
                                  {32, 64, 1}, {64, 64, 1}, {96, 32, 1}, {32, 32, 1},
                                  {48, 16, 1}, {16, 16, 1}, {16, 2, 0}};
enum { E1A, E1B, E2A, E2B, B3A, B3B, D2A, D2B, D1A, D1B, OUT, NL };

int r16(int c) { return (c + 15) / 16 * 16; }

long long param_count() {
  long long n = 0;
  for (const auto& L : kLayers) n += (long long)L.cout * L.cin * 27 + L.cout;
  return n;
}

}  // namespace
}  // namespace h6

struct h6_net_s {
  h6::Grid3 g1{}, g2{}, g3{};
  long long np = 0;
  // parameters
  float* w32 = nullptr;     // master (parameter layout)
  float* grad = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  long long off[h6::NL] = {};          // weight offset of each layer in the parameter array
  h6::bf16* wf[h6::NL] = {};           // packed BF16 forward weights
  h6::bf16* wb[h6::NL] = {};           // packed BF16 input-gradient weights
  int adam_t = 0;
  // activations (channels-last BF16)
  h6::bf16 *X0 = nullptr, *T1 = nullptr, *C1 = nullptr, *T1b = nullptr, *D1 = nullptr;
  h6::bf16 *Pl1 = nullptr, *T2 = nullptr, *C2 = nullptr, *T2b = nullptr, *D2 = nullptr;
  h6::bf16 *Pl2 = nullptr, *T3 = nullptr, *B3 = nullptr;
  float* Y = nullptr;
  // gradients (allocated for training)
  h6::bf16 *dY = nullptr, *dD1 = nullptr, *dT1b = nullptr, *dC1 = nullptr, *dT1 = nullptr;
  h6::bf16 *dD2 = nullptr, *dT2b = nullptr, *dC2 = nullptr, *dT2 = nullptr, *dPl1 = nullptr;
  h6::bf16 *dB3 = nullptr, *dT3 = nullptr, *dPl2 = nullptr;
  float* part = nullptr;
  float* bpart = nullptr;
  // operator-weighted loss: three complex128 work vectors (allocated on first use)
  double2* opbuf = nullptr;
  // scalars: [0] |r|^2, [1] |t|^2 (or |A t|^2), [2] loss numerator
  double* d_scal = nullptr;
  double* partials = nullptr;
  double* h_scal = nullptr;     // pinned
  std::vector<void*> allocs;
};

namespace h6 {
namespace {

template <typename T>
hipError_t dalloc(h6_net N, T** p, size_t count) {
  void* q = nullptr;
  hipError_t e = hipMalloc(&q, count * sizeof(T) + 64);
  if (e != hipSuccess) return e;
  N->allocs.push_back(q);
  *p = static_cast<T*>(q);
  return hipMemset(q, 0, count * sizeof(T) + 64);
}

// Workgroups below which a convolution takes blocks of 4 rows instead of 8: two per
// CU.  Smaller blocks read more halo (48 -> 16 at 128 x 130 x 130: 109 against 98 us),
// larger ones leave CUs idle (64 -> 64 at 16 x 17 x 17 would run on 36).
constexpr int kConvBlocks = 512;

unsigned nblk(long long n, int b = 256) { return unsigned((n + b - 1) / b); }

// out = act(conv(in)); with cu > 0 the first cu 16-channel chunks of the input are
// the nearest-neighbour upsampling of `up` (grid gu = half(g)) and the rest come from `in`
// cu < 0: the input is the features of the residual fr (first layer, cinp = 16);
// pout.p != nullptr: the output's 2 x 2 x 2 average pool also goes to pout on the
// half grid gp; out32: two output channels in FP32
hipError_t conv(View in, int cinp, const bf16* W, int coutp, const float* bias, View out, float* out32,
                int cout, int relu, Grid3 g, hipStream_t s, View up = View{nullptr, 0, 0}, Grid3 gu = Grid3{0, 0, 0},
                int cu = 0, const double2* fr = nullptr, const double* fnrm = nullptr, float fkh = 0.f,
                View pout = View{nullptr, 0, 0}, Grid3 gp = Grid3{0, 0, 0}, View mask = View{nullptr, 0, 0}) {
  if (cinp % 16 || coutp % 16 || cu >= cinp / 16 || (cu < 0 && cinp != 16)) return hipErrorInvalidValue;
  if (mask.p && (cu != 0 || out32)) return hipErrorInvalidValue;
  if (out32 ? cout != 2 || coutp != 16 || pout.p : cout != coutp) return hipErrorInvalidValue;
  const int ntx = (g.X + kTX - 1) / kTX, ntz = (g.Z + kTZ - 1) / kTZ, ntall = coutp / 16, chunks = cinp / 16;
  auto rows = [&](int mt) { return (g.Y + mt - 1) / mt; };
  const int mt = ntx * rows(8) * ntz * ntall < kConvBlocks ? 4 : 8;
  const int nblocks = ntx * rows(mt) * ntz;
  auto go = [&](auto MT, auto MODE, auto MULTI) {
    hipLaunchKernelGGL((conv_kernel<MT(), MODE(), MULTI()>), dim3(nblocks * ntall), dim3(256), 0, s, in, W, bias, out,
                       out32, chunks, ntall, relu, g, ntx, rows(mt), up, gu, cu, fr, fnrm, fkh, pout, gp, mask);
    return hipGetLastError();
  };
  auto mode = [&](auto MT) {
    constexpr std::integral_constant<int, 0> plain{};
    constexpr std::integral_constant<int, 1> upsampled{};
    constexpr std::integral_constant<int, 2> features{};
    constexpr std::integral_constant<int, 3> masked{};
    if (cu < 0) return go(MT, features, std::false_type{});
    if (cu > 0) return go(MT, upsampled, std::true_type{});
    if (mask.p) return chunks > 1 ? go(MT, masked, std::true_type{}) : go(MT, masked, std::false_type{});
    return chunks > 1 ? go(MT, plain, std::true_type{}) : go(MT, plain, std::false_type{});
  };
  return mt == 8 ? mode(std::integral_constant<int, 8>{}) : mode(std::integral_constant<int, 4>{});
}

// Partial rows of a layer with coutp x cinp channels: about kWgRows workgroups,
// blockIdx.y taking the 16-channel input chunks and the output channels by 16 or
// 32, with whole rounds of blocks per workgroup.
int wgrad_chunks(int cinp, int coutp) { return cinp / 16 * (coutp == 16 ? 1 : coutp / 32); }
int wgrad_rows(int nblocks, int chunks) {
  const int most = kWgRows / chunks, rounds = (nblocks + most - 1) / most;
  return (nblocks + rounds - 1) / rounds;
}
// floats of the partial rows of any layer: kWgRows / chunks rows of 27 coutp cinp,
// and coutp cinp <= 512 chunks
constexpr size_t kWgPartFloats = size_t(kWgRows) * 27 * 512;

// weight-gradient partials of one layer; *groups = the number of partial rows
hipError_t wgrad(View dz, View xin, int cinp, int coutp, float* part, float* bpart, Grid3 g,
                 hipStream_t s, int* groups) {
  if (cinp % 16 || (coutp != 16 && coutp % 32)) return hipErrorInvalidValue;
  const int ntx = (g.X + kTX - 1) / kTX, nty = (g.Y + kTY - 1) / kTY, ntz = (g.Z + kTZ - 1) / kTZ;
  const int nblocks = ntx * nty * ntz, chunks = wgrad_chunks(cinp, coutp);
  *groups = wgrad_rows(nblocks, chunks);
  const dim3 grid(*groups, chunks);
  if (coutp == 16)
    hipLaunchKernelGGL(wgrad_kernel<1>, grid, dim3(kWgThreads), 0, s, dz, xin, part, bpart, g, ntx, nty, nblocks, cinp,
                       coutp);
  else
    hipLaunchKernelGGL(wgrad_kernel<2>, grid, dim3(kWgThreads), 0, s, dz, xin, part, bpart, g, ntx, nty, nblocks, cinp,
                       coutp);
  return hipGetLastError();
}

View vw(bf16* p, int cs, int coff = 0) { return View{p, cs, coff}; }

// one layer: out = act(conv(in)) with the layer's packed weights
hipError_t layer_fwd(h6_net N, int L, View in, View out, float* out32, Grid3 g, hipStream_t s,
                     View up = View{nullptr, 0, 0}, Grid3 gu = Grid3{0, 0, 0}, int cu = 0,
                     const double2* fr = nullptr, float fkh = 0.f, View pout = View{nullptr, 0, 0},
                     Grid3 gp = Grid3{0, 0, 0}) {
  const LayerDef& d = kLayers[L];
  return conv(in, r16(d.cin), N->wf[L], r16(d.cout), N->w32 + N->off[L] + (long long)d.cout * d.cin * 27,
              out, out32, d.cout, d.relu, g, s, up, gu, cu, fr, N->d_scal, fkh, pout, gp);
}

// fuse_up (inference): the first convolution forms the input features from r
// itself, and the decoder convolutions read the upsampled coarser level
// directly instead of the materialised concatenations C2 / C1, whose memory
// then holds the encoder's skip outputs compactly; training keeps the
// features and the concatenations for the weight gradients
hipError_t forward(h6_net N, const double2* r, double kh, hipStream_t s, bool fuse_up = false) {
  const Grid3 g1 = N->g1, g2 = N->g2, g3 = N->g3;
  hipError_t e = launch_norm2(r, size_t(g1.P()), N->partials, N->d_scal, s);
  if (e != hipSuccess) return e;
  if (!fuse_up)
    hipLaunchKernelGGL(features_kernel, dim3(nblk(g1.P())), dim3(256), 0, s, r, N->d_scal, g1.P(),
                       float(kh), N->X0);
#define TRY(x) do { if ((e = (x)) != hipSuccess) return e; } while (0)
  // skip outputs of the encoder: channels 32..47 of C1 / 64..95 of C2 when the
  // concatenations are materialised, else compact 16- / 32-channel arrays at
  // the start of C1 / C2 (no partly read cache lines)
  const View skip1 = fuse_up ? vw(N->C1, 16) : vw(N->C1, 48, 32);
  const View skip2 = fuse_up ? vw(N->C2, 32) : vw(N->C2, 96, 64);
  if (fuse_up) {
    TRY(layer_fwd(N, E1A, vw(N->X0, 16), vw(N->T1, 16), nullptr, g1, s, View{nullptr, 0, 0}, Grid3{0, 0, 0}, -1,
                  r, float(kh)));
  } else {
    TRY(layer_fwd(N, E1A, vw(N->X0, 16), vw(N->T1, 16), nullptr, g1, s));
  }
  // in inference the encoder's pools come from the convolutions' epilogues
  if (fuse_up) {
    TRY(layer_fwd(N, E1B, vw(N->T1, 16), skip1, nullptr, g1, s, View{nullptr, 0, 0}, Grid3{0, 0, 0}, 0, nullptr,
                  0.f, vw(N->Pl1, 16), g2));
  } else {
    TRY(layer_fwd(N, E1B, vw(N->T1, 16), skip1, nullptr, g1, s));
    hipLaunchKernelGGL(pool8_kernel, dim3(nblk(g2.P() * 2)), dim3(256), 0, s, skip1, g1, vw(N->Pl1, 16), g2, 16);
  }
  TRY(layer_fwd(N, E2A, vw(N->Pl1, 16), vw(N->T2, 32), nullptr, g2, s));
  if (fuse_up) {
    TRY(layer_fwd(N, E2B, vw(N->T2, 32), skip2, nullptr, g2, s, View{nullptr, 0, 0}, Grid3{0, 0, 0}, 0, nullptr,
                  0.f, vw(N->Pl2, 32), g3));
  } else {
    TRY(layer_fwd(N, E2B, vw(N->T2, 32), skip2, nullptr, g2, s));
    hipLaunchKernelGGL(pool8_kernel, dim3(nblk(g3.P() * 4)), dim3(256), 0, s, skip2, g2, vw(N->Pl2, 32), g3, 32);
  }
  TRY(layer_fwd(N, B3A, vw(N->Pl2, 32), vw(N->T3, 64), nullptr, g3, s));
  TRY(layer_fwd(N, B3B, vw(N->T3, 64), vw(N->B3, 64), nullptr, g3, s));
  if (fuse_up) {
    TRY(layer_fwd(N, D2A, skip2, vw(N->T2b, 32), nullptr, g2, s, vw(N->B3, 64), g3, 4));
  } else {
    hipLaunchKernelGGL(up8_kernel, dim3(nblk(g2.P() * 8)), dim3(256), 0, s, vw(N->B3, 64), g3,
                       vw(N->C2, 96, 0), g2, 64);
    TRY(layer_fwd(N, D2A, vw(N->C2, 96), vw(N->T2b, 32), nullptr, g2, s));
  }
  TRY(layer_fwd(N, D2B, vw(N->T2b, 32), vw(N->D2, 32), nullptr, g2, s));
  if (fuse_up) {
    TRY(layer_fwd(N, D1A, skip1, vw(N->T1b, 16), nullptr, g1, s, vw(N->D2, 32), g2, 2));
  } else {
    hipLaunchKernelGGL(up8_kernel, dim3(nblk(g1.P() * 4)), dim3(256), 0, s, vw(N->D2, 32), g2,
                       vw(N->C1, 48, 0), g1, 32);
    TRY(layer_fwd(N, D1A, vw(N->C1, 48), vw(N->T1b, 16), nullptr, g1, s));
  }
  TRY(layer_fwd(N, D1B, vw(N->T1b, 16), vw(N->D1, 16), nullptr, g1, s));
  TRY(layer_fwd(N, OUT, vw(N->D1, 16), View{nullptr, 0, 0}, N->Y, g1, s));
#undef TRY
  return hipGetLastError();
}

// backward of one layer given the gradient gout of its output before the
// activation: accumulates the weight gradients and (gin.p != nullptr) writes the
// input gradient; mask: the input xin is an activation's output, so gin goes on to
// the gradient before that
hipError_t layer_bwd(h6_net N, int L, View gout, View xin, View gin, bool mask, Grid3 g, hipStream_t s) {
  const LayerDef& d = kLayers[L];
  const int cinp = r16(d.cin), coutp = r16(d.cout);
  hipError_t e;
  int G = 0;
  if ((e = wgrad(gout, xin, cinp, coutp, N->part, N->bpart, g, s, &G)) != hipSuccess) return e;
  const long long nw = (long long)d.cout * d.cin * 27;
  const unsigned nrb = unsigned((27 * coutp * cinp + kWrW - 1) / kWrW + (coutp + kWrW - 1) / kWrW);
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(nrb), dim3(kWrW * kWrS), 0, s, N->part, N->bpart, G, d.cin,
                     d.cout, cinp, coutp, N->grad + N->off[L], N->grad + N->off[L] + nw);
  if (gin.p)
    return conv(gout, coutp, N->wb[L], cinp, nullptr, gin, nullptr, cinp, 0, g, s, View{nullptr, 0, 0}, Grid3{0, 0, 0},
                0, nullptr, nullptr, 0.f, View{nullptr, 0, 0}, Grid3{0, 0, 0}, mask ? xin : View{nullptr, 0, 0});
  return hipGetLastError();
}

hipError_t backward(h6_net N, hipStream_t s) {
  const Grid3 g1 = N->g1, g2 = N->g2, g3 = N->g3;
  hipError_t e;
#define TRY(x) do { if ((e = (x)) != hipSuccess) return e; } while (0)
  TRY(layer_bwd(N, OUT, vw(N->dY, 16), vw(N->D1, 16), vw(N->dD1, 16), true, g1, s));
  TRY(layer_bwd(N, D1B, vw(N->dD1, 16), vw(N->T1b, 16), vw(N->dT1b, 16), true, g1, s));
  TRY(layer_bwd(N, D1A, vw(N->dT1b, 16), vw(N->C1, 48), vw(N->dC1, 48), false, g1, s));
  hipLaunchKernelGGL(up_back_kernel, dim3(nblk(g2.P() * 4)), dim3(256), 0, s, vw(N->dC1, 48, 0), g1,
                     vw(N->dD2, 32), g2, 32, vw(N->D2, 32));
  TRY(layer_bwd(N, D2B, vw(N->dD2, 32), vw(N->T2b, 32), vw(N->dT2b, 32), true, g2, s));
  TRY(layer_bwd(N, D2A, vw(N->dT2b, 32), vw(N->C2, 96), vw(N->dC2, 96), false, g2, s));
  hipLaunchKernelGGL(up_back_kernel, dim3(nblk(g3.P() * 8)), dim3(256), 0, s, vw(N->dC2, 96, 0), g2,
                     vw(N->dB3, 64), g3, 64, vw(N->B3, 64));
  TRY(layer_bwd(N, B3B, vw(N->dB3, 64), vw(N->T3, 64), vw(N->dT3, 64), true, g3, s));
  TRY(layer_bwd(N, B3A, vw(N->dT3, 64), vw(N->Pl2, 32), vw(N->dPl2, 32), false, g3, s));
  hipLaunchKernelGGL(pool_back_kernel, dim3(nblk(g2.P() * 4)), dim3(256), 0, s, vw(N->dPl2, 32), g3,
                     vw(N->dC2, 96, 64), g2, 32, vw(N->C2, 96, 64));
  TRY(layer_bwd(N, E2B, vw(N->dC2, 96, 64), vw(N->T2, 32), vw(N->dT2, 32), true, g2, s));
  TRY(layer_bwd(N, E2A, vw(N->dT2, 32), vw(N->Pl1, 16), vw(N->dPl1, 16), false, g2, s));
  hipLaunchKernelGGL(pool_back_kernel, dim3(nblk(g1.P() * 2)), dim3(256), 0, s, vw(N->dPl1, 16), g2,
                     vw(N->dC1, 48, 32), g1, 16, vw(N->C1, 48, 32));
  TRY(layer_bwd(N, E1B, vw(N->dC1, 48, 32), vw(N->T1, 16), vw(N->dT1, 16), true, g1, s));
  TRY(layer_bwd(N, E1A, vw(N->dT1, 16), vw(N->X0, 16), View{nullptr, 0, 0}, false, g1, s));
#undef TRY
  return hipGetLastError();
}

hipError_t pack_all(h6_net N, hipStream_t s) {
  for (int L = 0; L < NL; ++L) {
    const LayerDef& d = kLayers[L];
    const int n = packed_weights(r16(d.cin), r16(d.cout));
    hipLaunchKernelGGL(pack_kernel, dim3(nblk(n)), dim3(256), 0, s, N->w32 + N->off[L], d.cin, d.cout,
                       r16(d.cin), r16(d.cout), N->wf[L], N->wb[L]);
  }
  return hipGetLastError();
}

hipError_t alloc_training(h6_net N) {
  if (N->dY) return hipSuccess;
  const long long p1 = N->g1.P(), p2 = N->g2.P(), p3 = N->g3.P();
  hipError_t e = hipSuccess;
  auto A = [&](bf16** p, long long n) { if (e == hipSuccess) e = dalloc(N, p, size_t(n)); };
  A(&N->dY, p1 * 16); A(&N->dD1, p1 * 16); A(&N->dT1b, p1 * 16); A(&N->dC1, p1 * 48); A(&N->dT1, p1 * 16);
  A(&N->dD2, p2 * 32); A(&N->dT2b, p2 * 32); A(&N->dC2, p2 * 96); A(&N->dT2, p2 * 32); A(&N->dPl1, p2 * 16);
  A(&N->dB3, p3 * 64); A(&N->dT3, p3 * 64); A(&N->dPl2, p3 * 32);
  if (e == hipSuccess) e = dalloc(N, &N->part, kWgPartFloats);
  if (e == hipSuccess) e = dalloc(N, &N->bpart, size_t(kWgRows) * 64);
  if (e == hipSuccess) e = dalloc(N, &N->m, size_t(N->np));
  if (e == hipSuccess) e = dalloc(N, &N->v, size_t(N->np));
  return e;
}

// loss of the current forward output against t; gradients into N->grad
hipError_t loss_backward(h6_net N, const double2* t, hipStream_t s) {
  const long long P = N->g1.P();
  hipError_t e = launch_norm2(t, size_t(P), N->partials, N->d_scal + 1, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(loss_kernel, dim3(kRedBlocks), dim3(256), 0, s, N->Y, N->d_scal, N->d_scal + 1, t, P,
                     N->dY, N->partials);
  if ((e = launch_reduce_sum(N->partials, kRedBlocks, N->d_scal + 2, s)) != hipSuccess) return e;
  return backward(N, s);
}

// operator-weighted loss |A (c - t)|^2 / |A t|^2 of the current forward
// output (A: the plan's operator); gradients into N->grad.  The adjoint is
// taken as conj(A conj(.)), exact for complex symmetric A (Dirichlet faces).
hipError_t op_loss_backward(h6_net N, h6_plan plan, const double2* t, hipStream_t s) {
  const long long P = N->g1.P();
  hipError_t e = hipSuccess;
  if (!N->opbuf) {
    if ((e = dalloc(N, &N->opbuf, size_t(3 * P))) != hipSuccess) return e;
  }
  double2* b0 = N->opbuf;
  double2* b1 = b0 + P;
  double2* b2 = b1 + P;
  const unsigned nb = nblk(P);
  // |A t|^2
  if ((e = launch_stencil(plan, t, b2, nullptr, nullptr, nullptr, s)) != hipSuccess) return e;
  if ((e = launch_norm2(b2, size_t(P), N->partials, N->d_scal + 1, s)) != hipSuccess) return e;
  // u = A (c - t), |u|^2
  hipLaunchKernelGGL(output_kernel, dim3(nb), dim3(256), 0, s, N->Y, N->d_scal, P, static_cast<void*>(b0), 0);
  hipLaunchKernelGGL(sub_kernel, dim3(nb), dim3(256), 0, s, b0, t, b0, P);
  if ((e = launch_stencil(plan, b0, b1, nullptr, nullptr, nullptr, s)) != hipSuccess) return e;
  if ((e = launch_norm2(b1, size_t(P), N->partials, N->d_scal + 2, s)) != hipSuccess) return e;
  // w = A conj(u)
  hipLaunchKernelGGL(conj_kernel, dim3(nb), dim3(256), 0, s, b1, b0, P);
  if ((e = launch_stencil(plan, b0, b2, nullptr, nullptr, nullptr, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(op_grad_kernel, dim3(nb), dim3(256), 0, s, b2, N->d_scal, N->d_scal + 1, P, N->dY);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return backward(N, s);
}

}  // namespace
}  // namespace h6

using namespace h6;

extern "C" {

long long h6net_param_count(void) { return param_count(); }

h6_status h6net_create(const int dims[3], void* hip_stream, h6_net* out) {
  if (!out) return H6_ERR_ARG;
  *out = nullptr;
  if (!dims || dims[0] < 1 || dims[1] < 1 || dims[2] < 1) return H6_ERR_ARG;
  // the convolutions gather with 32-bit element offsets into the widest
  // activation buffers (48 channels on the grid, 96 on the half grid)
  {
    const Grid3 a{dims[0], dims[1], dims[2]}, b = half(a);
    if (a.P() * 48 >= (1LL << 31) || b.P() * 96 >= (1LL << 31)) return H6_ERR_ARG;
  }
  h6_net N = new (std::nothrow) h6_net_s();
  if (!N) return H6_ERR_ALLOC;
  N->g1 = Grid3{dims[0], dims[1], dims[2]};
  N->g2 = half(N->g1);
  N->g3 = half(N->g2);
  N->np = param_count();
  long long o = 0;
  for (int L = 0; L < NL; ++L) {
    N->off[L] = o;
    o += (long long)kLayers[L].cout * kLayers[L].cin * 27 + kLayers[L].cout;
  }
  const long long p1 = N->g1.P(), p2 = N->g2.P(), p3 = N->g3.P();
  hipError_t e = hipSuccess;
  auto B = [&](bf16** p, long long n) { if (e == hipSuccess) e = dalloc(N, p, size_t(n)); };
  B(&N->X0, p1 * 16); B(&N->T1, p1 * 16); B(&N->C1, p1 * 48); B(&N->T1b, p1 * 16); B(&N->D1, p1 * 16);
  B(&N->Pl1, p2 * 16); B(&N->T2, p2 * 32); B(&N->C2, p2 * 96); B(&N->T2b, p2 * 32); B(&N->D2, p2 * 32);
  B(&N->Pl2, p3 * 32); B(&N->T3, p3 * 64); B(&N->B3, p3 * 64);
  if (e == hipSuccess) e = dalloc(N, &N->Y, size_t(p1) * 2);
  if (e == hipSuccess) e = dalloc(N, &N->w32, size_t(N->np));
  if (e == hipSuccess) e = dalloc(N, &N->grad, size_t(N->np));
  for (int L = 0; L < NL && e == hipSuccess; ++L) {
    const size_t n = packed_weights(r16(kLayers[L].cin), r16(kLayers[L].cout));
    e = dalloc(N, &N->wf[L], n);
    if (e == hipSuccess) e = dalloc(N, &N->wb[L], n);
  }
  if (e == hipSuccess) e = dalloc(N, &N->d_scal, 8);
  if (e == hipSuccess) e = dalloc(N, &N->partials, size_t(kRedBlocks));
  if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void**>(&N->h_scal), 8 * sizeof(double));
  if (e == hipSuccess) e = hipStreamSynchronize(static_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) {
    h6net_destroy(N);
    return e == hipErrorOutOfMemory ? H6_ERR_ALLOC : H6_ERR_HIP;
  }
  *out = N;
  return H6_OK;
}

h6_status h6net_set_params(h6_net N, const float* params, long long count, void* hip_stream) {
  if (!N || !params || count != N->np) return H6_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (hipMemcpyAsync(N->w32, params, size_t(count) * sizeof(float), hipMemcpyHostToDevice, s) != hipSuccess ||
      pack_all(N, s) != hipSuccess)
    return H6_ERR_HIP;
  if (N->m && (hipMemsetAsync(N->m, 0, size_t(N->np) * 4, s) != hipSuccess ||
               hipMemsetAsync(N->v, 0, size_t(N->np) * 4, s) != hipSuccess))
    return H6_ERR_HIP;
  N->adam_t = 0;
  return hipStreamSynchronize(s) == hipSuccess ? H6_OK : H6_ERR_HIP;
}

h6_status h6net_get_params(h6_net N, float* params, long long count, void* hip_stream) {
  if (!N || !params || count != N->np) return H6_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (hipMemcpyAsync(params, N->w32, size_t(count) * sizeof(float), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return H6_ERR_HIP;
  return H6_OK;
}

h6_status h6net_forward(h6_net N, const void* r, double kh, void* c, void* hip_stream) {
  if (!N || !r || !c || r == c) return H6_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (forward(N, static_cast<const double2*>(r), kh, s, true) != hipSuccess) return H6_ERR_HIP;
  hipLaunchKernelGGL(output_kernel, dim3(nblk(N->g1.P())), dim3(256), 0, s, N->Y, N->d_scal, N->g1.P(), c, 0);
  return hipGetLastError() == hipSuccess ? H6_OK : H6_ERR_HIP;
}

h6_status h6net_gradients(h6_net N, const void* r, double kh, const void* t, float* grads, double* loss,
                          void* hip_stream) {
  if (!N || !r || !t) return H6_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (alloc_training(N) != hipSuccess) return H6_ERR_ALLOC;
  if (forward(N, static_cast<const double2*>(r), kh, s) != hipSuccess ||
      loss_backward(N, static_cast<const double2*>(t), s) != hipSuccess)
    return H6_ERR_HIP;
  if (hipMemcpyAsync(N->h_scal, N->d_scal, 3 * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess)
    return H6_ERR_HIP;
  if (grads && hipMemcpyAsync(grads, N->grad, size_t(N->np) * 4, hipMemcpyDeviceToHost, s) != hipSuccess)
    return H6_ERR_HIP;
  if (hipStreamSynchronize(s) != hipSuccess) return H6_ERR_HIP;
  if (loss) *loss = N->h_scal[1] > 0.0 ? N->h_scal[2] / N->h_scal[1] : 0.0;
  return H6_OK;
}

h6_status h6net_train_step(h6_net N, const void* r, double kh, const void* t, float lr, double* loss,
                           void* hip_stream) {
  if (!N || !r || !t) return H6_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (alloc_training(N) != hipSuccess) return H6_ERR_ALLOC;
  if (forward(N, static_cast<const double2*>(r), kh, s) != hipSuccess ||
      loss_backward(N, static_cast<const double2*>(t), s) != hipSuccess)
    return H6_ERR_HIP;
  N->adam_t += 1;
  const float c1 = float(1.0 / (1.0 - std::pow(0.9, N->adam_t)));
  const float c2 = float(1.0 / (1.0 - std::pow(0.999, N->adam_t)));
  hipLaunchKernelGGL(adam_kernel, dim3(nblk(N->np)), dim3(256), 0, s, N->w32, N->grad, N->m, N->v, N->np,
                     lr, c1, c2);
  if (pack_all(N, s) != hipSuccess) return H6_ERR_HIP;
  if (loss) {
    if (hipMemcpyAsync(N->h_scal, N->d_scal, 3 * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return H6_ERR_HIP;
    *loss = N->h_scal[1] > 0.0 ? N->h_scal[2] / N->h_scal[1] : 0.0;
  }
  return hipGetLastError() == hipSuccess ? H6_OK : H6_ERR_HIP;
}

static bool op_args_ok(h6_net N, h6_plan plan) {
  return N && plan && net_matches(N, plan->dims);
}

h6_status h6net_gradients_op(h6_net N, h6_plan plan, const void* r, const void* t, float* grads, double* loss,
                             void* hip_stream) {
  if (!op_args_ok(N, plan) || !r || !t) return H6_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (alloc_training(N) != hipSuccess) return H6_ERR_ALLOC;
  const double kh = plan->k.real() * plan->p.h;
  if (forward(N, static_cast<const double2*>(r), kh, s) != hipSuccess ||
      op_loss_backward(N, plan, static_cast<const double2*>(t), s) != hipSuccess)
    return H6_ERR_HIP;
  if (hipMemcpyAsync(N->h_scal, N->d_scal, 3 * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess)
    return H6_ERR_HIP;
  if (grads && hipMemcpyAsync(grads, N->grad, size_t(N->np) * 4, hipMemcpyDeviceToHost, s) != hipSuccess)
    return H6_ERR_HIP;
  if (hipStreamSynchronize(s) != hipSuccess) return H6_ERR_HIP;
  if (loss) *loss = N->h_scal[1] > 0.0 ? N->h_scal[2] / N->h_scal[1] : 0.0;
  return H6_OK;
}

h6_status h6net_train_step_op(h6_net N, h6_plan plan, const void* r, const void* t, float lr, double* loss,
                              void* hip_stream) {
  if (!op_args_ok(N, plan) || !r || !t) return H6_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (alloc_training(N) != hipSuccess) return H6_ERR_ALLOC;
  const double kh = plan->k.real() * plan->p.h;
  if (forward(N, static_cast<const double2*>(r), kh, s) != hipSuccess ||
      op_loss_backward(N, plan, static_cast<const double2*>(t), s) != hipSuccess)
    return H6_ERR_HIP;
  N->adam_t += 1;
  const float c1 = float(1.0 / (1.0 - std::pow(0.9, N->adam_t)));
  const float c2 = float(1.0 / (1.0 - std::pow(0.999, N->adam_t)));
  hipLaunchKernelGGL(adam_kernel, dim3(nblk(N->np)), dim3(256), 0, s, N->w32, N->grad, N->m, N->v, N->np,
                     lr, c1, c2);
  if (pack_all(N, s) != hipSuccess) return H6_ERR_HIP;
  if (loss) {
    if (hipMemcpyAsync(N->h_scal, N->d_scal, 3 * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return H6_ERR_HIP;
    *loss = N->h_scal[1] > 0.0 ? N->h_scal[2] / N->h_scal[1] : 0.0;
  }
  return hipGetLastError() == hipSuccess ? H6_OK : H6_ERR_HIP;
}

h6_status h6net_training_pair(h6_plan plan, const void* F, const void* Ustar, const void* U, void* r, void* t,
                              void* hip_stream) {
  if (!plan || !F || !Ustar || !U || !r || !t || r == t) return H6_ERR_ARG;
  for (const void* in : {F, Ustar, U})
    if (in == r || in == t) return H6_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const long long P = (long long)plan->N;
  double2* rr = static_cast<double2*>(r);
  double2* tt = static_cast<double2*>(t);
  if (launch_stencil(plan, static_cast<const double2*>(U), rr, static_cast<const double2*>(F), plan->partials,
                     nullptr, s) != hipSuccess ||
      launch_pinv(plan, rr, tt, s) != hipSuccess)
    return H6_ERR_HIP;
  hipLaunchKernelGGL(pair_target_kernel, dim3(nblk(P)), dim3(256), 0, s, static_cast<const double2*>(Ustar),
                     static_cast<const double2*>(U), tt, P);
  return hipGetLastError() == hipSuccess ? H6_OK : H6_ERR_HIP;
}

void h6net_destroy(h6_net N) {
  if (!N) return;
  for (void* p : N->allocs) (void)hipFree(p);
  if (N->h_scal) (void)hipHostFree(N->h_scal);
  delete N;
}

}  // extern "C"

namespace h6 {

// z += correction(q) for the solver (complex64 z in mixed plans)
hipError_t net_apply_add(h6_net N, const double2* q, double kh, void* z, bool z_f32, hipStream_t s) {
  hipError_t e = forward(N, q, kh, s, true);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(output_kernel, dim3(nblk(N->g1.P())), dim3(256), 0, s, N->Y, N->d_scal, N->g1.P(), z,
                     z_f32 ? 2 : 1);
  return hipGetLastError();
}

bool net_matches(h6_net N, const int dims[3]) {
  return N && N->g1.X == dims[0] && N->g1.Y == dims[1] && N->g1.Z == dims[2];
}

}  // namespace h6
