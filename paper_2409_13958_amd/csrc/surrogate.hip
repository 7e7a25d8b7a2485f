// Kernels and host object of the learned surrogate of the AIM grid
// convolution (layout and conventions in surrogate.h).
#include "surrogate.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace pmfem {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kT = 256;
constexpr int kSgMT = 512;         // threads of a middle layer's workgroup
constexpr int kRedBlocks = 1024;   // blocks of the device reductions (partials in dred)

constexpr int kSgThin = kSgC * 32;   // a thin layer's partial sums: 27 offsets, the bias, 4 unused

// FP32 -> BF16, round to nearest even (finite inputs)
__device__ __forceinline__ uint32_t bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ float bf16_float(uint32_t h) { return __uint_as_float(h << 16); }

// v in [-1, n] on a circular axis of n points; a tile's points past n, which
// nothing reads or meets only zeros, take the last one's. A remainder here took
// 40 instructions per staged value.
__device__ __forceinline__ int wrapi(int v, int n) {
  return v < 0 ? n - 1 : v == n ? 0 : min(v, n - 1);
}

__device__ __forceinline__ int64_t vox_of(const SgGrid& g, int z, int y, int x) {
  return ((int64_t)z * g.ny + y) * g.nx + x;
}

// ---------------------------------------------------------------------------
// First-layer form (one input channel -> kSgC outputs), FP32 FMA. Also the
// data gradient of the last layer (weights flipped). Tile: 8 rows of 32
// points of one z-plane per 256-thread workgroup; the 3 input planes of the
// tile with a one-point halo staged in LDS. A thread forms 4 channels of 8
// consecutive points, so that the ten values of a row serve 24 products each
// of their channels and eight lanes store (and read the mask of) 128
// contiguous bytes; with a thread for all channels of one point the 16-byte
// stores, 128 bytes apart, and 216 weight reads bound it. 128 x 128 x 8 points:
// 11.1 us, before 18.8; weights through the scalar cache 19.6.
__global__ __launch_bounds__(kT) void k_sg_in(SgGrid g, const float* __restrict__ x, float xs,
                                               const float* __restrict__ w,
                                               const float* __restrict__ b,
                                               float* __restrict__ out, int relu,
                                               const float* __restrict__ mask) {
  __shared__ float sx[3 * kSgHalo];
  __shared__ __align__(16) float sw[kSgC * 27];
  const int tiles_x = (g.nx + kSgTX - 1) / kSgTX;
  const int x0 = (int)(blockIdx.x % tiles_x) * kSgTX, y0 = (int)(blockIdx.x / tiles_x) * kSgTY;
  const int z = blockIdx.y, t = threadIdx.x;
  const int q = t & 7, ty = t >> 5, tx = ((t >> 3) & 3) * 8;  // channels 4 q .., points tx .. tx + 7
  const int gy = y0 + ty;
  const int64_t v0 = vox_of(g, z, min(gy, g.ny - 1), 0);
  float4 mk[8];
  if (mask) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      mk[i] = reinterpret_cast<const float4*>(mask + (v0 + min(x0 + tx + i, g.nx - 1)) * kSgC)[q];
  }
  for (int i = t; i < kSgC * 27; i += kT) sw[(i % 27) * kSgC + i / 27] = w[i];  // [o][co]
  for (int i = t; i < 3 * kSgHalo; i += kT) {
    const int pl = i / kSgHalo, h = i - pl * kSgHalo;
    const int hy = h / kSgHX, hx = h - hy * kSgHX, gz = z + pl - 1;
    float v = 0.f;
    if (gz >= 0 && gz < g.nz)
      v = x[vox_of(g, gz, wrapi(y0 + hy - 1, g.ny), wrapi(x0 + hx - 1, g.nx))] * xs;
    sx[i] = v;
  }
  __syncthreads();
  const float4 b4 = b ? reinterpret_cast<const float4*>(b)[q] : make_float4(0.f, 0.f, 0.f, 0.f);
  float4 acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = b4;
#pragma unroll 3
  for (int k = 0; k < 9; ++k) {  // dz, dy
    const float* s = &sx[(k / 3) * kSgHalo + (ty + k % 3) * kSgHX + tx];
    float v[10];
#pragma unroll
    for (int i = 0; i < 10; ++i) v[i] = s[i];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      const float4 ww = reinterpret_cast<const float4*>(&sw[(k * 3 + dx) * kSgC])[q];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        acc[i].x = fmaf(ww.x, v[i + dx], acc[i].x);
        acc[i].y = fmaf(ww.y, v[i + dx], acc[i].y);
        acc[i].z = fmaf(ww.z, v[i + dx], acc[i].z);
        acc[i].w = fmaf(ww.w, v[i + dx], acc[i].w);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float4 r = acc[i];
    if (mask) {
      r.x = mk[i].x > 0.f ? r.x : 0.f;
      r.y = mk[i].y > 0.f ? r.y : 0.f;
      r.z = mk[i].z > 0.f ? r.z : 0.f;
      r.w = mk[i].w > 0.f ? r.w : 0.f;
    }
    if (relu) {
      r.x = fmaxf(r.x, 0.f);
      r.y = fmaxf(r.y, 0.f);
      r.z = fmaxf(r.z, 0.f);
      r.w = fmaxf(r.w, 0.f);
    }
    const int gx = x0 + tx + i;
    if (gx < g.nx && gy < g.ny) reinterpret_cast<float4*>(out + (v0 + gx) * kSgC)[q] = r;
  }
}

// Last-layer form (kSgC inputs -> one output), FP32 FMA: y = (conv + b) ys.
// A thread sums 4 channels of 8 consecutive points over the 27 offsets, then
// eight lanes add their channels; the ten float4 of a row, eight lanes 128
// contiguous bytes, serve 24 products each of their channels. Each is read
// from the cache where it lies (by up to nine threads of a workgroup): staged
// in LDS with a thread per point, its 216 reads per thread bound the kernel.
// 128 x 128 x 8 points: 12.0 us, before 19.6.
__global__ __launch_bounds__(kT) void k_sg_out(SgGrid g, const float* __restrict__ a,
                                                const float* __restrict__ w,
                                                const float* __restrict__ b, float ys,
                                                float* __restrict__ y) {
  __shared__ __align__(16) float sw[kSgC * 27];
  const int tiles_x = (g.nx + kSgTX - 1) / kSgTX;
  const int x0 = (int)(blockIdx.x % tiles_x) * kSgTX, y0 = (int)(blockIdx.x / tiles_x) * kSgTY;
  const int z = blockIdx.y, t = threadIdx.x;
  const int q = t & 7, ty = t >> 5, tx = ((t >> 3) & 3) * 8;
  for (int i = t; i < kSgC * 27; i += kT) sw[(i % 27) * kSgC + i / 27] = w[i];  // [o][ci]
  const int gy = y0 + ty;
  int cx[10];  // the columns x0 + tx - 1 .. x0 + tx + 8, as float4 of a row
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    const int gx = x0 + tx + i - 1;
    cx[i] = wrapi(gx, g.nx) * (kSgC / 4) + q;
  }
  __syncthreads();
  float acc[8] = {};
#pragma unroll 3
  for (int k = 0; k < 9; ++k) {
    const int gz = z + k / 3 - 1;
    if (gz < 0 || gz >= g.nz) continue;  // the same for the whole workgroup
    int yy = gy + k % 3 - 1;             // rows past the grid's end are not stored
    yy = wrapi(yy, g.ny);
    const float4* row = reinterpret_cast<const float4*>(a + vox_of(g, gz, yy, 0) * kSgC);
    float4 v[10];
#pragma unroll
    for (int i = 0; i < 10; ++i) v[i] = row[cx[i]];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      const float4 ww = reinterpret_cast<const float4*>(&sw[(k * 3 + dx) * kSgC])[q];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        acc[i] = fmaf(ww.x, v[i + dx].x, acc[i]);
        acc[i] = fmaf(ww.y, v[i + dx].y, acc[i]);
        acc[i] = fmaf(ww.z, v[i + dx].z, acc[i]);
        acc[i] = fmaf(ww.w, v[i + dx].w, acc[i]);
      }
    }
  }
  // lane q ends with point tx + q: halves are exchanged three times
  float s4[4], s2[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float keep = q & 4 ? acc[4 + i] : acc[i], send = q & 4 ? acc[i] : acc[4 + i];
    s4[i] = keep + __shfl_xor(send, 4);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float keep = q & 2 ? s4[2 + i] : s4[i], send = q & 2 ? s4[i] : s4[2 + i];
    s2[i] = keep + __shfl_xor(send, 2);
  }
  const float keep = q & 1 ? s2[1] : s2[0], send = q & 1 ? s2[0] : s2[1];
  const float sum = keep + __shfl_xor(send, 1);
  const int gx = x0 + tx + q;
  if (gx < g.nx && gy < g.ny) y[vox_of(g, z, gy, gx)] = (sum + b[0]) * ys;
}

// Middle layer (kSgC -> kSgC) on the matrix cores, as an implicit GEMM: M =
// grid points, N = output channels, K = 27 offsets x kSgC input channels,
// with v_mfma_f32_16x16x32_bf16 (A: 16 points x 32 channels of one offset;
// B: 32 input x 16 output channels). A workgroup computes 8 rows x 32 points
// of two consecutive z-planes; each of its eight waves owns two rows (four
// 16-point M tiles) times one 16-channel N tile of both planes, eight
// independent accumulators. The layer's weights (54 KB) are staged in LDS
// once, the input planes z0-1 .. z0+2 one at a time as BF16 (and, with SPLIT,
// the BF16 remainder x - bf16(x), which a second product adds); every A
// fragment read from LDS serves both output planes, and the next plane's loads
// are in flight (in registers) while the current one is multiplied. The nine
// offsets of a plane are straight-line code, each one's LDS reads issued before
// the products of the one before. A 16-byte read of a wavefront takes four
// turns, the first of lanes 0-3, 12-15 and 20-27: the chunk of a point is
// XORed with twice bit 2 of its column, which leaves every turn without a bank
// conflict (with bits 2 and 3: 1.3 M conflict cycles of 3.1 M, now none), and
// as it does not depend on the row, all reads of a plane lie at fixed distances
// from three addresses.
// 128 x 128 x 8 points: 23.3 us; with four waves of both N tiles and addresses
// formed for every read 27.4; with the weights read from global memory under a
// branch per offset and the mask one value at a time 45. 256 workgroups leave
// two wavefronts per SIMD there, so staging and its barriers are only partly
// hidden: the matrix cores are busy for 5.8 us of it.
// Also the data gradient (weights transposed and flipped, no bias) with the
// ReLU mask of the layer below.
constexpr int kSgMP = kSgHX + 2;   // staged row: a multiple of four points
constexpr int kSgMPlane = kSgHY * kSgMP * 4;
// chunk swizzle of the point of column h, or of output channel h
__device__ __forceinline__ int swz(int h) { return (h >> 1) & 2; }

template <bool SPLIT>
struct SgMidLds {
  uint4 w[27 * kSgC * 4];                     // [offset][output][chunk of 8 inputs]
  uint4 hi[kSgMPlane], lo[SPLIT ? kSgMPlane : 1];
};

// products of the staged plane: offset plane dz of output z0 (ON0), dz - 1 of
// output z0 + 1 (ON1)
template <bool SPLIT, bool ON0, bool ON1>
__device__ __forceinline__ void sg_mid_plane(const SgMidLds<SPLIT>& sh, int dz, int wv, int li,
                                             int kg, int nt, f32x4 (&acc)[2][4]) {
  const uint4* w = &sh.w[(dz * 9 * kSgC + nt * 16 + li) * 4 + (kg ^ swz(li))];
  struct Frags {
    bf16x8 ah[4], al[4], bw[2];  // points' high parts and remainders, weights [zo]
  };
  int at[3];  // of the wavefront's first row at dx; the other rows and columns lie at fixed distances
#pragma unroll
  for (int dx = 0; dx < 3; ++dx) at[dx] = (2 * wv * kSgMP + li + dx) * 4 + (kg ^ swz(li + dx));
  auto load = [&](int j, Frags& f) {
#pragma unroll
    for (int zo = 0; zo < 2; ++zo)
      if (zo == 0 ? ON0 : ON1) f.bw[zo] = __builtin_bit_cast(bf16x8, w[(j - 9 * zo) * kSgC * 4]);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const int h = at[j % 3] + (((mt >> 1) + j / 3) * kSgMP + (mt & 1) * 16) * 4;
      f.ah[mt] = __builtin_bit_cast(bf16x8, sh.hi[h]);
      if (SPLIT) f.al[mt] = __builtin_bit_cast(bf16x8, sh.lo[h]);
    }
  };
  auto multiply = [&](const Frags& f) {
#pragma unroll
    for (int zo = 0; zo < 2; ++zo) {
      if (!(zo == 0 ? ON0 : ON1)) continue;
#pragma unroll
      for (int part = 0; part < (SPLIT ? 2 : 1); ++part)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
          acc[zo][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(part ? f.al[mt] : f.ah[mt],
                                                                f.bw[zo], acc[zo][mt], 0, 0, 0);
    }
  };
  Frags f[2];
  load(0, f[0]);
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    if (j < 8) load(j + 1, f[(j + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);
    multiply(f[j & 1]);
  }
}

template <bool SPLIT>
__global__ __launch_bounds__(kSgMT) void k_sg_mid(SgGrid g, const float* __restrict__ a,
                                                const uint16_t* __restrict__ w,
                                                const float* __restrict__ b,
                                                float* __restrict__ out, int relu,
                                                const float* __restrict__ mask) {
  constexpr int kLoads = (kSgHalo * (kSgC / 4) + kSgMT - 1) / kSgMT;  // float4 per thread per plane
  constexpr int kWts = 27 * kSgC * 4, kWLoads = (kWts + kSgMT - 1) / kSgMT;  // uint4 of the weights
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  extern __shared__ uint4 mid_lds[];
  SgMidLds<SPLIT>& sh = *reinterpret_cast<SgMidLds<SPLIT>*>(mid_lds);
  const int tiles_x = (g.nx + kSgTX - 1) / kSgTX;
  const int x0 = (int)(blockIdx.x % tiles_x) * kSgTX, y0 = (int)(blockIdx.x / tiles_x) * kSgTY;
  const int z0 = 2 * (int)blockIdx.y, nout = min(2, g.nz - z0);
  const int t = threadIdx.x;
  const int lane = t & 63, wv = (t >> 6) & 3, nt = t >> 8, li = lane & 15, kg = lane >> 4;
  // input planes of the two outputs inside the grid
  const int p_lo = max(0, z0 - 1), p_hi = min(g.nz - 1, z0 + nout);
  int off[kLoads];  // of the thread's values in a plane, the same in every plane
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {
    const int i = t + k * kSgMT, h = i >> 3, hy = h / kSgHX, hx = h - hy * kSgHX;
    off[k] = (wrapi(y0 + hy - 1, g.ny) * g.nx + wrapi(x0 + hx - 1, g.nx)) * (kSgC / 4) + (i & 7);
  }
  float4 pre[kLoads];
  auto load_plane = [&](int gz) {
    const float4* src = reinterpret_cast<const float4*>(a + vox_of(g, gz, 0, 0) * kSgC);
#pragma unroll
    for (int k = 0; k < kLoads; ++k)
      if (t + k * kSgMT < kSgHalo * (kSgC / 4)) pre[k] = src[off[k]];
  };
  auto store_plane = [&]() {
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const int i = t + k * kSgMT;
      if (i < kSgHalo * (kSgC / 4)) {
        const int p = i >> 3, q = i & 7, hy = p / kSgHX, hx = p - hy * kSgHX;
        const int at = (hy * kSgMP + hx) * 4 + ((q >> 1) ^ swz(hx));
        const float4 v = pre[k];
        const bf16x4 hv = {(__bf16)v.x, (__bf16)v.y, (__bf16)v.z, (__bf16)v.w};
        reinterpret_cast<bf16x4*>(&sh.hi[at])[q & 1] = hv;
        if (SPLIT) {
          const bf16x4 lv = {(__bf16)(v.x - (float)hv[0]), (__bf16)(v.y - (float)hv[1]),
                             (__bf16)(v.z - (float)hv[2]), (__bf16)(v.w - (float)hv[3])};
          reinterpret_cast<bf16x4*>(&sh.lo[at])[q & 1] = lv;
        }
      }
    }
  };
  f32x4 acc[2][4];
#pragma unroll
  for (int zo = 0; zo < 2; ++zo)
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) acc[zo][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  load_plane(p_lo);
  {
    const uint4* w4 = reinterpret_cast<const uint4*>(w);
#pragma unroll
    for (int k = 0; k < kWLoads; ++k) {
      const int i = t + k * kSgMT;
      if ((k + 1) * kSgMT <= kWts || i < kWts) sh.w[i ^ swz(i >> 2)] = w4[i];
    }
  }
  for (int p = p_lo; p <= p_hi; ++p) {
    __syncthreads();  // the previous plane has been multiplied
    store_plane();
    __syncthreads();
    if (p < p_hi) load_plane(p + 1);  // the next plane, in flight meanwhile
    // offset dz of this plane for output z0, dz - 1 for output z0 + 1
    const int dz = p - z0 + 1;
    if (dz == 3)
      sg_mid_plane<SPLIT, false, true>(sh, dz, wv, li, kg, nt, acc);
    else if (dz == 0 || nout == 1)
      sg_mid_plane<SPLIT, true, false>(sh, dz, wv, li, kg, nt, acc);
    else
      sg_mid_plane<SPLIT, true, true>(sh, dz, wv, li, kg, nt, acc);
  }
  // D tile of 16 points x 16 channels: lane holds points 4 kg + r, channel li.
  // The mask values of a plane are all requested before the first is used.
  const int co = nt * 16 + li;
  const float bias = b ? b[co] : 0.f;
#pragma unroll
  for (int zo = 0; zo < 2; ++zo) {
    if (zo >= nout) continue;
    const int64_t plane = vox_of(g, z0 + zo, 0, 0) * kSgC;
    float mk[4][4];
    if (mask) {
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int gy = min(y0 + 2 * wv + (mt >> 1), g.ny - 1);
          const int gx = min(x0 + (mt & 1) * 16 + kg * 4 + r, g.nx - 1);
          mk[mt][r] = mask[plane + (gy * g.nx + gx) * kSgC + co];
        }
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const int gy = y0 + 2 * wv + (mt >> 1);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gx = x0 + (mt & 1) * 16 + kg * 4 + r;
        float v = acc[zo][mt][r] + bias;
        if (mask && !(mk[mt][r] > 0.f)) v = 0.f;
        if (relu) v = fmaxf(v, 0.f);
        if (gx < g.nx && gy < g.ny) out[plane + (gy * g.nx + gx) * kSgC + co] = v;
      }
    }
  }
}

// Weight gradient of a kSgC -> kSgC layer: gW[co][ci][o] = sum over points v
// of gr[v][co] a[v + o][ci] (circular in x, y; zero outside in z), and the
// bias gradient, the sum of gr[v][co]. On the matrix cores, M = 16 output
// channels, N = 16 input channels, K = 32 points, each FP32 operand split into
// three BF16 parts x = h + m + l that hold all its 24 bits; of the nine
// products the six above 2^-26 of the whole are formed (v_mfma_f32_16x16x32_bf16),
// 96 cycles for what FP32 operands take 256. The 32 points' sum is formed from
// the smallest products on and then added to the running FP32 sum, one
// rounding for 32 points where FP32 operands round eight times. The split holds
// every bit of operands from about 2^-110 (below, the third part is a subnormal
// BF16 number) to 3.39e38 (above, the first part rounds to infinity and leaves
// a remainder that is not a number, as an infinite operand does).
//
// A workgroup walks tiles of 16 x 8 points up the planes of a column, a share
// of the (tile, plane) steps in order, so that each input plane is staged once
// for its three dz, in a ring of three; the next planes' loads are in flight
// while the current ones are multiplied. Tiles are staged transposed,
// [x][channel] with the eight y of a column as one 16-byte operand (K: four
// columns of eight rows), so that a shift by dx is another column and a shift
// by dy the same operand funnel-shifted with the two halo rows, and 16 lanes
// read 256 contiguous bytes. Each of its twelve wavefronts owns one dz and one
// 16 x 16 channel block for all nine (dy, dx): 54 matrix instructions for 21
// LDS reads. 128 KB of LDS, one workgroup of three wavefronts per SIMD on a
// compute unit.
// 128 x 128 x 8 points: 44.2 us, and 5.5 for the sums; a workgroup per dz, two
// on a compute unit, each staging its planes for itself, took 48.5; FP32
// operands (v_mfma_f32_16x16x4f32) 91 and 20. Without five of the six products
// it takes 24: the rest is the operands' shifts, staging and barriers. Error of
// the gradient against 64 bits 2.8e-8 (256 x 250 x 9 points, depth 3), with
// FP32 operands 3.5e-8, and with one running sum for all products 4.5e-8.
constexpr int kSgWTX = 16, kSgWTY = 8, kSgWHX = kSgWTX + 2;   // its tile
constexpr int kSgWT = 768;                                     // its threads
constexpr int kSgWBlocks = 256;                                // most workgroups, one per compute unit
constexpr int kSgWRow = kSgC * kSgC * 27 + kSgC;               // a row of partial sums: [o][co][ci], bias

struct Bf3 {
  uint32_t p[3];   // two neighbouring rows of one part each
};

__device__ __forceinline__ Bf3 split3(float v0, float v1) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  Bf3 r;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const bf16x2 h = {(__bf16)v0, (__bf16)v1};
    r.p[k] = __builtin_bit_cast(uint32_t, h);
    v0 -= (float)h[0];
    v1 -= (float)h[1];
  }
  return r;
}

struct SgWgradLds {
  static constexpr int kG = kSgWTX * kSgC, kA = kSgWHX * kSgC;  // columns of the tile and its plane
  uint4 g[3][kG];           // [part]
  uint4 a[3][3][kA];        // [plane mod 3][part] rows 0 .. 7
  uint32_t e[3][3][kA];     // halo rows 8 and 9
};

__global__ __launch_bounds__(kSgWT, 3) void k_sg_wgrad(SgGrid g, int each,
                                                        const float* __restrict__ gr,
                                                        const float* __restrict__ a,
                                                        float* __restrict__ part) {
  constexpr int kG = SgWgradLds::kG, kA = SgWgradLds::kA;
  static_assert(kG % 64 == 0 && kG < kSgWT && kG + kA <= 2 * kSgWT, "two items of a thread");
  extern __shared__ uint4 wgrad_lds[];
  SgWgradLds& sh = *reinterpret_cast<SgWgradLds*>(wgrad_lds);
  const int t = threadIdx.x, lane = t & 63, li = lane & 15, kg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int dz = wv >> 2, mt = (wv >> 1) & 1, nt = wv & 1;
  const int tiles_x = (g.nx + kSgWTX - 1) / kSgWTX, tiles_y = (g.ny + kSgWTY - 1) / kSgWTY;
  const int steps = tiles_x * tiles_y * g.nz;
  const int first = blockIdx.x * each, last = min(first + each, steps);
  // A stage brings input plane z + 1 + lead; with lead 0 also the tile of plane
  // z, which is then multiplied. A column's first step is led by the planes
  // below it that lie inside the grid.
  struct Stage {
    int step, x0, y0, z, lead;
  };
  auto column = [&](int step) {
    const int tl = step / g.nz, z = step - tl * g.nz;
    return Stage{step, (tl % tiles_x) * kSgWTX, (tl / tiles_x) * kSgWTY, z, z == 0 ? -1 : -2};
  };
  auto next = [&](Stage s) {
    if (s.lead < 0) {
      ++s.lead;
      return s;
    }
    if (s.z + 1 == g.nz) return column(s.step + 1);
    ++s.step;
    ++s.z;
    return s;
  };
  // Item 0 of the first kG threads is a column of the tile, the others'
  // and item 1 a column of the plane. Every load lies inside its array: out
  // of range, the nearest column or row is read (those of gr become zero when
  // they are staged, those of a meet its zeros).
  float pre[2][kSgWTY + 2];
  auto of_gr = [&](int k) { return k == 0 && wv < kG / 64; };
  auto load = [&](const Stage& s) {
    const uint32_t stride = g.nx * kSgC * sizeof(float);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int i = t + k * kSgWT, c = i & (kSgC - 1);
      if (of_gr(k)) {
        if (s.lead < 0) continue;
        const char* row = reinterpret_cast<const char*>(gr + vox_of(g, s.z, s.y0, 0) * kSgC);
        const uint32_t at = (min(s.x0 + i / kSgC, g.nx - 1) * kSgC + c) * sizeof(float);
#pragma unroll
        for (int r = 0; r < kSgWTY; ++r) {
          pre[k][r] = *reinterpret_cast<const float*>(row + at);
          row += s.y0 + r + 1 < g.ny ? stride : 0;
        }
      } else if (s.z + 1 + s.lead < g.nz && i < kG + kA) {
        int gx = s.x0 + (i - kG) / kSgC - 1;  // x0 - 1 .. x0 + 16
        gx = wrapi(gx, g.nx);
        const uint32_t at = (gx * kSgC + c) * sizeof(float);
        const char* plane = reinterpret_cast<const char*>(a + vox_of(g, s.z + 1 + s.lead, 0, 0) * kSgC);
        int gy = s.y0 == 0 ? g.ny - 1 : s.y0 - 1;
        const char* row = plane + (int64_t)gy * stride;
#pragma unroll
        for (int r = 0; r < kSgWTY + 2; ++r) {
          pre[k][r] = *reinterpret_cast<const float*>(row + at);
          const bool wrap = ++gy == g.ny;
          gy = wrap ? 0 : gy;
          row = wrap ? plane : row + stride;
        }
      }
    }
  };
  double bsum = 0.0;
  auto store = [&](const Stage& s) {
    const int slot = (s.z + 1 + s.lead) % 3;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int i = t + k * kSgWT;
      float* v = pre[k];
      if (of_gr(k)) {
        if (s.lead < 0) continue;
        const bool in = s.x0 + i / kSgC < g.nx;
#pragma unroll
        for (int r = 0; r < kSgWTY; ++r) v[r] = in && s.y0 + r < g.ny ? v[r] : 0.f;
        bsum += (double)(((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])));
        Bf3 p4[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) p4[q] = split3(v[2 * q], v[2 * q + 1]);
#pragma unroll
        for (int p = 0; p < 3; ++p)
          sh.g[p][i] = make_uint4(p4[0].p[p], p4[1].p[p], p4[2].p[p], p4[3].p[p]);
      } else if (s.z + 1 + s.lead < g.nz && i < kG + kA) {
        Bf3 p5[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) p5[q] = split3(v[2 * q], v[2 * q + 1]);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          sh.a[slot][p][i - kG] = make_uint4(p5[0].p[p], p5[1].p[p], p5[2].p[p], p5[3].p[p]);
          sh.e[slot][p][i - kG] = p5[4].p[p];
        }
      }
    }
  };
  f32x4 acc[3][3] = {};   // [dy][dx]
  if (first < last) {
    Stage s = column(first);
    load(s);
    while (s.step < last) {
      __syncthreads();  // the previous stage has been multiplied
      store(s);
      __syncthreads();
      const Stage n = next(s);
      if (n.step < last) load(n);
      const int pz = s.z + dz - 1;  // this wavefront's input plane
      const bool mult = s.lead == 0 && pz >= 0 && pz < g.nz;
      const int slot = (pz + 3) % 3;
      s = n;
      if (!mult) continue;  // the barriers are met by every wavefront
#pragma unroll 1
      for (int st = 0; st < kSgWTX / 4; ++st) {
        const int x = 4 * st + kg;
        bf16x8 A[3];
#pragma unroll
        for (int p = 0; p < 3; ++p)
          A[p] = __builtin_bit_cast(bf16x8, sh.g[p][x * kSgC + mt * 16 + li]);
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
          const int col = (x + dx) * kSgC + nt * 16 + li;
          bf16x8 Bm[3][3];  // [dy][part]
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            const uint4 q = sh.a[slot][p][col];
            const uint32_t e = sh.e[slot][p][col];
            Bm[0][p] = __builtin_bit_cast(bf16x8, q);
            Bm[1][p] = __builtin_bit_cast(
                bf16x8, make_uint4(__builtin_amdgcn_alignbit(q.y, q.x, 16),
                                   __builtin_amdgcn_alignbit(q.z, q.y, 16),
                                   __builtin_amdgcn_alignbit(q.w, q.z, 16),
                                   __builtin_amdgcn_alignbit(e, q.w, 16)));
            Bm[2][p] = __builtin_bit_cast(bf16x8, make_uint4(q.y, q.z, q.w, e));
          }
          // h l, l h, m m, h m, m h, h h of 32 points, then onto the sum
          constexpr int pa[6] = {0, 2, 1, 0, 1, 0}, pb[6] = {2, 0, 1, 1, 0, 0};
          f32x4 s32[3] = {};
#pragma unroll
          for (int j = 0; j < 6; ++j)
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
              s32[dy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[pa[j]], Bm[dy][pb[j]], s32[dy],
                                                                0, 0, 0);
#pragma unroll
          for (int dy = 0; dy < 3; ++dy) acc[dy][dx] += s32[dy];
        }
      }
    }
  }
  // D block: lane holds output channels 16 mt + 4 kg + r, input channel 16 nt + li
  float* P = part + (int64_t)blockIdx.x * kSgWRow;
#pragma unroll
  for (int j = 0; j < 9; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      P[((dz * 9 + j) * kSgC + mt * 16 + 4 * kg + r) * kSgC + nt * 16 + li] = acc[j / 3][j % 3][r];
  double* red = reinterpret_cast<double*>(wgrad_lds);
  __syncthreads();
  if (t < kG) red[t] = bsum;
  __syncthreads();
  if (t < kSgC) {
    double s = 0.0;
    for (int k = 0; k < kG / kSgC; ++k) s += red[k * kSgC + t];
    P[27 * kSgC * kSgC + t] = (float)s;
  }
}

// Weight gradient of the layers with one channel on a side, from their wide
// array a[v][C] and their narrow one x[v]: part[P][o][c] = sum over points v
// of a[v][c] x[v + o] xs (circular in x, y; zero outside in z) for the 27
// offsets, and at o = 27 the plain sum of a[v][c]. The first layer has a =
// its output gradient, x = Q; the last layer a = its input, x = dL/dy, and
// the offsets reversed. FP32 products and sums on the matrix cores
// (v_mfma_f32_16x16x4f32: M = 16 channels, N = 16 offsets, K = 4 points): 32
// channels x 32 columns in four accumulators. A is read once, straight into
// the operand layout (lane li holds channels 2 li and 2 li + 1, so that four
// points are one 512-byte load of the wavefront), x with its halo from LDS.
// A workgroup takes the 32 x 8 tiles blockIdx.x, + P, ..., each of its four
// wavefronts two rows with all sixteen loads in flight, and adds the four
// wavefronts in a fixed order. Bound by reading A: 131 k points in 8.7 us
// (2 TB/s; the sums after it 5 us), where the 32 x 32 kernel of the middle
// layers, fed the narrow array padded to 32 channels, took 91 and 20.
__global__ __launch_bounds__(kT) void k_sg_wgrad_thin(SgGrid g, const float* __restrict__ a,
                                                       const float* __restrict__ x, float xs,
                                                       float* __restrict__ part) {
  __shared__ float sx[3 * kSgHalo];
  __shared__ float red[4][kSgThin];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, li = lane & 15, kq = lane >> 4;
  const int tiles_x = (g.nx + kSgTX - 1) / kSgTX, tiles_y = (g.ny + kSgTY - 1) / kSgTY;
  const int tpp = tiles_x * tiles_y, ntiles = tpp * g.nz;
  // staged position of offset o relative to that of a point's (dz, dy, dx) = (-1, -1, -1)
  auto rel = [](int o) { return (o / 9) * kSgHalo + ((o % 9) / 3) * kSgHX + o % 3; };
  const int r0 = rel(li), r1 = rel(min(16 + li, 26));
  const bool o1 = li < 11;
  const float c1 = li == 11 ? 1.f : 0.f;  // columns 27 (plain sum) and 28 .. 31
  f32x4 acc[2][2] = {};
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int z = tile / tpp, r = tile - z * tpp;
    const int x0 = (r % tiles_x) * kSgTX, y0 = (r / tiles_x) * kSgTY;
    float2 av[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int gy = y0 + 2 * wv + k / 8, gx = x0 + (k % 8) * 4 + kq;
      av[k] = make_float2(0.f, 0.f);
      if (gx < g.nx && gy < g.ny)
        av[k] = reinterpret_cast<const float2*>(a + vox_of(g, z, gy, gx) * kSgC)[li];
    }
    __syncthreads();  // the previous tile has been used
    for (int i = t; i < 3 * kSgHalo; i += kT) {
      const int pl = i / kSgHalo, h = i - pl * kSgHalo;
      const int hy = h / kSgHX, hx = h - hy * kSgHX, gz = z + pl - 1;
      float v = 0.f;
      if (gz >= 0 && gz < g.nz)
        v = x[vox_of(g, gz, wrapi(y0 + hy - 1, g.ny), wrapi(x0 + hx - 1, g.nx))] * xs;
      sx[i] = v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int base = (2 * wv + k / 8) * kSgHX + (k % 8) * 4 + kq;
      const float b0 = sx[base + r0], bx = sx[base + r1], b1 = o1 ? bx : c1;
      acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[k].x, b0, acc[0][0], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[k].y, b0, acc[1][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[k].x, b1, acc[0][1], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[k].y, b1, acc[1][1], 0, 0, 0);
    }
  }
  // D block: lane holds rows 4 kq + r of the (even or odd) channels, column li
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[wv][(c * 16 + li) * kSgC + 2 * (4 * kq + r) + h] = acc[h][c][r];
  __syncthreads();
  for (int e = t; e < kSgThin; e += kT)
    part[(int64_t)blockIdx.x * kSgThin + e] = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
}

// Sum of the thin layers' partial sums part[P][o][c] into W[c][27] (offsets
// reversed for the last layer) and, where bias is given, the plain sums. One
// workgroup per offset, 32 shares of the P sums added in a fixed order (FP64).
__global__ __launch_bounds__(1024) void k_sg_reduce_thin(int P, const float* __restrict__ part,
                                                          int reversed, float* __restrict__ w,
                                                          float* __restrict__ bias) {
  __shared__ double red[32][kSgC];
  const int o = blockIdx.x, c = threadIdx.x & 31, sh = threadIdx.x >> 5;
  double sum = 0.0;
#pragma unroll 8
  for (int p = sh; p < P; p += 32) sum += part[(int64_t)p * kSgThin + o * kSgC + c];
  red[sh][c] = sum;
  __syncthreads();
  if (sh) return;
  sum = 0.0;
  for (int k = 0; k < 32; ++k) sum += red[k][c];
  if (o < 27)
    w[c * 27 + (reversed ? 26 - o : o)] = (float)sum;
  else if (bias)
    bias[c] = (float)sum;
}

// Sum of a middle layer's partial sums part[P][kSgWRow] into its W[co][ci][27]
// and b. A workgroup takes 64 consecutive entries (contiguous loads) and eight shares
// of the rows, added in a fixed order (FP64 throughout).
__global__ __launch_bounds__(512) void k_sg_reduce_w(int P, const float* __restrict__ part,
                                                      float* __restrict__ dst,
                                                      float* __restrict__ bias) {
  __shared__ double red[8][64];
  const int el = threadIdx.x & 63, sh = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + el;
  const int o = e / (kSgC * kSgC), co = (e / kSgC) % kSgC, ci = e % kSgC;
  double sum = 0.0;
  if (e < kSgWRow) {
#pragma unroll 8
    for (int p = sh; p < P; p += 8) sum += part[(int64_t)p * kSgWRow + e];
  }
  red[sh][el] = sum;
  __syncthreads();
  if (sh || e >= kSgWRow) return;
  sum = 0.0;
  for (int k = 0; k < 8; ++k) sum += red[k][el];
  if (o < 27)
    dst[(co * kSgC + ci) * 27 + o] = (float)sum;
  else
    bias[ci] = (float)sum;
}

__device__ __forceinline__ double block_sum(double v, double* red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int s = kT / 2; s > 0; s >>= 1) {
    if (t < s) red[t] += red[t + s];
    __syncthreads();
  }
  return red[0];
}

// Mean-squared loss against t tscale: gy = dL/dy = 2 (y - t tscale) / V;
// per-workgroup sums of squares to part[0 .. P) and of gy to part[P .. 2 P).
__global__ __launch_bounds__(kT) void k_sg_loss(int64_t V, const float* __restrict__ y,
                                                 const float* __restrict__ tg, float tscale,
                                                 float* __restrict__ gy,
                                                 double* __restrict__ part) {
  __shared__ double red[kT];
  double s = 0.0, sg = 0.0;
  const float k = 2.f / (float)V;
  for (int64_t v = (int64_t)blockIdx.x * kT + threadIdx.x; v < V; v += (int64_t)gridDim.x * kT) {
    const float d = y[v] - tg[v] * tscale, kd = k * d;
    s += (double)d * d;
    sg += (double)kd;
    gy[v] = kd;
  }
  s = block_sum(s, red);
  __syncthreads();
  sg = block_sum(sg, red);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = s;
    part[gridDim.x + blockIdx.x] = sg;
  }
}

// block 0: the loss, the mean of squares; block 1: the last layer's bias gradient
__global__ __launch_bounds__(kT) void k_sg_loss_sum(int P, const double* __restrict__ part,
                                                     double scale, double* __restrict__ loss,
                                                     float* __restrict__ bias) {
  __shared__ double red[kT];
  double s = 0.0;
  for (int p = threadIdx.x; p < P; p += kT) s += part[(int64_t)blockIdx.x * P + p];
  s = block_sum(s, red);
  if (threadIdx.x) return;
  if (blockIdx.x == 0)
    *loss = s * scale;
  else
    *bias = (float)s;
}

// per-workgroup sums of |a - b|^2 (b may be null: |a|^2) and |b|^2
__global__ __launch_bounds__(kT) void k_sg_sq2(int64_t n, const float* __restrict__ a,
                                                const float* __restrict__ b,
                                                double* __restrict__ part) {
  __shared__ double red[kT];
  double s0 = 0.0, s1 = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
    const double bv = b ? (double)b[i] : 0.0, d = (double)a[i] - bv;
    s0 += d * d;
    s1 += bv * bv;
  }
  s0 = block_sum(s0, red);
  __syncthreads();
  s1 = block_sum(s1, red);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = s0;
    part[2 * blockIdx.x + 1] = s1;
  }
}

__global__ void k_sg_adam(int64_t n, float* __restrict__ p, const float* __restrict__ g,
                          float* __restrict__ m1, float* __restrict__ m2, float lr_t, float b1,
                          float b2, float eps) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float a = b1 * m1[i] + (1.f - b1) * gi, v = b2 * m2[i] + (1.f - b2) * gi * gi;
  m1[i] = a;
  m2[i] = v;
  p[i] -= lr_t * a / (sqrtf(v) + eps);
}

// middle-layer weights W[co][ci][27] -> forward [27][co][ci] and, for the
// data gradient, [27][ci][co] with the offset reversed; both BF16
__global__ void k_sg_pack_mid(const float* __restrict__ W, uint16_t* __restrict__ wf,
                              uint16_t* __restrict__ wt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 27 * kSgC * kSgC) return;
  const int o = i / (kSgC * kSgC), r = i % (kSgC * kSgC), u = r / kSgC, v = r % kSgC;
  wf[i] = (uint16_t)bf16_bits(W[(u * kSgC + v) * 27 + o]);
  wt[i] = (uint16_t)bf16_bits(W[(v * kSgC + u) * 27 + 26 - o]);
}

// first/last-layer weights [C][27] -> BF16 values (and reversed offsets)
__global__ void k_sg_pack_io(const float* __restrict__ W, float* __restrict__ w,
                             float* __restrict__ wflip) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kSgC * 27) return;
  const int c = i / 27, o = i % 27;
  w[i] = bf16_float(bf16_bits(W[i]));
  if (wflip) wflip[i] = bf16_float(bf16_bits(W[c * 27 + 26 - o]));
}

// SplitMix64 finaliser (Steele, Lea and Flood, 2014) as a counter-based hash
__device__ __host__ __forceinline__ uint64_t mix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__global__ void k_sg_texture(int64_t n, const double* __restrict__ pos, SgTexture tx,
                             double* __restrict__ m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = pos[3 * i], y = pos[3 * i + 1];
  double mx, my, mz;
  if (tx.kind == 0) {
    const uint64_t h1 = mix64(((uint64_t)tx.seed << 32) ^ (uint64_t)(2 * i));
    const uint64_t h2 = mix64(((uint64_t)tx.seed << 32) ^ (uint64_t)(2 * i + 1));
    const double u1 = (double)(h1 >> 11) * 0x1p-53, u2 = (double)(h2 >> 11) * 0x1p-53;
    mz = 2.0 * u1 - 1.0;
    const double r = sqrt(fmax(0.0, 1.0 - mz * mz)), ph = 2.0 * 3.14159265358979323846 * u2;
    mx = r * cos(ph);
    my = r * sin(ph);
  } else if (tx.kind == 1) {
    double dx = x - tx.cx, dy = y - tx.cy;
    dx -= tx.Lx * rint(dx / tx.Lx);
    dy -= tx.Ly * rint(dy / tx.Ly);
    const double r = sqrt(dx * dx + dy * dy);
    mz = tx.pol * exp(-(r * r) / (tx.rc * tx.rc));
    const double ip = sqrt(fmax(0.0, 1.0 - mz * mz));
    if (r > 0.0) {
      mx = -tx.chir * dy / r * ip;
      my = tx.chir * dx / r * ip;
    } else {
      mx = my = 0.0;
      mz = tx.pol;
    }
  } else {
    const double L = tx.nx != 0.0 ? tx.Lx : tx.Ly;
    const double u = x * tx.nx + y * tx.ny - tx.cx;
    const double d1 = u - L * rint(u / L), d2 = (u - 0.5 * L) - L * rint((u - 0.5 * L) / L);
    const double th = fabs(d1) < fabs(d2) ? 2.0 * atan(exp(d1 / tx.rc)) : 2.0 * atan(exp(-d2 / tx.rc));
    const double c = cos(th), s = sin(th);
    mx = c * tx.ed[0] + s * tx.er[0];
    my = c * tx.ed[1] + s * tx.er[1];
    mz = c * tx.ed[2] + s * tx.er[2];
  }
  const double nrm = 1.0 / sqrt(mx * mx + my * my + mz * mz);
  m[3 * i] = mx * nrm;
  m[3 * i + 1] = my * nrm;
  m[3 * i + 2] = mz * nrm;
}

__global__ void k_sg_f32(int64_t n3, const double* __restrict__ a, float* __restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n3) b[i] = (float)a[i];
}

unsigned blocks(int64_t n, int t = kT) { return (unsigned)((n + t - 1) / t); }

dim3 tile_grid(const SgGrid& g) {
  return dim3((unsigned)(((g.nx + kSgTX - 1) / kSgTX) * ((g.ny + kSgTY - 1) / kSgTY)),
              (unsigned)g.nz);
}

template <class T>
hipError_t alloc(T** p, int64_t count) {
  *p = nullptr;
  return hipMalloc((void**)p, (size_t)count * sizeof(T));
}

void launch_mid(const Surrogate* s, hipStream_t st, const float* a, const uint16_t* w,
                const float* b, float* out, int relu, const float* mask) {
  const dim3 grid(tile_grid(s->gd).x, (unsigned)((s->gd.nz + 1) / 2));  // two planes per workgroup
  if (s->split)
    hipLaunchKernelGGL(k_sg_mid<true>, grid, dim3(kSgMT), sizeof(SgMidLds<true>), st, s->gd, a, w, b,
                       out, relu, mask);
  else
    hipLaunchKernelGGL(k_sg_mid<false>, grid, dim3(kSgMT), sizeof(SgMidLds<false>), st, s->gd, a, w, b,
                       out, relu, mask);
}

float* act_of(const Surrogate* s, int l, bool train) {
  return s->act + (int64_t)(train ? l : (l & 1)) * s->nvox * kSgC;
}

// forward pass; the output grid gets (net + b) * ys. ev (or null): events
// recorded before and after every layer, [2 * depth].
void forward(Surrogate* s, hipStream_t st, const float* Q, bool train, float* yout, float ys,
             hipEvent_t* ev = nullptr) {
  const int D = s->depth;
  const dim3 grid = tile_grid(s->gd);
  if (ev) (void)hipEventRecord(ev[0], st);
  hipLaunchKernelGGL(k_sg_in, grid, dim3(kT), 0, st, s->gd, Q, s->s_in, s->win, s->p + s->boff[0],
                     act_of(s, 0, train), 1, (const float*)nullptr);
  if (ev) (void)hipEventRecord(ev[1], st);
  for (int l = 1; l <= D - 2; ++l) {
    if (ev) (void)hipEventRecord(ev[2 * l], st);
    launch_mid(s, st, act_of(s, l - 1, train), s->wmid + (int64_t)(l - 1) * 27 * kSgC * kSgC,
               s->p + s->boff[l], act_of(s, l, train), 1, nullptr);
    if (ev) (void)hipEventRecord(ev[2 * l + 1], st);
  }
  if (ev) (void)hipEventRecord(ev[2 * (D - 1)], st);
  hipLaunchKernelGGL(k_sg_out, grid, dim3(kT), 0, st, s->gd, act_of(s, D - 2, train), s->wout,
                     s->p + s->boff[D - 1], ys, yout);
  if (ev) (void)hipEventRecord(ev[2 * D - 1], st);
}

// weight and bias gradients of a middle layer from its output gradient g
// [V][C] and its input a [V][C]
void layer_grads(Surrogate* s, hipStream_t st, int l, const float* g, const float* a) {
  const SgGrid& gd = s->gd;
  const int steps = ((gd.nx + kSgWTX - 1) / kSgWTX) * ((gd.ny + kSgWTY - 1) / kSgWTY) * gd.nz;
  const int each = (steps + kSgWBlocks - 1) / kSgWBlocks, P = (steps + each - 1) / each;
  hipLaunchKernelGGL(k_sg_wgrad, dim3((unsigned)P), dim3(kSgWT), sizeof(SgWgradLds), st, gd, each, g,
                     a, s->part);
  hipLaunchKernelGGL(k_sg_reduce_w, dim3((unsigned)((kSgWRow + 63) / 64)), dim3(512), 0, st, P,
                     s->part, s->grad + s->woff[l], s->grad + s->boff[l]);
}

// weight gradient of the first (l = 0, with its bias) or last layer from its
// 32-channel array a and its one-channel array x, scaled by xs
void thin_grads(Surrogate* s, hipStream_t st, int l, const float* a, const float* x, float xs) {
  const SgGrid& gd = s->gd;
  const int P = std::min(kSgWPart, (int)tile_grid(gd).x * gd.nz);
  hipLaunchKernelGGL(k_sg_wgrad_thin, dim3((unsigned)P), dim3(kT), 0, st, gd, a, x, xs, s->part);
  hipLaunchKernelGGL(k_sg_reduce_thin, dim3(l == 0 ? 28 : 27), dim3(1024), 0, st, P, s->part,
                     (int)(l != 0), s->grad + s->woff[l], l == 0 ? s->grad + s->boff[0] : nullptr);
}

}  // namespace

hipError_t sg_create(Surrogate* s, int depth, SgGrid gd, int64_t n, const double* pos_host,
                     bool split) {
  s->depth = depth;
  s->split = split;
  s->gd = gd;
  s->nvox = (int64_t)gd.nx * gd.ny * gd.nz;
  s->n = n;
  s->woff.assign(depth, 0);
  s->boff.assign(depth, 0);
  int64_t cur = 0;
  for (int l = 0; l < depth; ++l) {
    const int ci = l == 0 ? 1 : kSgC, co = l == depth - 1 ? 1 : kSgC;
    s->woff[l] = cur;
    cur += (int64_t)co * ci * 27;
    s->boff[l] = cur;
    cur += co;
  }
  s->nparam = cur;
  hipError_t e;
  const int nmid = std::max(0, depth - 2);
  if ((e = alloc(&s->p, cur)) || (e = alloc(&s->grad, cur)) || (e = alloc(&s->m1, cur)) ||
      (e = alloc(&s->m2, cur)))
    return e;
  if ((e = hipMemset(s->m1, 0, cur * 4)) || (e = hipMemset(s->m2, 0, cur * 4))) return e;
  if ((e = alloc(&s->wmid, std::max<int64_t>(1, (int64_t)nmid * 27 * kSgC * kSgC))) ||
      (e = alloc(&s->wmidt, std::max<int64_t>(1, (int64_t)nmid * 27 * kSgC * kSgC))) ||
      (e = alloc(&s->win, kSgC * 27)) || (e = alloc(&s->wout, kSgC * 27)) ||
      (e = alloc(&s->woutt, kSgC * 27)))
    return e;
  if ((e = hipFuncSetAttribute((const void*)k_sg_mid<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sizeof(SgMidLds<true>))) ||
      (e = hipFuncSetAttribute((const void*)k_sg_wgrad, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sizeof(SgWgradLds))) ||
      (e = hipFuncSetAttribute((const void*)k_sg_mid<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sizeof(SgMidLds<false>))))
    return e;
  if ((e = alloc(&s->act, 2 * s->nvox * kSgC))) return e;
  if ((e = alloc(&s->dred, 2 * kRedBlocks + 8))) return e;
  if ((e = alloc(&s->pos, 3 * n)) || (e = alloc(&s->m64, 3 * n)) || (e = alloc(&s->m32, 3 * n)) ||
      (e = alloc(&s->ha, 3 * n)) || (e = alloc(&s->hs, 3 * n)))
    return e;
  return hipMemcpy(s->pos, pos_host, (size_t)n * 3 * sizeof(double), hipMemcpyHostToDevice);
}

hipError_t sg_ensure_training(Surrogate* s, int n_loss) {
  hipError_t e;
  if (!s->trained_buffers) {
    (void)hipFree(s->act);
    s->act = nullptr;
    const int64_t nb = (int64_t)std::max(2, s->depth - 1) * s->nvox * kSgC;
    const int64_t vc = s->nvox * kSgC;
    if ((e = alloc(&s->act, nb)) || (e = alloc(&s->gA, vc)) || (e = alloc(&s->gB, vc)) ||
        (e = alloc(&s->y, s->nvox)) ||
        (e = alloc(&s->gy, s->nvox)) || (e = alloc(&s->qbuf, s->nvox)) ||
        (e = alloc(&s->ubuf, s->nvox)) ||
        (e = alloc(&s->part, std::max<int64_t>((int64_t)kSgWBlocks * kSgWRow, (int64_t)kSgWPart * kSgThin)))) {
      // back to the buffers of inference (none held: sg_apply refuses)
      float** bufs[] = {&s->act, &s->gA, &s->gB, &s->y, &s->gy, &s->qbuf, &s->ubuf, &s->part};
      for (float** b : bufs) {
        (void)hipFree(*b);
        *b = nullptr;
      }
      (void)alloc(&s->act, 2 * s->nvox * kSgC);
      (void)hipGetLastError();
      return e;
    }
    s->trained_buffers = true;
  }
  if (n_loss > s->loss_cap) {
    (void)hipFree(s->loss);
    s->loss = nullptr;
    s->loss_cap = 0;
    if ((e = alloc(&s->loss, n_loss))) return e;
    s->loss_cap = n_loss;
  }
  return hipSuccess;
}

void sg_destroy(Surrogate* s) {
  void* bufs[] = {s->p,   s->grad, s->m1,   s->m2,   s->wmid, s->wmidt, s->win, s->wout,
                  s->woutt, s->act, s->gA,  s->gB,   s->y,    s->gy,
                  s->qbuf, s->ubuf, s->part, s->dred, s->loss, s->pos,  s->m64, s->m32,
                  s->ha,  s->hs};
  for (void* b : bufs)
    if (b) (void)hipFree(b);
  *s = Surrogate{};
}

void sg_default_params(const Surrogate* s, uint64_t seed, std::vector<float>& out) {
  // He-normal weights (variance 2 / fan-in; 1 / fan-in for the linear last
  // layer), zero biases; normal deviates by Box-Muller from the hash above
  out.assign((size_t)s->nparam, 0.f);
  uint64_t ctr = 0;
  auto uni = [&]() { return ((double)(mix64(seed * 0x100000001B3ull + ctr++) >> 11) + 0.5) * 0x1p-53; };
  for (int l = 0; l < s->depth; ++l) {
    const int ci = l == 0 ? 1 : kSgC, co = l == s->depth - 1 ? 1 : kSgC;
    const double sd = std::sqrt((l == s->depth - 1 ? 1.0 : 2.0) / (27.0 * ci));
    for (int64_t k = 0; k < (int64_t)co * ci * 27; ++k) {
      const double u1 = uni(), u2 = uni();
      const double gsn = std::sqrt(-2.0 * std::log(u1)) * std::cos(2.0 * 3.14159265358979323846 * u2);
      out[(size_t)(s->woff[l] + k)] = (float)(sd * gsn);
    }
  }
}

hipError_t sg_set_params(Surrogate* s, const float* host, hipStream_t st) {
  hipError_t e = hipMemcpyAsync(s->p, host, (size_t)s->nparam * 4, hipMemcpyHostToDevice, st);
  if (e) return e;
  if ((e = hipMemsetAsync(s->m1, 0, (size_t)s->nparam * 4, st)) ||
      (e = hipMemsetAsync(s->m2, 0, (size_t)s->nparam * 4, st)))
    return e;
  s->adam_t = 0;
  return sg_pack(s, st);
}

hipError_t sg_pack(Surrogate* s, hipStream_t st) {
  const int D = s->depth;
  hipLaunchKernelGGL(k_sg_pack_io, dim3(blocks(kSgC * 27)), dim3(kT), 0, st, s->p + s->woff[0],
                     s->win, (float*)nullptr);
  hipLaunchKernelGGL(k_sg_pack_io, dim3(blocks(kSgC * 27)), dim3(kT), 0, st, s->p + s->woff[D - 1],
                     s->wout, s->woutt);
  for (int l = 1; l <= D - 2; ++l) {
    const int64_t off = (int64_t)(l - 1) * 27 * kSgC * kSgC;
    hipLaunchKernelGGL(k_sg_pack_mid, dim3(blocks(27 * kSgC * kSgC)), dim3(kT), 0, st,
                       s->p + s->woff[l], s->wmid + off, s->wmidt + off);
  }
  return hipGetLastError();
}

hipError_t sg_get_params(const Surrogate* s, float* host, hipStream_t st) {
  hipError_t e = hipMemcpyAsync(host, s->p, (size_t)s->nparam * 4, hipMemcpyDeviceToHost, st);
  if (e) return e;
  return hipStreamSynchronize(st);
}

hipError_t sg_apply(Surrogate* s, hipStream_t st, const float* Q, float* U) {
  if (!s->act) return hipErrorOutOfMemory;
  forward(s, st, Q, s->trained_buffers, U, s->s_out);
  return hipGetLastError();
}

hipError_t sg_profile(Surrogate* s, hipStream_t st, const float* Q, float* U, int reps, double* ms) {
  if (!s->act) return hipErrorOutOfMemory;
  const int D = s->depth;
  std::vector<hipEvent_t> ev(2 * D, nullptr);
  hipError_t e = hipSuccess;
  for (auto& x : ev)
    if ((e = hipEventCreate(&x))) break;
  for (int l = 0; l < D; ++l) ms[l] = 0.0;
  for (int r = 0; r < reps && e == hipSuccess; ++r) {
    forward(s, st, Q, s->trained_buffers, U, s->s_out, ev.data());
    if ((e = hipGetLastError()) || (e = hipStreamSynchronize(st))) break;
    for (int l = 0; l < D; ++l) {
      float t = 0.f;
      if ((e = hipEventElapsedTime(&t, ev[2 * l], ev[2 * l + 1]))) break;
      ms[l] += (double)t / reps;
    }
  }
  for (auto& x : ev)
    if (x) (void)hipEventDestroy(x);
  return e;
}

hipError_t sg_loss_grad(Surrogate* s, hipStream_t st, const float* Q, const float* tg, float tscale,
                        int slot) {
  const int D = s->depth;
  const SgGrid& gd = s->gd;
  const dim3 grid = tile_grid(gd);
  forward(s, st, Q, true, s->y, 1.f);
  hipLaunchKernelGGL(k_sg_loss, dim3(kRedBlocks), dim3(kT), 0, st, s->nvox, s->y, tg, tscale, s->gy,
                     s->dred);
  hipLaunchKernelGGL(k_sg_loss_sum, dim3(2), dim3(kT), 0, st, kRedBlocks, s->dred,
                     1.0 / (double)s->nvox, s->loss + slot, s->grad + s->boff[D - 1]);
  // last layer
  thin_grads(s, st, D - 1, act_of(s, D - 2, true), s->gy, 1.f);
  hipLaunchKernelGGL(k_sg_in, grid, dim3(kT), 0, st, gd, s->gy, 1.f, s->woutt, (const float*)nullptr,
                     s->gB, 0, act_of(s, D - 2, true));
  float *gcur = s->gB, *gnext = s->gA;
  for (int l = D - 2; l >= 1; --l) {
    layer_grads(s, st, l, gcur, act_of(s, l - 1, true));
    launch_mid(s, st, gcur, s->wmidt + (int64_t)(l - 1) * 27 * kSgC * kSgC, nullptr, gnext, 0,
               act_of(s, l - 1, true));
    std::swap(gcur, gnext);
  }
  thin_grads(s, st, 0, gcur, Q, s->s_in);
  return hipGetLastError();
}

hipError_t sg_adam(Surrogate* s, hipStream_t st, double lr) {
  const double b1 = 0.9, b2 = 0.999;
  s->adam_t++;
  const double lr_t = lr * std::sqrt(1.0 - std::pow(b2, (double)s->adam_t)) /
                      (1.0 - std::pow(b1, (double)s->adam_t));
  hipLaunchKernelGGL(k_sg_adam, dim3(blocks(s->nparam)), dim3(kT), 0, st, s->nparam, s->p, s->grad,
                     s->m1, s->m2, (float)lr_t, (float)b1, (float)b2, 1e-8f);
  return sg_pack(s, st);
}

hipError_t sg_texture(Surrogate* s, hipStream_t st, const SgTexture& tx, double* m_dev) {
  hipLaunchKernelGGL(k_sg_texture, dim3(blocks(s->n)), dim3(kT), 0, st, s->n, s->pos, tx, m_dev);
  return hipGetLastError();
}

hipError_t sg_to_f32(Surrogate* s, hipStream_t st, const double* m64, float* m32) {
  hipLaunchKernelGGL(k_sg_f32, dim3(blocks(3 * s->n)), dim3(kT), 0, st, 3 * s->n, m64, m32);
  return hipGetLastError();
}

hipError_t sg_field_error(Surrogate* s, hipStream_t st, const float* a, const float* b,
                          double* out2) {
  hipLaunchKernelGGL(k_sg_sq2, dim3(kRedBlocks), dim3(kT), 0, st, 3 * s->n, a, b, s->dred);
  std::vector<double> h(2 * kRedBlocks);
  hipError_t e = hipMemcpyAsync(h.data(), s->dred, h.size() * sizeof(double), hipMemcpyDeviceToHost, st);
  if (e || (e = hipStreamSynchronize(st))) return e;
  out2[0] = out2[1] = 0.0;
  for (int i = 0; i < kRedBlocks; ++i) {
    out2[0] += h[2 * i];
    out2[1] += h[2 * i + 1];
  }
  return hipSuccess;
}

hipError_t sg_sumsq(Surrogate* s, hipStream_t st, const float* x, int64_t count, double* out) {
  hipLaunchKernelGGL(k_sg_sq2, dim3(kRedBlocks), dim3(kT), 0, st, count, x, (const float*)nullptr,
                     s->dred);
  std::vector<double> h(2 * kRedBlocks);
  hipError_t e = hipMemcpyAsync(h.data(), s->dred, h.size() * sizeof(double), hipMemcpyDeviceToHost, st);
  if (e || (e = hipStreamSynchronize(st))) return e;
  *out = 0.0;
  for (int i = 0; i < kRedBlocks; ++i) *out += h[2 * i];
  return hipSuccess;
}

}  // namespace pmfem
