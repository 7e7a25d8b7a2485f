// gfx950 FFT kernels of the grid convolution (step 2 of Sec. 3.2.2):
//   k_fft_xy_fwd   real-to-complex FFT along x, FFT along y, per z-plane
//   k_fft_z_mul    FFT along z, multiply by the PGF spectrum, inverse along z
//   k_fft_yx_inv   inverse FFT along y, complex-to-real along x
//   k_r2c_x, k_fft_y, k_c2r_x   the plane passes one axis at a time
//
// Any extent whose prime factors are 2, 3, 5 and 7. Every transform is a
// Stockham autosort in LDS between two buffers, natural order in and out, of
// as few passes as the radices 2 .. 10 allow (FftAxis). Pass with Ns = product
// of the radices done so far and radix R: butterfly j of the n / R reads a_q =
// src[j + q n / R], q < R, multiplies a_q by w^(q k), k = j mod Ns, w = exp(-2 pi i / (Ns R)),
// forms the R-point DFT in registers and writes b_p to
// dst[(j / Ns) Ns R + k + p Ns]. The inverse is the conjugate of the transform
// of the conjugate, so the z pass holds one copy of the passes: on a small grid
// it runs its code once per workgroup, and with two copies took 12.4 us instead
// of 9.3 (64 x 64 x 128, padded). Lanes run over the lines, whose stride
// is odd, so LDS is read and written without bank conflicts and a wavefront
// shares its twiddles; index splits use a float reciprocal, no division.
//
// These transforms move little (60 MB of the 1.03 M unknown composite's 2 GB)
// and are bound by the latency of their LDS passes, so the passes are few, a
// thread has one or two butterflies in each, and where a grid has few planes
// several workgroups share one. Radices above 10 gain a pass at 128 and 256
// points but leave too few threads (radix 16: 52 us at 128^3 against 45 then).
// A workgroup of a small grid spends a third of its time on its one round trip
// to memory, so tables and lines are requested together (Tables).
//
// Radix 2 in place with stride-8 passes (16-way bank conflicts) and mixed
// radices with integer divisions took, us per convolution: 57 at 128^3 points,
// against 43 now; 96^3 70 and 29; 64^3 20.2 and 19.3; 42 x 40 x 15 30 and 16;
// 64 x 64 x 128, z alone periodic, 50 and 40; 256 x 256 x 4 57 and 27. Small
// grids of powers of two are the exception: 32^3 14.3 and 15.6, 16^3 13.2 and
// 13.7, 16 x 16 x 64 15.4 and 16.1.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"
#include "kernels.h"

namespace pmfem {

// ---------------------------------------------------------------------------
// R-point DFTs in registers, exp(-2 pi i / R)

struct Cs {
  float c, s;
};

// cos and sin of 2 pi m / N
template <int N>
__device__ constexpr Cs cs(int m) {
  if constexpr (N == 3) {
    constexpr float c[] = {1.f, -0.49999999999999978f, -0.50000000000000044f};
    constexpr float s[] = {0.f, 0.86602540378443871f, -0.86602540378443837f};
    return Cs{c[m], s[m]};
  } else if constexpr (N == 5) {
    constexpr float c[] = {1.f, 0.30901699437494745f, -0.80901699437494734f, -0.80901699437494756f,
                           0.30901699437494723f};
    constexpr float s[] = {0.f, 0.95105651629515353f, 0.58778525229247325f, -0.58778525229247303f,
                           -0.95105651629515364f};
    return Cs{c[m], s[m]};
  } else if constexpr (N == 6) {
    constexpr float c[] = {1.f, 0.50000000000000011f, -0.49999999999999978f};
    constexpr float s[] = {0.f, 0.8660254037844386f, 0.86602540378443871f};
    return Cs{c[m], s[m]};
  } else if constexpr (N == 7) {
    constexpr float c[] = {1.f, 0.62348980185873359f, -0.22252093395631434f, -0.90096886790241903f,
                           -0.90096886790241915f, -0.22252093395631459f, 0.62348980185873337f};
    constexpr float s[] = {0.f, 0.7818314824680298f, 0.97492791218182362f, 0.43388373911755823f,
                           -0.43388373911755801f, -0.97492791218182362f, -0.78183148246802991f};
    return Cs{c[m], s[m]};
  } else if constexpr (N == 8) {
    constexpr float c[] = {1.f, 0.70710678118654757f, 0.f, -0.70710678118654746f};
    constexpr float s[] = {0.f, 0.70710678118654746f, 1.f, 0.70710678118654757f};
    return Cs{c[m], s[m]};
  } else if constexpr (N == 9) {
    constexpr float c[] = {1.f, 0.76604444311897801f, 0.17364817766693041f, -0.49999999999999978f,
                           -0.93969262078590832f};
    constexpr float s[] = {0.f, 0.64278760968653925f, 0.98480775301220802f, 0.86602540378443871f,
                           0.34202014332566888f};
    return Cs{c[m], s[m]};
  } else if constexpr (N == 10) {
    constexpr float c[] = {1.f, 0.80901699437494745f, 0.30901699437494745f, -0.30901699437494734f,
                           -0.80901699437494734f};
    constexpr float s[] = {0.f, 0.58778525229247314f, 0.95105651629515353f, 0.95105651629515364f,
                           0.58778525229247325f};
    return Cs{c[m], s[m]};
  }
}

__device__ __forceinline__ float2 conj(float2 v) { return make_float2(v.x, -v.y); }

// v times -i
__device__ __forceinline__ float2 quarter(float2 v) { return make_float2(v.y, -v.x); }

// v exp(-2 pi i m / N)
template <int N>
__device__ __forceinline__ float2 twist(float2 v, int m) {
  const Cs w = cs<N>(m);
  if (w.c == 0.f) return quarter(v);  // m = N / 4
  return make_float2(v.x * w.c + v.y * w.s, v.y * w.c - v.x * w.s);
}

__device__ __forceinline__ float2 operator+(float2 a, float2 b) {
  return make_float2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ float2 operator-(float2 a, float2 b) {
  return make_float2(a.x - b.x, a.y - b.y);
}

template <int R>
__device__ __forceinline__ void dft(float2* v);

// R = N1 N2: N2-point DFTs over the stride-N1 subsequences, twiddles, N1-point
// DFTs across them
template <int N1, int N2>
__device__ __forceinline__ void dft_split(float2* v) {
  float2 a[N1][N2];
#pragma unroll
  for (int i = 0; i < N1; ++i) {
#pragma unroll
    for (int k = 0; k < N2; ++k) a[i][k] = v[i + N1 * k];
    dft<N2>(a[i]);
#pragma unroll
    for (int k = 1; k < N2; ++k)
      if (i > 0) a[i][k] = twist<N1 * N2>(a[i][k], i * k);
  }
#pragma unroll
  for (int k = 0; k < N2; ++k) {
    float2 b[N1];
#pragma unroll
    for (int i = 0; i < N1; ++i) b[i] = a[i][k];
    dft<N1>(b);
#pragma unroll
    for (int i = 0; i < N1; ++i) v[k + N2 * i] = b[i];
  }
}

// odd prime R: sums and differences of the pairs (q, R - q)
template <int R>
__device__ __forceinline__ void dft_odd(float2* v) {
  constexpr int H = (R - 1) / 2;
  float2 sum[H], dif[H];
#pragma unroll
  for (int q = 0; q < H; ++q) {
    sum[q] = v[q + 1] + v[R - 1 - q];
    dif[q] = v[q + 1] - v[R - 1 - q];
  }
  float2 all = v[0];
  float2 out[R];
#pragma unroll
  for (int p = 0; p < H; ++p) {
    float2 e = v[0], o = make_float2(0.f, 0.f);
#pragma unroll
    for (int q = 0; q < H; ++q) {
      const Cs w = cs<R>((p + 1) * (q + 1) % R);
      e = make_float2(e.x + w.c * sum[q].x, e.y + w.c * sum[q].y);
      o = make_float2(o.x + w.s * dif[q].x, o.y + w.s * dif[q].y);
    }
    const float2 r = quarter(o);
    out[p + 1] = e + r;
    out[R - 1 - p] = e - r;
    all = all + sum[p];
  }
  out[0] = all;
#pragma unroll
  for (int p = 0; p < R; ++p) v[p] = out[p];
}

template <int R>
__device__ __forceinline__ void dft(float2* v) {
  if constexpr (R == 2) {
    const float2 a = v[0], b = v[1];
    v[0] = a + b;
    v[1] = a - b;
  } else if constexpr (R == 4) {
    const float2 a = v[0] + v[2], b = v[0] - v[2], c = v[1] + v[3], d = quarter(v[1] - v[3]);
    v[0] = a + c;
    v[1] = b + d;
    v[2] = a - c;
    v[3] = b - d;
  } else if constexpr (R == 6) {
    dft_split<2, 3>(v);
  } else if constexpr (R == 8) {
    dft_split<2, 4>(v);
  } else if constexpr (R == 9) {
    dft_split<3, 3>(v);
  } else if constexpr (R == 10) {
    dft_split<2, 5>(v);
  } else {
    dft_odd<R>(v);
  }
}

// ---------------------------------------------------------------------------
// lines in LDS

// line l, element i at l ld + i, the stride ld between lines odd
struct Lines {
  float2* p;
  int ld;
  __device__ __forceinline__ float2& at(int l, int i) const { return p[l * ld + i]; }
};

template <int R>
__device__ __forceinline__ void fft_pass(const Lines& src, const Lines& dst, int Ns, int step,
                                         int lines, const float2* tw) {
  const int nR = step * Ns, total = lines * nR;  // step = n / (Ns R)
  const float iln = recip(lines), iNs = recip(Ns);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int j = fdiv(idx, lines, iln), l = idx - j * lines;
    const int jj = fdiv(j, Ns, iNs), k = j - jj * Ns;
    const float2* s0 = &src.at(l, j);
    float2 v[R];
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = s0[q * nR];
    if (Ns > 1) {
      const int ks = k * step;
#pragma unroll
      for (int q = 1; q < R; ++q) {
        const float2 w = tw[q * ks];  // q k step < n
        v[q] = make_float2(v[q].x * w.x - v[q].y * w.y, v[q].x * w.y + v[q].y * w.x);
      }
    }
    dft<R>(v);
    float2* d0 = &dst.at(l, jj * Ns * R + k);
#pragma unroll
    for (int p = 0; p < R; ++p) d0[p * Ns] = v[p];
  }
}

// Transform of `lines` lines of an axis with passes f, from a to b and back
// pass by pass; the result is in a (the two are swapped as needed).
__device__ __forceinline__ void fft_lines(Lines& a, Lines& b, const FftAxis& f, int lines,
                                          const float2* tw) {
  int Ns = 1;
  for (int p = 0; p < f.np; ++p) {
    const int R = f.rad[p], step = f.step[p];
    switch (R) {
      case 2: fft_pass<2>(a, b, Ns, step, lines, tw); break;
      case 3: fft_pass<3>(a, b, Ns, step, lines, tw); break;
      case 4: fft_pass<4>(a, b, Ns, step, lines, tw); break;
      case 5: fft_pass<5>(a, b, Ns, step, lines, tw); break;
      case 6: fft_pass<6>(a, b, Ns, step, lines, tw); break;
      case 7: fft_pass<7>(a, b, Ns, step, lines, tw); break;
      case 8: fft_pass<8>(a, b, Ns, step, lines, tw); break;
      case 9: fft_pass<9>(a, b, Ns, step, lines, tw); break;
      default: fft_pass<10>(a, b, Ns, step, lines, tw); break;
    }
    Ns *= R;
    __syncthreads();
    const Lines t = a;
    a = b;
    b = t;
  }
}

// The twiddle tables at the start of LDS (a of na values, then b of nb): each
// thread's first value is requested before the lines' loads and stored after
// them, so that a workgroup waits for memory once. With the tables copied
// first a convolution took 17.2 us instead of 15.6 at 32^3 points, 14.9 instead
// of 13.7 at 16^3, 44.9 instead of 42.8 at 128^3.
struct Tables {
  const float2 *a, *b;
  int na, n;
  float2 first;
  __device__ __forceinline__ Tables(const float2* __restrict__ a_, int na_,
                                    const float2* __restrict__ b_, int nb_)
      : a(a_), b(b_), na(na_), n(na_ + nb_), first(make_float2(0.f, 0.f)) {
    if ((int)threadIdx.x < n) first = at(threadIdx.x);
  }
  __device__ __forceinline__ float2 at(int i) const { return i < na ? a[i] : b[i - na]; }
  __device__ __forceinline__ void store(float2* sh) const {
    if ((int)threadIdx.x < n) sh[threadIdx.x] = first;
    for (int i = threadIdx.x + blockDim.x; i < n; i += blockDim.x) sh[i] = at(i);
  }
};

// spectrum of row y (odd: y + 1 of the pair) at k from the complex line of
// the pair: X_y = (Z[k] + conj Z[-k]) / 2, X_{y+1} = (Z[k] - conj Z[-k]) / (2i)
__device__ __forceinline__ float2 row_even(float2 a, float2 b) {
  return make_float2(0.5f * (a.x + b.x), 0.5f * (a.y - b.y));
}
__device__ __forceinline__ float2 row_odd(float2 a, float2 b) {
  return make_float2(0.5f * (a.y + b.y), -0.5f * (a.x - b.x));
}
// conj Z[k], Z = X_y + i X_{y+1}, of a row pair from a = conj X_y[k] and
// b = conj X_{y+1}[k], or in the upper half from their mirror values
__device__ __forceinline__ float2 pair_line(float2 a, float2 b, bool upper) {
  if (upper) {
    a.y = -a.y;
    b.y = -b.y;
  }
  return make_float2(a.x + b.y, a.y - b.x);
}

// ---------------------------------------------------------------------------
// Whole z-planes in LDS. Forward: real rows y < Ny are paired into complex
// lines along x, their half spectra kx < Hx unpacked into columns (zero past
// the rows) and transformed along y; Q[z][y][x] -> spec[z][ky][kx]. nsplit
// workgroups share a plane: each does the x pass and its share of the columns.

__device__ __forceinline__ void fft_xy_fwd_body(const GridParams& g, const float* __restrict__ Q,
                                                float2* __restrict__ spec,
                                                const float2* __restrict__ twx,
                                                const float2* __restrict__ twy, FftPlane pl,
                                                const int blk) {
  extern __shared__ float2 sh[];
  const int Mx = g.M[0], My = g.M[1], Hx = Mx / 2 + 1, Nx = g.N[0], Ny = g.N[1];
  const int pairs = (Ny + 1) / 2, z = blk / pl.nsplit, part = blk - z * pl.nsplit;
  const int kw = (Hx + pl.nsplit - 1) / pl.nsplit, k0 = part * kw, nk = min(Hx, k0 + kw) - k0;
  if (nk <= 0) return;  // the whole workgroup
  float2 *tx = sh, *ty = sh + Mx;
  Lines A = {ty + My, pl.ldx}, B = {ty + My + pl.cap, pl.ldx};
  const Tables tw(twx, Mx, twy, My);
  const int64_t qz = (int64_t)z * Ny * Nx;
  const float iMx = recip(Mx);
  batched<4>(
      pairs * Mx,
      [&](int idx) {
        const int l = fdiv(idx, Mx, iMx), x = idx - l * Mx, y = 2 * l;
        float2 v = make_float2(0.f, 0.f);
        if (x < Nx) {
          v.x = grid_load(Q, qz + (int64_t)y * Nx + x, g);
          if (y + 1 < Ny) v.y = grid_load(Q, qz + (int64_t)(y + 1) * Nx + x, g);
        }
        return v;
      },
      [&](int idx, float2 v) {
        const int l = fdiv(idx, Mx, iMx);
        A.at(l, idx - l * Mx) = v;
      });
  tw.store(sh);
  const float ipr = recip(pairs);
  // the x lines, then (from their buffer into the other one) the columns
#pragma unroll
  for (int axis = 0; axis < 2; ++axis) {
    if (axis == 1) {
      const Lines C = {B.p, pl.ldy};
      for (int idx = threadIdx.x; idx < nk * pairs; idx += blockDim.x) {
        const int c = fdiv(idx, pairs, ipr), l = idx - c * pairs, k = k0 + c, y = 2 * l;
        const float2 a = A.at(l, k), b = A.at(l, k == 0 ? 0 : Mx - k);
        C.at(c, y) = row_even(a, b);
        if (y + 1 < My) C.at(c, y + 1) = y + 1 < Ny ? row_odd(a, b) : make_float2(0.f, 0.f);
      }
      const int pad = My - 2 * pairs;  // rows of zero padding
      if (pad > 0) {
        const float ip = recip(pad);
        for (int idx = threadIdx.x; idx < nk * pad; idx += blockDim.x) {
          const int c = fdiv(idx, pad, ip);
          C.at(c, 2 * pairs + idx - c * pad) = make_float2(0.f, 0.f);
        }
      }
      B = {A.p, pl.ldy};
      A = C;
    }
    __syncthreads();
    fft_lines(A, B, g.fa[axis], axis == 0 ? pairs : nk, axis == 0 ? tx : ty);
  }
  float2* Sz = spec + (int64_t)z * My * Hx;
  const float ink = recip(nk);
  for (int idx = threadIdx.x; idx < My * nk; idx += blockDim.x) {
    const int ky = fdiv(idx, nk, ink), c = idx - ky * nk;
    Sz[ky * Hx + k0 + c] = A.at(c, ky);
  }
}

// Inverse of fft_xy_fwd: inverse FFT along y of the half spectrum columns, the
// rows y < Ny paired into complex lines with their Hermitian half, inverse FFT
// along x; spec[z] -> U[z][y][x]. nsplit workgroups share a plane: each does
// the y pass and its share of the row pairs.
__device__ __forceinline__ void fft_yx_inv_body(const GridParams& g,
                                                const float2* __restrict__ spec,
                                                float* __restrict__ U,
                                                const float2* __restrict__ twx,
                                                const float2* __restrict__ twy, FftPlane pl,
                                                const int blk) {
  extern __shared__ float2 sh[];
  const int Mx = g.M[0], My = g.M[1], Hx = Mx / 2 + 1, Nx = g.N[0], Ny = g.N[1];
  const int pairs = (Ny + 1) / 2, z = blk / pl.nsplit, part = blk - z * pl.nsplit;
  const int lw = (pairs + pl.nsplit - 1) / pl.nsplit, l0 = part * lw, nl = min(pairs, l0 + lw) - l0;
  if (nl <= 0) return;  // the whole workgroup
  float2 *tx = sh, *ty = sh + Mx;
  Lines A = {ty + My, pl.ldy}, B = {ty + My + pl.cap, pl.ldy};
  const Tables tw(twx, Mx, twy, My);
  const float2* Sz = spec + (int64_t)z * My * Hx;
  const float iHx = recip(Hx), inl = recip(nl);
  batched<8>(
      My * Hx, [&](int idx) { return Sz[idx]; },
      [&](int idx, float2 v) {
        const int ky = fdiv(idx, Hx, iHx);
        A.at(idx - ky * Hx, ky) = conj(v);
      });
  tw.store(sh);
#pragma unroll
  for (int axis = 1; axis >= 0; --axis) {
    if (axis == 0) {
      const Lines X = {B.p, pl.ldx};
      for (int idx = threadIdx.x; idx < nl * Mx; idx += blockDim.x) {
        const int k = fdiv(idx, nl, inl), l = idx - k * nl, y = 2 * (l0 + l);
        const int kk = k < Hx ? k : Mx - k;
        const float2 a = A.at(kk, y), b = y + 1 < Ny ? A.at(kk, y + 1) : make_float2(0.f, 0.f);
        X.at(l, k) = pair_line(a, b, k >= Hx);
      }
      B = {A.p, pl.ldx};
      A = X;
    }
    __syncthreads();
    fft_lines(A, B, g.fa[axis], axis == 1 ? Hx : nl, axis == 1 ? ty : tx);
  }
  const int64_t uz = (int64_t)z * Ny * Nx;
  const float iNx = recip(Nx);
  for (int idx = threadIdx.x; idx < nl * Nx; idx += blockDim.x) {
    const int l = fdiv(idx, Nx, iNx), x = idx - l * Nx, y = 2 * (l0 + l);
    const float2 v = A.at(l, x);
    grid_store(U, uz + (int64_t)y * Nx + x, v.x, g);
    if (y + 1 < Ny) grid_store(U, uz + (int64_t)(y + 1) * Nx + x, -v.y, g);
  }
}

// ---------------------------------------------------------------------------
// one axis at a time; LDS: the axis' table and two buffers of `B` lines

// R2C along x: pairs of real rows (y, y + 1) of plane z form one complex line.
// grid [Nz][Ny][Nx] real -> spec [Nz][My][Hx] complex (rows y < Ny written).
__device__ __forceinline__ void r2c_x_body(const GridParams& g, const float* __restrict__ Q,
                                           float2* __restrict__ spec,
                                           const float2* __restrict__ twx, int B, const int blk) {
  extern __shared__ float2 sh[];
  const int Mx = g.M[0], Hx = Mx / 2 + 1, Nx = g.N[0], Ny = g.N[1], ld = fft_stride(Mx);
  Lines A = {sh + Mx, ld}, D = {sh + Mx + B * ld, ld};
  const Tables tw(twx, Mx, nullptr, 0);
  const int pairs = (Ny + 1) / 2;
  const int l0 = blk * B, nl = min(pairs * g.N[2] - l0, B);
  const float iMx = recip(Mx), iHx = recip(Hx), ipr = recip(pairs);
  batched<4>(
      nl * Mx,
      [&](int idx) {
        const int l = fdiv(idx, Mx, iMx), x = idx - l * Mx;
        const int z = fdiv(l0 + l, pairs, ipr), y = 2 * (l0 + l - z * pairs);
        float2 v = make_float2(0.f, 0.f);
        if (x < Nx) {
          v.x = grid_load(Q, ((int64_t)z * Ny + y) * Nx + x, g);
          if (y + 1 < Ny) v.y = grid_load(Q, ((int64_t)z * Ny + y + 1) * Nx + x, g);
        }
        return v;
      },
      [&](int idx, float2 v) {
        const int l = fdiv(idx, Mx, iMx);
        A.at(l, idx - l * Mx) = v;
      });
  tw.store(sh);
  __syncthreads();
  fft_lines(A, D, g.fa[0], nl, sh);
  for (int idx = threadIdx.x; idx < nl * Hx; idx += blockDim.x) {
    const int l = fdiv(idx, Hx, iHx), k = idx - l * Hx;
    const int z = fdiv(l0 + l, pairs, ipr), y = 2 * (l0 + l - z * pairs);
    const float2 a = A.at(l, k), b = A.at(l, k == 0 ? 0 : Mx - k);
    spec[((int64_t)z * g.M[1] + y) * Hx + k] = row_even(a, b);
    if (y + 1 < Ny) spec[((int64_t)z * g.M[1] + y + 1) * Hx + k] = row_odd(a, b);
  }
}

// C2R along x: rows (y, y + 1) of plane z from their half spectra -> U[z][y][x].
__device__ __forceinline__ void c2r_x_body(const GridParams& g, const float2* __restrict__ spec,
                                           float* __restrict__ U, const float2* __restrict__ twx,
                                           int B, const int blk) {
  extern __shared__ float2 sh[];
  const int Mx = g.M[0], Hx = Mx / 2 + 1, Nx = g.N[0], Ny = g.N[1], ld = fft_stride(Mx);
  Lines A = {sh + Mx, ld}, D = {sh + Mx + B * ld, ld};
  const Tables tw(twx, Mx, nullptr, 0);
  const int pairs = (Ny + 1) / 2;
  const int l0 = blk * B, nl = min(pairs * g.N[2] - l0, B);
  const float iHx = recip(Hx), iNx = recip(Nx), ipr = recip(pairs);
  // a thread takes k and its mirror Mx - k of one row pair
  for (int idx = threadIdx.x; idx < nl * Hx; idx += blockDim.x) {
    const int l = fdiv(idx, Hx, iHx), k = idx - l * Hx;
    const int z = fdiv(l0 + l, pairs, ipr), y = 2 * (l0 + l - z * pairs);
    const float2* row = spec + ((int64_t)z * g.M[1] + y) * Hx + k;
    const float2 a = conj(row[0]), b = y + 1 < Ny ? conj(row[Hx]) : make_float2(0.f, 0.f);
    A.at(l, k) = pair_line(a, b, false);
    if (k > 0 && Mx - k >= Hx) A.at(l, Mx - k) = pair_line(a, b, true);
  }
  tw.store(sh);
  __syncthreads();
  fft_lines(A, D, g.fa[0], nl, sh);
  for (int idx = threadIdx.x; idx < nl * Nx; idx += blockDim.x) {
    const int l = fdiv(idx, Nx, iNx), x = idx - l * Nx;
    const int z = fdiv(l0 + l, pairs, ipr), y = 2 * (l0 + l - z * pairs);
    const float2 v = A.at(l, x);
    grid_store(U, ((int64_t)z * Ny + y) * Nx + x, v.x, g);
    if (y + 1 < Ny) grid_store(U, ((int64_t)z * Ny + y + 1) * Nx + x, -v.y, g);
  }
}

// FFT along y of B consecutive columns kx of plane z, in place. Forward: rows
// y < Ny in (the others zero), all My out; inverse: all in, y < Ny out.
__device__ __forceinline__ void fft_y_body(const GridParams& g, float2* __restrict__ spec,
                                           const float2* __restrict__ twy, int B, int inverse,
                                           const int blk) {
  extern __shared__ float2 sh[];
  const int My = g.M[1], Hx = g.M[0] / 2 + 1, ld = fft_stride(My);
  const int n_in = inverse ? My : g.N[1], n_out = inverse ? g.N[1] : My;
  Lines A = {sh + My, ld}, D = {sh + My + B * ld, ld};
  const Tables tw(twy, My, nullptr, 0);
  const int groups = (Hx + B - 1) / B, z = blk / groups;
  const int k0 = (blk - z * groups) * B, nb = min(Hx - k0, B);
  const float inb = recip(nb);
  float2* S = spec + (int64_t)z * My * Hx + k0;
  batched<4>(
      nb * My,
      [&](int idx) {
        const int y = fdiv(idx, nb, inb);
        return y < n_in ? S[y * Hx + idx - y * nb] : make_float2(0.f, 0.f);
      },
      [&](int idx, float2 v) {
        const int y = fdiv(idx, nb, inb);
        A.at(idx - y * nb, y) = inverse ? conj(v) : v;
      });
  tw.store(sh);
  __syncthreads();
  fft_lines(A, D, g.fa[1], nb, sh);
  for (int idx = threadIdx.x; idx < nb * n_out; idx += blockDim.x) {
    const int y = fdiv(idx, nb, inb), c = idx - y * nb;
    const float2 v = A.at(c, y);
    S[y * Hx + c] = inverse ? conj(v) : v;
  }
}

// FFT along z of the lines c = ky Hx + kx (B consecutive per workgroup),
// multiply by the real spectrum khat[kz][c], inverse FFT, write z < Nz.
__device__ __forceinline__ void fft_z_mul_body(const GridParams& g, float2* __restrict__ spec,
                                               const float* __restrict__ khat,
                                               const float2* __restrict__ twz, int B,
                                               const int blk) {
  extern __shared__ float2 sh[];
  const int Mz = g.M[2], Hx = g.M[0] / 2 + 1, ld = fft_stride(Mz), Nz = g.N[2];
  const int64_t plane = (int64_t)g.M[1] * Hx, c0 = (int64_t)blk * B;
  Lines A = {sh + Mz, ld}, D = {sh + Mz + B * ld, ld};
  const Tables tw(twz, Mz, nullptr, 0);
  const int nb = (int)((plane - c0) < B ? (plane - c0) : B);
  const float inb = recip(nb);
  // the first values of the spectrum of K, requested with the lines
  constexpr int KK = 4;
  float kk[KK];
#pragma unroll
  for (int j = 0; j < KK; ++j) {
    const int idx = threadIdx.x + j * blockDim.x;
    const int kz = fdiv(idx, nb, inb);
    kk[j] = idx < nb * Mz ? khat[(int64_t)kz * plane + c0 + idx - kz * nb] : 0.f;
  }
  batched<8>(
      nb * Mz,
      [&](int idx) {
        const int z = fdiv(idx, nb, inb);
        return z < Nz ? spec[(int64_t)z * plane + c0 + idx - z * nb] : make_float2(0.f, 0.f);
      },
      [&](int idx, float2 v) {
        const int z = fdiv(idx, nb, inb);
        A.at(idx - z * nb, z) = v;
      });
  tw.store(sh);
  // the product with K, conjugated for the inverse
  auto scale = [&](int idx, float k) {
    const int kz = fdiv(idx, nb, inb);
    float2& v = A.at(idx - kz * nb, kz);
    v = make_float2(v.x * k, -v.y * k);
  };
#pragma nounroll  // one copy of the passes
  for (int inverse = 0; inverse < 2; ++inverse) {
    if (inverse) {
#pragma unroll
      for (int j = 0; j < KK; ++j) {
        const int idx = threadIdx.x + j * blockDim.x;
        if (idx < nb * Mz) scale(idx, kk[j]);
      }
      for (int idx = threadIdx.x + KK * blockDim.x; idx < nb * Mz; idx += blockDim.x) {
        const int kz = fdiv(idx, nb, inb);
        scale(idx, khat[(int64_t)kz * plane + c0 + idx - kz * nb]);
      }
    }
    __syncthreads();
    fft_lines(A, D, g.fa[2], nb, sh);
  }
  for (int idx = threadIdx.x; idx < nb * Nz; idx += blockDim.x) {
    const int z = fdiv(idx, nb, inb), c = idx - z * nb;
    spec[(int64_t)z * plane + c0 + c] = conj(A.at(c, z));
  }
}

// ---------------------------------------------------------------------------
// kernels: one cell, and the cells of a batch (each workgroup's cell from a
// block-to-cell table)

__global__ void __launch_bounds__(1024) k_fft_xy_fwd(GridParams g, const float* __restrict__ Q,
                                                     float2* __restrict__ spec,
                                                     const float2* __restrict__ twx,
                                                     const float2* __restrict__ twy, FftPlane pl) {
  fft_xy_fwd_body(g, Q, spec, twx, twy, pl, blockIdx.x);
}

__global__ void __launch_bounds__(1024) k_fft_yx_inv(GridParams g, const float2* __restrict__ spec,
                                                     float* __restrict__ U,
                                                     const float2* __restrict__ twx,
                                                     const float2* __restrict__ twy, FftPlane pl) {
  fft_yx_inv_body(g, spec, U, twx, twy, pl, blockIdx.x);
}

__global__ void __launch_bounds__(256) k_r2c_x(GridParams g, const float* __restrict__ Q,
                                               float2* __restrict__ spec,
                                               const float2* __restrict__ twx, int B) {
  r2c_x_body(g, Q, spec, twx, B, blockIdx.x);
}

__global__ void __launch_bounds__(256) k_c2r_x(GridParams g, const float2* __restrict__ spec,
                                               float* __restrict__ U,
                                               const float2* __restrict__ twx, int B) {
  c2r_x_body(g, spec, U, twx, B, blockIdx.x);
}

__global__ void __launch_bounds__(256) k_fft_y(GridParams g, float2* __restrict__ spec,
                                               const float2* __restrict__ twy, int B,
                                               int inverse) {
  fft_y_body(g, spec, twy, B, inverse, blockIdx.x);
}

__global__ void __launch_bounds__(256) k_fft_z_mul(GridParams g, float2* __restrict__ spec,
                                                   const float* __restrict__ khat,
                                                   const float2* __restrict__ twz, int B) {
  fft_z_mul_body(g, spec, khat, twz, B, blockIdx.x);
}

__global__ void __launch_bounds__(1024) k_fft_xy_fwd_cells(const CellTab* __restrict__ tab,
                                                           const int32_t* __restrict__ bcell,
                                                           const int32_t* __restrict__ boff) {
  const int c = bcell[blockIdx.x];
  const CellTab& t = tab[c];
  fft_xy_fwd_body(t.g, t.grid, t.spec, t.twx, t.twy, t.fp, blockIdx.x - boff[c]);
}

__global__ void __launch_bounds__(1024) k_fft_yx_inv_cells(const CellTab* __restrict__ tab,
                                                           const int32_t* __restrict__ bcell,
                                                           const int32_t* __restrict__ boff) {
  const int c = bcell[blockIdx.x];
  const CellTab& t = tab[c];
  fft_yx_inv_body(t.g, t.spec, t.grid, t.twx, t.twy, t.fp, blockIdx.x - boff[c]);
}

__global__ void __launch_bounds__(256) k_r2c_x_cells(const CellTab* __restrict__ tab,
                                                     const int32_t* __restrict__ bcell,
                                                     const int32_t* __restrict__ boff) {
  const int c = bcell[blockIdx.x];
  const CellTab& t = tab[c];
  r2c_x_body(t.g, t.grid, t.spec, t.twx, t.bx, blockIdx.x - boff[c]);
}

__global__ void __launch_bounds__(256) k_c2r_x_cells(const CellTab* __restrict__ tab,
                                                     const int32_t* __restrict__ bcell,
                                                     const int32_t* __restrict__ boff) {
  const int c = bcell[blockIdx.x];
  const CellTab& t = tab[c];
  c2r_x_body(t.g, t.spec, t.grid, t.twx, t.bx, blockIdx.x - boff[c]);
}

__global__ void __launch_bounds__(256) k_fft_y_cells(const CellTab* __restrict__ tab,
                                                     const int32_t* __restrict__ bcell,
                                                     const int32_t* __restrict__ boff,
                                                     int inverse) {
  const int c = bcell[blockIdx.x];
  const CellTab& t = tab[c];
  fft_y_body(t.g, t.spec, t.twy, t.by, inverse, blockIdx.x - boff[c]);
}

__global__ void __launch_bounds__(256) k_fft_z_mul_cells(const CellTab* __restrict__ tab,
                                                         const int32_t* __restrict__ bcell,
                                                         const int32_t* __restrict__ boff) {
  const int c = bcell[blockIdx.x];
  const CellTab& t = tab[c];
  fft_z_mul_body(t.g, t.spec, t.khat, t.twz, t.bz, blockIdx.x - boff[c]);
}

}  // namespace pmfem
