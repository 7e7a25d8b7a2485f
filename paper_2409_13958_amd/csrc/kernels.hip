// gfx950 kernels of the PM-FEM effective-field evaluation.
//
// One H_eff evaluation (paper Eqs. heff, hex, hms_d1 - hms_d3):
//   k_rowdot3      q = D m (Eq. hms_d1); on a second stream u_Z = Z0 m (Eq. hms_d2b)
//   k_anterp_scatter, k_anterp_sum  Q = W^T q      (Sec. 3.2.2, step 1; other forms:
//                  k_anterp_line by grid lines, k_anterp by tiles, both gathers)
//   (fft.hip)      U = (1/4 pi) K * Q             (step 2)
//   k_interp_tile  u = W U + P q + u_Z            (steps 3 and 4)
//   k_exch         H_ex = L m, as differences     (Eqs. hex, lapl_2; second stream)
//   k_mprod        q, u_Z and H_ex in one launch  (small cells; no second stream)
//   k_gsum         H = H_ex - G u (+ H_applied)   (Eq. hms_d3, heff)
// All arithmetic is FP32; every reduction is done in a fixed order inside a
// wavefront or a thread, so results are bitwise reproducible (no atomics).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"
#include "kernels.h"

namespace pmfem {

// ---------------------------------------------------------------------------
// helpers

__device__ __forceinline__ float lagrange(int a, float xi, int p) {
  // basis function a of the Lagrange interpolant through 0..p at xi:
  // prod_{c != a} (xi - c) times 1 / prod_{c != a} (a - c) = (-1)^(p-a) / (a! (p-a)!)
  const float invf[6] = {1.0f, 1.0f, 0.5f, 1.0f / 6.0f, 1.0f / 24.0f, 1.0f / 120.0f};
  float v = ((p - a) & 1 ? -1.0f : 1.0f) * invf[a] * invf[p - a];
  for (int c = 0; c <= p; ++c)
    if (c != a) v *= (xi - (float)c);
  return v;
}

// Cubic (p = 3) Lagrange basis through xi = 0, 1, 2, 3 as a polynomial in the
// centred variable t = xi - 3/2 (|t| <= 3/2, so no cancellation beyond a few
// ulps): L_a(t) = c0 + c1 t + c2 t^2 + c3 t^3.
struct Cubic {
  float c0, c1, c2, c3;
};

__device__ __forceinline__ Cubic cubic_basis(int a) {
  Cubic c;
  c.c0 = (a == 0 || a == 3) ? -0.0625f : 0.5625f;
  c.c1 = a == 0 ? (1.0f / 24.0f) : a == 1 ? -1.125f : a == 2 ? 1.125f : -(1.0f / 24.0f);
  c.c2 = (a == 0 || a == 3) ? 0.25f : -0.25f;
  c.c3 = a == 0 ? -(1.0f / 6.0f) : a == 1 ? 0.5f : a == 2 ? -0.5f : (1.0f / 6.0f);
  return c;
}

__device__ __forceinline__ float cubic_eval(const Cubic& c, float xi) {
  const float t = xi - 1.5f;
  return fmaf(fmaf(fmaf(c.c3, t, c.c2), t, c.c1), t, c.c0);
}

__device__ __forceinline__ void wave_lds_sync() {
  // make this wavefront's LDS writes visible to its own other lanes
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int st_of(uint32_t packed, int axis) {
  return (int)((packed >> (10 * axis)) & 1023u);
}

// cumulative node index of source row `srow` at unwrapped box x (the node
// index of its first node, continued across a periodic wrap)
__device__ __forceinline__ int row_cum(const int32_t* box_start, int64_t srow, int nbx, int per,
                                       int tot, int x) {
  if (per) {
    int wrap = 0;
    if (x < 0) {
      x += nbx;
      wrap = -1;
    } else if (x > nbx) {
      x -= nbx;
      wrap = 1;
    }
    return wrap * tot + box_start[srow + x];
  }
  return box_start[srow + min(max(x, 0), nbx)];
}

// node index of staged element e: rows [base[j], base[j+1]) hold the nodes
// of box row j from cumulative index c0[j] on (wrapping inside the row on a
// periodic x axis, where the row has tot[j] nodes starting at b0[j])
__device__ __forceinline__ int staged_node(int e, int nrow, const int* base, const int* c0,
                                           const int* b0, const int* tot, int per, int& row) {
  int lo = 0, hi = nrow;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (base[mid] <= e) lo = mid;
    else hi = mid;
  }
  row = lo;
  const int c = c0[lo] + (e - base[lo]);
  if (!per) return c;
  int rel = (c - b0[lo]) % tot[lo];
  if (rel < 0) rel += tot[lo];
  return b0[lo] + rel;
}

template <int W>
__device__ __forceinline__ float group_sum(float v) {
  // butterfly sum over groups of W consecutive lanes (W divides 64)
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, W);
  return v;
}

// Entries e0 + lane, e0 + lane + G, ... of a row, K records of a lane in
// flight at once: all K record loads, then the K uses (which issue their
// gathers together). A record past the row end re-reads entry e (valid) and
// is passed on with ok = false; the sum order is the entry order.
template <int G, int K, class Rec, class Use>
__device__ __forceinline__ void row_entries(int e0, int e1, int lane, const Rec* __restrict__ rec,
                                            Use&& use) {
  for (int e = e0 + lane; e < e1; e += K * G) {
    Rec r[K];
#pragma unroll
    for (int k = 0; k < K; ++k) r[k] = rec[e + k * G < e1 ? e + k * G : e];
#pragma unroll
    for (int k = 0; k < K; ++k) use(r[k], e + k * G < e1);
  }
}

// ---------------------------------------------------------------------------
// charges and element-exact correction, G lanes per row, one 16-byte record
// {column, x, y, z} per entry (one vector load):
//   k_charges:  q_n   = sum_k D_nk . m_k     (local pattern)
//   k_zcorr:    u_Z,n = sum_j Z0_nj . m_j     (element-correction pattern)
// The two are independent; the library runs k_zcorr on a second stream,
// beside anterpolation and the FFT.

template <int G>
__device__ __forceinline__ void rowdot3_body(int64_t row, int lane, const float* __restrict__ m,
                                             const int32_t* __restrict__ rp,
                                             const int4* __restrict__ rec,
                                             float* __restrict__ out) {
  float acc = 0.f;
  row_entries<G, 4>(rp[row], rp[row + 1], lane, rec, [&](const int4& r, bool ok) {
    const float* mk = m + 3 * (int64_t)r.x;
    const float m0 = mk[0], m1 = mk[1], m2 = mk[2];
    acc = fmaf(ok ? __int_as_float(r.y) : 0.f, m0, acc);
    acc = fmaf(ok ? __int_as_float(r.z) : 0.f, m1, acc);
    acc = fmaf(ok ? __int_as_float(r.w) : 0.f, m2, acc);
  });
  acc = group_sum<G>(acc);
  if (lane == 0) out[row] = acc;
}

template <int G>
__global__ void __launch_bounds__(256) k_rowdot3(int64_t n, const float* __restrict__ m,
                                                 const int32_t* __restrict__ rp,
                                                 const int4* __restrict__ rec,
                                                 float* __restrict__ out) {
  const int64_t row = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
  if (row >= n) return;  // whole groups leave together
  rowdot3_body<G>(row, threadIdx.x & (G - 1), m, rp, rec, out);
}

template __global__ void k_rowdot3<4>(int64_t, const float*, const int32_t*, const int4*, float*);
template __global__ void k_rowdot3<8>(int64_t, const float*, const int32_t*, const int4*, float*);
template __global__ void k_rowdot3<16>(int64_t, const float*, const int32_t*, const int4*, float*);

// ---------------------------------------------------------------------------
// anterpolation: one workgroup per tile of kAntTX x kAntTY x kAntTZ grid
// points. The nodes of every box whose stencil can reach the tile (the
// tile's halo) are staged once in LDS; then each thread gathers, in a fixed
// order, the contributions of the boxes covering its grid point (per-axis
// box ranges precomputed on the host). No atomics; the sum order per grid
// point is fixed, so the result is reproducible bit for bit.

__device__ void block_exclusive_scan(int* a, int n, int* tmp) {
  // in-place exclusive scan of a[0..n) by blockDim.x threads; tmp holds
  // blockDim.x ints; a[n] receives the total
  const int T = blockDim.x, t = threadIdx.x;
  const int per = (n + T - 1) / T;
  const int lo = t * per, hi = min(n, lo + per);
  int sum = 0;
  for (int i = lo; i < hi; ++i) sum += a[i];
  tmp[t] = sum;
  __syncthreads();
  for (int d = 1; d < T; d <<= 1) {
    int v = (t >= d) ? tmp[t - d] : 0;
    __syncthreads();
    tmp[t] += v;
    __syncthreads();
  }
  int run = tmp[t] - sum;
  for (int i = lo; i < hi; ++i) {
    int c = a[i];
    a[i] = run;
    run += c;
  }
  if (t == T - 1) a[n] = tmp[T - 1];
  __syncthreads();
}

// stencil start of box b along an axis (unwrapped for periodic axes)
__device__ __forceinline__ int box_stencil_start(int b, int N, int p, int per) {
  const int s0 = b - (p - 1) / 2;
  return per ? s0 : min(max(s0, 0), N - p - 1);
}

__global__ void __launch_bounds__(256) k_anterp(
    GridParams g, const float* __restrict__ q, const float4* __restrict__ pos4,
    const int32_t* __restrict__ box_start, const int2* __restrict__ brx,
    const int2* __restrict__ bry, const int2* __restrict__ brz, float* __restrict__ Q) {
  __shared__ int s_off[kAntHalo];
  __shared__ int s_tmp[256];
  __shared__ float4 s_nd[kAntCap];  // xi_x, xi_y, xi_z, q of the staged nodes
  const int ntx = (g.N[0] + kAntTX - 1) / kAntTX, nty = (g.N[1] + kAntTY - 1) / kAntTY;
  const int tile = blockIdx.x;
  const int t0[3] = {(tile % ntx) * kAntTX, ((tile / ntx) % nty) * kAntTY,
                     (tile / (ntx * nty)) * kAntTZ};
  const int te[3] = {min(kAntTX, g.N[0] - t0[0]), min(kAntTY, g.N[1] - t0[1]),
                     min(kAntTZ, g.N[2] - t0[2])};
  const int2* br[3] = {brx, bry, brz};
  int hs[3], hc[3];
  for (int a = 0; a < 3; ++a) {
    const int2 f = br[a][t0[a]], l = br[a][t0[a] + te[a] - 1];
    hs[a] = f.x;
    hc[a] = g.per[a] ? (te[a] - 1) + g.p + 1 : l.x + l.y - f.x;
  }
  const int H = hc[0] * hc[1] * hc[2];
  auto box_of = [&](int h) -> int64_t {
    const int ix = h % hc[0], iy = (h / hc[0]) % hc[1], iz = h / (hc[0] * hc[1]);
    const int bx = (hs[0] + ix) % g.nbox[0], by = (hs[1] + iy) % g.nbox[1],
              bz = (hs[2] + iz) % g.nbox[2];
    return ((int64_t)bz * g.nbox[1] + by) * g.nbox[0] + bx;
  };
  for (int h = threadIdx.x; h < H; h += blockDim.x) {
    const int64_t b = box_of(h);
    s_off[h] = box_start[b + 1] - box_start[b];
  }
  __syncthreads();
  block_exclusive_scan(s_off, H, s_tmp);
  const int total = s_off[H];
  const int lx = threadIdx.x % kAntTX, ly = (threadIdx.x / kAntTX) % kAntTY,
            lz = threadIdx.x / (kAntTX * kAntTY);
  const bool inside = lx < te[0] && ly < te[1] && lz < te[2];
  const int gx = t0[0] + lx, gy = t0[1] + ly, gz = t0[2] + lz;
  if (total == 0) {  // no node reaches this tile (uniform across the block)
    if (inside) grid_store(Q, ((int64_t)gz * g.N[1] + gy) * g.N[0] + gx, 0.f, g);
    return;
  }
  const bool staged = total <= kAntCap;
  if (staged) {
    for (int h = threadIdx.x; h < H; h += blockDim.x) {
      const int64_t b = box_of(h);
      const int k0 = box_start[b], k1 = box_start[b + 1], o = s_off[h];
      for (int k = k0; k < k1; ++k) {
        const float4 pp = pos4[k];
        s_nd[o + k - k0] = make_float4(pp.x, pp.y, pp.z, q[k]);
      }
    }
  }
  __syncthreads();
  if (!inside) return;
  const int2 rx = brx[gx], ry = bry[gy], rz = brz[gz];
  // halo-relative first box of this point's ranges
  const int ox = g.per[0] ? lx : rx.x - hs[0];
  const int oy = g.per[1] ? ly : ry.x - hs[1];
  const int oz = g.per[2] ? lz : rz.x - hs[2];
  float acc = 0.f;
  // stencil index of the point in the k-th box of its range: on a periodic
  // axis the k-th box starts its stencil k - p points before the point; on a
  // non-periodic axis the (clamped) stencil start of that box decides
  for (int iz = 0; iz < rz.y; ++iz) {
    const int az = g.per[2] ? g.p - iz : gz - box_stencil_start(rz.x + iz, g.N[2], g.p, 0);
    for (int iy = 0; iy < ry.y; ++iy) {
      const int ay = g.per[1] ? g.p - iy : gy - box_stencil_start(ry.x + iy, g.N[1], g.p, 0);
      const int hrow = ((oz + iz) * hc[1] + (oy + iy)) * hc[0] + ox;
      for (int ix = 0; ix < rx.y; ++ix) {
        const int ax = g.per[0] ? g.p - ix : gx - box_stencil_start(rx.x + ix, g.N[0], g.p, 0);
        const int k0 = s_off[hrow + ix], k1 = s_off[hrow + ix + 1];
        if (k0 == k1) continue;
        // nodes of one box: all share (ax, ay, az)
        const bool cubic = g.p == 3;
        Cubic cx, cy, cz;
        if (cubic) {
          cx = cubic_basis(ax);
          cy = cubic_basis(ay);
          cz = cubic_basis(az);
        }
        for (int k = k0; k < k1; ++k) {
          float4 nd;
          if (staged) {
            nd = s_nd[k];
          } else {
            const int64_t b = box_of(hrow + ix);
            const int kg = box_start[b] + (k - k0);
            const float4 pp = pos4[kg];
            nd = make_float4(pp.x, pp.y, pp.z, q[kg]);
          }
          const float w = cubic ? cubic_eval(cx, nd.x) * cubic_eval(cy, nd.y) * cubic_eval(cz, nd.z)
                                : lagrange(ax, nd.x, g.p) * lagrange(ay, nd.y, g.p) *
                                      lagrange(az, nd.z, g.p);
          acc = fmaf(nd.w, w, acc);
        }
      }
    }
  }
  grid_store(Q, ((int64_t)gz * g.N[1] + gy) * g.N[0] + gx, acc, g);
}

// ---------------------------------------------------------------------------
// anterpolation by grid lines. A workgroup takes `xa` consecutive points of
// one (y, z) grid line, one thread per point. The boxes whose stencils reach
// the line form at most (p + 1)^2 box rows. Their nodes in the segment's x
// range are listed on the host, column-major (x box outermost, then box row,
// then node order), each entry tagged with its box row; the box table does
// not change between evaluations, so the list is built once. The workgroup
// stages the listed nodes in LDS, each reduced to what the line needs: its
// xi_x and the product c = q L_ay(xi_y) L_az(xi_z) of its charge with its y
// and z weights at the line (a_y, a_z are fixed per box row). A point then
// sums c L_ax(xi_x) over the p + 1 box columns covering it; a_x is fixed per
// column, so the inner loop runs over one contiguous LDS range per column.
// The sum order is fixed (no atomics).

__device__ __forceinline__ float basis(int a, float xi, int p) {
  return p == 3 ? cubic_eval(cubic_basis(a), xi) : lagrange(a, xi, p);
}

__global__ void __launch_bounds__(128) k_anterp_line(
    GridParams g, AntPlan pl, const float* __restrict__ q, const float4* __restrict__ pos4,
    const int32_t* __restrict__ list, const int32_t* __restrict__ lstart,
    const int32_t* __restrict__ colst, const int2* __restrict__ brx,
    const int2* __restrict__ bry, const int2* __restrict__ brz, float* __restrict__ Q) {
  extern __shared__ float4 smem4[];
  unsigned char* smem = reinterpret_cast<unsigned char*>(smem4);
  float2* s_nd = reinterpret_cast<float2*>(smem + pl.o_x);  // (xi_x, c) per listed node
  int* s_col0 = reinterpret_cast<int*>(smem + pl.o_off);    // [sbx + 1] column starts
  int* s_ayz = reinterpret_cast<int*>(smem + pl.o_meta);    // [nrow] a_y | a_z << 8
  const int tid = threadIdx.x, T = blockDim.x;
  const int w = blockIdx.x;
  const int sx = w % pl.nsx, line = w / pl.nsx;
  const int gy = line % g.N[1], gz = line / g.N[1];
  const int x0 = sx * pl.xa, xa = min(pl.xa, g.N[0] - x0);
  const int2 ry = bry[gy], rz = brz[gz];
  const int nrow = ry.y * rz.y;
  const int p = g.p, shift = (p - 1) / 2;
  const int fb = g.per[0] ? x0 - p + shift : brx[x0].x;  // first listed box column
  const int l0 = lstart[w];
  const int n = min(lstart[w + 1] - l0, pl.ncap);
  if (tid < nrow) {
    const int iy = tid % ry.y, iz = tid / ry.y;
    int by = ry.x + iy, bz = rz.x + iz;
    if (by >= g.nbox[1]) by -= g.nbox[1];
    if (bz >= g.nbox[2]) bz -= g.nbox[2];
    int ay = gy - box_stencil_start(by, g.N[1], p, g.per[1]);
    int az = gz - box_stencil_start(bz, g.N[2], p, g.per[2]);
    if (g.per[1]) ay = ((ay % g.N[1]) + g.N[1]) % g.N[1];
    if (g.per[2]) az = ((az % g.N[2]) + g.N[2]) % g.N[2];
    s_ayz[tid] = ay | (az << 8);
  }
  for (int k = tid; k <= pl.sbx; k += T) s_col0[k] = colst[(int64_t)w * (pl.sbx + 1) + k];
  __syncthreads();
  // stage the listed nodes with their y/z weights at this line, K in flight
  {
    constexpr int K = 8;
    for (int e0 = tid; e0 < n; e0 += K * T) {
      int ent[K];
#pragma unroll
      for (int j = 0; j < K; ++j) ent[j] = e0 + j * T < n ? list[l0 + e0 + j * T] : 0;
      float4 nd[K];
      float qq[K];
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int gi = ent[j] & 0x3FFFFFF;
        nd[j] = pos4[gi];
        qq[j] = q[gi];
      }
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int e = e0 + j * T;
        if (e < n) {
          const int ayz = s_ayz[(unsigned)ent[j] >> 26];
          s_nd[e] = make_float2(nd[j].x, qq[j] * basis(ayz & 255, nd[j].y, p) *
                                             basis(ayz >> 8, nd[j].z, p));
        }
      }
    }
  }
  __syncthreads();
  if (tid >= xa) return;
  // gather for the point gx, column by column
  const int gx = x0 + tid;
  const int2 rx = brx[gx];
  const int k0 = g.per[0] ? tid : rx.x - fb;
  const int kc = g.per[0] ? p + 1 : rx.y;
  float acc = 0.f;
  for (int c4 = 0; c4 < kc; ++c4) {
    const int k = k0 + c4;
    const int a = g.per[0] ? p - c4 : gx - box_stencil_start(fb + k, g.N[0], p, 0);
    const int n1 = min(s_col0[k + 1], n);
    if (p == 3) {
      const Cubic cb = cubic_basis(a);
#pragma unroll 2
      for (int e = s_col0[k]; e < n1; ++e) {
        const float2 v = s_nd[e];
        acc = fmaf(v.y, cubic_eval(cb, v.x), acc);
      }
    } else {
      for (int e = s_col0[k]; e < n1; ++e) {
        const float2 v = s_nd[e];
        acc = fmaf(v.y, lagrange(a, v.x, p), acc);
      }
    }
  }
  grid_store(Q, ((int64_t)gz * g.N[1] + gy) * g.N[0] + gx, acc, g);
}

// ---------------------------------------------------------------------------
// anterpolation by scatter. One workgroup of four wavefronts per tile of boxes
// (only tiles with nodes are launched, the fullest first). The tile's nodes,
// listed on the host in box order, are dealt to the four wavefronts in turn
// and taken in batches of 64 per wavefront: each lane forms the p + 1 weights
// per axis of one node of the batch (q times those of x) and leaves them in
// LDS; then the wavefront takes the nodes one by one, a lane owning one
// (a, b, c) point of the stencil (p = 3: 64 points, 64 lanes; larger p: several
// points per lane) and adding q L_a(xi_x) L_b(xi_y) L_c(xi_z) to it in the
// wavefront's own LDS copy of the tile footprint (the grid points the stencils
// of the tile's boxes cover), the next node's weights being read meanwhile.
// Within an instruction the lanes address distinct points, and a wavefront
// takes its nodes in a fixed order, so the sums do not depend on timing. The
// copies are then added in wavefront order and the footprint written out (where
// four copies do not fit in LDS, ScPlan::nw wavefronts take nodes);
// k_anterp_sum adds, for every grid point, the footprints of the (at most two
// per axis) tiles that cover it.
//
// What bounds it is LDS: a read-add-write per node and its latency, so a node
// costs one conflict-free read and write (ScPlan's strides put the 32 points
// of half a wavefront into 32 banks) besides three broadcast reads, and twenty
// wavefronts per compute unit hide the latency. With one wavefront per tile,
// 16 lanes per node and four points per lane, two- to threefold bank conflicts
// and nine wavefronts per compute unit, the composite of 1.03 M unknowns took
// 63 us alone, against 39 us now (25 MB of nodes, 28 MB of footprints); the
// 138 k composite 18 us against 12; a 44 k unknown box, where a wavefront's 61
// nodes in a row are what counts, 17 us against 11.

// L_a(xi) for compile-time p and a
template <int P>
__device__ __forceinline__ float basis_ct(int a, float xi) {
  if constexpr (P == 3) return cubic_eval(cubic_basis(a), xi);
  else return lagrange(a, xi, P);
}

template <int P>
__device__ __forceinline__ void anterp_scatter_body(
    GridParams g, ScPlan pl, const float* __restrict__ q, const float4* __restrict__ rec,
    const int32_t* __restrict__ node, const int32_t* __restrict__ lstart,
    const int32_t* __restrict__ tile, float* __restrict__ part, const int blk) {
  constexpr int P1 = P + 1, NP = P1 * P1 * P1, K = (NP + 63) / 64;
  constexpr int WS = P1 <= 4 ? 4 : 8;           // weights of one axis, padded
  constexpr int NB = P1 <= 4 ? 64 : 32;         // nodes whose weights are held at a time
  extern __shared__ float4 smem4[];
  __shared__ float s_w[kScWaves][3][NB * WS];
  const int lane = threadIdx.x & 63, T = 64 * kScWaves, nw = pl.nw;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l0 = lstart[blk], cnt = lstart[blk + 1] - l0;
  float* out = part + (int64_t)tile[blk] * pl.fsize;
  // thread (wv, lane) holds entry f0 + nw lane + wv of the list: its record
  // {xi_x, xi_y, xi_z, LDS offset of its stencil} lies in list order, only its
  // charge is gathered. The next batch's records and charges and the node
  // indices of the one after are requested while a batch is added.
  const int step = NB * nw;
  const int slot = nw * (lane & (NB - 1)) + wv;
  auto entry = [&](int f0) { return l0 + (f0 + slot < cnt ? f0 + slot : 0); };
  float4 ps = rec[entry(0)];
  int nd = node[entry(0)];
  float qq = slot < cnt ? q[nd] : 0.f;
  nd = node[entry(step)];
  for (int i = threadIdx.x; i < nw * pl.lsize / 4; i += T)
    smem4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  // the lane's stencil points (a, b, c)
  float* acc = reinterpret_cast<float*>(smem4) + (wv < nw ? wv : 0) * pl.lsize;
  int pt[K], pa[K], pb[K], pc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = min(lane + 64 * k, NP - 1);
    pa[k] = i % P1;
    pb[k] = i / P1 % P1;
    pc[k] = i / (P1 * P1);
    pt[k] = pc[k] * pl.sz + pb[k] * pl.sy + pa[k];
  }
  float *wx = s_w[wv][0], *wy = s_w[wv][1], *wz = s_w[wv][2];
  for (int f0 = 0; f0 < cnt && wv < nw; f0 += step) {
    const float4 psn = rec[entry(f0 + step)];
    const float qn = q[nd];
    const float qqn = f0 + step + slot < cnt ? qn : 0.f;
    nd = node[entry(f0 + 2 * step)];
    // this wavefront's nodes of the batch
    const int nb = min(NB, (cnt - f0 - wv + nw - 1) / nw);
    wave_lds_sync();  // the previous batch's weights have been read
    if (lane < NB) {
#pragma unroll
      for (int c = 0; c < P1; ++c) {
        wx[lane * WS + c] = qq * basis_ct<P>(c, ps.x);
        wy[lane * WS + c] = basis_ct<P>(c, ps.y);
        wz[lane * WS + c] = basis_ct<P>(c, ps.z);
      }
    }
    wave_lds_sync();
    float x[K], y[K], z[K];
    auto weights = [&](int i) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        x[k] = wx[i * WS + pa[k]];
        y[k] = wy[i * WS + pb[k]];
        z[k] = wz[i * WS + pc[k]];
      }
    };
    weights(0);
#pragma unroll 4
    for (int i = 0; i < nb; ++i) {
      float* base = acc + __builtin_amdgcn_readlane(__float_as_int(ps.w), i);
      float v[K];
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = base[pt[k]];
      float wxy[K], cz[K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        wxy[k] = x[k] * y[k];
        cz[k] = z[k];
      }
      weights(min(i + 1, NB - 1));
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (lane + 64 * k < NP) base[pt[k]] = fmaf(wxy[k], cz[k], v[k]);
      // keep the next node's reads behind these writes (other lanes' points)
      __builtin_amdgcn_wave_barrier();
    }
    ps = psn;
    qq = qqn;
  }
  __syncthreads();
  const float* s = reinterpret_cast<const float*>(smem4);
  const int FX = pl.fd[0], FXY = FX * pl.fd[1];
  const float ifx = recip(FX), ifxy = recip(FXY);
  for (int i = threadIdx.x; i < pl.fsize; i += T) {
    const int cz = fdiv(i, FXY, ifxy), r = i - cz * FXY, cy = fdiv(r, FX, ifx);
    const int o = cz * pl.sz + cy * pl.sy + (r - cy * FX);
    float v = s[o];
    for (int k = 1; k < nw; ++k) v += s[k * pl.lsize + o];
    out[i] = v;
  }
}

template <int P>
__global__ void __launch_bounds__(64 * kScWaves) k_anterp_scatter(
    GridParams g, ScPlan pl, const float* __restrict__ q, const float4* __restrict__ rec,
    const int32_t* __restrict__ node, const int32_t* __restrict__ lstart,
    const int32_t* __restrict__ tile, float* __restrict__ part) {
  anterp_scatter_body<P>(g, pl, q, rec, node, lstart, tile, part, blockIdx.x);
}

template <int P>
__global__ void __launch_bounds__(64 * kScWaves) k_anterp_scatter_cells(
    const CellTab* __restrict__ tab, const int32_t* __restrict__ bcell,
    const int32_t* __restrict__ boff) {
  const int c = bcell[blockIdx.x];
  const CellTab& t = tab[c];
  anterp_scatter_body<P>(t.g, t.sp, t.q, t.sc_rec, t.sc_node, t.sc_lstart, t.sc_tile,
                         t.sc_part, blockIdx.x - boff[c]);
}

#define PMFEM_ANTERP_SCATTER(P)                                                               \
  template __global__ void k_anterp_scatter<P>(GridParams, ScPlan, const float*, const float4*, \
                                               const int32_t*, const int32_t*,               \
                                               const int32_t*, float*);                      \
  template __global__ void k_anterp_scatter_cells<P>(const CellTab*, const int32_t*,          \
                                                     const int32_t*);
PMFEM_ANTERP_SCATTER(1)
PMFEM_ANTERP_SCATTER(2)
PMFEM_ANTERP_SCATTER(3)
PMFEM_ANTERP_SCATTER(4)
PMFEM_ANTERP_SCATTER(5)

// Q at every grid point: the sum, z tile outermost, then y, then x, of the
// footprint values of the tiles covering it; tab_a[2 g + i] = (tile, offset)
// along axis a, tile < 0 when absent. A thread takes PT consecutive x points
// of one grid line (PT divides Nx), sharing their y and z entries.
template <int PT>
__device__ __forceinline__ void anterp_sum_body(GridParams g, ScPlan pl,
                                                    const int2* __restrict__ tabx,
                                                    const int2* __restrict__ taby,
                                                    const int2* __restrict__ tabz,
                                                    const float* __restrict__ part,
                                                    float* __restrict__ Q, const int blk) {
  const int Nx = g.N[0], Ny = g.N[1];
  const int64_t i0 = ((int64_t)blk * blockDim.x + threadIdx.x) * PT;
  if (i0 >= (int64_t)Nx * Ny * g.N[2]) return;
  const int gx0 = (int)(i0 % Nx);
  const int64_t r = i0 / Nx;
  const int gy = (int)(r % Ny), gz = (int)(r / Ny);
  int2 ex[PT][2];
#pragma unroll
  for (int k = 0; k < PT; ++k) {
    ex[k][0] = tabx[2 * (gx0 + k)];
    ex[k][1] = tabx[2 * (gx0 + k) + 1];
  }
  const int2 ey0 = taby[2 * gy], ey1 = taby[2 * gy + 1];
  const int2 ez0 = tabz[2 * gz], ez1 = tabz[2 * gz + 1];
  const int FX = pl.fd[0], FY = pl.fd[1];
  // all 8 PT candidate values are loaded at once (an absent tile reads entry
  // 0 and counts as zero), so that no load waits behind a branch
  float val[2][2][PT][2];
#pragma unroll
  for (int kz = 0; kz < 2; ++kz) {
    const int2 ez = kz ? ez1 : ez0;
#pragma unroll
    for (int ky = 0; ky < 2; ++ky) {
      const int2 ey = ky ? ey1 : ey0;
      const int64_t t0 = ((int64_t)ez.x * pl.nt[1] + ey.x) * pl.nt[0];
      const int o0 = (ez.y * FY + ey.y) * FX;
#pragma unroll
      for (int k = 0; k < PT; ++k)
#pragma unroll
        for (int kx = 0; kx < 2; ++kx) {
          const int2 e = ex[k][kx];
          const bool ok = ez.x >= 0 && ey.x >= 0 && e.x >= 0;
          val[kz][ky][k][kx] = part[ok ? (t0 + e.x) * pl.fsize + o0 + e.y : 0];
          if (!ok) val[kz][ky][k][kx] = 0.f;
        }
    }
  }
  float sum[PT];
#pragma unroll
  for (int k = 0; k < PT; ++k) {
    sum[k] = 0.f;
#pragma unroll
    for (int kz = 0; kz < 2; ++kz)
#pragma unroll
      for (int ky = 0; ky < 2; ++ky)
#pragma unroll
        for (int kx = 0; kx < 2; ++kx) sum[k] += val[kz][ky][k][kx];
  }
#pragma unroll
  for (int k = 0; k < PT; ++k) grid_store(Q, i0 + k, sum[k], g);
}

template <int PT>
__global__ void __launch_bounds__(256) k_anterp_sum(GridParams g, ScPlan pl,
                                                    const int2* __restrict__ tabx,
                                                    const int2* __restrict__ taby,
                                                    const int2* __restrict__ tabz,
                                                    const float* __restrict__ part,
                                                    float* __restrict__ Q) {
  anterp_sum_body<PT>(g, pl, tabx, taby, tabz, part, Q, blockIdx.x);
}

template <int PT>
__global__ void __launch_bounds__(256) k_anterp_sum_cells(const CellTab* __restrict__ tab,
                                                         const int32_t* __restrict__ bcell,
                                                         const int32_t* __restrict__ boff) {
  const int c = bcell[blockIdx.x];
  const CellTab& t = tab[c];
  anterp_sum_body<PT>(t.g, t.sp, t.sc_tab[0], t.sc_tab[1], t.sc_tab[2], t.sc_part, t.grid,
                      blockIdx.x - boff[c]);
}

template __global__ void k_anterp_sum<1>(GridParams, ScPlan, const int2*, const int2*,
                                         const int2*, const float*, float*);
template __global__ void k_anterp_sum<4>(GridParams, ScPlan, const int2*, const int2*,
                                         const int2*, const float*, float*);
template __global__ void k_anterp_sum_cells<1>(const CellTab*, const int32_t*, const int32_t*);
template __global__ void k_anterp_sum_cells<4>(const CellTab*, const int32_t*, const int32_t*);

// ---------------------------------------------------------------------------
// interpolation + precorrection (steps 3 and 4), tile form. A workgroup
// takes the observer boxes x in [x0, x0 + xs), y = by, z in [z0, z0 + tz).
// Every source box their near regions touch lies in the block
//   x in [x0 - r_b, x0 + xs + r_b), y in [by - r_b, by + r_b],
//   z in [z0 - r_b, z0 + tz + r_b)
// whose nodes are listed on the host column-major: x box column outermost,
// then z, then y, then node order (the box table is fixed, so the list is
// built once). The workgroup stages the charges of its list in LDS. The
// precorrection values of every row are stored in the matching order (x
// offset, then z, then y), so the near columns of a row are 2 r_b + 1
// contiguous runs of the staged charges, one per x offset; each row carries
// the (start, length) of its runs. The (p + 1) y-lines of U over the tile's z
// range are staged too. Each group of G lanes then takes one observer row:
// u_n = W_n U + sum over the runs of P q + u_Z, in a fixed order.
//
// A row's values are one padded array (each run rounded up to 4 values with
// zeros), read as 4-value chunks: lane l of the group takes chunks l, l + G,
// ..., the first KC of them held in registers at once, so the lanes stay busy
// whatever the run lengths are; a chunk finds its run from the cumulative
// chunk counts of the row.

// five waves per SIMD (at most 96 registers) where the row state fits them
// without spilling, else four
#define PMFEM_IC_OCC __attribute__((amdgpu_waves_per_eu(WT * KC <= 30 ? 5 : 4)))
template <int WT, int KC>
__device__ __forceinline__ void interp_tile_body(
    GridParams g, IcPlan pl, const float* __restrict__ U, const float4* __restrict__ pos4,
    const int32_t* __restrict__ list, const int32_t* __restrict__ lstart,
    const int32_t* __restrict__ wseg, const uint32_t* __restrict__ rdesc,
    const int32_t* __restrict__ prp, const float* __restrict__ pval,
    const float* __restrict__ q, const float* __restrict__ uz, float* __restrict__ u, const int blk) {
  extern __shared__ float4 smem4[];
  unsigned char* smem = reinterpret_cast<unsigned char*>(smem4);
  float* s_q = reinterpret_cast<float*>(smem + pl.o_q);   // staged charges
  float* s_U = reinterpret_cast<float*>(smem + pl.o_u);   // [uzl][p + 1][ux]
  int* s_seg = reinterpret_cast<int*>(smem + pl.o_seg);   // [tz + 1] row prefix, [tz] first row
  const int tid = threadIdx.x, T = blockDim.x;
  const int nby = g.nbox[1];
  const int p = g.p, p1 = p + 1;
  // [0, pl.tz]: row prefix over the z segments; [pl.tz + 1, 2 pl.tz]: first
  // row of each; then the tile (only tiles with rows are launched, the
  // fullest first)
  const int segw = 2 * pl.tz + 2;
  const int w = wseg[(int64_t)blk * segw + segw - 1];
  const int sx = w % pl.nsx, rest = w / pl.nsx;
  const int by = rest % nby, sz = rest / nby;
  const int x0 = sx * pl.xs, z0 = sz * pl.tz;
  const int tz = min(pl.tz, g.nbox[2] - z0);
  for (int i = tid; i < segw - 1; i += T) s_seg[i] = wseg[(int64_t)blk * segw + i];
  const int l0 = lstart[blk];
  const int n = min(lstart[blk + 1] - l0, pl.qcap);
  // the first list entries are requested before the potential lines are
  // staged, so that both wait on memory together
  constexpr int KQ = 8;
  int gi[KQ];
#pragma unroll
  for (int j = 0; j < KQ; ++j) gi[j] = tid + j * T < n ? list[l0 + tid + j * T] : 0;
  // stencil lines of U: z-lines [stz(z0), stz(z0) + tz + p), y-lines [sty, sty + p]
  const int ux0 = box_stencil_start(x0, g.N[0], p, g.per[0]);
  const int sty = box_stencil_start(by, g.N[1], p, g.per[1]);
  const int stz = box_stencil_start(z0, g.N[2], p, g.per[2]);
  {
    // thread -> one x point t of the lines l = l00, l00 + lpp, ... (lpp whole
    // lines per pass); y and z follow l incrementally, so no division per value
    const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
    const int ux = pl.ux, nl = pl.uzl * p1, lpp = T / ux;
    const int l00 = tid / ux, t = tid - l00 * ux;
    if (l00 < lpp) {
      // a periodic line wraps at most once (ux, p + 1 and uzl never exceed N)
      int x = ux0 + t;
      if (g.per[0]) x = x < 0 ? x + Nx : (x >= Nx ? x - Nx : x);
      const bool okx = x < Nx;
      const int wy = g.per[1] ? Ny : 0, wz = g.per[2] ? Nz : 0;
      const int dly = lpp % p1, dlz = lpp / p1;
      int ly = l00 % p1, lz = l00 / p1;
      constexpr int KU = 8;
      for (int l0 = l00; l0 < nl; l0 += KU * lpp) {
        float v[KU];
#pragma unroll
        for (int k = 0; k < KU; ++k) {
          int y = sty + ly, z = stz + lz;
          y += y < 0 ? wy : 0;
          y -= y >= Ny ? wy : 0;
          z += z < 0 ? wz : 0;
          z -= z >= Nz ? wz : 0;
          const bool ok = okx && z < Nz && l0 + k * lpp < nl;
          v[k] = ok ? grid_load(U, (int64_t)(z * Ny + y) * Nx + x, g) : 0.f;
          ly += dly;
          lz += dlz;
          if (ly >= p1) {
            ly -= p1;
            ++lz;
          }
        }
#pragma unroll
        for (int k = 0; k < KU; ++k)
          if (l0 + k * lpp < nl) s_U[(l0 + k * lpp) * ux + t] = v[k];
      }
    }
  }
  // stage the listed charges, KQ loads in flight, the next list entries
  // requested while the charges arrive; 4 zeros after them
  if (tid < 4) s_q[n + tid] = 0.f;
  for (int e0 = tid; e0 < n; e0 += KQ * T) {
    float v[KQ];
#pragma unroll
    for (int j = 0; j < KQ; ++j) v[j] = q[gi[j]];
    const int e1 = e0 + KQ * T;
#pragma unroll
    for (int j = 0; j < KQ; ++j) gi[j] = e1 + j * T < n ? list[l0 + e1 + j * T] : 0;
#pragma unroll
    for (int j = 0; j < KQ; ++j)
      if (e0 + j * T < n) s_q[e0 + j * T] = v[j];
  }
  __syncthreads();
  const int nrows = s_seg[tz];
  const int* s_first = s_seg + pl.tz + 1;

  // rows: G lanes per row; the next row's descriptors are fetched while the
  // current row is formed
  constexpr int G = kIcLanes;
  constexpr int W = WT;                 // 2 r_b + 1
  const int lane = tid & (G - 1), grp = tid / G, ngrp = T / G;
  const bool cubic = p == 3;
  // lane-constant parts of the interpolation weights (p = 3): lane -> x point
  // ax = lane % 4 and the NY = 16 / G y points from ay0 = NY (lane / 4)
  constexpr int NY = 16 / G;
  const int ax = lane & 3, ay0 = (lane >> 2) * NY;
  const Cubic cbx = cubic_basis(ax);
  Cubic cby[NY];
#pragma unroll
  for (int i = 0; i < NY; ++i) cby[i] = cubic_basis(ay0 + i);
  // slot sl of the tile -> its row: segment kz by bisection over the prefix
  // (pl.tz is a power of two; prefix entries past the tile equal nrows)
  auto fetch = [&](int sl, uint32_t* dsc, int& pp, float4& xi, int& r) {
    int kz = 0;
    for (int s = pl.tz >> 1; s > 0; s >>= 1) kz = s_seg[kz + s] <= sl ? kz + s : kz;
    r = s_first[kz] + (sl - s_seg[kz]);
#pragma unroll
    for (int dx = 0; dx < W; ++dx) dsc[dx] = rdesc[(int64_t)r * W + dx];
    pp = prp[r];
    xi = pos4[r];
  };
  uint32_t dsc[W];
  int pp = 0, r = 0;
  float4 xi = make_float4(0.f, 0.f, 0.f, 0.f);
  if (grp < nrows) fetch(grp, dsc, pp, xi, r);
  for (int sl = grp; sl < nrows; sl += ngrp) {
    // cumulative chunk counts cb of the runs and the staged index of chunk j
    // of run d, qb_d + 4 j with qb_d = start_d - 4 cb_d, kept as qb_0 and the
    // steps dq_d = qb_d - qb_(d-1) (a sum of selects, not an indexed array)
    int cb[W + 1], dq[W];
    cb[0] = 0;
    int qprev = 0;
#pragma unroll
    for (int d = 0; d < W; ++d) {
      const int qbd = (int)(dsc[d] & 0xFFFFu) - 4 * cb[d];
      dq[d] = qbd - qprev;
      qprev = qbd;
      cb[d + 1] = cb[d] + (((int)(dsc[d] >> 16) + 3) >> 2);
    }
    const int C = cb[W];
    // the first KC chunks of every lane in flight at once; a chunk past the
    // row reads valid (finite) values of the next rows, or the zeros that pad
    // the matrix, and pairs them with the zeros after the staged charges
    const float4* prow = reinterpret_cast<const float4*>(pval + pp) + lane;
    float4 v[KC];
#pragma unroll
    for (int t = 0; t < KC; ++t) v[t] = prow[G * t];
    uint32_t dn[W];
    int ppn = 0, rn = 0;
    float4 xin = make_float4(0.f, 0.f, 0.f, 0.f);
    if (sl + ngrp < nrows) fetch(sl + ngrp, dn, ppn, xin, rn);
    float acc = 0.f;
    // padding values are zero and 4 zeros follow the staged charges, so the
    // 4 products of a chunk need no per-value test
    auto chunk = [&](int j, const float4& pv) {
      int b = dq[0] + 4 * j;
#pragma unroll
      for (int d = 1; d < W; ++d) b += j >= cb[d] ? dq[d] : 0;
      const float* sq = s_q + (j < C ? b : n);
      acc = fmaf(pv.x, sq[0], acc);
      acc = fmaf(pv.y, sq[1], acc);
      acc = fmaf(pv.z, sq[2], acc);
      acc = fmaf(pv.w, sq[3], acc);
    };
#pragma unroll
    for (int t = 0; t < KC; ++t) chunk(lane + G * t, v[t]);
    for (int j = lane + G * KC; j < C; j += G) chunk(j, prow[j - lane]);
    // W U from the staged lines; the box of the row from its packed coordinates
    const uint32_t bc = __float_as_uint(xi.w);
    const int bx = (int)(bc & 1023u), bz = (int)((bc >> 20) & 1023u);
    const int relx = g.per[0] ? bx - x0 : box_stencil_start(bx, g.N[0], p, 0) - ux0;
    const int relz = g.per[2] ? bz - z0 : box_stencil_start(bz, g.N[2], p, 0) - stz;
    if (cubic) {
      const int zs = p1 * pl.ux;
      const float* su = s_U + (relz * p1 + ay0) * pl.ux + relx + ax;
      const float wz0 = cubic_eval(cubic_basis(0), xi.z), wz1 = cubic_eval(cubic_basis(1), xi.z);
      const float wz2 = cubic_eval(cubic_basis(2), xi.z), wz3 = cubic_eval(cubic_basis(3), xi.z);
      float sy = 0.f;
#pragma unroll
      for (int i = 0; i < NY; ++i) {
        const float* s0 = su + i * pl.ux;
        const float t = wz0 * s0[0] + wz1 * s0[zs] + wz2 * s0[2 * zs] + wz3 * s0[3 * zs];
        sy = fmaf(cubic_eval(cby[i], xi.y), t, sy);
      }
      acc = fmaf(cubic_eval(cbx, xi.x), sy, acc);
    } else {
      const int nst = p1 * p1 * p1;
      for (int l = lane; l < nst; l += G) {
        const int lx = l % p1, ly = (l / p1) % p1, lz = l / (p1 * p1);
        acc = fmaf(lagrange(lx, xi.x, p) * lagrange(ly, xi.y, p) * lagrange(lz, xi.z, p),
                   s_U[((relz + lz) * p1 + ly) * pl.ux + relx + lx], acc);
      }
    }
    acc = group_sum<G>(acc);
    if (lane == 0) u[r] = acc + uz[r];
#pragma unroll
    for (int dx = 0; dx < W; ++dx) dsc[dx] = dn[dx];
    pp = ppn;
    xi = xin;
    r = rn;
  }
}

template <int WT, int KC>
__global__ void __launch_bounds__(256) PMFEM_IC_OCC k_interp_tile(
    GridParams g, IcPlan pl, const float* __restrict__ U, const float4* __restrict__ pos4,
    const int32_t* __restrict__ list, const int32_t* __restrict__ lstart,
    const int32_t* __restrict__ wseg, const uint32_t* __restrict__ rdesc,
    const int32_t* __restrict__ prp, const float* __restrict__ pval,
    const float* __restrict__ q, const float* __restrict__ uz, float* __restrict__ u) {
  interp_tile_body<WT, KC>(g, pl, U, pos4, list, lstart, wseg, rdesc, prp, pval, q, uz, u,
                           blockIdx.x);
}

template <int WT, int KC>
__global__ void __launch_bounds__(256) PMFEM_IC_OCC k_interp_tile_cells(
    const CellTab* __restrict__ tab, const int32_t* __restrict__ bcell,
    const int32_t* __restrict__ boff) {
  const int c = bcell[blockIdx.x];
  const CellTab& t = tab[c];
  interp_tile_body<WT, KC>(t.g, t.icp, t.grid, t.pos4, t.ic_list, t.ic_lstart, t.ic_wseg,
                           t.ic_rdesc, t.prp, t.pv, t.q, t.uz, t.u, blockIdx.x - boff[c]);
}

#define PMFEM_INTERP_TILE(WT, KC)                                                             \
  template __global__ void k_interp_tile<WT, KC>(                                             \
      GridParams, IcPlan, const float*, const float4*, const int32_t*, const int32_t*,        \
      const int32_t*, const uint32_t*, const int32_t*, const float*, const float*, const float*, \
      float*);                                                                                \
  template __global__ void k_interp_tile_cells<WT, KC>(const CellTab*, const int32_t*,        \
                                                       const int32_t*);
#define PMFEM_INTERP_TILES(WT) \
  PMFEM_INTERP_TILE(WT, 2)     \
  PMFEM_INTERP_TILE(WT, 4)     \
  PMFEM_INTERP_TILE(WT, 6)     \
  PMFEM_INTERP_TILE(WT, 8)
PMFEM_INTERP_TILES(1)
PMFEM_INTERP_TILES(3)
PMFEM_INTERP_TILES(5)
PMFEM_INTERP_TILES(7)
#undef PMFEM_INTERP_TILE

// ---------------------------------------------------------------------------
// exchange and gradient over the shared local pattern, G lanes per row:
//   k_exch:  H_ex,n = sum_k L_nk (m_k - m_n)         (records {col, L})
//   k_gsum:  H_n = H_ex,n - sum_k G_nk u_k + H_applied  (records {col, Gx, Gy, Gz})
// The exchange needs only m, so the library runs it on the second stream
// beside the grid steps; k_gsum then adds the magnetostatic gradient.

template <int G, typename MT>
__device__ __forceinline__ void exch_body(int64_t row, int lane, const int32_t* __restrict__ rp,
                                          const int2* __restrict__ lrec,
                                          const MT* __restrict__ m, float* __restrict__ hex) {
  // difference form: the rows of L sum to zero (constants are in its null
  // space), so H_ex,n = sum_k L_nk (m_k - m_n); a uniform m gives exactly
  // zero and the FP32 rounding scales with the variation of m, not with m.
  // With an FP64 m (MT = double) the differences are formed before the one
  // rounding to FP32, so the rounding of m itself, which the exchange
  // operator would amplify by its largest eigenvalue, never enters.
  const MT* mn = m + 3 * row;
  const MT n0 = mn[0], n1 = mn[1], n2 = mn[2];
  float hx = 0.f, hy = 0.f, hz = 0.f;
  row_entries<G, 4>(rp[row], rp[row + 1], lane, lrec, [&](const int2& r, bool ok) {
    const MT* mk = m + 3 * (int64_t)r.x;
    const float d0 = (float)(mk[0] - n0), d1 = (float)(mk[1] - n1), d2 = (float)(mk[2] - n2);
    const float w = ok ? __int_as_float(r.y) : 0.f;
    hx = fmaf(w, d0, hx);
    hy = fmaf(w, d1, hy);
    hz = fmaf(w, d2, hz);
  });
  hx = group_sum<G>(hx);
  hy = group_sum<G>(hy);
  hz = group_sum<G>(hz);
  if (lane == 0) {
    hex[3 * row] = hx;
    hex[3 * row + 1] = hy;
    hex[3 * row + 2] = hz;
  }
}

template <int G, typename MT>
__global__ void __launch_bounds__(256) k_exch(int64_t n, const int32_t* __restrict__ rp,
                                              const int2* __restrict__ lrec,
                                              const MT* __restrict__ m,
                                              float* __restrict__ hex) {
  const int64_t row = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
  if (row >= n) return;  // whole groups leave together
  exch_body<G, MT>(row, threadIdx.x & (G - 1), rp, lrec, m, hex);
}

// Every product that needs only m in one launch: workgroups [0, nbl) the
// charges, [nbl, nbl + nbz) the element correction, the rest (none without
// exchange) the exchange, each row summed as in its own kernel, so the
// results are the same bits. For cells whose stages are shorter than the
// events that fork a second stream and join it again (a fork and join around
// three empty kernels takes 31 us against 4.6 us in line): on the 20 x 20 x
// 2 nm film three launches of 2.7 us and the events become one of 3 us.
template <int GL, int GZ, typename MT>
__global__ void __launch_bounds__(256) k_mprod(int64_t n, unsigned nbl, unsigned nbz, MProd a,
                                               const float* __restrict__ m,
                                               const MT* __restrict__ mx) {
  const unsigned b = blockIdx.x;
  if (b >= nbl && b < nbl + nbz) {
    const int64_t row = ((int64_t)(b - nbl) * blockDim.x + threadIdx.x) / GZ;
    if (row < n) rowdot3_body<GZ>(row, threadIdx.x & (GZ - 1), m, a.zrp, a.zrec, a.uz);
    return;
  }
  const unsigned bl = b < nbl ? b : b - nbl - nbz;
  const int64_t row = ((int64_t)bl * blockDim.x + threadIdx.x) / GL;
  if (row >= n) return;
  if (b < nbl) rowdot3_body<GL>(row, threadIdx.x & (GL - 1), m, a.lrp, a.drec, a.q);
  else exch_body<GL, MT>(row, threadIdx.x & (GL - 1), a.lrp, a.lrec, mx, a.hex);
}

template <int G>
__global__ void __launch_bounds__(256) k_gsum(int64_t n, const int32_t* __restrict__ rp,
                                              const int4* __restrict__ grec,
                                              const float* __restrict__ u,
                                              const float* __restrict__ hex,
                                              float* __restrict__ h, float hax, float hay,
                                              float haz, int with_hex, int with_ms) {
  const int64_t row = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
  const int lane = threadIdx.x & (G - 1);
  if (row >= n) return;  // whole groups leave together
  float hx = 0.f, hy = 0.f, hz = 0.f;
  if (with_ms) {
    row_entries<G, 4>(rp[row], rp[row + 1], lane, grec, [&](const int4& r, bool ok) {
      const float uv = u[r.x];
      const float uk = ok ? uv : 0.f;
      hx = fmaf(-__int_as_float(r.y), uk, hx);
      hy = fmaf(-__int_as_float(r.z), uk, hy);
      hz = fmaf(-__int_as_float(r.w), uk, hz);
    });
    hx = group_sum<G>(hx);
    hy = group_sum<G>(hy);
    hz = group_sum<G>(hz);
  }
  if (lane == 0) {
    if (with_hex) {
      hx += hex[3 * row];
      hy += hex[3 * row + 1];
      hz += hex[3 * row + 2];
    }
    h[3 * row] = hx + hax;
    h[3 * row + 1] = hy + hay;
    h[3 * row + 2] = hz + haz;
  }
}

#define PMFEM_LOCAL_KERNELS(G)                                                                  \
  template __global__ void k_exch<G, float>(int64_t, const int32_t*, const int2*, const float*,   \
                                            float*);                                             \
  template __global__ void k_exch<G, double>(int64_t, const int32_t*, const int2*, const double*, \
                                             float*);                                            \
  template __global__ void k_gsum<G>(int64_t, const int32_t*, const int4*, const float*,         \
                                     const float*, float*, float, float, float, int, int);
PMFEM_LOCAL_KERNELS(4)
PMFEM_LOCAL_KERNELS(8)
PMFEM_LOCAL_KERNELS(16)
#undef PMFEM_LOCAL_KERNELS

#define PMFEM_MPROD(GL, GZ)                                                                  \
  template __global__ void k_mprod<GL, GZ, float>(int64_t, unsigned, unsigned, MProd,         \
                                                  const float*, const float*);               \
  template __global__ void k_mprod<GL, GZ, double>(int64_t, unsigned, unsigned, MProd,        \
                                                   const float*, const double*);
PMFEM_MPROD(4, 4)
PMFEM_MPROD(4, 8)
PMFEM_MPROD(4, 16)
PMFEM_MPROD(8, 4)
PMFEM_MPROD(8, 8)
PMFEM_MPROD(8, 16)
PMFEM_MPROD(16, 4)
PMFEM_MPROD(16, 8)
PMFEM_MPROD(16, 16)
#undef PMFEM_MPROD

// ---------------------------------------------------------------------------
// LLG (unit-vector Landau-Lifshitz form), classic RK4 in FP64

// the FP32 copy of m
__global__ void k_rk_stage(int64_t n, const double* __restrict__ m, float* __restrict__ m32) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 3 * n) m32[i] = (float)m[i];
}

// The slope of stage k and the vector of the next one: the slope at mst goes into
// acc, and m + c k into the next stage's mst (in place of this one's) and m32.
// One launch instead of two, and the slope itself goes to no array of its own:
// with small cells a step is bound by its launches.
__global__ void k_rk_next(int64_t n, const double* __restrict__ m, const double* mcur,
                          const float* __restrict__ h, double pref, double alpha, double weight,
                          int first, double c, double* mst, float* __restrict__ m32,
                          double* __restrict__ acc) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double mx = mcur[3 * i], my = mcur[3 * i + 1], mz = mcur[3 * i + 2];
  double hx = h[3 * i], hy = h[3 * i + 1], hz = h[3 * i + 2];
  double cx = my * hz - mz * hy, cy = mz * hx - mx * hz, cz = mx * hy - my * hx;   // m x H
  double dx = my * cz - mz * cy, dy = mz * cx - mx * cz, dz = mx * cy - my * cx;   // m x (m x H)
  double kx = pref * (cx + alpha * dx), ky = pref * (cy + alpha * dy), kz = pref * (cz + alpha * dz);
  if (first) {
    acc[3 * i] = weight * kx;
    acc[3 * i + 1] = weight * ky;
    acc[3 * i + 2] = weight * kz;
  } else {
    acc[3 * i] += weight * kx;
    acc[3 * i + 1] += weight * ky;
    acc[3 * i + 2] += weight * kz;
  }
  const double x = m[3 * i] + c * kx, y = m[3 * i + 1] + c * ky, z = m[3 * i + 2] + c * kz;
  mst[3 * i] = x;
  mst[3 * i + 1] = y;
  mst[3 * i + 2] = z;
  m32[3 * i] = (float)x;
  m32[3 * i + 1] = (float)y;
  m32[3 * i + 2] = (float)z;
}

// the last stage's slope, the step m + dt / 6 (acc + k) and its norm, and the
// FP32 copy that the next step starts from
__global__ void k_rk_last(int64_t n, double* __restrict__ m, const double* __restrict__ mst,
                          const float* __restrict__ h, double pref, double alpha,
                          const double* __restrict__ acc, double dt6, float* __restrict__ m32) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double mx = mst[3 * i], my = mst[3 * i + 1], mz = mst[3 * i + 2];
  double hx = h[3 * i], hy = h[3 * i + 1], hz = h[3 * i + 2];
  double cx = my * hz - mz * hy, cy = mz * hx - mx * hz, cz = mx * hy - my * hx;
  double dx = my * cz - mz * cy, dy = mz * cx - mx * cz, dz = mx * cy - my * cx;
  double kx = pref * (cx + alpha * dx), ky = pref * (cy + alpha * dy), kz = pref * (cz + alpha * dz);
  double x = m[3 * i] + dt6 * (acc[3 * i] + kx);
  double y = m[3 * i + 1] + dt6 * (acc[3 * i + 1] + ky);
  double z = m[3 * i + 2] + dt6 * (acc[3 * i + 2] + kz);
  double r = 1.0 / sqrt(x * x + y * y + z * z);
  x *= r;
  y *= r;
  z *= r;
  m[3 * i] = x;
  m[3 * i + 1] = y;
  m[3 * i + 2] = z;
  m32[3 * i] = (float)x;
  m32[3 * i + 1] = (float)y;
  m32[3 * i + 2] = (float)z;
}

// energy partial sums: block b writes {sum mu m.Hex, sum q u}
// ---------------------------------------------------------------------------
// Implicit LLG steps (Sec. 2.2: implicit time stepping with a Newton
// iteration and a preconditioned Krylov solver). One step solves
//   G(x) = x - r - dt f(mb) = 0,   mb = (1 - theta) m + theta x,
//   f(v) = c [v x H(v) + alpha v x (v x H(v))],  c = -gamma0 / (1 + alpha^2),
// with r = m, theta = 1/2 for the midpoint rule and r a combination of past
// states, dt the step times the BDF coefficient, theta = 1 for BDF; by
// Newton, the linear systems dG/dx d = G by GMRES with the Jacobian applied
// matrix-free (the field is linear in m, H(v) = A v + H_app):
//   dG/dx w = w - theta dt c [w x H + mb x (A w)
//                            + alpha (w x (mb x H) + mb x (w x H) + mb x (mb x (A w)))].
// All vectors are FP64; A w is one FP32 field evaluation. (Below, "m" of
// the residual kernel is r.)

__device__ __forceinline__ void cross3(double ax, double ay, double az, double bx, double by,
                                       double bz, double& cx, double& cy, double& cz) {
  cx = ay * bz - az * by;
  cy = az * bx - ax * bz;
  cz = ax * by - ay * bx;
}

// the evaluation point mb = (1 - theta) m + theta x (theta = 1/2: the
// midpoint rule; theta = 1: BDF, mb = x) and its FP32 copy for the field
__global__ void k_mid_point(int64_t n3, const double* __restrict__ m, const double* __restrict__ x,
                            double theta, double* __restrict__ mb, float* __restrict__ mb32) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n3) return;
  const double v = theta == 1.0 ? x[i] : (1.0 - theta) * m[i] + theta * x[i];
  mb[i] = v;
  mb32[i] = (float)v;
}

// Residual G at the field H of the evaluation point and, per node, the inverse of the 3x3
// diagonal block of dG/dx with A replaced by its exchange diagonal a_n
// (the block-inverse preconditioner); part[b] = block b's share of |G|^2,
// summed in a fixed order (grid-stride, then a tree in LDS).
__global__ void __launch_bounds__(256) k_mid_residual(int64_t n, const double* __restrict__ m,
                                                      const double* __restrict__ x,
                                                      const double* __restrict__ mb,
                                                      const float* __restrict__ H,
                                                      const double* __restrict__ adiag, double dt,
                                                      double c, double alpha, double theta,
                                                      double* __restrict__ G,
                                                      double* __restrict__ Minv,
                                                      double* __restrict__ part) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double bx = mb[3 * i], by = mb[3 * i + 1], bz = mb[3 * i + 2];
    const double hx = H[3 * i], hy = H[3 * i + 1], hz = H[3 * i + 2];
    double px, py, pz, qx, qy, qz;
    cross3(bx, by, bz, hx, hy, hz, px, py, pz);   // mb x H
    cross3(bx, by, bz, px, py, pz, qx, qy, qz);   // mb x (mb x H)
    const double gx = x[3 * i] - m[3 * i] - dt * c * (px + alpha * qx);
    const double gy = x[3 * i + 1] - m[3 * i + 1] - dt * c * (py + alpha * qy);
    const double gz = x[3 * i + 2] - m[3 * i + 2] - dt * c * (pz + alpha * qz);
    G[3 * i] = gx;
    G[3 * i + 1] = gy;
    G[3 * i + 2] = gz;
    acc += gx * gx + gy * gy + gz * gz;
    // columns of the block: D e_k = e_k x H + a mb x e_k
    //   + alpha (e_k x (mb x H) + mb x (e_k x H) + a mb x (mb x e_k))
    const double a = adiag[i];
    double B[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double ex = k == 0, ey = k == 1, ez = k == 2;
      double t1x, t1y, t1z, t2x, t2y, t2z, t3x, t3y, t3z, t4x, t4y, t4z, t5x, t5y, t5z, ux, uy, uz;
      cross3(ex, ey, ez, hx, hy, hz, t1x, t1y, t1z);        // e x H
      cross3(bx, by, bz, ex, ey, ez, t2x, t2y, t2z);        // mb x e
      cross3(ex, ey, ez, px, py, pz, t3x, t3y, t3z);        // e x (mb x H)
      cross3(bx, by, bz, t1x, t1y, t1z, t4x, t4y, t4z);     // mb x (e x H)
      cross3(bx, by, bz, t2x, t2y, t2z, t5x, t5y, t5z);     // mb x (mb x e)
      ux = t1x + a * t2x + alpha * (t3x + t4x + a * t5x);
      uy = t1y + a * t2y + alpha * (t3y + t4y + a * t5y);
      uz = t1z + a * t2z + alpha * (t3z + t4z + a * t5z);
      const double s = -theta * dt * c;
      B[0][k] = (k == 0) + s * ux;
      B[1][k] = (k == 1) + s * uy;
      B[2][k] = (k == 2) + s * uz;
    }
    // inverse by the adjugate
    const double c00 = B[1][1] * B[2][2] - B[1][2] * B[2][1];
    const double c01 = B[1][2] * B[2][0] - B[1][0] * B[2][2];
    const double c02 = B[1][0] * B[2][1] - B[1][1] * B[2][0];
    const double det = B[0][0] * c00 + B[0][1] * c01 + B[0][2] * c02;
    const double r = 1.0 / det;
    double* Mi = Minv + 9 * i;
    Mi[0] = c00 * r;
    Mi[1] = (B[0][2] * B[2][1] - B[0][1] * B[2][2]) * r;
    Mi[2] = (B[0][1] * B[1][2] - B[0][2] * B[1][1]) * r;
    Mi[3] = c01 * r;
    Mi[4] = (B[0][0] * B[2][2] - B[0][2] * B[2][0]) * r;
    Mi[5] = (B[0][2] * B[1][0] - B[0][0] * B[1][2]) * r;
    Mi[6] = c02 * r;
    Mi[7] = (B[0][1] * B[2][0] - B[0][0] * B[2][1]) * r;
    Mi[8] = (B[0][0] * B[1][1] - B[0][1] * B[1][0]) * r;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// x / |x| per node (an accepted adaptive step: the rule keeps |m| only up to
// the Newton residual, which is an rms over all nodes, so a few nodes could
// otherwise drift over many steps)
__global__ void k_mid_normalize(int64_t n, double* __restrict__ x) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double a = x[3 * i], b = x[3 * i + 1], c = x[3 * i + 2];
  const double r = 1.0 / sqrt(a * a + b * b + c * c);
  x[3 * i] = a * r;
  x[3 * i + 1] = b * r;
  x[3 * i + 2] = c * r;
}

// GMRES of the implicit solver. The Krylov basis V is held in FP32 (its
// rounding, 6e-8 relative, lies below the relative residual GMRES is asked
// for, and each basis vector is one FP32 field evaluation's input anyway); w
// and every sum are FP64, each sum in a fixed order (grid-stride per thread, a
// fixed shuffle tree per wavefront, the four wavefronts in order, then
// sum_rows over the workgroups).
//
// Around a field evaluation a vector takes five launches and one wait of the
// host. What bounds them on the cells that such steps are made of (a few ten
// thousand unknowns) is their number and the host's waits, not their bytes:
// nothing sums the workgroups' shares in a launch of its own - each workgroup
// of the reader sums all of them, in the same order - and whether the second
// pass of the Gram-Schmidt is needed is read on the device.
// Film of 12 k unknowns, one step of 7 vectors: 1120 us with a launch per
// operation, a copy and a wait per pass, 805 us so; 138 k unknowns and 25
// vectors 5150 and 4570, 1.03 M and 26 vectors 21.4 and 19.6 ms.
//
// Rows of part (stride nparts), for nv basis vectors: [0, nv) V_j . w,
// nv: |w|^2, nv + 1: |w|^2 after the first pass, nv + 2: after the second,
// nv + 3 + j: V_j . w of the second pass.
constexpr int kGsChunk = 16;

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
  return v;
}

// out[r] = sum over b < nparts of part[r * nparts + b] for r < rows, by all 256
// threads: 16 lanes a row, each with 16 loads in flight. With one load behind
// the other's addition a kernel waited some 10 us for the shares of 512
// workgroups: k_gs_update at 138 k nodes and 8 vectors took 17 us, now 8.
__device__ __forceinline__ void sum_rows(const double* __restrict__ part, int nparts, int rows,
                                         double* out) {
  const int l = threadIdx.x & 15;
  for (int r = threadIdx.x >> 4; r < rows; r += 16) {
    const double* p = part + (int64_t)r * nparts;
    double v = 0.0;
    for (int b = l; b < nparts; b += 16 * 16) {
      double x[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) x[k] = b + 16 * k < nparts ? p[b + 16 * k] : 0.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) v += x[k];
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 16);
    if (l == 0) out[r] = v;
  }
  __syncthreads();
}

// the first pass removed more than half of |w|^2: w has lost orthogonality
__device__ __forceinline__ bool gs_again(double ww, double w2) { return w2 < 0.5 * ww; }

// w = dG/dx z of one node, with Az = A z from one FP32 field evaluation
__device__ __forceinline__ void mid_jvp(const MidJvp& a, int64_t i, double* __restrict__ w) {
  const double bx = a.mb[3 * i], by = a.mb[3 * i + 1], bz = a.mb[3 * i + 2];
  const double hx = a.H[3 * i], hy = a.H[3 * i + 1], hz = a.H[3 * i + 2];
  const double zx = a.z[3 * i], zy = a.z[3 * i + 1], zz = a.z[3 * i + 2];
  const double ax = a.Az[3 * i], ay = a.Az[3 * i + 1], az = a.Az[3 * i + 2];
  double px, py, pz, t1x, t1y, t1z, t2x, t2y, t2z, t3x, t3y, t3z, t4x, t4y, t4z, t5x, t5y, t5z;
  cross3(bx, by, bz, hx, hy, hz, px, py, pz);          // mb x H
  cross3(zx, zy, zz, hx, hy, hz, t1x, t1y, t1z);       // z x H
  cross3(bx, by, bz, ax, ay, az, t2x, t2y, t2z);       // mb x (A z)
  cross3(zx, zy, zz, px, py, pz, t3x, t3y, t3z);       // z x (mb x H)
  cross3(bx, by, bz, t1x, t1y, t1z, t4x, t4y, t4z);    // mb x (z x H)
  cross3(bx, by, bz, t2x, t2y, t2z, t5x, t5y, t5z);    // mb x (mb x (A z))
  w[0] = zx + a.s * (t1x + t2x + a.alpha * (t3x + t4x + t5x));
  w[1] = zy + a.s * (t1y + t2y + a.alpha * (t3y + t4y + t5y));
  w[2] = zz + a.s * (t1z + t2z + a.alpha * (t3z + t4z + t5z));
}

// block b's share of V_j . w for j < nv, a node's three components per thread;
// JVP: w = dG/dx z is formed first, and |w|^2 is one more row (j = nv)
template <bool JVP>
__device__ __forceinline__ void gs_dots_body(int64_t n, const MidJvp& a,
                                             const float* __restrict__ V, int64_t ldv, int nv,
                                             double* __restrict__ w, double* __restrict__ part) {
  __shared__ double red[4][kGsChunk];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int rows = nv + (JVP ? 1 : 0);
  for (int j0 = 0; j0 < rows; j0 += kGsChunk) {
    const int jn = min(kGsChunk, rows - j0);
    double acc[kGsChunk];
#pragma unroll
    for (int k = 0; k < kGsChunk; ++k) acc[k] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
      double x[3];
      if (JVP && j0 == 0) {
        mid_jvp(a, i, x);
        w[3 * i] = x[0];
        w[3 * i + 1] = x[1];
        w[3 * i + 2] = x[2];
      } else {
        x[0] = w[3 * i];
        x[1] = w[3 * i + 1];
        x[2] = w[3 * i + 2];
      }
#pragma unroll
      for (int k = 0; k < kGsChunk; ++k) {
        const int j = j0 + k;
        if (k < jn) {
          if (j < nv) {
            const float* Vj = V + (int64_t)j * ldv + 3 * i;
            acc[k] = fma((double)Vj[0], x[0], acc[k]);
            acc[k] = fma((double)Vj[1], x[1], acc[k]);
            acc[k] = fma((double)Vj[2], x[2], acc[k]);
          } else {
            acc[k] = fma(x[0], x[0], acc[k]);
            acc[k] = fma(x[1], x[1], acc[k]);
            acc[k] = fma(x[2], x[2], acc[k]);
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kGsChunk; ++k) {
      if (k < jn) {
        const double sv = wave_sum_d(acc[k]);
        if (lane == 0) red[wv][k] = sv;
      }
    }
    __syncthreads();
    if ((int)threadIdx.x < jn)
      part[(int64_t)(j0 + threadIdx.x) * gridDim.x + blockIdx.x] =
          ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
    __syncthreads();
  }
}

// w = dG/dx z and its products with the basis
__global__ void __launch_bounds__(256) k_gs_jvp_dots(int64_t n, MidJvp a,
                                                     const float* __restrict__ V, int64_t ldv,
                                                     int nv, double* __restrict__ w,
                                                     double* __restrict__ part) {
  gs_dots_body<true>(n, a, V, ldv, nv, w, part);
}

// the products of the second pass, where it is needed
__global__ void __launch_bounds__(256) k_gs_dots_again(int64_t n, const float* __restrict__ V,
                                                       int64_t ldv, int nv,
                                                       double* __restrict__ w,
                                                       double* __restrict__ part) {
  __shared__ double nrm[2];
  sum_rows(part + (int64_t)nv * gridDim.x, gridDim.x, 2, nrm);
  if (!gs_again(nrm[0], nrm[1])) return;
  gs_dots_body<false>(n, MidJvp{}, V, ldv, nv, w, part + (int64_t)(nv + 3) * gridDim.x);
}

// w -= sum_j h[j] V_j (j < nv, ascending) with the first (pass 0) or second
// pass's products, and block b's share of |w|^2 after it; out[j] = h[j]
__global__ void __launch_bounds__(256) k_gs_update(int64_t n3, const float* __restrict__ V,
                                                   int64_t ldv, int nv, int pass,
                                                   double* __restrict__ w,
                                                   double* __restrict__ part,
                                                   double* __restrict__ out) {
  __shared__ double hs[kGsMaxVectors];
  __shared__ double red[4];
  const int64_t P = gridDim.x;
  if (pass) {
    sum_rows(part + nv * P, (int)P, 2, hs);
    const bool again = gs_again(hs[0], hs[1]);
    __syncthreads();
    if (!again) return;
  }
  sum_rows(part + (pass ? nv + 3 : 0) * P, (int)P, nv, hs);
  if (blockIdx.x == 0)
    for (int j = threadIdx.x; j < nv; j += blockDim.x) out[j] = hs[j];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n3;
       i += (int64_t)gridDim.x * blockDim.x) {
    double v = w[i];
    for (int j = 0; j < nv; ++j) v = fma(-hs[j], (double)V[(int64_t)j * ldv + i], v);
    w[i] = v;
    acc = fma(v, v, acc);
  }
  const double sv = wave_sum_d(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sv;
  __syncthreads();
  if (threadIdx.x == 0)
    part[(nv + 1 + pass) * P + blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// the next basis vector v = w / |w| in FP32 and its preconditioned
// z = Minv v with its FP32 copy. |w|^2 is the one row of part (nv = 0: the
// residual) or, of the rows nv, nv + 1 and nv + 2, the last pass's.
// out: |w|^2 before, after the first and after the second pass (nv = 0: out[0])
__global__ void __launch_bounds__(256) k_gs_next(int64_t n, const double* __restrict__ w,
                                                 const double* __restrict__ Minv,
                                                 const double* __restrict__ part, int nparts,
                                                 int nv, float* __restrict__ v,
                                                 double* __restrict__ z, float* __restrict__ z32,
                                                 double* __restrict__ out) {
  __shared__ double nrm[3];
  sum_rows(part + (int64_t)nv * nparts, nparts, nv ? 3 : 1, nrm);
  if (blockIdx.x == 0 && (int)threadIdx.x < (nv ? 3 : 1)) out[threadIdx.x] = nrm[threadIdx.x];
  const double w2 = nv == 0 ? nrm[0] : gs_again(nrm[0], nrm[1]) ? nrm[2] : nrm[1];
  const double s = 1.0 / sqrt(fmax(w2, 0.0));
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float fx = (float)(s * w[3 * i]), fy = (float)(s * w[3 * i + 1]),
                fz = (float)(s * w[3 * i + 2]);
    v[3 * i] = fx;
    v[3 * i + 1] = fy;
    v[3 * i + 2] = fz;
    const double* Mi = Minv + 9 * i;
    const double vx = fx, vy = fy, vz = fz;
    const double a = Mi[0] * vx + Mi[1] * vy + Mi[2] * vz;
    const double b = Mi[3] * vx + Mi[4] * vy + Mi[5] * vz;
    const double d = Mi[6] * vx + Mi[7] * vy + Mi[8] * vz;
    z[3 * i] = a;
    z[3 * i + 1] = b;
    z[3 * i + 2] = d;
    z32[3 * i] = (float)a;
    z32[3 * i + 1] = (float)b;
    z32[3 * i + 2] = (float)d;
  }
}

// Newton's correction x -= Minv sum_j y[j] V_j (j < nv, ascending) and the next
// evaluation point as in k_mid_point
__global__ void __launch_bounds__(256) k_mid_correct(int64_t n, const float* __restrict__ V,
                                                     int64_t ldv, int nv, GsCoef y,
                                                     const double* __restrict__ Minv,
                                                     const double* __restrict__ m, double theta,
                                                     double* __restrict__ x,
                                                     double* __restrict__ mb,
                                                     float* __restrict__ mb32) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double vx = 0.0, vy = 0.0, vz = 0.0;
  for (int j = 0; j < nv; ++j) {
    const float* Vj = V + (int64_t)j * ldv + 3 * i;
    vx = fma(y.c[j], (double)Vj[0], vx);
    vy = fma(y.c[j], (double)Vj[1], vy);
    vz = fma(y.c[j], (double)Vj[2], vz);
  }
  const double* Mi = Minv + 9 * i;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double xn = x[3 * i + k] - (Mi[3 * k] * vx + Mi[3 * k + 1] * vy + Mi[3 * k + 2] * vz);
    x[3 * i + k] = xn;
    const double b = theta == 1.0 ? xn : (1.0 - theta) * m[3 * i + k] + theta * xn;
    mb[3 * i + k] = b;
    mb32[3 * i + k] = (float)b;
  }
}

// part[j * gridDim.x + b] = block b's share of V_j . w for j < nv (fixed
// order: grid-stride per thread, then a tree in LDS)
__global__ void __launch_bounds__(256) k_mdot(int64_t n3, const double* __restrict__ V,
                                              int64_t ldv, int nv, const double* __restrict__ w,
                                              double* __restrict__ part) {
  __shared__ double red[256];
  for (int j = 0; j < nv; ++j) {
    const double* Vj = V + (int64_t)j * ldv;
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n3;
         i += (int64_t)gridDim.x * blockDim.x)
      acc = fma(Vj[i], w[i], acc);
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) part[(int64_t)j * gridDim.x + blockIdx.x] = red[0];
    __syncthreads();
  }
}

// out[j] = sum over b < nparts of part[j * nparts + b], one block per j,
// fixed order
__global__ void __launch_bounds__(256) k_sum_parts(const double* __restrict__ part, int nparts,
                                                   double* __restrict__ out) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int b = threadIdx.x; b < nparts; b += blockDim.x) acc += part[(int64_t)blockIdx.x * nparts + b];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// out = aw w + sum_j coef[j] V_j (j < nv); out may alias w
__global__ void k_lincomb(int64_t n3, const double* __restrict__ V, int64_t ldv, int nv,
                          const double* __restrict__ coef, double aw, const double* w,
                          double* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n3) return;
  double v = aw != 0.0 ? aw * w[i] : 0.0;
  for (int j = 0; j < nv; ++j) v = fma(coef[j], V[(int64_t)j * ldv + i], v);
  out[i] = v;
}

__global__ void __launch_bounds__(256) k_energy(int64_t n, const double* __restrict__ m,
                                                const double* __restrict__ mu,
                                                const float* __restrict__ hex,
                                                const float* __restrict__ q,
                                                const float* __restrict__ u,
                                                double* __restrict__ part) {
  __shared__ double s0[256], s1[256];
  double a = 0.0, b = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    a += mu[i] * (m[3 * i] * hex[3 * i] + m[3 * i + 1] * hex[3 * i + 1] +
                  m[3 * i + 2] * hex[3 * i + 2]);
    b += (double)q[i] * (double)u[i];
  }
  s0[threadIdx.x] = a;
  s1[threadIdx.x] = b;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      s0[threadIdx.x] += s0[threadIdx.x + o];
      s1[threadIdx.x] += s1[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = s0[0];
    part[2 * blockIdx.x + 1] = s1[0];
  }
}

}  // namespace pmfem
