// Batched blip-orbital evaluation for gfx950 (the paper's Sec. 2.4: orbitals
// re-represented in a blip (B-spline) basis; evaluating them after a move is a
// grid lookup, a few cubic polynomials, and the multiplication of the 64
// blip functions that are nonzero at the point by every orbital's
// coefficients, which the paper sends through 64-element BLAS calls one
// point at a time, Sec. 5.3).  Here one wave serves one point and a slice of
// the orbitals:
//   - lane p < 64 finds grid point p of the 4 x 4 x 4 window around the
//     point and forms its blip product, the product's Cartesian gradient and
//     its Laplacian (five weights), parked in LDS;
//   - the wave then streams the 64 coefficient rows (orbital index fastest),
//     eight in flight, each row's address read from its lane into scalar
//     registers and its weights from LDS, and accumulates value, gradient and
//     Laplacian of the lane's orbitals.
// (Weights read from their lanes as well, ten reads per row, spare the LDS but
// cost more vector issue than they save: 40,000 points, gradients, 33 orbitals 156 us against
// 94; 130 orbitals 341 and 209; 512 on a 40^3 grid in the order below 707 and
// 505.  One wave for all orbitals of a point takes 512 orbitals at 500
// points 54 us, a wave per slice 16.)
// The work is a gather of 64 n_orb coefficients per point with 5 FMAs per
// coefficient, not a dense contraction (each point takes its own 64 rows),
// bound by where the rows come from.  Points in any order take every row from
// the last-level cache or HBM (262 KB per point at 512 orbitals).  A large batch
// over a coefficient set beyond the L2s is therefore served in the order of
// the points' places on the grid (bricks of BRICK^3 cells, each L2 taking a
// contiguous range), so that the points that share a row (64 windows of the
// grid hold it) find it in the L2.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <string>

#include "ewald.h"
#include "ewald_internal.h"

namespace ewald {
// thread-local message shared with the rest of the library
void set_last_error(const std::string& msg);
}  // namespace ewald

struct ewald_blip {
  int grid[3];
  int n_orb;
  double ainv[9];   // s = r Ainv (row vectors)
  double J[9];      // J[e][d] = d x_d / d r_e = Ainv[e][d] n_d
  double M[6];      // sum_e J[e][d] J[e][d'] for (d, d') = 00, 11, 22, 01, 02, 12
};

namespace ewald {
namespace {

struct BlipK {
  int n[3];
  int n_orb;
  double ainv[9];
  double J[9];
  double M[6];
};

// Blip function Th(x) = 1 - 3/2 x^2 + 3/4 |x|^3 (|x| <= 1), 1/4 (2 - |x|)^3
// (1 < |x| < 2), and its first two derivatives.
__device__ __forceinline__ void blip_fn(double x, double& f, double& f1, double& f2) {
  const double ax = fabs(x), sg = x < 0.0 ? -1.0 : 1.0;
  if (ax <= 1.0) {
    f = fma(0.75 * ax, x * x, fma(-1.5, x * x, 1.0));
    f1 = fma(2.25 * sg, x * x, -3.0 * x);
    f2 = fma(4.5, ax, -3.0);
  } else {
    const double t = ax < 2.0 ? 2.0 - ax : 0.0;
    f = 0.25 * t * t * t;
    f1 = -0.75 * sg * t * t;
    f2 = 1.5 * t;
  }
}

constexpr int BLIP_WAVES = 4;  // waves per workgroup
constexpr int BRICK = 4;       // cells along each side of a brick (ordering of large batches)
constexpr int BRICKS_MAX = 16384;

struct __align__(16) BlipW {
  double b, gx, gy, gz, l;
  double pad_;
};

// A point's grid coordinates x_d = n_d s_d, s wrapped into [0, 1).
__device__ __forceinline__ void grid_coords(const BlipK& K, const double* __restrict__ pos, size_t p, double* x) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < 3; ++e) s = fma(pos[p * 3 + e], K.ainv[e * 3 + d], s);
    s -= floor(s);
    x[d] = s * K.n[d];
  }
}

// VW = 2: orbital pairs read as 16-byte loads (n_orb even); 1: single loads.
// A wave serves 64 VW orbitals of one point and `slices` waves (consecutive, so
// that they run together) all of them.
// order: NULL (points p_lo .. p_hi - 1 in turn), or the points' order; those
// from p_hi on are left to a later launch (their outputs hold the order).
template <int VW, bool DER>
__global__ __launch_bounds__(64 * BLIP_WAVES) void k_blip(BlipK K, const double* __restrict__ coef, int p_lo, int p_hi,
                                                            int n_items, int slices,
                                                            const int* order, const double* __restrict__ pos,
                                                            double* val, double* grad, double* lap) {
  __shared__ BlipW wts[BLIP_WAVES][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  int blk = blockIdx.x;
  if (order) {
    // consecutive workgroups go to the eight L2s in turn: give each a
    // contiguous range (the grid is a multiple of 8)
    const int per = gridDim.x / 8;
    blk = (blk & 7) * per + (blk >> 3);
  }
  const int item = blk * BLIP_WAVES + wave;
  if (item >= n_items) return;  // uniform per wave; no block-level barrier below
  const int it = item / slices, slice = item - it * slices;
  const int p = order ? __builtin_amdgcn_readfirstlane(order[it]) : p_lo + it;
  if (p >= p_hi) return;
  const int n_orb = K.n_orb;
  BlipW* W = wts[wave];
  uint64_t row;  // byte offset of the lane's coefficient row
  {
    double x[3];
    grid_coords(K, pos, size_t(p), x);
    const int a[3] = {lane >> 4, (lane >> 2) & 3, lane & 3};
    double f[3], f1[3], f2[3];
    int idx[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double fl = floor(x[d]);
      const int g = int(fl) - 1 + a[d];  // grid points floor(x) - 1 .. floor(x) + 2
      blip_fn(x[d] - double(g), f[d], f1[d], f2[d]);
      const int gw = g % K.n[d];
      idx[d] = gw < 0 ? gw + K.n[d] : gw;
    }
    BlipW w;
    w.b = f[0] * f[1] * f[2];
    if (DER) {
      const double dx[3] = {f1[0] * f[1] * f[2], f[0] * f1[1] * f[2], f[0] * f[1] * f1[2]};
      // second derivatives in x: diagonal and mixed
      const double h00 = f2[0] * f[1] * f[2], h11 = f[0] * f2[1] * f[2], h22 = f[0] * f[1] * f2[2];
      const double h01 = f1[0] * f1[1] * f[2], h02 = f1[0] * f[1] * f1[2], h12 = f[0] * f1[1] * f1[2];
      double g[3];
#pragma unroll
      for (int e = 0; e < 3; ++e) g[e] = fma(K.J[e * 3 + 2], dx[2], fma(K.J[e * 3 + 1], dx[1], K.J[e * 3] * dx[0]));
      w.gx = g[0];
      w.gy = g[1];
      w.gz = g[2];
      w.l = fma(K.M[0], h00, fma(K.M[1], h11, fma(K.M[2], h22,
            2.0 * fma(K.M[3], h01, fma(K.M[4], h02, K.M[5] * h12)))));
    } else {
      w.gx = w.gy = w.gz = w.l = 0.0;
    }
    w.pad_ = 0.0;
    W[lane] = w;
    row = ((uint64_t(idx[0]) * uint32_t(K.n[1]) + uint32_t(idx[1])) * uint32_t(K.n[2]) + uint32_t(idx[2])) * uint32_t(n_orb) * 8;
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const size_t out0 = size_t(p) * n_orb;
  for (int o0 = slice * 64 * VW; o0 < n_orb; o0 += slices * 64 * VW) {
    double v[VW], gx[VW], gy[VW], gz[VW], l[VW];
    const int o = o0 + lane * VW;
    const int oo = o < n_orb ? o : 0;  // (clamped: every load is in bounds)
#pragma unroll
    for (int c = 0; c < VW; ++c) v[c] = gx[c] = gy[c] = gz[c] = l[c] = 0.0;
    constexpr int RB = 8;  // rows in flight
#pragma unroll 1
    for (int r0 = 0; r0 < 64; r0 += RB) {
      double a[RB][VW];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const uint64_t at = uint64_t(uint32_t(__builtin_amdgcn_readlane(int(row >> 32), r0 + r))) << 32 |
                            uint32_t(__builtin_amdgcn_readlane(int(uint32_t(row)), r0 + r));
        const double* src = reinterpret_cast<const double*>(reinterpret_cast<const char*>(coef) + at);
        if (VW == 2) {
          const double2 t = *reinterpret_cast<const double2*>(src + oo);
          a[r][0] = t.x;
          a[r][VW - 1] = t.y;
        } else {
          a[r][0] = src[oo];
        }
      }
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const BlipW w = W[r0 + r];
#pragma unroll
        for (int c = 0; c < VW; ++c) {
          v[c] = fma(w.b, a[r][c], v[c]);
          if (DER) {
            gx[c] = fma(w.gx, a[r][c], gx[c]);
            gy[c] = fma(w.gy, a[r][c], gy[c]);
            gz[c] = fma(w.gz, a[r][c], gz[c]);
            l[c] = fma(w.l, a[r][c], l[c]);
          }
        }
      }
    }
    if (o < n_orb)
#pragma unroll
      for (int c = 0; c < VW; ++c) {
        val[out0 + o + c] = v[c];
        if (DER) {
          grad[3 * out0 + o + c] = gx[c];
          grad[3 * out0 + n_orb + o + c] = gy[c];
          grad[3 * out0 + 2 * size_t(n_orb) + o + c] = gz[c];
          lap[out0 + o + c] = l[c];
        }
      }
  }
}

// ---- ordering of a large batch by brick: a counting sort ----------------------
// Workgroups of 1024 points count in LDS first and add each brick's count to
// the batch's once (points in one brick would otherwise queue up at one address,
// 12 ns each: 40,000 of them took 1 ms).  Dynamic LDS: one int per brick.

struct Bricks {
  int n[3];  // bricks along each axis
  int total;
};

__device__ __forceinline__ int brick_of(const BlipK& K, const Bricks& B, const double* __restrict__ pos, size_t p) {
  double x[3];
  grid_coords(K, pos, p, x);
  int b[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    // (a NaN position converts to some integer: clamped, any brick will do)
    const int c = int(x[d]) / BRICK;
    b[d] = min(max(c, 0), B.n[d] - 1);
  }
  return (b[0] * B.n[1] + b[1]) * B.n[2] + b[2];
}

__global__ void k_brick_zero(int* count, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) count[i] = 0;
}

constexpr int SORT_NT = 1024;

__global__ __launch_bounds__(SORT_NT) void k_brick_count(BlipK K, Bricks B, const double* __restrict__ pos, int n_pts,
                                                         int* count) {
  extern __shared__ int own[];
  for (int i = threadIdx.x; i < B.total; i += SORT_NT) own[i] = 0;
  __syncthreads();
  const int p = blockIdx.x * SORT_NT + threadIdx.x;
  if (p < n_pts) atomicAdd(&own[brick_of(K, B, pos, size_t(p))], 1);
  __syncthreads();
  for (int i = threadIdx.x; i < B.total; i += SORT_NT)
    if (own[i] != 0) atomicAdd(&count[i], own[i]);
}

// Counts to first places, by one workgroup of 1024.
__global__ __launch_bounds__(1024) void k_brick_scan(int* count, int n) {
  __shared__ int part[1024];
  const int per = (n + 1023) / 1024, i0 = threadIdx.x * per, i1 = min(i0 + per, n);
  int s = 0;
  for (int i = i0; i < i1; ++i) s += count[i];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int t = int(threadIdx.x) >= off ? part[threadIdx.x - off] : 0;
    __syncthreads();
    part[threadIdx.x] += t;
    __syncthreads();
  }
  int first = part[threadIdx.x] - s;
  for (int i = i0; i < i1; ++i) {
    const int c = count[i];
    count[i] = first;
    first += c;
  }
}

// (points of one brick come in any order: no output depends on it)
__global__ __launch_bounds__(SORT_NT) void k_brick_place(BlipK K, Bricks B, const double* __restrict__ pos, int n_pts,
                                                         int* first, int* order) {
  extern __shared__ int own[];
  for (int i = threadIdx.x; i < B.total; i += SORT_NT) own[i] = 0;
  __syncthreads();
  const int p = blockIdx.x * SORT_NT + threadIdx.x;
  int b = 0, rank = 0;
  if (p < n_pts) {
    b = brick_of(K, B, pos, size_t(p));
    rank = atomicAdd(&own[b], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < B.total; i += SORT_NT)
    if (own[i] != 0) own[i] = atomicAdd(&first[i], own[i]);
  __syncthreads();
  if (p < n_pts) order[own[b] + rank] = p;
}

// One launch over `count` points (order: of all of them; else p_lo, p_lo + 1, ...).
void blip_launch(const BlipK& K, bool vec, bool der, const double* coef, int p_lo, int p_hi, int count,
                 const int* order, const double* pos, double* val, double* grad, double* lap, hipStream_t s) {
  const int per = vec ? 128 : 64;
  const int slices = (K.n_orb + per - 1) / per;
  const long long items = (long long)count * slices;
  // several passes over the orbitals per wave where the items would not fit the grid
  const int sl = items > (1ll << 30) ? 1 : slices;
  const int n_items = count * sl;
  int grid = (n_items + BLIP_WAVES - 1) / BLIP_WAVES;
  if (order) grid = (grid + 7) & ~7;
#define EW_BLIP(VW, DER)                                                                                          \
  hipLaunchKernelGGL((k_blip<VW, DER>), dim3(grid), dim3(64 * BLIP_WAVES), 0, s, K, coef, p_lo, p_hi, n_items, sl, \
                     order, pos, val, grad, lap)
  if (vec) {
    if (der) EW_BLIP(2, true); else EW_BLIP(2, false);
  } else {
    if (der) EW_BLIP(1, true); else EW_BLIP(1, false);
  }
#undef EW_BLIP
}

}  // namespace
}  // namespace ewald

extern "C" {

ewald_status ewald_blip_create(const double lattice[3][3], const int grid[3], int n_orb, ewald_blip** out) try {
  if (!out) {
    ewald::set_last_error("out is NULL");
    return EWALD_E_ARG;
  }
  *out = nullptr;
  if (!lattice || !grid) {
    ewald::set_last_error("lattice/grid is NULL");
    return EWALD_E_ARG;
  }
  if (n_orb < 1) {
    ewald::set_last_error("n_orb must be >= 1");
    return EWALD_E_ARG;
  }
  for (int d = 0; d < 3; ++d)
    if (grid[d] < 4 || grid[d] > 4096) {
      ewald::set_last_error("every grid dimension must be in [4, 4096]");
      return EWALD_E_ARG;
    }
  const double* A = &lattice[0][0];
  for (int i = 0; i < 9; ++i)
    if (!std::isfinite(A[i])) {
      ewald::set_last_error("non-finite lattice");
      return EWALD_E_LATTICE;
    }
  const double det = A[0] * (A[4] * A[8] - A[5] * A[7]) - A[1] * (A[3] * A[8] - A[5] * A[6]) +
                     A[2] * (A[3] * A[7] - A[4] * A[6]);
  double norm = 1.0;
  for (int i = 0; i < 3; ++i) norm *= std::sqrt(A[3 * i] * A[3 * i] + A[3 * i + 1] * A[3 * i + 1] + A[3 * i + 2] * A[3 * i + 2]);
  if (!(std::fabs(det) > 1e-10 * norm)) {
    ewald::set_last_error("singular lattice");
    return EWALD_E_LATTICE;
  }
  ewald_blip* b = new ewald_blip();
  for (int d = 0; d < 3; ++d) b->grid[d] = grid[d];
  b->n_orb = n_orb;
  // inverse by cofactors: Ainv[e][d] with sum_e A[i][e] Ainv[e][d] = delta_id
  const double c[9] = {A[4] * A[8] - A[5] * A[7], A[2] * A[7] - A[1] * A[8], A[1] * A[5] - A[2] * A[4],
                       A[5] * A[6] - A[3] * A[8], A[0] * A[8] - A[2] * A[6], A[2] * A[3] - A[0] * A[5],
                       A[3] * A[7] - A[4] * A[6], A[1] * A[6] - A[0] * A[7], A[0] * A[4] - A[1] * A[3]};
  for (int i = 0; i < 9; ++i) b->ainv[i] = c[i] / det;
  for (int e = 0; e < 3; ++e)
    for (int d = 0; d < 3; ++d) b->J[e * 3 + d] = b->ainv[e * 3 + d] * grid[d];
  const int pd[6][2] = {{0, 0}, {1, 1}, {2, 2}, {0, 1}, {0, 2}, {1, 2}};
  for (int t = 0; t < 6; ++t) {
    double m = 0.0;
    for (int e = 0; e < 3; ++e) m += b->J[e * 3 + pd[t][0]] * b->J[e * 3 + pd[t][1]];
    b->M[t] = m;
  }
  *out = b;
  return EWALD_OK;
} catch (const std::bad_alloc&) {
  ewald::set_last_error("host allocation failed");
  return EWALD_E_NOMEM;
}

void ewald_blip_destroy(ewald_blip* b) { delete b; }

ewald_status ewald_blip_eval_batch(const ewald_blip* b, const double* coef, int n_points, const double* pos,
                                   double* val, double* grad, double* lap, void* stream) {
  ewald::CallTimer timer("ewald_blip_eval_batch", stream);
  if (!b) {
    ewald::set_last_error("blip handle is NULL");
    return EWALD_E_ARG;
  }
  if (n_points < 0) {
    ewald::set_last_error("n_points must be >= 0");
    return EWALD_E_ARG;
  }
  if (n_points == 0) return EWALD_OK;
  if (!coef || !pos || !val) {
    ewald::set_last_error("coef, pos and val must be non-NULL");
    return EWALD_E_ARG;
  }
  if ((grad == nullptr) != (lap == nullptr)) {
    ewald::set_last_error("grad and lap must be given together");
    return EWALD_E_ARG;
  }
  const bool vec = (b->n_orb % 2) == 0 && (reinterpret_cast<uintptr_t>(coef) % 16) == 0;
  ewald::BlipK K;
  for (int d = 0; d < 3; ++d) K.n[d] = b->grid[d];
  K.n_orb = b->n_orb;
  std::memcpy(K.ainv, b->ainv, sizeof K.ainv);
  std::memcpy(K.J, b->J, sizeof K.J);
  std::memcpy(K.M, b->M, sizeof K.M);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool der = grad != nullptr;
  // Ordered where the coefficients exceed the L2s (4 MB each, and a row that
  // one of them holds is shared by points that all run there), the points
  // are enough for rows to be shared and the gather is long enough for the sort's
  // five launches (20 to 35 us).  Spread points, us without and with the order: 128
  // orbitals, 10,000 points on 40^3 (0.66 GB of rows) 95 and 66, 256 on 24^3, 4000 points
  // (0.52 GB), values 66 and 44; 100 orbitals, 4000 points (0.2 GB) 33 and 52.  Points
  // that all lie in a few bricks find their rows in the L2s anyway and pay for the sort
  // (10,000 points, 256 orbitals 63 and 87, 40,000 points, 512 orbitals 480 and 500).  The order (one int per point and per
  // brick) sits at the end of `val` until the main launch has read it, and the
  // points whose values lie there are evaluated last.  48 orbitals at least
  // keep these few (and shorter rows gain nothing: 33 orbitals, 65,536 points 147 us
  // and 174).
  const double rows = double(b->grid[0]) * b->grid[1] * b->grid[2];
  ewald::Bricks B;
  for (int d = 0; d < 3; ++d) B.n[d] = (b->grid[d] + ewald::BRICK - 1) / ewald::BRICK;
  const bool ordered = rows * b->n_orb * 8.0 > 16e6 && b->n_orb >= 48 && n_points >= 2048 && n_points >= rows / 16 &&
                       512.0 * n_points * b->n_orb >= 0.5e9 && double(B.n[0]) * B.n[1] * B.n[2] <= ewald::BRICKS_MAX;
  if (ordered) {
    B.total = B.n[0] * B.n[1] * B.n[2];
    const size_t ints = size_t(n_points) + size_t(B.total);
    const int late = int((ints * 4 + size_t(b->n_orb) * 8 - 1) / (size_t(b->n_orb) * 8));  // points that are evaluated last
    if (late < n_points) {
      const int p_hi = n_points - late;
      int* count = reinterpret_cast<int*>(val + size_t(p_hi) * b->n_orb);
      int* order = count + B.total;
      const dim3 sort_grid((n_points + ewald::SORT_NT - 1) / ewald::SORT_NT), sort_block(ewald::SORT_NT);
      const size_t sort_lds = size_t(B.total) * sizeof(int);
      hipLaunchKernelGGL(ewald::k_brick_zero, dim3((B.total + 255) / 256), dim3(256), 0, s, count, B.total);
      hipLaunchKernelGGL(ewald::k_brick_count, sort_grid, sort_block, sort_lds, s, K, B, pos, n_points, count);
      hipLaunchKernelGGL(ewald::k_brick_scan, dim3(1), dim3(1024), 0, s, count, B.total);
      hipLaunchKernelGGL(ewald::k_brick_place, sort_grid, sort_block, sort_lds, s, K, B, pos, n_points, count, order);
      ewald::blip_launch(K, vec, der, coef, 0, p_hi, n_points, order, pos, val, grad, lap, s);
      ewald::blip_launch(K, vec, der, coef, p_hi, n_points, late, nullptr, pos, val, grad, lap, s);
    } else {
      ewald::blip_launch(K, vec, der, coef, 0, n_points, n_points, nullptr, pos, val, grad, lap, s);
    }
  } else {
    ewald::blip_launch(K, vec, der, coef, 0, n_points, n_points, nullptr, pos, val, grad, lap, s);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    ewald::set_last_error(std::string("blip launch failed: ") + hipGetErrorString(e));
    return EWALD_E_HIP;
  }
  return EWALD_OK;
}

}  // extern "C"
