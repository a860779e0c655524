// The optimizer around the guarded state solve: the minimum-compliance loop
// of Sec. 3.1 (Eq. to_problem) with the linear-hat density filter, the
// smoothed Heaviside projection (Eq. projection), the optimality-criteria
// update with a move limit and a bisection on the volume multiplier, and the
// two-stage continuation of Tab. trajectory-settings; the floor is chosen at
// every outer iteration by the guarded policy (Alg. floor_policy), optionally
// reusing the previous decision until the guard rejects it (the cost
// reduction Sec. 5.2 names as untested), or fixed without acceptance test
// (the controls of Sec. 4.1.2).
//
// Every kernel here is a small stencil over the element grid (x fastest); a
// workgroup stages its tile of elements and their halo in LDS.  Sums run in a
// fixed order.  The bisection's decisions are taken on the device, several
// multipliers per launch; the loop runs on the host around the kernels.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "tg_internal.h"

namespace tg {
namespace {

constexpr int TO_BLOCK = 256;
constexpr int TO_MAX_R = 3;       // stencil half-width: r_min < 4

// Weights of the hat filter by squared distance |d|^2 (0 where r_min <= |d|)
// and the sum of all of them in the order dz, dy, dx (W of an element whose
// stencil lies inside the grid); passed to the kernels by value, so that the
// weights come in scalar registers.
struct Hat {
  double wsum;
  double w[3 * TO_MAX_R * TO_MAX_R + 1];
};

// Tile of 16 x 4 x 4 elements and its halo of R elements on every side.
template <int R>
struct Tile {
  static constexpr int X = 16, Y = 4, Z = 4;
  static constexpr int SX = X + 2 * R, SY = Y + 2 * R, SZ = Z + 2 * R, N = SX * SY * SZ;
};
static_assert(Tile<0>::X * Tile<0>::Y * Tile<0>::Z == TO_BLOCK, "one thread per element of a tile");

struct Dims {
  int nx, ny, nz;
  int tx, ty, tz;                 // tiles per dimension
  long long n;
};

// W_e: the weights of the in-grid offsets of element (i, j, k), in order
template <int R>
__device__ __forceinline__ double weight_sum(const Hat& h, const Dims& D, int i, int j, int k) {
  if (i >= R && i < D.nx - R && j >= R && j < D.ny - R && k >= R && k < D.nz - R) return h.wsum;
  double W = 0.0;
#pragma unroll
  for (int dz = -R; dz <= R; ++dz) {
    if (k + dz < 0 || k + dz >= D.nz) continue;
#pragma unroll
    for (int dy = -R; dy <= R; ++dy) {
      if (j + dy < 0 || j + dy >= D.ny) continue;
#pragma unroll
      for (int dx = -R; dx <= R; ++dx)
        W += i + dx >= 0 && i + dx < D.nx ? h.w[dx * dx + dy * dy + dz * dz] : 0.0;
    }
  }
  return W;
}

// v(e, i, j, k) of every element of tile t and its halo into sv (0 outside the grid)
template <int R, class F>
__device__ __forceinline__ void stage_tile(const Dims& D, int t, double* sv, F&& v) {
  using T = Tile<R>;
  const int tk = t / (D.tx * D.ty), r = t - tk * D.tx * D.ty, tj = r / D.tx, ti = r - tj * D.tx;
  for (int q = threadIdx.x; q < T::N; q += TO_BLOCK) {
    const int sk = q / (T::SX * T::SY), sr = q - sk * T::SX * T::SY, sj = sr / T::SX, si = sr - sj * T::SX;
    const int i = ti * T::X + si - R, j = tj * T::Y + sj - R, k = tk * T::Z + sk - R;
    const bool in = i >= 0 && i < D.nx && j >= 0 && j < D.ny && k >= 0 && k < D.nz;
    sv[q] = in ? v(i + (long long)D.nx * (j + (long long)D.ny * k), i, j, k) : 0.0;
  }
}
// this thread's element of tile t and its place in the staged tile
template <int R>
__device__ __forceinline__ bool tile_elem(const Dims& D, int t, int& i, int& j, int& k, int& at) {
  using T = Tile<R>;
  const int tk = t / (D.tx * D.ty), r = t - tk * D.tx * D.ty, tj = r / D.tx, ti = r - tj * D.tx;
  const int x = threadIdx.x & 15, y = (threadIdx.x >> 4) & 3, z = threadIdx.x >> 6;
  i = ti * T::X + x;
  j = tj * T::Y + y;
  k = tk * T::Z + z;
  at = ((z + R) * T::SY + y + R) * T::SX + x + R;
  return i < D.nx && j < D.ny && k < D.nz;
}
// sum of w v over the offsets with w > 0, in order (the halo outside the grid
// holds 0)
template <int R>
__device__ __forceinline__ double hat_sum(const Hat& h, const double* sv, int at) {
  using T = Tile<R>;
  double s = 0.0;
#pragma unroll
  for (int dz = -R; dz <= R; ++dz)
#pragma unroll
    for (int dy = -R; dy <= R; ++dy)
#pragma unroll
      for (int dx = -R; dx <= R; ++dx) {
        const double w = h.w[dx * dx + dy * dy + dz * dz];
        const double v = sv[at + (dz * T::SY + dy) * T::SX + dx];
        s += w > 0.0 ? w * v : 0.0;
      }
  return s;
}

// xt = H x (and, if xbar, xbar = project(xt), dxbar its derivative); t1 =
// tanh(beta eta), den = t1 + tanh(beta (1 - eta)).  Bound by the stencil's
// LDS reads and the tanh; with the neighbours read from global memory and
// their weights recomputed (a square root each) it took 11 us at 64x32x32 and
// r_min = 1.5, 5.6 us so.
template <int R>
__global__ __launch_bounds__(TO_BLOCK) void k_filter(Hat h, Dims D, const double* __restrict__ x, double beta,
                                                     double eta, double t1, double den, double* __restrict__ xt,
                                                     double* __restrict__ xbar, double* __restrict__ dxbar) {
  __shared__ double sv[Tile<R>::N];
  const int t = blockIdx.x;
  stage_tile<R>(D, t, sv, [&](long long e, int, int, int) { return x[e]; });
  __syncthreads();
  int i, j, k, at;
  if (!tile_elem<R>(D, t, i, j, k, at)) return;
  const long long e = i + (long long)D.nx * (j + (long long)D.ny * k);
  const double v = hat_sum<R>(h, sv, at) / weight_sum<R>(h, D, i, j, k);
  if (xt) xt[e] = v;
  if (xbar) {
    const double th = tanh(beta * (v - eta));
    xbar[e] = fmin(1.0, fmax(0.0, (t1 + th) / den));   // rounding stays in [0, 1]
    if (dxbar) dxbar[e] = beta * (1.0 - th * th) / den;
  }
}

// y_j = sum_e w_ej a_e b_e / W_e (b may be NULL: 1).  The quotients are formed
// once per element while the tile is staged (the stencil is symmetric, so e
// runs over j's own stencil).  Recomputing W_e for every pair took 70 us at
// 64x32x32 and r_min = 1.5; this form takes 5.2 us.
template <int R>
__global__ __launch_bounds__(TO_BLOCK) void k_filter_adj(Hat h, Dims D, const double* __restrict__ a,
                                                         const double* __restrict__ b, double* __restrict__ y) {
  __shared__ double sv[Tile<R>::N];
  const int t = blockIdx.x;
  stage_tile<R>(D, t, sv, [&](long long e, int i, int j, int k) {
    return (b ? a[e] * b[e] : a[e]) / weight_sum<R>(h, D, i, j, k);
  });
  __syncthreads();
  int i, j, k, at;
  if (tile_elem<R>(D, t, i, j, k, at)) y[i + (long long)D.nx * (j + (long long)D.ny * k)] = hat_sum<R>(h, sv, at);
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// the workgroup's part of sum_e tanh(beta ((H v)_e - eta)) over tiles b, b + nb, ...
template <int R, class F>
__device__ __forceinline__ double volume_part(const Hat& h, const Dims& D, int b, int nb, double beta, double eta,
                                              double* sv, double* sh, F&& v) {
  double acc = 0.0;
  const int nt = D.tx * D.ty * D.tz;
  for (int t = b; t < nt; t += nb) {
    __syncthreads();              // the previous tile's reads
    stage_tile<R>(D, t, sv, v);
    __syncthreads();
    int i, j, k, at;
    if (tile_elem<R>(D, t, i, j, k, at))
      acc += tanh(beta * (hat_sum<R>(h, sv, at) / weight_sum<R>(h, D, i, j, k) - eta));
  }
  __syncthreads();
  return block_sum(acc, sh);
}

template <int R>
__global__ __launch_bounds__(TO_BLOCK) void k_volume(Hat h, Dims D, const double* __restrict__ x, double beta,
                                                     double eta, double* __restrict__ part) {
  __shared__ double sv[Tile<R>::N], sh[4];
  const double s = volume_part<R>(h, D, blockIdx.x, gridDim.x, beta, eta, sv, sh,
                                  [&](long long e, int, int, int) { return x[e]; });
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// per-block maxima of |a - b|
__global__ __launch_bounds__(TO_BLOCK) void k_max_change(const double* __restrict__ a, const double* __restrict__ b,
                                                         long long n, double* __restrict__ part) {
  __shared__ double red[TO_BLOCK / 64];
  double acc = 0.0;
  for (long long e = (long long)blockIdx.x * TO_BLOCK + threadIdx.x; e < n; e += (long long)gridDim.x * TO_BLOCK)
    acc = fmax(acc, fabs(a[e] - b[e]));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc = fmax(acc, __shfl_xor(acc, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// ---- the OC step.  The bisection of the multiplier from [0, 1e9] takes about
// 70 halvings, each needing the volume of the design at its midpoint.  A
// launch evaluates several midpoints at once, one set of workgroups per
// midpoint, and the next launch (every workgroup for itself, from the
// partial sums) takes the decisions, so nothing returns to the host on the
// way.  With a bracket [l1, l2], l1 > 0, whose ends' volumes are known, the
// midpoints are those along the way to the multiplier that the two volumes
// predict (the design goes as its inverse root, so that is where they are
// interpolated): a launch takes as many halvings as the prediction is right
// for, one more where it is not, and the nearer the ends the more of them.
// Without the volumes (l2 as it was given) they are those of the next levels of
// the bisection, 2^depth - 1 of them.  While l1 = 0 the
// midpoints are l2 / 2, l2 / 4, ...: the volume does not increase with the
// multiplier, so one that is not above the target decides every larger one,
// and the midpoints are taken `stride` halvings apart until one is above.
// The halvings, their order, the stop test and the midpoints are those of
// one evaluation at a time; 64x32x32 took 31 us per halving with the volume
// read back after each, 2.0 ms in all; 14 launches with three levels of the
// bisection in each, 0.20 ms; 7 or 8 with the prediction, 0.12 ms.
constexpr int OC_MAX_CAND = 7;    // depth 3
constexpr int OC_STRIDE = 6;
constexpr int OC_MAX_HALVINGS = 200;
struct OcState {
  double l1, l2, lm;
  double it, done, stride;        // halvings taken; stop test met; left-phase stride
  double v1, v2;                  // volumes at l1 and l2 (NaN: not known)
};
constexpr int OC_STATE_W = 8;
static_assert(sizeof(OcState) <= OC_STATE_W * sizeof(double), "state words");

__device__ __forceinline__ bool oc_more(const OcState& s) {
  return s.it < OC_MAX_HALVINGS && (s.l2 - s.l1) / (s.l1 + s.l2) > 1e-9;
}
// the multiplier that the volumes at the bracket's ends predict; 0: none
__device__ __forceinline__ double oc_guess(const OcState& s, double target) {
  if (s.l1 == 0.0 || !(s.v1 > s.v2)) return 0.0;
  const double u1 = 1.0 / sqrt(s.l1), u2 = 1.0 / sqrt(s.l2);
  const double u = u1 + (u2 - u1) * ((s.v1 - target) / (s.v1 - s.v2));
  return 1.0 / (u * u);
}
// the c-th midpoint (c < nc) the launch after state s evaluates; 0: none
__device__ __forceinline__ double oc_midpoint(const OcState& s, int c, double target) {
  if (s.l1 == 0.0) {
    const double lev = s.stride * (c + 1);
    return s.it + lev <= OC_MAX_HALVINGS ? ldexp(s.l2, -(int)lev) : 0.0;
  }
  double l1 = s.l1, l2 = s.l2;
  const double guess = oc_guess(s, target);
  if (guess > 0.0) {
    for (int q = 0; q < c; ++q) {
      const double m = 0.5 * (l1 + l2);
      if (guess > m) l1 = m;
      else l2 = m;
    }
    return 0.5 * (l1 + l2);
  }
  // node c + 1 of the heap-ordered tree of halvings: its path from the top bit
  for (int b = 30 - __clz(c + 1); b >= 0; --b) {
    const double m = 0.5 * (l1 + l2);
    if ((c + 1) >> b & 1) l1 = m;
    else l2 = m;
  }
  return 0.5 * (l1 + l2);
}
// the state after the volumes of those midpoints
__device__ __forceinline__ OcState oc_advance(OcState s, const double* vol, int nc, double target) {
  if (s.l1 == 0.0) {
    const int stride = (int)s.stride;
    for (int c = 0; c < nc; ++c) {
      if (s.it + stride > OC_MAX_HALVINGS) {
        // the last halvings before the cap one by one
        if (stride == 1) break;
        s.stride = 1.0;
        break;
      }
      if (vol[c] > target) {
        if (stride == 1) {
          s.l1 = s.lm = 0.5 * s.l2;
          s.v1 = vol[c];
          s.it += 1.0;
        } else {
          s.stride = 1.0;         // within the next `stride` halvings
        }
        break;
      }
      s.l2 = s.lm = ldexp(s.l2, -stride);
      s.v2 = vol[c];
      s.it += stride;
    }
  } else {
    const double guess = oc_guess(s, target);
    for (int c = 0; c < nc && oc_more(s);) {
      s.lm = 0.5 * (s.l1 + s.l2);
      s.it += 1.0;
      const bool above = vol[c] > target;
      if (above) s.l1 = s.lm, s.v1 = vol[c];
      else s.l2 = s.lm, s.v2 = vol[c];
      if (guess == 0.0) c = 2 * c + 1 + (above ? 1 : 0);
      else if (above == (guess > s.lm)) ++c;
      else break;
    }
  }
  if (!oc_more(s)) s.done = 1.0;
  return s;
}

// the state this launch starts from: the previous launch's state advanced by
// its partial sums (prev NULL: the first launch), the same in every workgroup
__device__ __forceinline__ OcState oc_state(const double* prev, int nb, int nc, double target, double* vol) {
  if (!prev) return {0.0, 1e9, 0.5e9, 0.0, 0.0, (double)OC_STRIDE, NAN, NAN};
  OcState s = *(const OcState*)prev;
  if (s.done != 0.0) return s;
  const int c = threadIdx.x >> 5, l = threadIdx.x & 31;
  double a = 0.0;
  if (c < nc)
    for (int b = l; b < nb; b += 32) a += prev[OC_STATE_W + c * nb + b];
#pragma unroll
  for (int off = 16; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
  if (l == 0) vol[c] = a;
  __syncthreads();
  return oc_advance(s, vol, nc, target);
}

// v within the move limit and [0, 1]
__device__ __forceinline__ double oc_clip(double x, double v, double move) {
  return fmin(fmin(1.0, x + move), fmax(fmax(0.0, x - move), v));
}

__device__ __forceinline__ double oc_ratio(double dc, double dv) { return fmax(0.0, -dc) / fmax(dv, 1e-300); }

// xs = x sqrt(max(0, -dc) / dv): the unclipped design at multiplier 1
__global__ __launch_bounds__(TO_BLOCK) void k_oc_unit(const double* __restrict__ x, const double* __restrict__ dc,
                                                      const double* __restrict__ dv, long long n,
                                                      double* __restrict__ xs) {
  const long long e = (long long)blockIdx.x * TO_BLOCK + threadIdx.x;
  if (e < n) xs[e] = x[e] * sqrt(oc_ratio(dc[e], dv[e]));
}

// grid (nb, nc): partial volumes of midpoint blockIdx.y into next (of the
// designs xs / sqrt(lam), one multiplication per element)
template <int R>
__global__ __launch_bounds__(TO_BLOCK) void k_oc_volumes(Hat h, Dims D, const double* __restrict__ x,
                                                         const double* __restrict__ xs, double move, double beta,
                                                         double eta, double target,
                                                         const double* __restrict__ prev, double* __restrict__ next) {
  __shared__ double sv[Tile<R>::N], sh[4], vol[TO_BLOCK / 32];
  const int nb = gridDim.x, nc = gridDim.y, c = blockIdx.y;
  const OcState s = oc_state(prev, nb, nc, target, vol);
  if (blockIdx.x == 0 && c == 0 && threadIdx.x == 0) *(OcState*)next = s;
  if (s.done != 0.0) return;
  const double lam = oc_midpoint(s, c, target);
  if (lam == 0.0) {
    if (threadIdx.x == 0) next[OC_STATE_W + c * nb + blockIdx.x] = 0.0;
    return;
  }
  const double il = 1.0 / sqrt(lam);
  const double a = volume_part<R>(h, D, blockIdx.x, nb, beta, eta, sv, sh, [&](long long e, int, int, int) {
    return oc_clip(x[e], xs[e] * il, move);
  });
  if (threadIdx.x == 0) next[OC_STATE_W + c * nb + blockIdx.x] = a;
}

// once the stop test is met: the design of the last midpoint,
// x sqrt(ratio / lam), over the unit designs
__global__ __launch_bounds__(TO_BLOCK) void k_oc_design(const double* __restrict__ x, const double* __restrict__ dc,
                                                        const double* __restrict__ dv, long long n, double move,
                                                        double target, int nb, int nc, const double* prev,
                                                        double* state, double* __restrict__ xn) {
  __shared__ double vol[TO_BLOCK / 32];
  const OcState s = oc_state(prev, nb, nc, target, vol);
  if (blockIdx.x == 0 && threadIdx.x == 0) *(OcState*)state = s;
  const long long e = (long long)blockIdx.x * TO_BLOCK + threadIdx.x;
  if (s.done != 0.0 && e < n) xn[e] = oc_clip(x[e], x[e] * sqrt(oc_ratio(dc[e], dv[e]) / s.lm), move);
}

int stencil_R(double r_min) { return (int)std::floor(r_min); }

int nblocks(long long n) { return (int)std::max<long long>(1, std::min<long long>(1024, (n + TO_BLOCK - 1) / TO_BLOCK)); }
unsigned nblocks_all(long long n) { return (unsigned)((n + TO_BLOCK - 1) / TO_BLOCK); }

long long n_elem(const tg_grid* g) { return (long long)g->nx * g->ny * g->nz; }

int check_grid(const tg_grid* g) {
  if (!g || !g->bound) return fail(TG_ESTATE, "grid has no bound workspace");
  return TG_OK;
}

int check_r(double r_min) {
  if (!(r_min > 0) || !(r_min < TO_MAX_R + 1)) return fail(TG_EINVAL, "need 0 < r_min < 4");
  return TG_OK;
}

Hat hat_of(double r) {
  Hat h = {};
  const int R = stencil_R(r);
  for (int q = 0; q <= 3 * R * R; ++q) h.w[q] = std::max(0.0, r - std::sqrt((double)q));
  for (int dz = -R; dz <= R; ++dz)
    for (int dy = -R; dy <= R; ++dy)
      for (int dx = -R; dx <= R; ++dx) h.wsum += h.w[dx * dx + dy * dy + dz * dz];
  return h;
}

Dims dims_of(const tg_grid* g) {
  using T = Tile<0>;
  return {g->nx, g->ny, g->nz, (g->nx + T::X - 1) / T::X, (g->ny + T::Y - 1) / T::Y, (g->nz + T::Z - 1) / T::Z,
          n_elem(g)};
}
unsigned n_tiles(const Dims& D) { return (unsigned)D.tx * D.ty * D.tz; }

struct Projection {
  double beta, eta, t1, den;
};
Projection projection_of(double beta, double eta) {
  const double t1 = std::tanh(beta * eta);
  return {beta, eta, t1, t1 + std::tanh(beta * (1.0 - eta))};
}

// LAUNCH(R) with the stencil half-width as a constant
#define TO_BY_R(r, LAUNCH)      \
  do {                          \
    switch (stencil_R(r)) {     \
      case 0: LAUNCH(0); break; \
      case 1: LAUNCH(1); break; \
      case 2: LAUNCH(2); break; \
      default: LAUNCH(3);       \
    }                           \
    TG_HIP(hipGetLastError());  \
  } while (0)

int launch_filter(const tg_grid* g, const double* x, double r, const Projection& pr, double* xt, double* xbar,
                  double* dxbar, hipStream_t s) {
  const Hat h = hat_of(r);
  const Dims D = dims_of(g);
#define TO_FILTER(R) k_filter<R><<<n_tiles(D), TO_BLOCK, 0, s>>>(h, D, x, pr.beta, pr.eta, pr.t1, pr.den, xt, xbar, dxbar)
  TO_BY_R(r, TO_FILTER);
#undef TO_FILTER
  return TG_OK;
}

int read_parts(const tg_grid* g, int nb, std::vector<double>& h, hipStream_t s) {
  h.resize(nb);
  TG_HIP(hipMemcpyAsync(h.data(), g->desc.part, sizeof(double) * nb, hipMemcpyDeviceToHost, s));
  TG_HIP(hipStreamSynchronize(s));
  return TG_OK;
}

// sum_e project(H x)_e through the grid's partial-sum scratch
int volume_host(const tg_grid* g, const double* x, double r, const Projection& pr, hipStream_t s, double* out) {
  const Hat h = hat_of(r);
  const Dims D = dims_of(g);
  const int nb = (int)std::min<long long>(n_tiles(D), std::min<long long>(256, (long long)TG_PART_W * g->lv[0].n_chunks));
#define TO_VOLUME(R) k_volume<R><<<nb, TO_BLOCK, 0, s>>>(h, D, x, pr.beta, pr.eta, g->desc.part)
  TO_BY_R(r, TO_VOLUME);
#undef TO_VOLUME
  std::vector<double> p;
  const int rc = read_parts(g, nb, p, s);
  if (rc) return rc;
  double th = 0.0;
  for (double v : p) th += v;
  *out = ((double)D.n * pr.t1 + th) / pr.den;
  return TG_OK;
}

// max_e |a_e - b_e|
int change_host(const tg_grid* g, const double* a, const double* b, hipStream_t s, double* out) {
  const long long n = n_elem(g);
  const int nb = (int)std::min<long long>(nblocks(n), (long long)TG_PART_W * g->lv[0].n_chunks);
  k_max_change<<<nb, TO_BLOCK, 0, s>>>(a, b, n, g->desc.part);
  TG_HIP(hipGetLastError());
  std::vector<double> p;
  const int rc = read_parts(g, nb, p, s);
  if (rc) return rc;
  *out = *std::max_element(p.begin(), p.end());
  return TG_OK;
}

int oc_update(const tg_grid* g, const double* x, const double* dc, const double* dv, double volfrac, double move,
              double r, const Projection& pr, double* xn, double* lam_out, hipStream_t s) {
  const Hat h = hat_of(r);
  const Dims D = dims_of(g);
  // the volume sum_e (t1 + tanh(...)_e) / den against volfrac n, as a bound on the sum of the tanh
  const double target = volfrac * (double)D.n * pr.den - (double)D.n * pr.t1;
  // Midpoints per launch: a launch costs about 7 us beside its work (its own
  // start and the previous launch's sums), and the work of one midpoint is
  // about 1 us per 65,536 elements (14 us per launch of seven there), so seven
  // at once (some 8 launches, against 14 with three and 35 to 40 with one) pay up
  // to 2^18 elements and three up to 2^20.
  const int nc = D.n <= (1 << 18) ? 7 : D.n <= (1 << 20) ? 3 : 1;
  // two buffers of one state and nc rows of partial sums each, and a state
  const long long cap = (long long)TG_PART_W * g->lv[0].n_chunks;
  const int nb = (int)std::min<long long>({(long long)n_tiles(D), 128, (cap - 3 * OC_STATE_W) / (2 * nc)});
  double* buf[2] = {g->desc.part, g->desc.part + OC_STATE_W + (long long)nc * nb};
  double* fin = buf[1] + OC_STATE_W + (long long)nc * nb;
  k_oc_unit<<<nblocks_all(D.n), TO_BLOCK, 0, s>>>(x, dc, dv, D.n, xn);
  TG_HIP(hipGetLastError());
  const double* prev = nullptr;
  int t = 0;
  // the launches that most updates need before the first look at the state (7 or 8,
  // 12 to 15, 33 to 42 over multipliers of 1e-12 to 1e6), then some more
  for (int more = nc == 7 ? 8 : nc == 3 ? 15 : 42;; more = nc == 1 ? 6 : 3) {
    for (int q = 0; q < more; ++q, ++t) {
      double* next = buf[t & 1];
#define TO_OC(R)                                                                                                    \
  k_oc_volumes<R><<<dim3(nb, nc), TO_BLOCK, 0, s>>>(h, D, x, xn, move, pr.beta, pr.eta, target, prev, next)
      TO_BY_R(r, TO_OC);
#undef TO_OC
      prev = next;
    }
    k_oc_design<<<nblocks_all(D.n), TO_BLOCK, 0, s>>>(x, dc, dv, D.n, move, target, nb, nc, prev, fin, xn);
    TG_HIP(hipGetLastError());
    OcState st;
    TG_HIP(hipMemcpyAsync(&st, fin, sizeof(st), hipMemcpyDeviceToHost, s));
    TG_HIP(hipStreamSynchronize(s));
    if (st.done != 0.0) {
      if (lam_out) *lam_out = st.lm;
      return TG_OK;
    }
  }
}

}  // namespace
}  // namespace tg

using namespace tg;

extern "C" {

int tg_density_filter(const tg_grid* g, const double* x_d, double r_min, double* xt_d, void* stream) {
  int rc = check_grid(g);
  if (rc) return rc;
  if ((rc = check_r(r_min))) return rc;
  if (!x_d || !xt_d) return fail(TG_EINVAL, "NULL argument");
  return launch_filter(g, x_d, r_min, {0.0, 0.5, 0.0, 1.0}, xt_d, nullptr, nullptr, (hipStream_t)stream);
}

int tg_density_filter_adjoint(const tg_grid* g, const double* a_d, const double* b_d, double r_min, double* y_d,
                              void* stream) {
  int rc = check_grid(g);
  if (rc) return rc;
  if ((rc = check_r(r_min))) return rc;
  if (!a_d || !y_d) return fail(TG_EINVAL, "NULL argument");
  if (a_d == y_d || b_d == y_d) return fail(TG_EINVAL, "output must not alias an input");
  hipStream_t s = (hipStream_t)stream;
  const Hat h = hat_of(r_min);
  const Dims D = dims_of(g);
#define TO_ADJ(R) k_filter_adj<R><<<n_tiles(D), TO_BLOCK, 0, s>>>(h, D, a_d, b_d, y_d)
  TO_BY_R(r_min, TO_ADJ);
#undef TO_ADJ
  return TG_OK;
}

int tg_filter_project(const tg_grid* g, const double* x_d, double r_min, double beta, double eta, double* xt_d,
                      double* xbar_d, double* dxbar_d, void* stream) {
  int rc = check_grid(g);
  if (rc) return rc;
  if ((rc = check_r(r_min))) return rc;
  if (!x_d || !xbar_d) return fail(TG_EINVAL, "NULL argument");
  if (!(beta > 0) || !(eta > 0 && eta < 1)) return fail(TG_EINVAL, "need beta > 0 and 0 < eta < 1");
  return launch_filter(g, x_d, r_min, projection_of(beta, eta), xt_d, xbar_d, dxbar_d, (hipStream_t)stream);
}

int tg_oc_update(const tg_grid* g, const double* x_d, const double* dc_d, const double* dv_d, double volfrac,
                 double move, double r_min, double beta, double eta, double* x_new_d, double* lambda_h,
                 void* stream) {
  int rc = check_grid(g);
  if (rc) return rc;
  if ((rc = check_r(r_min))) return rc;
  if (!x_d || !dc_d || !dv_d || !x_new_d) return fail(TG_EINVAL, "NULL argument");
  if (!(volfrac > 0 && volfrac < 1) || !(move > 0) || !(beta > 0) || !(eta > 0 && eta < 1))
    return fail(TG_EINVAL, "need 0 < volfrac < 1, move > 0, beta > 0, 0 < eta < 1");
  return oc_update(g, x_d, dc_d, dv_d, volfrac, move, r_min, projection_of(beta, eta), x_new_d, lambda_h,
                   (hipStream_t)stream);
}

void tg_default_topopt(tg_topopt_opts* o) {
  if (!o) return;
  std::memset(o, 0, sizeof(*o));
  o->max_iters = 40;
  o->min_iters = 20;
  o->tol = 0.01;
  o->volfrac = 0.30;
  o->r_min = 1.5;
  o->eta = 0.5;
  o->n_stages = 2;
  o->stages[0] = {1, 1.5, 1.0, 0.20};
  o->stages[1] = {16, 3.5, 4.0, 0.15};
  o->mode = TG_LOOP_GUARDED;
  o->fixed_floor = 1e-3;
  tg_default_policy(&o->policy);
  o->policy.n_rungs = 3;
  o->policy.rungs[0] = 1e-12;
  o->policy.rungs[1] = 1e-3;
  o->policy.rungs[2] = 1e-2;
}

int tg_topopt_workspace_bytes(const tg_grid* g, size_t* bytes) {
  if (!g || !bytes) return fail(TG_EINVAL, "NULL argument");
  const size_t ne = (size_t)g->nx * g->ny * g->nz, nd = (size_t)g->lv[0].n_dof;
  auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
  *bytes = 7 * al(ne * sizeof(double)) + al(nd * sizeof(double));
  return TG_OK;
}

int tg_topopt_run(tg_grid* g, const double* f_d, const tg_topopt_opts* o, void* ws_d, size_t ws_bytes,
                  double* x_d, tg_topopt_record* rec, int* n_rec, void* stream) {
  int rc = check_grid(g);
  if (rc) return rc;
  if (!f_d || !o || !ws_d || !x_d || !rec || !n_rec) return fail(TG_EINVAL, "NULL argument");
  if ((rc = check_r(o->r_min))) return rc;
  if (o->n_stages < 1 || o->n_stages > 4 || o->stages[0].first_iter != 1 || o->max_iters < 1)
    return fail(TG_EINVAL, "need 1..4 continuation stages, the first starting at iteration 1");
  if (o->mode < TG_LOOP_GUARDED || o->mode > TG_LOOP_FIXED) return fail(TG_EINVAL, "bad loop mode");
  size_t need = 0;
  tg_topopt_workspace_bytes(g, &need);
  if (ws_bytes < need) return fail(TG_EWORKSPACE, "topopt workspace too small");
  hipStream_t s = (hipStream_t)stream;
  const size_t ne = (size_t)n_elem(g);
  auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
  char* w = (char*)ws_d;
  double* B[7];
  for (int i = 0; i < 7; ++i, w += al(ne * sizeof(double))) B[i] = (double*)w;
  double *xt = B[0], *xbar = B[1], *dxbar = B[2], *dcp = B[3], *dcd = B[4], *dv = B[5], *xn = B[6];
  double* u = (double*)w;
  const double r = o->r_min, eta = o->eta;
  const tg_policy& pol0 = o->policy;
  int prev_rung = -1;
  *n_rec = 0;
  for (int t = 1; t <= o->max_iters; ++t) {
    const auto t0 = std::chrono::steady_clock::now();
    int st = 0;
    for (int q = 0; q < o->n_stages; ++q)
      if (t >= o->stages[q].first_iter) st = q;
    const double p = o->stages[st].p, beta = o->stages[st].beta, move = o->stages[st].move;
    tg_topopt_record& R = rec[t - 1];
    std::memset(&R, 0, sizeof(R));
    R.iter = t;
    R.p = p;
    R.beta = beta;
    if ((rc = tg_filter_project(g, x_d, r, beta, eta, xt, xbar, dxbar, stream))) return rc;
    // the state solve
    tg_policy pol = pol0;
    pol.p = p;
    double floor = -1.0;
    if (o->mode == TG_LOOP_FIXED) {
      if ((rc = tg_set_density(g, xbar, p, o->fixed_floor, stream))) return rc;
      tg_solve_result sr;
      if ((rc = tg_fgmres_solve(g, f_d, u, &pol.solve, &sr, nullptr, stream))) return rc;
      if ((rc = tg_true_residual(g, f_d, u, &R.true_eta, stream))) return rc;
      R.solve_iters = sr.iterations;
      R.accepted = -1;           // no acceptance test
      R.rung = -1;
      floor = o->fixed_floor;
    } else {
      bool done = false;
      if (o->mode == TG_LOOP_REUSE && prev_rung >= 0) {
        // the previous decision, kept while the guard accepts it
        if ((rc = tg_set_density(g, xbar, p, pol.rungs[prev_rung], stream))) return rc;
        tg_solve_result sr;
        if ((rc = tg_fgmres_solve(g, f_d, u, &pol.solve, &sr, nullptr, stream))) return rc;
        double eta_t = 1.0;
        if ((rc = tg_true_residual(g, f_d, u, &eta_t, stream))) return rc;
        R.solve_iters += sr.iterations;
        if (eta_t <= pol.tau) {
          done = true;
          R.rung = prev_rung;
          R.true_eta = eta_t;
          R.accepted = 1;
          floor = pol.rungs[prev_rung];
        }
      }
      if (!done) {
        tg_policy_result pr;
        if ((rc = tg_select_floor(g, xbar, f_d, &pol, u, &pr, stream))) return rc;
        R.probed = 1;
        R.solve_iters += pr.iters_probe + pr.iters_selected + pr.iters_rejected;
        R.rung = pr.rung;
        if (pr.rung < 0) {
          R.accepted = 0;
          *n_rec = t;
          return TG_OK;          // no admissible floor: the loop stops here
        }
        R.true_eta = pr.attempts[pr.n_attempts - 1].true_eta;
        R.accepted = 1;
        floor = pr.floor;
        prev_rung = pr.rung;
      }
    }
    R.floor = floor;
    // compliance and its gradient with respect to the design
    if ((rc = tg_compliance_sensitivity(g, xbar, p, floor, f_d, u, nullptr, dcp, &R.compliance, stream))) return rc;
    if ((rc = tg_density_filter_adjoint(g, dcp, dxbar, r, dcd, stream))) return rc;
    if ((rc = tg_density_filter_adjoint(g, dxbar, nullptr, r, dv, stream))) return rc;
    if ((rc = oc_update(g, x_d, dcd, dv, o->volfrac, move, r, projection_of(beta, eta), xn, nullptr, s))) return rc;
    double vol = 0.0;
    // volume of the physical density this iteration solved with, and the
    // largest design change of the step
    if ((rc = volume_host(g, x_d, r, projection_of(beta, eta), s, &vol))) return rc;
    R.volume = vol / (double)ne;
    if ((rc = change_host(g, xn, x_d, s, &R.change))) return rc;
    TG_HIP(hipMemcpyAsync(x_d, xn, ne * sizeof(double), hipMemcpyDeviceToDevice, s));
    TG_HIP(hipStreamSynchronize(s));
    R.ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    *n_rec = t;
    if (t >= o->min_iters && R.change < o->tol) break;
  }
  return TG_OK;
}

}  // extern "C"
