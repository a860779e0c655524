// Device kernels of the guarded SIMP state solve (gfx950).
//
// All kernels take the batch descriptor array and a work list; workgroup b
// serves problem work[b].x, tile work[b].y.  Vectors are full length
// (3 * nodes, AoS) and hold zeros on the clamped x = 0 nodes.
#include <climits>
#include <mutex>

#include "tg_internal.h"

namespace tg {

// ---------------------------------------------------------------------------
// small device helpers
template <class T> __device__ __forceinline__ T* pool(const LevelDesc& L);
template <> __device__ __forceinline__ double* pool<double>(const LevelDesc& L) { return L.vec64; }
template <> __device__ __forceinline__ float* pool<float>(const LevelDesc& L) { return L.vec32; }

// slot >= 0: slot of the pool of type T at this level; slot < 0: external pointer
template <class T>
__device__ __forceinline__ T TG_GLOBAL* vslot(const LevelDesc& L, int slot, const void* ext) {
  return gp(slot < 0 ? (T*)ext : pool<T>(L) + (long long)slot * L.stride);
}
template <class T> __device__ __forceinline__ const T* Dinv(const LevelDesc& L);
template <> __device__ __forceinline__ const double* Dinv<double>(const LevelDesc& L) { return L.Dinv64; }
template <> __device__ __forceinline__ const float* Dinv<float>(const LevelDesc& L) { return L.Dinv32; }
template <class T> __device__ __forceinline__ const T* CinvP(const ProbDesc& P);
template <> __device__ __forceinline__ const double* CinvP<double>(const ProbDesc& P) { return P.Cinv64; }
template <> __device__ __forceinline__ const float* CinvP<float>(const ProbDesc& P) { return P.Cinv32; }

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sixteen wave sums at once: each butterfly stage pairs a lane with its
// partner across one lane bit and keeps half of the values, so 15 exchanges
// leave every lane with one value summed over 16 lanes, and two more finish the
// sum over the wave.  Lane l < 16 returns the total of value rev4(l), where
// rev4 reverses the four low bits (a fixed order: deterministic).
template <int H, int M>
__device__ __forceinline__ void sum16_stage(double* v, int lane) {
  const bool up = lane & M;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double keep = up ? v[i + H] : v[i];
    const double send = up ? v[i] : v[i + H];
    v[i] = keep + __shfl_xor(send, M, 64);
  }
}
__device__ __forceinline__ double wave_sum16(double* v, int lane) {
  sum16_stage<8, 1>(v, lane);
  sum16_stage<4, 2>(v, lane);
  sum16_stage<2, 4>(v, lane);
  sum16_stage<1, 8>(v, lane);
  double r = v[0];
  r += __shfl_xor(r, 16, 64);
  r += __shfl_xor(r, 32, 64);
  return r;
}
__device__ __forceinline__ int rev4(int l) {
  return ((l & 1) << 3) | ((l & 2) << 1) | ((l & 4) >> 1) | ((l & 8) >> 3);
}

// Deterministic block sum over 256 threads (4 waves); result valid in thread 0.
__device__ __forceinline__ double block_sum256(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) r = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  __syncthreads();
  return r;
}

// ---------------------------------------------------------------------------
// set_density: E_e = rho_min + (1 - rho_min) rho^p   (Eq. floor_scaling)
__global__ __launch_bounds__(256) void k_young(const ProbDesc* __restrict__ probs,
                                               const int2* __restrict__ work, double p,
                                               int* __restrict__ bad) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  const LevelDesc& L = P.lv[0];
  const long long n_e = (long long)L.ex * L.ey * L.ez;
  const long long e = (long long)wi.y * 256 + threadIdx.x;
  if (e >= n_e) return;
  const double r = P.ext0[e];
  if (!(r >= 0.0 && r <= 1.0)) {   // also catches NaN
    atomicOr(bad + wi.x, 1);
  }
  const double rc = fmin(fmax(r, 0.0), 1.0);
  const double E = P.rho_min + (1.0 - P.rho_min) * pow(rc, p);
  P.E64[e] = E;
  P.E32[e] = (float)E;
}

// Memory ordering between the lanes of one wave
// (the wave is in lockstep; the fence keeps the compiler and the LDS queue
// from moving a lane's reads above another lane's writes)
#define TG_WAVE_SYNC()                                       \
  do {                                                       \
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");   \
    __builtin_amdgcn_wave_barrier();                         \
  } while (0)

// Level-1 Galerkin element matrices: Kel1[C] = sum_c E[child c] * G_c, where
// G_c = P_c^T Ke P_c and P_c interpolates the coarse element's 24 DOFs to
// those of child c (trilinear, exact for nested hex8 spaces).  A thread keeps
// its three columns of G for the workgroup's elements, so what is left is to
// write the matrices.  The bytes written bound a large level: 2.4 GB at 128x64x64 in 538 us (one element per
// workgroup and G read from the cache for each: 1540).
__global__ __launch_bounds__(192) void k_galerkin1(const ProbDesc* __restrict__ probs,
                                                   const int2* __restrict__ work) {
  __shared__ double sE[TG_SETUP_CHUNK][8];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  const LevelDesc& Lf = P.lv[0];
  const LevelDesc& Lc = P.lv[1];
  const long long ne = (long long)Lc.ex * Lc.ey * Lc.ez, C0 = (long long)wi.y * setup_chunk(ne);
  const int nC = (int)(ne - C0 < setup_chunk(ne) ? ne - C0 : setup_chunk(ne));
  double G[3][8];
#pragma unroll
  for (int u = 0; u < 3; ++u)
#pragma unroll
    for (int c = 0; c < 8; ++c) G[u][c] = P.G64[c * 576 + 192 * u + threadIdx.x];
  if ((int)threadIdx.x < 8 * nC) {
    const int c = threadIdx.x & 7;
    const long long C = C0 + (threadIdx.x >> 3);
    const int cx = (int)(C % Lc.ex), cy = (int)((C / Lc.ex) % Lc.ey), cz = (int)(C / ((long long)Lc.ex * Lc.ey));
    const int fx = 2 * cx + (c & 1), fy = 2 * cy + ((c >> 1) & 1), fz = 2 * cz + (c >> 2);
    sE[threadIdx.x >> 3][c] = P.E64[fx + (long long)Lf.ex * (fy + (long long)Lf.ey * fz)];
  }
  __syncthreads();
  for (int q = 0; q < nC; ++q) {
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      double s = 0.0;
#pragma unroll
      for (int c = 0; c < 8; ++c) s += sE[q][c] * G[u][c];
      Lc.Kel64[(C0 + q) * 576 + 192 * u + threadIdx.x] = s;
    }
  }
}

// Weight of parent node A at node a of child c: the product over the
// dimensions of 1, 1/2 or 0 for a node at 0, 1/2 or 1 of the parent's edge.
__device__ constexpr double child_weight(int c, int a, int A) {
  double w = 1.0;
  for (int d = 0; d < 3; ++d) {
    const int pos = ((c >> d) & 1) + ((a >> d) & 1), q = (A >> d) & 1;
    w *= pos == 1 ? 0.5 : pos == 2 * q ? 1.0 : 0.0;
  }
  return w;
}
// X = (W^T x I3) Kel (W x I3) of child C by one wave, X in its LDS: the row
// products one item per (row, component), the column products one per
// (component, column), eight entries in and eight out, over the 27 nonzero
// weights of 64 and in the order of the child's nodes.
template <int C>
__device__ __forceinline__ void galerkin_child(const double* K, double* X, int lane) {
  const auto* Kg = gp(K);
  for (int it = lane; it < 72; it += 64) {
    const int r = it / 3, j = it - 3 * r;
    double k[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) k[a] = Kg[24 * r + 3 * a + j];
#pragma unroll
    for (int A = 0; A < 8; ++A) {
      double t = 0.0;
#pragma unroll
      for (int a = 0; a < 8; ++a)
        if (child_weight(C, a, A) != 0.0) t += k[a] * child_weight(C, a, A);
      X[24 * r + 3 * A + j] = t;
    }
  }
  TG_WAVE_SYNC();
  for (int it = lane; it < 72; it += 64) {
    const int i = it / 24, col = it - 24 * i;
    double t[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) t[b] = X[24 * (3 * b + i) + col];
#pragma unroll
    for (int B = 0; B < 8; ++B) {
      double x = 0.0;
#pragma unroll
      for (int b = 0; b < 8; ++b)
        if (child_weight(C, b, B) != 0.0) x += child_weight(C, b, B) * t[b];
      X[24 * (3 * B + i) + col] = x;
    }
  }
}
// Level l -> l+1 (l >= 1): Kel_{l+1}[C] = sum_c P_c^T Kel_l[child c] P_c, a wave
// per child, the eight products added in the children's order.  Each P_c is a
// scalar trilinear weight matrix times I_3, so both products sum over the 8
// nodes of a component, not over 24 DOFs.  Bounded by latency on small levels
// (6.2 us where eight children in turn, each entry's products read from LDS, took
// 22.2) and by reading the children on large ones (the levels of 256x128x128:
// 711 us together, 1688 before).
__global__ __launch_bounds__(512) void k_galerkin_up(const ProbDesc* __restrict__ probs,
                                                     const int2* __restrict__ work, int lc) {
  __shared__ double sX[8][576];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  const LevelDesc& Lf = P.lv[lc - 1];
  const LevelDesc& Lc = P.lv[lc];
  const long long ne = (long long)Lc.ex * Lc.ey * Lc.ez, C0 = (long long)wi.y * setup_chunk(ne);
  const int nC = (int)(ne - C0 < setup_chunk(ne) ? ne - C0 : setup_chunk(ne));
  const int lane = threadIdx.x & 63, c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (long long C = C0; C < C0 + nC; ++C) {
    const int cx = (int)(C % Lc.ex), cy = (int)((C / Lc.ex) % Lc.ey), cz = (int)(C / ((long long)Lc.ex * Lc.ey));
    const int fx = 2 * cx + (c & 1), fy = 2 * cy + ((c >> 1) & 1), fz = 2 * cz + (c >> 2);
    const double* K = Lf.Kel64 + 576 * (fx + (long long)Lf.ex * (fy + (long long)Lf.ey * fz));
    switch (c) {
      case 0: galerkin_child<0>(K, sX[0], lane); break;
      case 1: galerkin_child<1>(K, sX[1], lane); break;
      case 2: galerkin_child<2>(K, sX[2], lane); break;
      case 3: galerkin_child<3>(K, sX[3], lane); break;
      case 4: galerkin_child<4>(K, sX[4], lane); break;
      case 5: galerkin_child<5>(K, sX[5], lane); break;
      case 6: galerkin_child<6>(K, sX[6], lane); break;
      default: galerkin_child<7>(K, sX[7], lane); break;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < 576; q += 512) {
      double s = 0.0;
#pragma unroll
      for (int m = 0; m < 8; ++m) s += sX[m][q];
      Lc.Kel64[C * 576 + q] = s;
    }
    if (C + 1 < C0 + nC) __syncthreads();
  }
}

// Mode-basis form of the level-l Galerkin element matrices (l > TG_MF_LEVELS):
// Khat = H Kel H^T / 64 with H the per-component 8-point +-1 transform of
// the node index (DOF 3 a + c -> 3 m + c, H[m][a] = prod over the bits b of m
// of (2 bit_b(a) - 1)), symmetrized, and its TG_GM_NU pattern entries stored
// at Km[e * TG_GM_STRIDE + v] (padding zero).  Entries off the pattern vanish
// in exact arithmetic.
__device__ __forceinline__ void mode_pack(const LevelDesc& L, long long e, double* sX) {
  auto H = [](int m, int a) { return (__popc(m & ~a) & 1) ? -1.0 : 1.0; };
  // X = (H x I3) Kel: eight entries of a column in, eight out
  if (threadIdx.x < 72) {
    const int i = threadIdx.x / 24, c = threadIdx.x - 24 * i;
    const auto* K = gp((const double*)L.Kel64) + e * 576;
    double k[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) k[a] = K[(3 * a + i) * 24 + c];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      double t = 0.0;
#pragma unroll
      for (int a = 0; a < 8; ++a) t += H(m, a) * k[a];
      sX[(3 * m + i) * 24 + c] = t;
    }
  }
  __syncthreads();
  if (threadIdx.x < TG_GM_STRIDE) {
    const int v = threadIdx.x;
    double k = 0.0;
    if (v < TG_GM_NU) {
      const int r = kGMPairs[v][0], c = kGMPairs[v][1];
      // Khat[r][c] = sum_b X[r][3 b + j] H[n][b] / 64, and its transpose
      const int n = c / 3, j = c % 3, m = r / 3, i = r % 3;
      double t1 = 0.0, t2 = 0.0;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        t1 += sX[r * 24 + 3 * b + j] * H(n, b);
        t2 += sX[c * 24 + 3 * b + i] * H(m, b);
      }
      k = 0.5 * (t1 + t2) / 64.0;
    }
    L.Km64[gm_index(e, v, 2)] = k;
    L.Km32[gm_index(e, v, 4)] = (float)k;
  }
}

// Node-block diagonal (3x3, coupling u_x, u_y, u_z of one node) and its inverse.
// The eight elements' entries are read together, those outside the grid count
// zero.
__device__ __forceinline__ void nodeblock(const ProbDesc& P, int l, int n) {
  const LevelDesc& L = P.lv[l];
  if (n >= L.n_nodes) return;
  const int i = n % L.NX, t = n / L.NX, j = t % L.NY, k = t / L.NY;
  const auto* Eg = gp((const double*)P.E64);
  const auto* Kg = gp(l == 0 ? P.Ke64 : (const double*)L.Kel64);
  double B[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int ex = i - (a & 1), ey = j - ((a >> 1) & 1), ez = k - ((a >> 2) & 1);
    const bool in = ex >= 0 && ex < L.ex && ey >= 0 && ey < L.ey && ez >= 0 && ez < L.ez;
    const long long e = in ? ex + (long long)L.ex * (ey + (long long)L.ey * ez) : 0;
    if (l == 0) {
      const double E = in ? Eg[e] : 0.0;
#pragma unroll
      for (int q = 0; q < 9; ++q) {
#pragma clang fp contract(off)
        const double v = E * Kg[(3 * a + q / 3) * 24 + 3 * a + q % 3];
        B[q] += v;
      }
    } else {
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const double v = Kg[e * 576 + (3 * a + q / 3) * 24 + 3 * a + q % 3];
        B[q] += in ? v : 0.0;
      }
    }
  }
  double D[9];
  if (i == 0) {
    for (int q = 0; q < 9; ++q) D[q] = (q % 4 == 0) ? 1.0 : 0.0;
  } else {
    const double c00 = B[4] * B[8] - B[5] * B[7];
    const double c01 = B[5] * B[6] - B[3] * B[8];
    const double c02 = B[3] * B[7] - B[4] * B[6];
    const double det = B[0] * c00 + B[1] * c01 + B[2] * c02;
    const double id = 1.0 / det;
    D[0] = c00 * id;
    D[1] = (B[2] * B[7] - B[1] * B[8]) * id;
    D[2] = (B[1] * B[5] - B[2] * B[4]) * id;
    D[3] = c01 * id;
    D[4] = (B[0] * B[8] - B[2] * B[6]) * id;
    D[5] = (B[2] * B[3] - B[0] * B[5]) * id;
    D[6] = c02 * id;
    D[7] = (B[1] * B[6] - B[0] * B[7]) * id;
    D[8] = (B[0] * B[4] - B[1] * B[3]) * id;
  }
  for (int q = 0; q < 9; ++q) {
    L.Dinv64[9LL * n + q] = D[q];
    L.Dinv32[9LL * n + q] = (float)D[q];
  }
}

// Node coordinates and component of a free DOF of the coarsest level, one byte
// each (i, j, k, component); a level of at most TG_MAX_COARSE free DOFs has
// fewer than 256 nodes in every dimension.
__device__ __forceinline__ int coarse_dof(const LevelDesc& L, int r) {
  const int nxm = L.NX - 1, f = r / 3, t = f / nxm, k = t / L.NY;
  return (f - t * nxm + 1) | (t - k * L.NY) << 8 | k << 16 | (r - 3 * f) << 24;
}
// Entry (r, c) of the coarsest level's assembled free-DOF matrix (dr, dc: the
// two DOFs' coarse_dof): the sum of the element entries that couple them, over
// the up to eight elements both nodes share, in ascending element order; the
// unit matrix beyond n.  The eight loads are issued together (absent elements
// read entry 0).
__device__ __forceinline__ double coarse_entry(const ProbDesc& P, const LevelDesc& L, bool fine, int n, int r,
                                               int c, int dr, int dc) {
  const bool pad = r >= n || c >= n;
  const double unit = pad && r == c ? 1.0 : 0.0;
  const int i = dr & 255, j = (dr >> 8) & 255, kr = (dr >> 16) & 255, cr = dr >> 24, cc = dc >> 24;
  const int di = (dc & 255) - i, dj = ((dc >> 8) & 255) - j, dk = ((dc >> 16) & 255) - kr;
  const bool near = !pad && di >= -1 && di <= 1 && dj >= -1 && dj <= 1 && dk >= -1 && dk <= 1;
  if (!__any(near)) return unit;
  const auto* Kg = gp(fine ? P.Ke64 : (const double*)L.Kel64);
  const auto* Eg = gp((const double*)P.E64);
  double k[8], E[8];
  bool in[8];
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    // the element in which node (i, j, kr) is corner a; the other node's corner
    const int ax = a & 1, ay = (a >> 1) & 1, az = a >> 2;
    const int bx = ax + di, by = ay + dj, bz = az + dk;
    const int ex = i - ax, ey = j - ay, ez = kr - az;   // ex >= 0: i >= 1
    in[a] = near && bx >= 0 && bx <= 1 && by >= 0 && by <= 1 && bz >= 0 && bz <= 1 && ex < L.ex && ey >= 0 &&
            ey < L.ey && ez >= 0 && ez < L.ez;
    const int e = in[a] ? ex + L.ex * (ey + L.ey * ez) : 0;
    const int q = in[a] ? (3 * a + cr) * 24 + 3 * (bx + 2 * by + 4 * bz) + cc : 0;
    k[a] = Kg[fine ? q : 576 * e + q];
    E[a] = fine ? Eg[e] : 1.0;
  }
  double s = 0.0;
#pragma unroll
  for (int a = 7; a >= 0; --a) s += in[a] ? E[a] * k[a] : 0.0;
  return pad ? unit : s;
}

// The node blocks of every level, the mode-basis elements of the stored ones and
// the assembled coarsest matrices, in one launch: all of them read the finished
// element matrices only.
// Workgroups [end of the list before, end[u]) take list u (level u's nodes
// for u < TG_MAXLEV, level u - TG_MAXLEV's elements from there), those behind them
// a 16 x 16 tile of a problem's coarsest matrix each, which k_coarse_inverse reads
// (assembled by that kernel's one workgroup, 322 us at n = 288 in place of 265).  At 48x24x24 14.9 us in place of
// six launches, 72 us; at 256x128x128 883 us, 1277 before.
struct SetupTail {
  const int2* list[2 * TG_MAXLEV];
  int end[2 * TG_MAXLEV];
  const int2* prob;
  int tiles;                // per problem, of the largest
};
// Tile t (row I, column J: t = I (I + 1) / 2 + J) to Cwork + 256 t, in the layout
// of the matrix cores' results.
__device__ __forceinline__ void coarse_tile(const ProbDesc& P, int t) {
  const int n = P.ncoarse, T = (n + 15) >> 4;
  if (t >= T * (T + 1) / 2) return;
  int I = 0;
  while ((I + 1) * (I + 2) / 2 <= t) ++I;
  const int J = t - I * (I + 1) / 2, lane = threadIdx.x & 63;
  const LevelDesc& L = P.lv[P.nlev - 1];
  const int r = 16 * I + (lane >> 4) + 4 * (threadIdx.x >> 6), c = 16 * J + (lane & 15);
  const int hi = max(r, c), lo = min(r, c);
  P.Cwork[t * 256 + threadIdx.x] = coarse_entry(P, L, P.nlev == 1, n, hi, lo, coarse_dof(L, hi), coarse_dof(L, lo));
}
__global__ __launch_bounds__(256) void k_setup_tail(const ProbDesc* __restrict__ probs, SetupTail w) {
  __shared__ double sX[576];
  const int nb = w.end[2 * TG_MAXLEV - 1];
  if ((int)blockIdx.x >= nb) {
    const int q = (int)blockIdx.x - nb;
    coarse_tile(probs[w.prob[q / w.tiles].x], q % w.tiles);
    return;
  }
  int u = 0, b0 = 0;
#pragma unroll
  for (int q = 0; q < 2 * TG_MAXLEV - 1; ++q)
    if ((int)blockIdx.x >= w.end[q]) {
      u = q + 1;
      b0 = w.end[q];
    }
  const int2* list = w.list[0];
#pragma unroll
  for (int q = 1; q < 2 * TG_MAXLEV; ++q)
    if (u == q) list = w.list[q];
  const int2 wi = list[blockIdx.x - b0];
  const ProbDesc& P = probs[wi.x];
  if (u < TG_MAXLEV) {
    nodeblock(P, u, wi.y * TG_NODE_TILE + threadIdx.x);
    return;
  }
  const LevelDesc& L = P.lv[u - TG_MAXLEV];
  const long long ne = (long long)L.ex * L.ey * L.ez, e0 = (long long)wi.y * setup_chunk(ne);
  const long long e1 = e0 + setup_chunk(ne) < ne ? e0 + setup_chunk(ne) : ne;
  for (long long e = e0; e < e1; ++e) {
    if (e > e0) __syncthreads();
    mode_pack(L, e, sX);
  }
}

// One 64-bit value of lane `lane` (a constant), in every lane of the wave.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(w.x, lane),
                                              __builtin_amdgcn_readlane(w.y, lane)));
}
// Lane K of each row of 16 lanes, in every lane of that row.
template <int K>
__device__ __forceinline__ double row_value(double v) {
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, w.x, 0x150 + K, 0xf, 0xf, false),
                                              __builtin_amdgcn_update_dpp(0, w.y, 0x150 + K, 0xf, 0xf, false)));
}

// Pivot K of the unit-lower elimination of a 16 x 16 symmetric block held by
// one wave (lane l: row l % 16, columns 4 (l / 16) + q): with m = the unit
// matrix at the start, all sixteen pivots leave m = M, the inverse of the unit
// lower factor of A = M^-1 diag(p) M^-T.  pinv: 1 / p of this lane's row.
template <int K>
__device__ __forceinline__ void ldl_pivot(double* a, double* m, int lane, double& pinv, bool& ok) {
  const int row = lane & 15;
  const double p = lane_value(a[K & 3], K + 16 * (K >> 2));
  ok = ok && p > 0.0;
  const double d = 1.0 / p;
  if (row == K) pinv = d;
  const double col = __shfl(a[K & 3], row + 16 * (K >> 2), 64);   // a[row][K]
  const double f = row > K ? col * d : 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    a[q] -= f * row_value<K>(a[q]);
    m[q] -= f * row_value<K>(m[q]);
  }
}
template <int K = 0>
__device__ __forceinline__ void ldl_block(double* a, double* m, int lane, double& pinv, bool& ok) {
  if constexpr (K < 16) {
    ldl_pivot<K>(a, m, lane, pinv, ok);
    ldl_block<K + 1>(a, m, lane, pinv, ok);
  }
}

// Coarsest level's explicit inverse, one workgroup per problem: the assembled
// free-DOF matrix, padded with the unit matrix to T x T tiles of 16, is swept
// block pivot by block pivot.  With A_KK = M^-1 diag(p) M^-T, G_I = A_IK
// (= A_KI^T) and G'_I = G_I M^T:
//   A_IJ -= G'_I diag(1/p) G'_J^T,  A_IK <- G'_I diag(1/p) M,
//   A_KK <- -M^T diag(1/p) M,
// which keeps the matrix symmetric, so only the tiles I >= J are held, and
// leaves -A^-1.  (The factored form of A_KK^-1 keeps the Schur complements as
// accurate as a Cholesky elimination; its explicit inverse would not.)  No
// pivoting: the pivots are diagonal entries of successive Schur complements,
// positive for an SPD matrix (a non-positive one flags the problem).
// What bounds it is the chain of n pivots at small n: each 16 of them are done by
// one wave in registers (row and column of the pivot by lane moves, 3 to 5 us),
// beside the other waves' matrix-core update of the previous block, so a block
// pivot costs two barriers; from n = 200 or so that update (171 tiles at n = 288,
// 4.6 us of one CU's FP64 matrix rate).  One element-by-element Gauss-Jordan
// pivot per barrier took 170 us at n = 108, and the global-memory Cholesky that
// n > 141 used took 22.9 ms at n = 288; this form takes 38 and 244 us (47 and 322
// with the matrix assembled by the one workgroup and no tile skipped).
// Where the tiles are: all in LDS, beside the panel, up to CI_LDS_N (ten tile rows,
// 141 KB, would fit too; at 150 unknowns the next form takes the same time: set-up of
// 4x8x8 103.5 us either way); up to CI_REG_N most of those left of the diagonal in
// registers, 8 a wave, the rest in LDS; beyond, in the problem's work array, which one workgroup's waves keep in
// cache (n = 288 that way: 265 us).
// Lane layouts of v_mfma_f64_16x16x4 (measured on gfx950): A[i][k] and
// B[k][j] at lane i (j) + 16 k; D[i][j] at lane 16 (i % 4) + j, element i / 4.
// A tile is stored in the D layout; slot s of lane group c is k = c + 4 s in
// every product.
#define CI_THREADS 1024
#define CI_LDS_N 144    // 45 tiles (92 KB) and a 20 KB panel
#define CI_REG_N 288    // 171 tiles: 120 in registers, 51 in LDS (105 KB) beside a 42 KB panel
#define CI_SLOTS 8      // tiles that a wave holds in registers
enum { CI_LDS = 0, CI_REG = 1, CI_MEM = 2 };
#define CI_LD 18        // panel row stride (16 columns, padded)
#define CI_M (16 * CI_LD + 16)   // M and 1 / p of a block pivot
typedef double f64x4 __attribute__((ext_vector_type(4)));
// tiles left of the diagonal that the register form holds in registers
__host__ __device__ inline int ci_reg_tiles(int T) {
  const int off = T * (T - 1) / 2, cap = CI_SLOTS * (CI_THREADS / 64 - 1);
  return off < cap ? off : cap;
}
__host__ __device__ inline size_t ci_lds_words(int n, int form) {
  const int T = (n + 15) / 16, NT = T * (T + 1) / 2;
  // panel, two M blocks, tile order and panel flags (32-bit each), tiles
  return (size_t)16 * T * CI_LD + 2 * CI_M + (NT + T + 1) / 2 +
         256 * (size_t)(form == CI_LDS ? NT : form == CI_REG ? NT - ci_reg_tiles(T) : 0);
}

// f(0), .., f(N - 1) with constant arguments (register arrays need constant indices)
template <int N, int I = 0, class F>
__device__ __forceinline__ void ci_each(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>());
    ci_each<N, I + 1>(f);
  }
}

template <int FORM>
__global__ __launch_bounds__(CI_THREADS) void k_coarse_inverse(const ProbDesc* __restrict__ probs,
                                                               const int2* __restrict__ work, int* bad, int nlo,
                                                               int nhi) {
  extern __shared__ double smem[];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  const int n = P.ncoarse;
  if (n == 0 || n < nlo || n > nhi) return;   // no direct coarsest level, or the other form's size
  const int T = (n + 15) >> 4, NT = T * (T + 1) / 2;
  double* G = smem;                       // panel: row r, column k at r CI_LD + k
  double* sM = G + 16 * T * CI_LD;        // M, same row stride, then 1 / p; of even and odd block pivots
  int* sT = (int*)(sM + 2 * CI_M);      // tile u in column order: I | J << 8
  int* sZ = sT + NT;                      // whether tile row I of the panel is not all zero
  double* A = FORM != CI_MEM ? sM + 2 * CI_M + (NT + T + 1) / 2 : P.Cwork;
  // (wave: uniform, so that tile indices and addresses stay scalar)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lj = lane & 15, lc = lane >> 4;
  constexpr int NW = CI_THREADS / 64;
  // Register form: the tiles left of the diagonal in column order; wave 1 + v % 15
  // has tile v, in slot v / 15 while v < NR, else in LDS behind the T diagonal
  // tiles.  Wave 0 has none: it factors.
  const int NO = NT - T, NR = ci_reg_tiles(T);
  auto off_of = [&](int v) -> int {   // I | J << 8
    int J = 0, u = v;
    while (u >= T - 1 - J) u -= T - 1 - J++;
    return (J + 1 + u) | J << 8;
  };
  auto place = [&](int I, int J) -> int {
    if (FORM != CI_REG) return I * (I + 1) / 2 + J;
    return I == J ? I : T + J * (T - 1) - J * (J - 1) / 2 + I - J - 1 - NR;
  };
  for (int q = threadIdx.x; q < T * T; q += CI_THREADS) {
    const int J = q / T, I = q - J * T;
    if (I >= J) sT[J * T - J * (J - 1) / 2 + I - J] = I | J << 8;
  }
  if (threadIdx.x < T) sZ[threadIdx.x] = 0;
  __syncthreads();
  auto tile_of = [&](int u) -> int { return __builtin_amdgcn_readfirstlane(sT[u]); };
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
  // the assembled tiles (k_setup_tail) from the work array; the register form's
  // waves fetch their own below
  if constexpr (FORM != CI_MEM)
    for (int u = wave; u < NT; u += NW) {
      const int ij = tile_of(u), I = ij & 255, J = ij >> 8, t = place(I, J);
      const bool reg = FORM == CI_REG && t < T && I != J;
      const double* w = P.Cwork + 256 * (I * (I + 1) / 2 + J);
      if (!reg)
#pragma unroll
        for (int v = 0; v < 4; ++v) A[t * 256 + 64 * v + lane] = w[64 * v + lane];
    }
  auto put = [&](int t, const f64x4& c) {
#pragma unroll
    for (int v = 0; v < 4; ++v) A[t * 256 + 64 * v + lane] = c[v];
  };
  __syncthreads();
  // tile entry (i, j) of tile t
  auto at = [&](int t, int i, int j) -> double { return A[t * 256 + 64 * (i >> 2) + 16 * (i & 3) + j]; };
  // wave 0: M and 1 / p of the block pivot K from tile (K, K), to LDS
  auto factor = [&](int K) {
    double a[4], m[4], pinv = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = at(place(K, K), lj, 4 * lc + q);
      m[q] = lj == 4 * lc + q ? 1.0 : 0.0;
    }
    bool ok = true;
    ldl_block(a, m, lane, pinv, ok);
    if (!ok && lane == 0) atomicOr(bad + wi.x, 2);
    double* o = sM + (K & 1) * CI_M;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[lj * CI_LD + 4 * lc + q] = m[q];
    if (lc == 0) o[16 * CI_LD + lj] = pinv;
  };
  auto mul = [&](const f64x4& a, const f64x4& b, f64x4 c) -> f64x4 {
#pragma unroll
    for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], c, 0, 0, 0);
    return c;
  };
  auto rows = [&](const double* X) -> f64x4 {   // X[lj][lc + 4 s]
    f64x4 g;
#pragma unroll
    for (int s = 0; s < 4; ++s) g[s] = X[lj * CI_LD + lc + 4 * s];
    return g;
  };
  auto blockM = [&](int K) -> const double* { return sM + (K & 1) * CI_M; };
  auto tile = [&](int t) -> f64x4 {
    f64x4 c;
#pragma unroll
    for (int v = 0; v < 4; ++v) c[v] = A[t * 256 + 64 * v + lane];
    return c;
  };
  // panel G' = G M^T, G = column K of the symmetric matrix; each wave turns
  // its own tiles into rows through their places in the panel.  x: entries
  // (lc + 4 v, lj) of the stored tile, (I, K) or (K, I)
  auto panel = [&](int K, int I, const f64x4& x) {
    double* X = G + 16 * I * CI_LD;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (I >= K)
        X[(lc + 4 * v) * CI_LD + lj] = x[v];
      else
        X[lj * CI_LD + lc + 4 * v] = x[v];
    }
    TG_WAVE_SYNC();
    const f64x4 g = mul(rows(X), rows(blockM(K)), zero);
    TG_WAVE_SYNC();
#pragma unroll
    for (int v = 0; v < 4; ++v) X[(lc + 4 * v) * CI_LD + lj] = g[v];
    const bool any = __any(!(x[0] == 0.0 && x[1] == 0.0 && x[2] == 0.0 && x[3] == 0.0));
    if (lane == 0) sZ[I] = any;
  };
  // A tile whose row or column of the panel is zero keeps its value (zero itself
  // in the pivot's row or column): beyond the band of the rows not yet swept,
  // nearly a third of all updates at n = 288.
  auto touched = [&](int K, int I, int J) -> bool {
    return __builtin_amdgcn_readfirstlane((I == K || sZ[I]) && (J == K || sZ[J])) != 0;
  };
  // tile (I, J) after block pivot K, from its old value c
  auto updated = [&](int K, int I, int J, const f64x4& c) -> f64x4 {
    const double *M = blockM(K), *gi = G + 16 * I * CI_LD, *gj = G + 16 * J * CI_LD;
    f64x4 ip;                               // 1 / p[lc + 4 s]
#pragma unroll
    for (int s = 0; s < 4; ++s) ip[s] = M[16 * CI_LD + lc + 4 * s];
    if (I != K && J != K) return mul(-rows(gi), rows(gj) * ip, c);   // A_IJ - G'_I diag(1/p) G'_J^T
    f64x4 Mc;                               // M[lc + 4 s][lj]
#pragma unroll
    for (int s = 0; s < 4; ++s) Mc[s] = M[(lc + 4 * s) * CI_LD + lj];
    if (I != K) return mul(rows(gi) * ip, Mc, zero);                 // G'_I diag(1/p) M
    if (J != K) return mul(Mc * ip, rows(gj), zero);                 // its transpose for a tile left of the diagonal
    return -mul(Mc * ip, Mc, zero);                                  // -M^T diag(1/p) M
  };
  // wave 0's part between two panels
  auto next_pivot = [&](int K) {
    if (K >= T) return;
    put(place(K, K), updated(K - 1, K, K, tile(place(K, K))));
    TG_WAVE_SYNC();                         // the tile is read back in another layout
    factor(K);
  };
  if constexpr (FORM == CI_REG) {
    // (the two roles' loops apart: wave 0 needs no room for tiles)
    if (wave == 0) {
      factor(0);
      __syncthreads();
      for (int K = 0; K < T; ++K) {
        __syncthreads();
        next_pivot(K + 1);
        __syncthreads();
      }
    } else {
      f64x4 R[CI_SLOTS];
      int rij[CI_SLOTS];                    // this wave's register tiles, -1: none
      ci_each<CI_SLOTS>([&](auto s) {
        const int v = wave - 1 + (NW - 1) * s;
        rij[s] = v < NR ? __builtin_amdgcn_readfirstlane(off_of(v)) : -1;
        const int I = rij[s] & 255, t = rij[s] >= 0 ? I * (I + 1) / 2 + (rij[s] >> 8) : 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) R[s][q] = P.Cwork[t * 256 + 64 * q + lane];
      });
      __syncthreads();
      for (int K = 0; K < T; ++K) {
        ci_each<CI_SLOTS>([&](auto s) {
          const int I = rij[s] & 255, J = rij[s] >> 8;
          if (rij[s] >= 0 && (I == K || J == K)) panel(K, J == K ? I : J, R[s]);
        });
        for (int v = NR + wave - 1; v < NO; v += NW - 1) {
          const int ij = __builtin_amdgcn_readfirstlane(off_of(v)), I = ij & 255, J = ij >> 8;
          if (I == K || J == K) panel(K, J == K ? I : J, tile(T + v - NR));
        }
        __syncthreads();
        ci_each<CI_SLOTS>([&](auto s) {
          const int I = rij[s] & 255, J = rij[s] >> 8;
          if (rij[s] >= 0 && touched(K, I, J)) R[s] = updated(K, I, J, R[s]);
        });
        for (int v = NR + wave - 1; v < NO; v += NW - 1) {
          const int ij = __builtin_amdgcn_readfirstlane(off_of(v)), I = ij & 255, J = ij >> 8;
          if (touched(K, I, J)) put(T + v - NR, updated(K, I, J, tile(T + v - NR)));
        }
        for (int I = NW - 1 - wave; I < T; I += NW - 1)
          if (I != K + 1 && touched(K, I, I)) put(I, updated(K, I, I, tile(I)));
        __syncthreads();
      }
      ci_each<CI_SLOTS>([&](auto s) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * (rij[s] & 255) + lc + 4 * v, c = 16 * (rij[s] >> 8) + lj;
          if (rij[s] >= 0 && r < n && c < n) {
            P.Cinv64[r * n + c] = P.Cinv64[c * n + r] = -R[s][v];
            P.Cinv32[r * n + c] = P.Cinv32[c * n + r] = (float)-R[s][v];
          }
        }
      });
    }
  } else {
    if (wave == 0) factor(0);
    __syncthreads();
    for (int K = 0; K < T; ++K) {
      for (int I = wave; I < T; I += NW) panel(K, I, tile(I >= K ? place(I, K) : place(K, I)));
      __syncthreads();
      if (wave == 0) {
        next_pivot(K + 1);
      } else {
        const int u0 = (wave - 1) * NT / (NW - 1), u1 = wave * NT / (NW - 1);
        f64x4 next = zero;
        int ij = 0, t = 0;
        auto fetch = [&](int u) {           // the next tile's values are loaded one update ahead
          ij = tile_of(u);
          t = place(ij & 255, ij >> 8);
          next = tile(t);
        };
        if (u0 < u1) fetch(u0);
        for (int u = u0; u < u1; ++u) {
          const f64x4 c = next;
          const int I = ij & 255, J = ij >> 8, tu = t;
          if (u + 1 < u1) fetch(u + 1);
          if ((I == K + 1 && J == K + 1) || !touched(K, I, J)) continue;   // (the former is wave 0's)
          put(tu, updated(K, I, J, c));
        }
      }
      __syncthreads();
    }
  }
  for (int u = wave; u < NT; u += NW) {
    const int ij = tile_of(u), I = ij & 255, J = ij >> 8, t = place(I, J);
    if (FORM == CI_REG && I != J && t < T) continue;   // (held in registers)
    const f64x4 c4 = tile(t);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * I + lc + 4 * v, c = 16 * J + lj;
      // (a diagonal tile holds both triangles, equal up to rounding)
      const double x = I == J ? -0.5 * (c4[v] + at(t, lj, lc + 4 * v)) : -c4[v];
      if (r < n && c < n) {
        P.Cinv64[r * n + c] = P.Cinv64[c * n + r] = x;
        P.Cinv32[r * n + c] = P.Cinv32[c * n + r] = (float)x;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Operator modes of the level kernels (the z-march kernels of tg_fine.hip):
//   OP_APPLY : y = K x
//   OP_RESID : y = b - K x
//   OP_SMOOTH: y = x + w D^-1 (b - K x)      (damped node-block Jacobi)
//   OP_RESTRICT: b_{l+1} = P^T (b - K x)     (residual fused with the restriction)
//   OP_SMOOTH1: level 0, the first two sweeps from x = 0 with b read from an
//               FP64 slot (x = scale offset, y2 = slot of b's FP32 copy)
//   OP_SMOOTH1E: the same with b read from an external vector of the level's type
//   OP_SMOOTHP: OP_SMOOTH of x + P e (y2 = slot of e at the next level)
enum { OP_APPLY = 0, OP_RESID = 1, OP_SMOOTH = 2, OP_RESTRICT = 3, OP_SMOOTH1 = 4, OP_SMOOTH1E = 5,
       OP_SMOOTHP = 6 };

// First pre-sweep from x = 0: x = w D^-1 b; optionally keep b in type T.
template <class TB, class T>
__global__ __launch_bounds__(256) void k_jacobi_first(const ProbDesc* __restrict__ probs,
                                                      const int2* __restrict__ work, int l, int sb,
                                                      const void* eb_, int sbT, int sx, T omega,
                                                      int scale_off) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const LevelDesc& L = P.lv[l];
  const int n = wi.y * TG_NODE_TILE + threadIdx.x;
  if (n >= L.n_nodes) return;
  const auto* b = vslot<TB>(L, sb, eb_);
  auto* x = vslot<T>(L, sx, nullptr);
  // optional per-problem input scale (small[scale_off]), applied in FP64
  const double sc = scale_off >= 0 ? P.small[scale_off] : 1.0;
  T b0 = T(double(b[3LL * n]) * sc), b1 = T(double(b[3LL * n + 1]) * sc), b2 = T(double(b[3LL * n + 2]) * sc);
  if (n % L.NX == 0) b0 = b1 = b2 = T(0);
  if (sbT != INT_MIN) {
    auto* bT = vslot<T>(L, sbT, nullptr);
    bT[3LL * n] = b0;
    bT[3LL * n + 1] = b1;
    bT[3LL * n + 2] = b2;
  }
  const T* D = Dinv<T>(L) + 9LL * n;
  x[3LL * n] = omega * (D[0] * b0 + D[1] * b1 + D[2] * b2);
  x[3LL * n + 1] = omega * (D[3] * b0 + D[4] * b1 + D[5] * b2);
  x[3LL * n + 2] = omega * (D[6] * b0 + D[7] * b1 + D[8] * b2);
}

// Prolongation and correction x_f += P e_c (trilinear); slots < 0 take the
// external vectors ee (coarse) and ex (fine).
template <class T>
__global__ __launch_bounds__(256) void k_prolong(const ProbDesc* __restrict__ probs,
                                                 const int2* __restrict__ work, int l, int sx,
                                                 int se, const void* ee, void* ex, int vbskip) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  if (vbskip && l >= (sizeof(T) == 8 ? P.vb_lb64 : P.vb_lb32)) return;   // run by k_vbottom
  const LevelDesc& Lf = P.lv[l];
  const LevelDesc& Lc = P.lv[l + 1];
  const int n = wi.y * TG_NODE_TILE + threadIdx.x;
  if (n >= Lf.n_nodes) return;
  const int i = n % Lf.NX, t = n / Lf.NX, j = t % Lf.NY, k = t / Lf.NY;
  if (i == 0) return;
  const auto* e = vslot<T>(Lc, se, ee);
  auto* x = vslot<T>(Lf, sx, ex);
  const int i0 = i >> 1, i1 = (i + 1) >> 1, j0 = j >> 1, j1 = (j + 1) >> 1, k0 = k >> 1, k1 = (k + 1) >> 1;
  const T wi_ = (i & 1) ? T(0.5) : T(1), wj = (j & 1) ? T(0.5) : T(1), wk = (k & 1) ? T(0.5) : T(1);
  T s0 = T(0), s1 = T(0), s2 = T(0);
  for (int c = 0; c < 8; ++c) {
    if ((c & 1) && !(i & 1)) continue;
    if ((c & 2) && !(j & 1)) continue;
    if ((c & 4) && !(k & 1)) continue;
    const int I = (c & 1) ? i1 : i0, J = (c & 2) ? j1 : j0, K = (c & 4) ? k1 : k0;
    const long long m = I + (long long)Lc.NX * (J + (long long)Lc.NY * K);
    const T w = wi_ * wj * wk;
    s0 += w * e[3 * m];
    s1 += w * e[3 * m + 1];
    s2 += w * e[3 * m + 2];
  }
  x[3LL * n] += s0;
  x[3LL * n + 1] += s1;
  x[3LL * n + 2] += s2;
}

// Coarsest solve x = K_c^-1 b with the explicit inverse (one workgroup per problem).
template <class TB, class T, class TY>
__global__ __launch_bounds__(256) void k_coarse_solve(const ProbDesc* __restrict__ probs,
                                                      const int2* __restrict__ work, int l, int sb,
                                                      const void* eb_, int sy, void* ey_, int vbskip) {
  __shared__ T sb_[TG_MAX_COARSE];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  if (vbskip && l >= (sizeof(TY) == 8 ? P.vb_lb64 : P.vb_lb32)) return;   // run by k_vbottom
  const LevelDesc& L = P.lv[l];
  const int n = P.ncoarse;
  const auto* b = vslot<TB>(L, sb, eb_);
  auto* y = vslot<TY>(L, sy, ey_);
  for (int q = threadIdx.x; q < n; q += blockDim.x) {
    const int c = q % 3, fn = q / 3;
    const int i = fn % (L.NX - 1) + 1, t = fn / (L.NX - 1);
    sb_[q] = T(b[3LL * (i + (long long)L.NX * t) + c]);
  }
  __syncthreads();
  const T* Ci = CinvP<T>(P);
  for (int q = threadIdx.x; q < n; q += blockDim.x) {
    T s = T(0);
    for (int c = 0; c < n; ++c) s += Ci[(long long)q * n + c] * sb_[c];
    const int cc = q % 3, fn = q / 3;
    const int i = fn % (L.NX - 1) + 1, t = fn / (L.NX - 1);
    y[3LL * (i + (long long)L.NX * t) + cc] = TY(s);
  }
  for (int node = threadIdx.x; node < L.n_nodes; node += blockDim.x) {
    if (node % L.NX == 0) {
      y[3LL * node] = TY(0);
      y[3LL * node + 1] = TY(0);
      y[3LL * node + 2] = TY(0);
    }
  }
}

// Copy between typed vectors at one level (masking the clamped nodes).
template <class TA, class TB>
__global__ __launch_bounds__(256) void k_copy_level(const ProbDesc* __restrict__ probs,
                                                    const int2* __restrict__ work, int l, int sa,
                                                    const void* ea, int sb, void* eb, int scale_off) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const LevelDesc& L = P.lv[l];
  const int n = wi.y * TG_NODE_TILE + threadIdx.x;
  if (n >= L.n_nodes) return;
  const auto* a = vslot<TA>(L, sa, ea);
  auto* b = vslot<TB>(L, sb, eb);
  const bool clamp = (n % L.NX) == 0;
  const double sc = scale_off >= 0 ? P.small[scale_off] : 1.0;
  for (int c = 0; c < 3; ++c) b[3LL * n + c] = clamp ? TB(0) : TB(double(a[3LL * n + c]) * sc);
}

// ---------------------------------------------------------------------------
// Vector kernels on the level-0 FP64 pool (work list: {problem, chunk}).
__device__ __forceinline__ void chunk_range(const LevelDesc& L, int c, long long& lo, long long& hi) {
  lo = (long long)c * TG_VCHUNK;
  hi = lo + TG_VCHUNK;
  const long long n = 3LL * L.n_nodes;
  if (hi > n) hi = n;
}

// dir 0: slot <- ext0 (masked); dir 1: ext1 <- slot
__global__ __launch_bounds__(256) void k_copy_ext_(const ProbDesc* __restrict__ probs,
                                                   const int2* __restrict__ work, int dir, int slot) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  auto* v = gp(L.vec64 + (long long)slot * L.stride);
  for (long long q = lo + threadIdx.x; q < hi; q += 256) {
    if (dir == 0) {
      const long long node = q / 3;
      v[q] = (node % L.NX == 0) ? 0.0 : P.ext0[q];
    } else {
      P.ext1[q] = v[q];
    }
  }
}

__global__ __launch_bounds__(256) void k_fill0_(const ProbDesc* __restrict__ probs,
                                                const int2* __restrict__ work, int slot, double val) {
  const int2 wi = work[blockIdx.x];
  const LevelDesc& L = probs[wi.x].lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  auto* v = gp(L.vec64 + (long long)slot * L.stride);
  for (long long q = lo + threadIdx.x; q < hi; q += 256) v[q] = val;
}

__global__ __launch_bounds__(256) void k_copy0_(const ProbDesc* __restrict__ probs,
                                                const int2* __restrict__ work, int src, int dst) {
  const int2 wi = work[blockIdx.x];
  const LevelDesc& L = probs[wi.x].lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  const auto* a = gp(L.vec64 + (long long)src * L.stride);
  auto* b = gp(L.vec64 + (long long)dst * L.stride);
  for (long long q = lo + threadIdx.x; q < hi; q += 256) b[q] = a[q];
}

// Partial dots: part[k * n_chunks + chunk] = sum_{q in chunk} V_{sbase+k}[q] * w[q]
// for k < nv; if with_self, entry nv holds w . w.
__global__ __launch_bounds__(256) void k_multidot_(const ProbDesc* __restrict__ probs,
                                                   const int2* __restrict__ work, int sbase, int nv,
                                                   int sw, int with_self) {
  __shared__ double sh[8][4];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  const auto* w = gp(L.vec64 + (long long)sw * L.stride);
  double wr[TG_VCHUNK / 256];
#pragma unroll
  for (int q = 0; q < TG_VCHUNK / 256; ++q) {
    const long long idx = lo + threadIdx.x + 256LL * q;
    wr[q] = idx < hi ? w[idx] : 0.0;
  }
  const int ntot = nv + (with_self ? 1 : 0);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int k0 = 0; k0 < ntot; k0 += 8) {
    double s[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      s[g] = 0.0;
      const int k = k0 + g;
      if (k < ntot) {
        const auto* v = (k < nv) ? gp(L.vec64 + (long long)(sbase + k) * L.stride) : w;
#pragma unroll
        for (int q = 0; q < TG_VCHUNK / 256; ++q) {
          const long long idx = lo + threadIdx.x + 256LL * q;
          if (idx < hi) s[g] += v[idx] * wr[q];
        }
      }
    }
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const double r = wave_sum(s[g]);
      if (lane == 0) sh[g][wv] = r;
    }
    __syncthreads();
    if (threadIdx.x < 8 && k0 + (int)threadIdx.x < ntot) {
      const int g = threadIdx.x;
      P.part[(long long)(k0 + g) * L.n_chunks + wi.y] = (sh[g][0] + sh[g][1]) + (sh[g][2] + sh[g][3]);
    }
    __syncthreads();
  }
}

// tmp[dst + k] = sum over chunks of part[k][.] in a fixed order.  mode 0 also
// assigns h[k], mode 1 adds into h[k], mode 2 touches only tmp.  Entry k ==
// save_k (if >= 0) goes to scal[SC_FLAG] instead.  Grid: (problems, nv).
__global__ __launch_bounds__(256) void k_reduce_(const ProbDesc* __restrict__ probs,
                                                 const int2* __restrict__ work, int h_off,
                                                 int tmp_off, int flag_off, int mode, int save_k) {
  __shared__ double sh[4];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const int nc = P.lv[0].n_chunks;
  const int k = blockIdx.y;
  double s = 0.0;
  for (int c = threadIdx.x; c < nc; c += 256) s += P.part[(long long)k * nc + c];
  s = block_sum256(s, sh);
  if (threadIdx.x == 0) {
    if (k == save_k) {
      P.small[flag_off] = s;
      return;
    }
    P.small[tmp_off + k] = s;
    if (mode == 0) P.small[h_off + k] = s;
    if (mode == 1) P.small[h_off + k] += s;
  }
}

// w -= sum_k coef[k] V_{sbase+k}
__global__ __launch_bounds__(256) void k_update_(const ProbDesc* __restrict__ probs,
                                                 const int2* __restrict__ work, int sbase, int nv,
                                                 int sw, int coef_off) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  auto* w = gp(L.vec64 + (long long)sw * L.stride);
  const double* coef = P.small + coef_off;
  double acc[TG_VCHUNK / 256];
#pragma unroll
  for (int q = 0; q < TG_VCHUNK / 256; ++q) acc[q] = 0.0;
  for (int k = 0; k < nv; ++k) {
    const double ck = coef[k];
    const auto* v = gp(L.vec64 + (long long)(sbase + k) * L.stride);
#pragma unroll
    for (int q = 0; q < TG_VCHUNK / 256; ++q) {
      const long long idx = lo + threadIdx.x + 256LL * q;
      if (idx < hi) acc[q] += ck * v[idx];
    }
  }
#pragma unroll
  for (int q = 0; q < TG_VCHUNK / 256; ++q) {
    const long long idx = lo + threadIdx.x + 256LL * q;
    if (idx < hi) w[idx] -= acc[q];
  }
}

// Fused Gram-Schmidt sweep: w -= sum_k coef[k] V_k over the chunk, then the
// chunk partials of V_k . w (k < ndot) and, if with_self, of w . w, written
// like k_multidot_.  The update of one chunk only needs that chunk, so the
// dots of the updated vector are exact chunk sums.
__global__ __launch_bounds__(256) void k_update_dots_(const ProbDesc* __restrict__ probs,
                                                      const int2* __restrict__ work, int sbase, int nv,
                                                      int sw, int coef_off, int ndot, int with_self) {
  __shared__ double sh[8][4];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  auto* w = gp(L.vec64 + (long long)sw * L.stride);
  const double* coef = P.small + coef_off;
  double wr[TG_VCHUNK / 256];
#pragma unroll
  for (int q = 0; q < TG_VCHUNK / 256; ++q) {
    const long long idx = lo + threadIdx.x + 256LL * q;
    wr[q] = idx < hi ? w[idx] : 0.0;
  }
  {
    double acc[TG_VCHUNK / 256];
#pragma unroll
    for (int q = 0; q < TG_VCHUNK / 256; ++q) acc[q] = 0.0;
    for (int k = 0; k < nv; ++k) {
      const double ck = coef[k];
      const auto* v = gp(L.vec64 + (long long)(sbase + k) * L.stride);
#pragma unroll
      for (int q = 0; q < TG_VCHUNK / 256; ++q) {
        const long long idx = lo + threadIdx.x + 256LL * q;
        if (idx < hi) acc[q] += ck * v[idx];
      }
    }
#pragma unroll
    for (int q = 0; q < TG_VCHUNK / 256; ++q) {
      const long long idx = lo + threadIdx.x + 256LL * q;
      wr[q] -= acc[q];
      if (idx < hi) w[idx] = wr[q];
    }
  }
  const int ntot = ndot + (with_self ? 1 : 0);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int k0 = 0; k0 < ntot; k0 += 8) {
    double sacc[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      sacc[g] = 0.0;
      const int k = k0 + g;
      if (k < ntot) {
        if (k < ndot) {
          const auto* v = gp(L.vec64 + (long long)(sbase + k) * L.stride);
#pragma unroll
          for (int q = 0; q < TG_VCHUNK / 256; ++q) {
            const long long idx = lo + threadIdx.x + 256LL * q;
            if (idx < hi) sacc[g] += v[idx] * wr[q];
          }
        } else {
#pragma unroll
          for (int q = 0; q < TG_VCHUNK / 256; ++q) sacc[g] += wr[q] * wr[q];
        }
      }
    }
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const double r = wave_sum(sacc[g]);
      if (lane == 0) sh[g][wv] = r;
    }
    __syncthreads();
    if (threadIdx.x < 8 && k0 + (int)threadIdx.x < ntot) {
      const int g = threadIdx.x;
      P.part[(long long)(k0 + g) * L.n_chunks + wi.y] = (sh[g][0] + sh[g][1]) + (sh[g][2] + sh[g][3]);
    }
    __syncthreads();
  }
}

// Single-read form of the fused sweep for nv <= NVR: each thread keeps its
// DOF's values of all V_k in registers, so V is read once for both the update
// and the dots of the updated vector.
template <int NVR>
__global__ __launch_bounds__(256) void k_update_dots_reg_(const ProbDesc* __restrict__ probs,
                                                          const int2* __restrict__ work, int sbase, int nv,
                                                          int sw, int coef_off, int ndot, int with_self) {
  __shared__ double sh[NVR + 1][4];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  auto* w = gp(L.vec64 + (long long)sw * L.stride);
  const auto* V0 = gp(L.vec64 + (long long)sbase * L.stride);
  const long long st = L.stride;
  const double* coef = P.small + coef_off;
  double cf[NVR], acc[NVR + 1];
#pragma unroll
  for (int k = 0; k < NVR; ++k) {
    cf[k] = k < nv ? coef[k] : 0.0;
    acc[k] = 0.0;
  }
  acc[NVR] = 0.0;
  for (int q = 0; q < TG_VCHUNK / 256; ++q) {
    const long long idx = lo + threadIdx.x + 256LL * q;
    if (idx >= hi) break;
    double v[NVR];
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < NVR; ++k) {
      v[k] = k < nv ? V0[k * st + idx] : 0.0;
      t += cf[k] * v[k];
    }
    const double wn = w[idx] - t;
    w[idx] = wn;
#pragma unroll
    for (int k = 0; k < NVR; ++k) acc[k] += v[k] * wn;
    acc[NVR] += wn * wn;
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NVR; ++k) {
    if (k < ndot) {
      const double r = wave_sum(acc[k]);
      if (lane == 0) sh[k][wv] = r;
    }
  }
  if (with_self) {
    const double r = wave_sum(acc[NVR]);
    if (lane == 0) sh[NVR][wv] = r;
  }
  __syncthreads();
  const int ntot = ndot + (with_self ? 1 : 0);
  if ((int)threadIdx.x < ntot) {
    const int k = threadIdx.x;
    const int src = k < ndot ? k : NVR;
    P.part[(long long)k * L.n_chunks + wi.y] = (sh[src][0] + sh[src][1]) + (sh[src][2] + sh[src][3]);
  }
}

struct SmallOffs {
  int mmax, H, g, cs, sn, y, h, tmp, scal, hist;
};
// CGS2 with delayed reorthogonalization, sweep A.  For k < nv the chunk
// partials of V_k . q and V_k . w, then q . q, q . w, w . w: 2 nv + 3 entries
// in the order [V.q (nv) | V.w (nv) | q.q, q.w, w.w].  One read of V, q, w.
// NT (both sweeps): V is read with non-temporal loads.  A basis that exceeds
// the L2 caches is not read again before it is evicted, and without the hint
// it also evicts what the V-cycle reads next: over the policy step of 24 64x32x32
// states sweep A went from 97 to 89 us per launch, B from 103 to 98.  One
// state's basis (29 MB at 15 vectors) stays cached, and is read the ordinary
// way (10 us against 13).
template <bool NT, class P>
__device__ __forceinline__ double basis_load(P p) {
  return NT ? __builtin_nontemporal_load(p) : *p;
}
template <bool NT>
__global__ __launch_bounds__(256) void k_dots2_(const ProbDesc* __restrict__ probs,
                                                const int2* __restrict__ work, int sbase, int nv, int sq,
                                                int sw) {
  // per group of eight basis vectors: the 16 wave sums of each wave (every
  // group has its own slots, so the waves only meet once, at the end)
  constexpr int NGRP = (TG_MAX_RESTART + 8) / 8;
  __shared__ double sh[NGRP][16][4];
  __shared__ double sh3[3][4];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  const long long nc = L.n_chunks;
  const auto* qv = gp(L.vec64 + (long long)sq * L.stride);
  const auto* wv = gp(L.vec64 + (long long)sw * L.stride);
  // whole chunks: the slot stride is a multiple of the chunk and the tail
  // beyond 3 n_nodes holds zeros
  constexpr int NQ = TG_VCHUNK / 256;
  double qr[NQ], wr[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const long long idx = lo + threadIdx.x + 256LL * q;
    qr[q] = qv[idx];
    wr[q] = wv[idx];
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int k0 = 0; k0 < nv; k0 += 8) {
    const int gi = k0 >> 3;
    double a[8], c[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      a[g] = c[g] = 0.0;
      const int k = k0 + g;
      if (k < nv) {
        const auto* v = gp(L.vec64 + (long long)(sbase + k) * L.stride);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const double x = basis_load<NT>(v + (lo + threadIdx.x + 256LL * q));
          a[g] += x * qr[q];
          c[g] += x * wr[q];
        }
      }
    }
    double v16[16];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      v16[g] = a[g];
      v16[8 + g] = c[g];
    }
    const double r = wave_sum16(v16, lane);
    if (lane < 16) sh[gi][rev4(lane)][wave] = r;
  }
  double qq = 0.0, qw = 0.0, ww = 0.0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    qq += qr[q] * qr[q];
    qw += qr[q] * wr[q];
    ww += wr[q] * wr[q];
  }
  qq = wave_sum(qq);
  qw = wave_sum(qw);
  ww = wave_sum(ww);
  if (lane == 0) {
    sh3[0][wave] = qq;
    sh3[1][wave] = qw;
    sh3[2][wave] = ww;
  }
  __syncthreads();
  // rows [V.q | V.w]: row which * nv + k from slot (k & 7) + 8 which of group k / 8
  for (int t = threadIdx.x; t < 2 * nv; t += 256) {
    const int which = t / nv, k = t - which * nv, gi = k >> 3, sl = (k & 7) + 8 * which;
    P.part[(long long)t * nc + wi.y] = (sh[gi][sl][0] + sh[gi][sl][1]) + (sh[gi][sl][2] + sh[gi][sl][3]);
  }
  if (threadIdx.x < 3) {
    const int t = threadIdx.x;
    P.part[(2LL * nv + t) * nc + wi.y] = (sh3[t][0] + sh3[t][1]) + (sh3[t][2] + sh3[t][3]);
  }
}

// CGS2 with delayed reorthogonalization, sweep B (coefficients at small+coef):
//   q     <- cq * q - sum_k a_k V_k        (the reorthogonalized, normalized q)
//   qnext <- w - sum_k c_k V_k - cw * q_old (the next vector, projected once)
// with a = coef[0, nv), c = coef[nv, 2 nv), cq = coef[2 nv], cw = coef[2 nv + 1];
// chunk partial of qnext . qnext into part row 0.  One read of V, q, w.
template <bool NT>
__global__ __launch_bounds__(256) void k_update2_(const ProbDesc* __restrict__ probs,
                                                  const int2* __restrict__ work, int sbase, int nv, int sq,
                                                  int sw, int snext, int coef_off) {
  __shared__ double sh[4];
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  const double* cf = P.small + coef_off;
  constexpr int NQ = TG_VCHUNK / 256;
  double ta[NQ], tc[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) ta[q] = tc[q] = 0.0;
  // whole chunks (see k_dots2_); on the zero tail every value written is 0
  for (int k = 0; k < nv; ++k) {
    const double ak = cf[k], ck = cf[nv + k];
    const auto* v = gp(L.vec64 + (long long)(sbase + k) * L.stride);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const double x = basis_load<NT>(v + (lo + threadIdx.x + 256LL * q));
      ta[q] += ak * x;
      tc[q] += ck * x;
    }
  }
  const double cq = cf[2 * nv], cw = cf[2 * nv + 1];
  auto* qv = gp(L.vec64 + (long long)sq * L.stride);
  const auto* wv = gp(L.vec64 + (long long)sw * L.stride);
  auto* nv_ = gp(L.vec64 + (long long)snext * L.stride);
  double nn = 0.0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const long long idx = lo + threadIdx.x + 256LL * q;
    const double qo = qv[idx];
    const double nx = wv[idx] - tc[q] - cw * qo;
    qv[idx] = cq * qo - ta[q];
    nv_[idx] = nx;
    nn += nx * nx;
  }
  nn = block_sum256(nn, sh);
  if (threadIdx.x == 0) P.part[wi.y] = nn;
}

// dst = src * small[scal + sc_index]
__global__ __launch_bounds__(256) void k_scale_(const ProbDesc* __restrict__ probs,
                                                const int2* __restrict__ work, int src, int dst,
                                                int sidx) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  const double a = P.small[sidx];
  const auto* s = gp(L.vec64 + (long long)src * L.stride);
  auto* d = gp(L.vec64 + (long long)dst * L.stride);
  for (long long q = lo + threadIdx.x; q < hi; q += 256) d[q] = s[q] * a;
}

// ---------------------------------------------------------------------------
// FGMRES scalar kernels: one thread per problem (work list {p, 0}).
__global__ void k_init_small_(const ProbDesc* __restrict__ probs, const int2* __restrict__ work,
                              int total) {
  const ProbDesc& P = probs[work[blockIdx.x].x];
  for (int q = threadIdx.x; q < total; q += blockDim.x) P.small[q] = 0.0;
}

// Cycle start: beta = ||r|| (tmp[0] holds r.r); history and stop tests.
__global__ void k_cycle_start_(const ProbDesc* __restrict__ probs, const int2* __restrict__ work,
                               SmallOffs o, int k, int cap, double tol, double* status_out) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  if (threadIdx.x != 0) return;
  double* S = P.small;
  double* sc = S + o.scal;
  const double beta = sqrt(S[o.tmp]);
  if (k == 0) {
    sc[SC_BNORM] = beta;
    S[o.hist] = (beta > 0.0) ? 1.0 : 0.0;
  }
  const double bnorm = sc[SC_BNORM];
  const double rel = bnorm > 0.0 ? beta / bnorm : 0.0;
  if (k > 0) S[o.hist + k] = rel;   // cycle-start true residual replaces the projection
  double st = TG_RUNNING;
  if (!isfinite(beta)) st = TG_NONFINITE;
  else if (rel <= tol) st = TG_PROJ_CONVERGED;
  else if (k >= cap) st = TG_MAXIT;
  sc[SC_BETA] = beta;
  sc[SC_STATUS] = st;
  sc[SC_ITERS] = k;
  sc[SC_JDONE] = 0;
  sc[SC_EST] = rel;
  sc[SC_INV] = beta > 0.0 ? 1.0 / beta : 0.0;
  sc[SC_RHO] = beta;   // delayed form: V_0 holds r itself, first-pass norm beta
  for (int q = 0; q <= o.mmax; ++q) S[o.g + q] = 0.0;
  S[o.g] = beta;
  status_out[wi.x] = st;
}

// Arnoldi column j: h (accumulated) and tmp[0] = ||w||^2 after projection,
// scal[SC_HN] <- ||w||; apply Givens rotations, new rotation, history, stop tests.
__global__ void k_arnoldi_(const ProbDesc* __restrict__ probs, const int2* __restrict__ work,
                           SmallOffs o, int j, int k, int cap, double tol, double brk,
                           double* status_out) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  if (threadIdx.x != 0) return;
  double* S = P.small;
  double* sc = S + o.scal;
  const int ldh = o.mmax + 1;
  double* Hc = S + o.H + (long long)ldh * j;
  const double hn = sqrt(S[o.tmp]);
  const double wn0 = sqrt(fmax(sc[SC_FLAG], 0.0));   // ||w|| before projection
  bool finite = isfinite(hn);
  for (int i = 0; i <= j; ++i) {
    Hc[i] = S[o.h + i];
    finite = finite && isfinite(Hc[i]);
  }
  Hc[j + 1] = hn;
  double st = TG_RUNNING;
  if (!finite) {
    st = TG_NONFINITE;
    sc[SC_STATUS] = st;
    status_out[wi.x] = st;
    return;   // column j unusable: jdone stays j
  }
  for (int i = 0; i < j; ++i) {
    const double c = S[o.cs + i], s = S[o.sn + i];
    const double t = c * Hc[i] + s * Hc[i + 1];
    Hc[i + 1] = -s * Hc[i] + c * Hc[i + 1];
    Hc[i] = t;
  }
  const double d = hypot(Hc[j], Hc[j + 1]);
  if (!(d > 0.0) || !isfinite(d)) {
    st = TG_NONFINITE;
    sc[SC_STATUS] = st;
    status_out[wi.x] = st;
    return;
  }
  const double c = Hc[j] / d, s = Hc[j + 1] / d;
  S[o.cs + j] = c;
  S[o.sn + j] = s;
  Hc[j] = d;
  Hc[j + 1] = 0.0;
  const double gj = S[o.g + j];
  S[o.g + j + 1] = -s * gj;
  S[o.g + j] = c * gj;
  const int kk = (int)sc[SC_ITERS] + 1;   // iterations so far live on the device (k: the host's count)
  (void)k;
  const double est = fabs(S[o.g + j + 1]) / sc[SC_BNORM];
  S[o.hist + kk] = est;
  sc[SC_EST] = est;
  sc[SC_ITERS] = kk;
  sc[SC_JDONE] = j + 1;
  sc[SC_HN] = hn;
  sc[SC_INV] = hn > 0.0 ? 1.0 / hn : 0.0;
  if (est <= tol) st = TG_PROJ_CONVERGED;
  else if (hn <= brk * wn0) st = TG_BREAKDOWN;
  else if (kk >= cap) st = TG_MAXIT;
  sc[SC_STATUS] = st;
  status_out[wi.x] = st;
}

// Delayed reorthogonalization, after sweep A of step j.  V_0..V_{j-1} hold
// the final orthonormal q_i, V_j the once-projected q~_j with first-pass norm
// rho = scal[SC_RHO]; tmp holds [Q^T q~ | Q^T w | q~.q~, q~.w, w.w] with
// w = K z_j, z_j = M^-1 (q~_j / rho).  With S = Q^T q~ / rho:
//   nu = sqrt(q~.q~ / rho^2 - |S|^2),  q_j = (q~_j / rho - Q S) / nu.
// Column j-1 of H becomes final: [h1 + rho S ; rho nu] (h1 = its first-pass
// coefficients), replacing the tentative column and rotation of step j-1.
// The first-pass coefficients of column j are h1 = [Q^T w ; q_j . w]; the
// coefficients of sweep B go to tmp (see k_update2_).
// The scalar state a part reads, in LDS: loaded by the workgroup while the
// chunk sums are formed, so that the one wave that runs the part does not wait
// for memory in between.
struct FinState {
  double h[TG_MAX_RESTART + 2], c[TG_MAX_RESTART + 1], s[TG_MAX_RESTART + 1];
  double sc[16];                // scalars SC_*
  double tmp[TG_PART_W];        // chunk sums
  int bad;
};
__device__ __forceinline__ void fin_load(const ProbDesc& P, const SmallOffs& o, int nh, int nrot, FinState& F) {
  const auto* S = gp((const double*)P.small);
  for (int i = threadIdx.x; i < nh; i += (int)blockDim.x) F.h[i] = S[o.h + i];
  for (int i = threadIdx.x; i < nrot; i += (int)blockDim.x) {
    F.c[i] = S[o.cs + i];
    F.s[i] = S[o.sn + i];
  }
  if (threadIdx.x < 16) F.sc[threadIdx.x] = S[o.scal + threadIdx.x];
}

__device__ void dcgs_a_wave(const ProbDesc& P, int p, const SmallOffs& o, int j, FinState& F, double* status_out) {
  // one wave: the column and the rotations are rotated in LDS by lane 0 (a
  // chain of register operations rather than of round trips through memory)
  const int lane = threadIdx.x;
  double* S = P.small;
  double* sc = S + o.scal;
  if (F.sc[SC_STATUS] != TG_RUNNING) return;
  const double* T = F.tmp;
  double* tmp = S + o.tmp;
  double* h1 = S + o.h;
  const int ldh = o.mmax + 1;
  const double rho = F.sc[SC_RHO];
  const double alpha = T[2 * j] / (rho * rho), qw = T[2 * j + 1] / rho, ww = T[2 * j + 2];
  double ss = 0.0, sz = 0.0;
  for (int k = lane; k < j; k += 64) {
    const double sk = T[k] / rho;
    ss += sk * sk;
    sz += sk * T[j + k];
  }
  ss = wave_sum(ss);
  sz = wave_sum(sz);
  const double nu2 = alpha - ss;
  double st = TG_RUNNING;
  if (!isfinite(nu2) || !isfinite(qw) || !isfinite(sz)) st = TG_NONFINITE;
  else if (!(nu2 > 0.0)) st = TG_BREAKDOWN;   // q~_j lies in span(Q): nothing new
  if (st != TG_RUNNING) {
    if (lane == 0) {
      sc[SC_STATUS] = st;
      status_out[p] = st;
    }
    return;
  }
  const double nu = sqrt(nu2);
  if (lane == 0) sc[SC_FLAG] = ww;
  if (j >= 1) {
    double* sH = F.h;
    double* Hc = S + o.H + (long long)ldh * (j - 1);
    for (int i = lane; i < j; i += 64) sH[i] = sH[i] + T[i];
    TG_WAVE_SYNC();
    if (lane == 0) {
      sH[j] = rho * nu;
      double carry = sH[0];
      for (int i = 0; i < j - 1; ++i) {
        const double c = F.c[i], sn = F.s[i], b = sH[i + 1];
        sH[i] = c * carry + sn * b;
        carry = -sn * carry + c * b;
      }
      sH[j - 1] = carry;
      const double d = hypot(sH[j - 1], sH[j]);
      F.bad = !(d > 0.0) || !isfinite(d);
      if (F.bad) {
        sc[SC_STATUS] = TG_NONFINITE;
        status_out[p] = TG_NONFINITE;
      } else {
        const double c = sH[j - 1] / d, sn = sH[j] / d;
        S[o.cs + j - 1] = c;
        S[o.sn + j - 1] = sn;
        sH[j - 1] = d;
        sH[j] = 0.0;
        const double gj = F.sc[SC_GJ];
        S[o.g + j - 1] = c * gj;
        S[o.g + j] = -sn * gj;
      }
    }
    TG_WAVE_SYNC();
    for (int i = lane; i <= j; i += 64) Hc[i] = sH[i];
    if (F.bad) return;
  }
  const double hjj = (qw - sz) / nu;
  for (int k = lane; k < j; k += 64) {
    const double sk = T[k] / rho, zk = T[j + k];
    h1[k] = zk;
    tmp[j + k] = zk - sk * hjj / nu;
    tmp[k] = sk / nu;
  }
  if (lane == 0) {
    h1[j] = hjj;
    tmp[2 * j] = 1.0 / (rho * nu);
    tmp[2 * j + 1] = hjj / (nu * rho);
  }
}

// After sweep B of step j: rho' = ||q~_{j+1}|| (tmp[0]).  Column j enters
// tentatively as [h1 ; rho'] (its reorthogonalization correction is known
// only after the next sweep A): rotations, projected residual estimate,
// history and stop tests as in the immediate form.
__device__ void dcgs_b_wave(const ProbDesc& P, int p, const SmallOffs& o, int j, int cap, double tol, double brk,
                            FinState& F, double* status_out) {
  const int lane = threadIdx.x;
  double* S = P.small;
  double* sc = S + o.scal;
  if (F.sc[SC_STATUS] != TG_RUNNING) return;   // stopped in sweep A of this step
  const int ldh = o.mmax + 1;
  const double rn = sqrt(F.tmp[0]);
  double* sH = F.h;
  double* Hc = S + o.H + (long long)ldh * j;
  bool finite = true;
  for (int i = lane; i <= j; i += 64) finite = finite && isfinite(sH[i]);
  finite = __all(finite) && isfinite(rn);
  if (!finite) {
    for (int i = lane; i <= j; i += 64) Hc[i] = sH[i];
    if (lane == 0) {
      Hc[j + 1] = rn;
      sc[SC_STATUS] = TG_NONFINITE;
      status_out[p] = TG_NONFINITE;
    }
    return;
  }
  TG_WAVE_SYNC();
  if (lane == 0) {
    sH[j + 1] = rn;
    double carry = sH[0];
    for (int i = 0; i < j; ++i) {
      const double c = F.c[i], sn = F.s[i], b = sH[i + 1];
      sH[i] = c * carry + sn * b;
      carry = -sn * carry + c * b;
    }
    sH[j] = carry;
    const double d = hypot(sH[j], sH[j + 1]);
    F.bad = !(d > 0.0) || !isfinite(d);
    if (F.bad) {
      sc[SC_STATUS] = TG_NONFINITE;
      status_out[p] = TG_NONFINITE;
    } else {
      const double c = sH[j] / d, sn = sH[j + 1] / d;
      S[o.cs + j] = c;
      S[o.sn + j] = sn;
      sH[j] = d;
      sH[j + 1] = 0.0;
      const double gj = S[o.g + j];
      sc[SC_GJ] = gj;
      S[o.g + j + 1] = -sn * gj;
      S[o.g + j] = c * gj;
      const int kk = (int)F.sc[SC_ITERS] + 1;   // iterations so far live on the device
      const double est = fabs(-sn * gj) / F.sc[SC_BNORM];
      S[o.hist + kk] = est;
      sc[SC_EST] = est;
      sc[SC_ITERS] = kk;
      sc[SC_JDONE] = j + 1;
      sc[SC_HN] = rn;
      sc[SC_RHO] = rn;
      sc[SC_INV] = rn > 0.0 ? 1.0 / rn : 0.0;
      double st = TG_RUNNING;
      if (est <= tol) st = TG_PROJ_CONVERGED;
      else if (rn <= brk * sqrt(fmax(F.sc[SC_FLAG], 0.0))) st = TG_BREAKDOWN;
      else if (kk >= cap) st = TG_MAXIT;
      sc[SC_STATUS] = st;
      status_out[p] = st;
    }
  }
  TG_WAVE_SYNC();
  for (int i = lane; i <= j + 1; i += 64) Hc[i] = sH[i];
}

// The scalar ends of the two sweeps of a delayed-CGS2 step, one workgroup per
// problem: the chunk partials summed in a fixed order, then the step's scalar
// part on one wave.  A: rows [V.q | V.w | q.q, q.w, w.w], each summed over the
// chunks in chunk order; B: ||q_next||^2 over the chunks.  Bound by latency:
// with the scalar state read in turn after the sums, A took 9.3 us between the
// sweeps of one 64x32x32 problem and 11.9 of 24, so 7.1 and 8.2 (B 4.7 and
// 7.0, now 4.6 and 6.1).
__global__ __launch_bounds__(256) void k_fin_a_(const ProbDesc* __restrict__ probs, const int2* __restrict__ work,
                                                SmallOffs o, int j, double* status_out) {
  __shared__ FinState F;
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  fin_load(P, o, j, j - 1, F);
  const int nc = P.lv[0].n_chunks;
  const auto* part = gp((const double*)P.part);
  for (int r = threadIdx.x; r < 2 * j + 3; r += 256) {
    const auto* pr = part + (long long)r * nc;
    double a = 0.0;
#pragma unroll 32
    for (int c = 0; c < nc; ++c) a += pr[c];
    F.tmp[r] = a;
  }
  __syncthreads();
  if (threadIdx.x < 64) dcgs_a_wave(P, wi.x, o, j, F, status_out);
}
__global__ __launch_bounds__(256) void k_fin_b_(const ProbDesc* __restrict__ probs, const int2* __restrict__ work,
                                                SmallOffs o, int j, int cap, double tol, double brk,
                                                double* status_out) {
  __shared__ double sh[4];
  __shared__ FinState F;
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  TG_GATE(P);
  fin_load(P, o, j + 1, j, F);
  const int nc = P.lv[0].n_chunks;
  const auto* part = gp((const double*)P.part);
  double a = 0.0;
  for (int c = threadIdx.x; c < nc; c += 256) a += part[c];
  a = block_sum256(a, sh);
  if (threadIdx.x == 0) F.tmp[0] = a;
  __syncthreads();
  if (threadIdx.x < 64) dcgs_b_wave(P, wi.x, o, j, cap, tol, brk, F, status_out);
}

// Least squares: y = R^{-1} g over the jdone columns (back substitution).
__global__ void k_lsq_(const ProbDesc* __restrict__ probs, const int2* __restrict__ work, SmallOffs o) {
  const ProbDesc& P = probs[work[blockIdx.x].x];
  if (threadIdx.x != 0) return;
  double* S = P.small;
  const int jd = (int)S[o.scal + SC_JDONE];
  const int ldh = o.mmax + 1;
  for (int i = jd - 1; i >= 0; --i) {
    double v = S[o.g + i];
    for (int c = i + 1; c < jd; ++c) v -= S[o.H + (long long)ldh * c + i] * S[o.y + c];
    S[o.y + i] = v / S[o.H + (long long)ldh * i + i];
  }
  for (int i = jd; i < o.mmax; ++i) S[o.y + i] = 0.0;
}

// x += sum_{j < jdone} y_j Z_j
__global__ __launch_bounds__(256) void k_xupdate_(const ProbDesc* __restrict__ probs,
                                                  const int2* __restrict__ work, SmallOffs o,
                                                  int sz0) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, wi.y, lo, hi);
  const int jd = (int)P.small[o.scal + SC_JDONE];
  auto* x = gp(L.vec64 + (long long)S_X * L.stride);
  double acc[TG_VCHUNK / 256];
#pragma unroll
  for (int q = 0; q < TG_VCHUNK / 256; ++q) acc[q] = 0.0;
  for (int jj = 0; jj < jd; ++jj) {
    const double yj = P.small[o.y + jj];
    const auto* z = gp(L.vec64 + (long long)(sz0 + jj) * L.stride);
#pragma unroll
    for (int q = 0; q < TG_VCHUNK / 256; ++q) {
      const long long idx = lo + threadIdx.x + 256LL * q;
      if (idx < hi) acc[q] += yj * z[idx];
    }
  }
#pragma unroll
  for (int q = 0; q < TG_VCHUNK / 256; ++q) {
    const long long idx = lo + threadIdx.x + 256LL * q;
    if (idx < hi) x[idx] += acc[q];
  }
}

// eta = sqrt(r.r / f.f) with tmp[0] = r.r, tmp[1] = f.f.  A zero right-hand
// side solved exactly (r.r = f.f = 0) gives 0; any other f.f that is not a
// finite positive number (a non-finite entry in f, or f.f = 0 with r != 0)
// gives NaN, which no acceptance test passes.
__global__ void k_true_eta_(const ProbDesc* __restrict__ probs, const int2* __restrict__ work,
                            SmallOffs o, double* out) {
  const int2 wi = work[blockIdx.x];
  const ProbDesc& P = probs[wi.x];
  if (threadIdx.x != 0) return;
  const double rr = P.small[o.tmp], ff = P.small[o.tmp + 1];
  double eta;
  if (rr == 0.0 && ff == 0.0)
    eta = 0.0;
  else if (ff > 0.0 && isfinite(ff))
    eta = sqrt(rr / ff);   // NaN when r.r is NaN, +inf when it overflows
  else
    eta = __builtin_nan("");
  P.small[o.scal + SC_TRUE] = eta;
  if (out) out[wi.x] = eta;
}

// ===========================================================================
// Launch wrappers.  Each launch of a timed class is bracketed by timer events
// (when the timer is on) and charged its algorithmic HBM bytes.
static inline dim3 nblk(const DevList& d) { return dim3((unsigned)d.n); }

static SmallOffs offs(const Batch* b) {
  const SmallLayout& s = b->grids[0]->sl;
  SmallOffs o;
  o.mmax = s.mmax;
  o.H = s.H;
  o.g = s.g;
  o.cs = s.cs;
  o.sn = s.sn;
  o.y = s.y;
  o.h = s.h;
  o.tmp = s.tmp;
  o.scal = s.scal;
  o.hist = s.hist;
  return o;
}

static int check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, what);
  return TG_OK;
}

// Sums over the active problems that take part in a level-l launch.
// mode 0: every problem with level l; 1: l is not its coarsest; 2: l is its coarsest
static void level_sums(const Batch* b, int l, int mode, double& nodes, double& elems, double& cdof2) {
  nodes = elems = cdof2 = 0;
  for (int p : b->active) {
    const tg_grid* g = b->grids[p];
    if (l >= g->nlev) continue;
    if (mode == 1 && l == g->nlev - 1) continue;
    if (mode == 2 && l != g->nlev - 1) continue;
    nodes += (double)g->lv[l].n_nodes;
    elems += (double)g->lv[l].n_elem;
    cdof2 += (double)g->ncoarse * g->ncoarse;
  }
}
static double dofs0(const Batch* b) {
  double n = 0;
  for (int p : b->active) n += 3.0 * b->grids[p]->lv[0].n_nodes;
  return n;
}

#define TG_TIMED(kind, bytes_expr, ...)                 \
  do {                                                  \
    void* _th = timer_begin((kind), s);                 \
    __VA_ARGS__;                                        \
    if (_th) timer_end(_th, (double)(bytes_expr), s);   \
  } while (0)

// Raises the dynamic-LDS limit of the coarsest-inverse kernels on the current
// device to what their largest problem takes, once per device.
static int coarse_lds_raise() {
  static bool done[64] = {};
  static std::mutex mu;   // batches on several host threads
  std::lock_guard<std::mutex> lk(mu);
  int dev = 0;
  TG_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return fail(TG_EINVAL, "device index out of range");
  if (done[dev]) return TG_OK;
  const void* f[3] = {(const void*)k_coarse_inverse<CI_LDS>, (const void*)k_coarse_inverse<CI_REG>,
                      (const void*)k_coarse_inverse<CI_MEM>};
  const int nmax[3] = {CI_LDS_N, CI_REG_N, TG_MAX_COARSE};
  for (int q = 0; q < 3; ++q)
    TG_HIP(hipFuncSetAttribute(f[q], hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(sizeof(double) * ci_lds_words(nmax[q], q))));
  done[dev] = true;
  return TG_OK;
}

int k_set_density(Batch* b, hipStream_t s) {
  int* bad = b->flag_d;
  const int rc = coarse_lds_raise();
  if (rc) return rc;
  TG_HIP(hipMemsetAsync(bad, 0, sizeof(int) * b->n, s));
  TG_TIMED(TG_KT_SETUP, 0, {
    if (b->elem[0].n) k_young<<<nblk(b->elem[0]), 256, 0, s>>>(b->desc_d, b->elem[0].ptr, b->p, bad);
    if (b->elem[1].n) k_galerkin1<<<nblk(b->elem[1]), 192, 0, s>>>(b->desc_d, b->elem[1].ptr);
    for (int l = 2; l < b->maxlev; ++l)
      if (b->elem[l].n) k_galerkin_up<<<nblk(b->elem[l]), 512, 0, s>>>(b->desc_d, b->elem[l].ptr, l);
    SetupTail w = {};
    long long blocks = 0;
    for (int u = 0; u < 2 * TG_MAXLEV; ++u) {
      const int l = u % TG_MAXLEV;
      const DevList& dl = u < TG_MAXLEV ? b->node[l] : b->elem[l];
      if (l < b->maxlev && (u < TG_MAXLEV || l > TG_MF_LEVELS)) {
        w.list[u] = dl.ptr;
        blocks += dl.n;
      }
      w.end[u] = (int)blocks;
    }
    for (int p : b->active) w.tiles = std::max(w.tiles, ci_tiles(b->grids[p]->ncoarse));
    w.prob = b->prob.ptr;
    blocks += (long long)b->prob.n * w.tiles;
    if (blocks) k_setup_tail<<<(unsigned)blocks, 256, 0, s>>>(b->desc_d, w);
    if (b->prob.n) {
      // which form inverts a problem's coarsest matrix depends only on its own
      // size, so a problem gets the same inverse alone or batched
      const int lim[4] = {0, CI_LDS_N, CI_REG_N, TG_MAX_COARSE};
      int nmax[3] = {0, 0, 0};
      for (int p : b->active) {
        const int n = b->grids[p]->ncoarse;
        for (int q = 0; q < 3; ++q)
          if (n > lim[q] && n <= lim[q + 1]) nmax[q] = std::max(nmax[q], n);
      }
      for (int q = 0; q < 3; ++q)
        if (nmax[q])
          (q == CI_LDS ? k_coarse_inverse<CI_LDS> : q == CI_REG ? k_coarse_inverse<CI_REG> : k_coarse_inverse<CI_MEM>)
              <<<nblk(b->prob), CI_THREADS, sizeof(double) * ci_lds_words(nmax[q], q), s>>>(
                  b->desc_d, b->prob.ptr, bad, lim[q] + 1, lim[q + 1]);
    }
  });
  return check_launch("set_density kernels");
}

// fine-level operator of type T on list dl (mode: 0 apply, 1 resid, 2 smooth)
template <class T>
static double op_bytes(const Batch* b, int l, int lmode, int op) {
  double nodes, elems, c2;
  level_sums(b, l, lmode, nodes, elems, c2);
  const double vec = 3.0 * nodes * sizeof(T);
  // fine level and matrix-free Galerkin levels read the fine moduli; deeper
  // levels read their stored mode-basis element matrices
  const double mat = (l <= TG_MF_LEVELS) ? elems * double(1 << (3 * l)) * sizeof(T) : elems * double(TG_GM_NU) * sizeof(T);
  const double dinv = (op == OP_SMOOTH || op == OP_SMOOTHP) ? 9.0 * nodes * sizeof(T) : 0.0;
  const int nvec = op == OP_APPLY ? 2 : 3;
  // the fused restriction reads x and b and writes the coarse right-hand side
  if (op == OP_RESTRICT) return 2 * vec + mat + vec / 8.0;
  // the fused first sweeps read b in FP64 and the node blocks, write x and b's copy
  if (op == OP_SMOOTH1) return 3.0 * nodes * 8.0 + 9.0 * nodes * sizeof(T) + mat + 2 * vec;
  if (op == OP_SMOOTH1E) return 9.0 * nodes * sizeof(T) + mat + 3 * vec;
  return nvec * vec + mat + dinv + (op == OP_SMOOTHP ? vec / 8.0 : 0.0);
}

int k_apply(Batch* b, int prec, int sx, const void* ex, int sy, void* ey, hipStream_t s) {
  // (measured heights serve the operator as well)
  if (b->op_zc[0] && !b->tuned && !b->active.empty())
    TG_TIMED(prec == TG_F64 ? TG_KT_APPLY_F64 : TG_KT_VCYCLE_FINE,
             (prec == TG_F64 ? op_bytes<double>(b, 0, 0, OP_APPLY) : op_bytes<float>(b, 0, 0, OP_APPLY)),
             launch_op_lone(b, prec, sx, ex, sy, ey, s));
  else if (prec == TG_BF16MFMA || prec == TG_BF16X3MFMA)
    TG_TIMED(TG_KT_VCYCLE_FINE, (op_bytes<float>(b, 0, 0, OP_APPLY)),
             launch_fine_mfma(b, b->fine, OP_APPLY, prec == TG_BF16X3MFMA, sx, ex, 0, nullptr, sy, ey, 0.0,
                              false, s));
  else if (prec == TG_F64)
    TG_TIMED(TG_KT_APPLY_F64, (op_bytes<double>(b, 0, 0, OP_APPLY)),
             launch_fine<double>(b, b->fine, 0, OP_APPLY, sx, ex, 0, nullptr, sy, ey, 0.0, s));
  else
    TG_TIMED(TG_KT_VCYCLE_FINE, (op_bytes<float>(b, 0, 0, OP_APPLY)),
             launch_fine<float>(b, b->fine, 0, OP_APPLY, sx, ex, 0, nullptr, sy, ey, 0.0, s));
  return check_launch("apply_K");
}

int k_residual64(Batch* b, int sb, int sx, int sy, hipStream_t s) {
  TG_TIMED(TG_KT_APPLY_F64, (op_bytes<double>(b, 0, 0, OP_RESID)),
           launch_fine<double>(b, b->fine, 0, OP_RESID, sx, nullptr, sb, nullptr, sy, nullptr, 0.0, s));
  return check_launch("residual");
}

// mf: 0 = vector mode-basis contraction, 1 = BF16 matrix cores, 2 = split BF16
template <class T, int OP>
// (y: slot of level l, or for OP_RESTRICT the right-hand-side slot of level
// l + 1, with y2 that level's first-sweep slot)
static void vc_op(Batch* b, int l, int x, int bs, int y, T om, hipStream_t s, int mf = 0, int y2 = -1,
                  int vbs = 0, const void* eb = nullptr, void* ey = nullptr) {
  const DevList& dl = (OP == OP_RESTRICT) ? b->zm_r[l] : b->zm_s[l];
  if (l == 0 && mf)
    TG_TIMED(TG_KT_VCYCLE_FINE, (op_bytes<T>(b, 0, 1, OP)),
             launch_fine_mfma(b, dl, OP, mf == 2, x, nullptr, bs, eb, y, ey, (double)om, false, s, y2));
  else if (l == 0)
    TG_TIMED(TG_KT_VCYCLE_FINE, (op_bytes<T>(b, 0, 1, OP)),
             launch_fine<T>(b, dl, 0, OP, x, nullptr, bs, eb, y, ey, (double)om, s, y2));
  else
    TG_TIMED(TG_KT_VCYCLE_COARSE, (op_bytes<T>(b, l, 1, OP)),
             launch_fine<T>(b, dl, l, OP, x, nullptr, bs, nullptr, y, nullptr, (double)om, s, y2, vbs));
}

// One fixed V-cycle.  Level-0 input b (slot sb of the FP64 pool or external
// eb, typed double unless in_is_f32) -> output (slot sy of the FP64 pool or
// external ey, double unless out_is_f32).
template <class T>
static int vcycle_t(Batch* b, int in_is_f32, int sb, const void* eb, int out_is_f32, int sy,
                    void* ey, hipStream_t s, int mf, int in_scale) {
  const tg_mg_opts& mg = b->grids[0]->mg;
  const T om = T(mg.omega);
  const bool f64 = sizeof(T) == 8;
  const int B0 = f64 ? S_VB : C_B, XA0 = f64 ? S_VXA : C_XA, XB0 = f64 ? S_VXB : C_XB;
  const int flips = (mg.nu_pre - 1) + mg.nu_post;
  const int FIN = (flips % 2 == 0) ? C_XA : C_XB;      // level >= 1 result slot
  const int FIN0 = (flips % 2 == 0) ? XA0 : XB0;
  int cur[TG_MAXLEV];
  const int L = b->maxlev;
  double nodes, elems, c2;
  const double sT = sizeof(T), sIn = in_is_f32 ? 4.0 : 8.0, sOut = out_is_f32 ? 4.0 : 8.0;
  // Fast level-0 boundary: FGMRES calls with an FP64 slot in, an FP64 slot out
  // and every problem multilevel.  The first sweep reads the FP64 vector
  // directly and the last sweep writes the FP64 output.
  bool all_multi = true;
  for (int p : b->active) all_multi = all_multi && b->grids[p]->nlev > 1;
  // An external vector (of type T) is read and written by the same two sweeps;
  // it may be one vector, since only the first of them reads the input.
  const bool ext_in = sb < 0 && in_is_f32 == (f64 ? 0 : 1) && all_multi && mg.nu_pre >= 2 && in_scale < 0;
  const bool ext_out = sy < 0 && out_is_f32 == (f64 ? 0 : 1) && all_multi && mg.nu_post >= 1;
  const bool fast_in = (!in_is_f32 && sb >= 0 && all_multi) || ext_in;
  const bool fast_out = !out_is_f32 && sy >= 0 && all_multi;
  // The bottom of the cycle (each problem's levels from its vb_lb down) runs
  // as one launch between the two passes; the level-by-level launches skip
  // those levels (vbs) and whole levels no problem needs.
  const int tv = f64 ? 1 : 0;
  const bool use_vb = b->vb[tv].n > 0;
  const int vbs = use_vb ? 1 : 0;
  auto level_needed = [&](int l) { return !use_vb || b->vb_need[tv][l]; };
  // ---- descend
  for (int l = 0; l < L; ++l) {
    if (!level_needed(l)) continue;
    const int Bs = l == 0 ? B0 : C_B, XA = l == 0 ? XA0 : C_XA, XB = l == 0 ? XB0 : C_XB;
    const DevList& sm = b->smooth[l];
    const DevList& co = b->coarse[l];
    if (l == 0 && b->node[0].n && !fast_in) {
      // b into the working slot of type T (also masks the clamped nodes)
      level_sums(b, 0, 0, nodes, elems, c2);
      if (in_is_f32)
        TG_TIMED(TG_KT_TRANSFER, 3.0 * nodes * (sIn + sT),
                 k_copy_level<float, T><<<nblk(b->node[0]), 256, 0, s>>>(b->desc_d, b->node[0].ptr, 0, sb, eb, Bs, nullptr, in_scale));
      else
        TG_TIMED(TG_KT_TRANSFER, 3.0 * nodes * (sIn + sT),
                 k_copy_level<double, T><<<nblk(b->node[0]), 256, 0, s>>>(b->desc_d, b->node[0].ptr, 0, sb, eb, Bs, nullptr, in_scale));
    }
    if (co.n) {
      const int fin = l == 0 ? FIN0 : FIN;
      level_sums(b, l, 2, nodes, elems, c2);
      TG_TIMED(TG_KT_TRANSFER, c2 * sT + 6.0 * nodes * sT,
               k_coarse_solve<T, T, T><<<nblk(co), 256, 0, s>>>(b->desc_d, co.ptr, l, Bs, nullptr, fin, nullptr,
                                                                vbs));
    }
    if (!sm.n) continue;
    level_sums(b, l, 1, nodes, elems, c2);
    int c = XA, o = XB;
    int it0 = 1;
    if (l == 0 && fast_in && mg.nu_pre >= 2) {
      // first sweep from zero computed while staging, second sweep in the same pass
      if (ext_in) vc_op<T, OP_SMOOTH1E>(b, 0, -1, -1, o, om, s, mf, Bs, vbs, eb);
      else vc_op<T, OP_SMOOTH1>(b, 0, in_scale, sb, o, om, s, mf, Bs, vbs);
      std::swap(c, o);
      it0 = 2;
    } else if (l == 0 && fast_in)
      TG_TIMED(TG_KT_TRANSFER, 3.0 * nodes * (8.0 + 2 * sT) + 9.0 * nodes * sT,
               k_jacobi_first<double, T><<<nblk(sm), 256, 0, s>>>(b->desc_d, sm.ptr, 0, sb, nullptr, Bs, XA, om,
                                                                    in_scale));
    else if (l == 0)
      TG_TIMED(TG_KT_TRANSFER, 3.0 * nodes * 2 * sT + 9.0 * nodes * sT,
               k_jacobi_first<T, T><<<nblk(sm), 256, 0, s>>>(b->desc_d, sm.ptr, l, Bs, nullptr, INT_MIN, XA, om, -1));
    // (levels >= 1: the restriction above already wrote the first sweep)
    for (int it = it0; it < mg.nu_pre; ++it) {
      vc_op<T, OP_SMOOTH>(b, l, c, Bs, o, om, s, mf, -1, vbs);
      std::swap(c, o);
    }
    // residual, restricted straight into the next level's right-hand side,
    // and that level's first Jacobi sweep from zero
    vc_op<T, OP_RESTRICT>(b, l, c, Bs, C_B, om, s, mf, C_XA, vbs);
    cur[l] = c;
  }
  if (use_vb)
    TG_TIMED(TG_KT_VCYCLE_COARSE, vbottom_bytes(b, tv),
             launch_vbottom<T>(b, b->vb[tv], b->vb_lds[tv], FIN, mg.omega, mg.nu_pre, mg.nu_post, b->vb_l1[tv], s));
  // ---- ascend
  for (int l = L - 1; l >= 0; --l) {
    const DevList& sm = b->smooth[l];
    if (!sm.n || !level_needed(l)) continue;
    const int Bs = l == 0 ? B0 : C_B, XA = l == 0 ? XA0 : C_XA, XB = l == 0 ? XB0 : C_XB;
    int c = cur[l];
    int o = (c == XA) ? XB : XA;
    level_sums(b, l, 1, nodes, elems, c2);
    // the first post-sweep forms x + P e itself (not where it is level 0's last
    // sweep, which writes the output)
    const bool pro = mg.nu_post >= (l == 0 ? 2 : 1) && fine_prolongs(b, l);
    if (!pro)
      TG_TIMED(TG_KT_TRANSFER, 3.0 * nodes * 2 * sT + 3.0 * nodes / 8 * sT,
               k_prolong<T><<<nblk(sm), 256, 0, s>>>(b->desc_d, sm.ptr, l, c, FIN, nullptr, nullptr, vbs));
    for (int it = 0; it < mg.nu_post; ++it) {
      if (it == 0 && pro) {
        vc_op<T, OP_SMOOTHP>(b, l, c, Bs, o, om, s, mf, FIN, vbs);
        std::swap(c, o);
        continue;
      }
      if (l == 0 && ext_out && it == mg.nu_post - 1) {
        vc_op<T, OP_SMOOTH>(b, 0, c, Bs, -1, om, s, mf, -1, vbs, nullptr, ey);
        c = -1;   // result is in the external vector
        break;
      }
      if (l == 0 && fast_out && it == mg.nu_post - 1) {
        if (f64)
          vc_op<T, OP_SMOOTH>(b, 0, c, Bs, sy, om, s, 0, -1, vbs);   // straight into the FP64 output slot
        else if (mf)
          TG_TIMED(TG_KT_VCYCLE_FINE, (op_bytes<T>(b, 0, 1, OP_SMOOTH) + 3.0 * nodes * (8.0 - sT)),
                   launch_fine_mfma(b, b->zm_s[0], OP_SMOOTH, mf == 2, c, nullptr, Bs, nullptr, sy, nullptr,
                                    (double)om, true, s));
        else
          TG_TIMED(TG_KT_VCYCLE_FINE, (op_bytes<T>(b, 0, 1, OP_SMOOTH) + 3.0 * nodes * (8.0 - sT)),
                   launch_fine_smooth_out64(b, b->zm_s[0], c, Bs, sy, (double)om, s));
        c = -1;   // result is in the output slot
        break;
      }
      vc_op<T, OP_SMOOTH>(b, l, c, Bs, o, om, s, mf, -1, vbs);
      std::swap(c, o);
    }
    cur[l] = c;
  }
  // ---- output (level 0): result in FIN0 for every problem
  if (b->node[0].n && !fast_out && !ext_out) {
    level_sums(b, 0, 0, nodes, elems, c2);
    if (out_is_f32)
      TG_TIMED(TG_KT_TRANSFER, 3.0 * nodes * (sOut + sT),
               k_copy_level<T, float><<<nblk(b->node[0]), 256, 0, s>>>(b->desc_d, b->node[0].ptr, 0, FIN0, nullptr, sy, ey, -1));
    else
      TG_TIMED(TG_KT_TRANSFER, 3.0 * nodes * (sOut + sT),
               k_copy_level<T, double><<<nblk(b->node[0]), 256, 0, s>>>(b->desc_d, b->node[0].ptr, 0, FIN0, nullptr, sy, ey, -1));
  }
  return check_launch("vcycle");
}

int k_vcycle(Batch* b, int prec, int in_is_f32, int sb, const void* eb, int out_is_f32, int sy,
             void* ey, hipStream_t s, int in_scale_sc) {
  const int in_scale = in_scale_sc >= 0 ? offs(b).scal + in_scale_sc : -1;
  if (prec == TG_F64) return vcycle_t<double>(b, in_is_f32, sb, eb, out_is_f32, sy, ey, s, 0, in_scale);
  const int mf = prec == TG_BF16MFMA ? 1 : prec == TG_BF16X3MFMA ? 2 : 0;
  return vcycle_t<float>(b, in_is_f32, sb, eb, out_is_f32, sy, ey, s, mf, in_scale);
}

// ---- level primitives of host-stepped cycles (FP64, external vectors of
// the level's full length, clamped nodes zero)
int level_op64(Batch* b, int l, int op, const double* x, const double* bb, double* y, double omega,
               hipStream_t s) {
  const bool all = (l == 0 && op == OP_APPLY);
  const DevList& dl = all ? b->fine : b->zm_s[l];
  TG_TIMED(l == 0 ? TG_KT_APPLY_F64 : TG_KT_VCYCLE_COARSE, (op_bytes<double>(b, l, all ? 0 : 1, op)),
           launch_fine<double>(b, dl, l, op, -1, x, -1, bb, -1, y, omega, s));
  return check_launch("level operator");
}
int level_restrict64(Batch* b, int l, const double* x, const double* bb, int slot_next, hipStream_t s) {
  TG_TIMED(l == 0 ? TG_KT_APPLY_F64 : TG_KT_VCYCLE_COARSE, (op_bytes<double>(b, l, 1, OP_RESTRICT)),
           launch_fine<double>(b, b->zm_r[l], l, OP_RESTRICT, -1, x, -1, bb, slot_next, nullptr, 0.0, s, -1));
  return check_launch("level restriction");
}
int level_prolong64(Batch* b, int l, const double* ec, double* xf, hipStream_t s) {
  const DevList& sm = b->smooth[l];
  if (sm.n) {
    double nodes, elems, c2;
    level_sums(b, l, 1, nodes, elems, c2);
    TG_TIMED(TG_KT_TRANSFER, 3.0 * nodes * 16.0 + 3.0 * nodes / 8 * 8.0,
             k_prolong<double><<<nblk(sm), 256, 0, s>>>(b->desc_d, sm.ptr, l, -1, -1, ec, xf, 0));
  }
  return check_launch("level prolongation");
}
int level_coarse64(Batch* b, int l, const double* bb, double* y, hipStream_t s) {
  const DevList& co = b->coarse[l];
  if (co.n) {
    double nodes, elems, c2;
    level_sums(b, l, 2, nodes, elems, c2);
    TG_TIMED(TG_KT_TRANSFER, c2 * 8.0 + 6.0 * nodes * 8.0,
             k_coarse_solve<double, double, double><<<nblk(co), 256, 0, s>>>(b->desc_d, co.ptr, l, -1, bb, -1, y,
                                                                             0));
  }
  return check_launch("coarsest solve");
}

int k_copy_ext(Batch* b, int dir, int slot, hipStream_t s) {
  if (b->vec.n)
    TG_TIMED(TG_KT_UPDATE, 16.0 * dofs0(b), k_copy_ext_<<<nblk(b->vec), 256, 0, s>>>(b->desc_d, b->vec.ptr, dir, slot));
  return check_launch("copy_ext");
}
int k_fill0(Batch* b, int slot, double v, hipStream_t s) {
  if (b->vec.n)
    TG_TIMED(TG_KT_UPDATE, 8.0 * dofs0(b), k_fill0_<<<nblk(b->vec), 256, 0, s>>>(b->desc_d, b->vec.ptr, slot, v));
  return check_launch("fill");
}
int k_copy0(Batch* b, int src, int dst, hipStream_t s) {
  if (b->vec.n)
    TG_TIMED(TG_KT_UPDATE, 16.0 * dofs0(b), k_copy0_<<<nblk(b->vec), 256, 0, s>>>(b->desc_d, b->vec.ptr, src, dst));
  return check_launch("copy");
}
int k_multidot(Batch* b, int sbase, int nv, int sw, int with_self, hipStream_t s) {
  if (b->vec.n)
    TG_TIMED(TG_KT_MULTIDOT, 8.0 * (nv + 1) * dofs0(b),
             k_multidot_<<<nblk(b->vec), 256, 0, s>>>(b->desc_d, b->vec.ptr, sbase, nv, sw, with_self));
  return check_launch("multidot");
}
int k_reduce(Batch* b, int nv, int mode, int dst, int save_k, hipStream_t s) {
  const SmallOffs o = offs(b);
  if (b->prob.n && nv > 0)
    TG_TIMED(TG_KT_SCALAR, 0,
             k_reduce_<<<dim3(b->prob.n, nv), 256, 0, s>>>(b->desc_d, b->prob.ptr, o.h, o.tmp + dst,
                                                          o.scal + SC_FLAG, mode, save_k));
  return check_launch("reduce");
}
int k_update(Batch* b, int sbase, int nv, int sw, int coef_is_tmp, hipStream_t s) {
  const SmallOffs o = offs(b);
  const int coef_off = coef_is_tmp ? o.tmp : o.h;
  if (b->vec.n)
    TG_TIMED(TG_KT_UPDATE, 8.0 * (nv + 2) * dofs0(b),
             k_update_<<<nblk(b->vec), 256, 0, s>>>(b->desc_d, b->vec.ptr, sbase, nv, sw, coef_off));
  return check_launch("update");
}
int k_update_dots(Batch* b, int sbase, int nv, int sw, int coef_is_tmp, int ndot, int with_self,
                  hipStream_t s) {
  const SmallOffs o = offs(b);
  const int coef_off = coef_is_tmp ? o.tmp : o.h;
  if (b->vec.n) {
    if (nv <= 32 && ndot <= 32)
      TG_TIMED(TG_KT_UPDATE, 8.0 * (nv + 2) * dofs0(b),
               k_update_dots_reg_<32><<<nblk(b->vec), 256, 0, s>>>(b->desc_d, b->vec.ptr, sbase, nv, sw,
                                                                  coef_off, ndot, with_self));
    else
      TG_TIMED(TG_KT_UPDATE, 8.0 * (nv + 2 + ndot) * dofs0(b),
               k_update_dots_<<<nblk(b->vec), 256, 0, s>>>(b->desc_d, b->vec.ptr, sbase, nv, sw, coef_off,
                                                          ndot, with_self));
  }
  return check_launch("update_dots");
}

// Whether a sweep over nv basis vectors of the running problems exceeds the L2
// caches (8 x 4 MB) well enough that non-temporal loads pay (k_dots2_).
static bool basis_streams(const Batch* b, int nv) { return 8.0 * (nv + 2) * dofs0(b) > 64e6; }

// Sweep A of the delayed CGS2 step j (nv = j basis vectors), then its
// scalar end (chunk sums and the first scalar part) in one per-problem launch.
int k_dots2(Batch* b, int sbase, int nv, int sq, int sw, hipStream_t s) {
  if (b->vec.n)
    TG_TIMED(TG_KT_MULTIDOT, 8.0 * (nv + 2) * dofs0(b),
             (basis_streams(b, nv) ? k_dots2_<true> : k_dots2_<false>)<<<nblk(b->vec), 256, 0, s>>>(
                 b->desc_d, b->vec.ptr, sbase, nv, sq, sw));
  if (b->prob.n)
    TG_TIMED(TG_KT_SCALAR, 0, k_fin_a_<<<nblk(b->prob), 256, 0, s>>>(b->desc_d, b->prob.ptr, offs(b), nv, b->sc_d));
  return check_launch("dots2");
}
// Sweep B, then its scalar end (the norm sum, the Givens update, the history
// entry and the stop tests) in one per-problem launch.
int k_update2(Batch* b, int sbase, int nv, int sq, int sw, int snext, int cap, double tol, double brk,
              hipStream_t s) {
  const SmallOffs o = offs(b);
  if (b->vec.n)
    TG_TIMED(TG_KT_UPDATE, 8.0 * (nv + 4) * dofs0(b),
             (basis_streams(b, nv) ? k_update2_<true> : k_update2_<false>)<<<nblk(b->vec), 256, 0, s>>>(
                 b->desc_d, b->vec.ptr, sbase, nv, sq, sw, snext, o.tmp));
  if (b->prob.n)
    TG_TIMED(TG_KT_SCALAR, 0,
             k_fin_b_<<<nblk(b->prob), 256, 0, s>>>(b->desc_d, b->prob.ptr, o, nv, cap, tol, brk, b->sc_d));
  return check_launch("update2");
}
int k_scale_to(Batch* b, int src, int dst, int sc_index, hipStream_t s) {
  const int sidx = offs(b).scal + sc_index;
  if (b->vec.n)
    TG_TIMED(TG_KT_UPDATE, 16.0 * dofs0(b), k_scale_<<<nblk(b->vec), 256, 0, s>>>(b->desc_d, b->vec.ptr, src, dst, sidx));
  return check_launch("scale");
}
int k_cycle_start(Batch* b, int k, int cap, double tol, hipStream_t s) {
  if (b->prob.n)
    TG_TIMED(TG_KT_SCALAR, 0,
             k_cycle_start_<<<nblk(b->prob), 64, 0, s>>>(b->desc_d, b->prob.ptr, offs(b), k, cap, tol, b->sc_d));
  return check_launch("cycle_start");
}
int k_arnoldi(Batch* b, int j, int k, int cap, double tol, double brk, hipStream_t s) {
  if (b->prob.n)
    TG_TIMED(TG_KT_SCALAR, 0,
             k_arnoldi_<<<nblk(b->prob), 64, 0, s>>>(b->desc_d, b->prob.ptr, offs(b), j, k, cap, tol, brk, b->sc_d));
  return check_launch("arnoldi");
}
int k_lsq_update(Batch* b, int mmax, int jmax, hipStream_t s) {
  const SmallOffs o = offs(b);
  if (b->prob.n) TG_TIMED(TG_KT_SCALAR, 0, k_lsq_<<<nblk(b->prob), 64, 0, s>>>(b->desc_d, b->prob.ptr, o));
  if (b->vec.n)
    TG_TIMED(TG_KT_UPDATE, 8.0 * (jmax + 2) * dofs0(b),
             k_xupdate_<<<nblk(b->vec), 256, 0, s>>>(b->desc_d, b->vec.ptr, o, slot_Z(mmax, 0)));
  return check_launch("lsq_update");
}
int k_true_eta(Batch* b, hipStream_t s, bool to_status) {
  if (b->prob.n)
    TG_TIMED(TG_KT_SCALAR, 0, k_true_eta_<<<nblk(b->prob), 64, 0, s>>>(b->desc_d, b->prob.ptr, offs(b),
                                                                        to_status ? b->sc_d : nullptr));
  return check_launch("true_eta");
}
int k_init_small(Batch* b, hipStream_t s) {
  if (b->prob.n)
    TG_TIMED(TG_KT_SCALAR, 0,
             k_init_small_<<<nblk(b->prob), 256, 0, s>>>(b->desc_d, b->prob.ptr, b->grids[0]->sl.total));
  return check_launch("init_small");
}


// ---------------------------------------------------------------------------
// One Krylov process on caller memory (KrylovOne).
// Bound by launches: a step is four of them, 25 us at 215 k unknowns, in place of
// eleven (two dot products of three launches each, the updates, the rotations).
static SmallOffs offs(const SmallLayout& s) {
  return {s.mmax, s.H, s.g, s.cs, s.sn, s.y, s.h, s.tmp, s.scal, s.hist};
}
// the descriptor and the work list, and the slots' tails cleared
__global__ __launch_bounds__(256) void k_kry_bind_(ProbDesc d, ProbDesc* desc, int2* list, int chunks, int slots) {
  const LevelDesc& L = d.lv[0];
  const long long n = 3LL * L.n_nodes;
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) *desc = d;
    for (int c = threadIdx.x; c < chunks; c += 256) list[c] = make_int2(0, c);
  }
  for (int v = blockIdx.x; v < slots; v += gridDim.x)
    for (long long q = n + threadIdx.x; q < L.stride; q += 256) L.vec64[v * L.stride + q] = 0.0;
}
int krylov_bind(const KrylovOne& K, hipStream_t s) {
  ProbDesc d = {};
  d.nlev = 1;
  d.small = K.small;
  d.part = K.part;
  d.lv[0].n_nodes = (int)(K.n / 3);
  d.lv[0].n_chunks = K.chunks;
  d.lv[0].stride = K.stride;
  d.lv[0].vec64 = K.pool;
  k_kry_bind_<<<std::min(64, K.q + 2), 256, 0, s>>>(d, K.desc, K.list, K.chunks, K.q + 2);
  return check_launch("krylov bind");
}
// V_0 = src and the chunk sums of src . src.  The tail is cleared as well: the
// sweeps of a process that has stopped (b = 0 among others) go on with whatever its
// coefficients hold, since a gate on its status, one more dependent load a launch,
// cost an application of the stack 1.2 %.  They leave nothing else behind: every
// other vector is written whole from V_0 and w before it is read.
__global__ __launch_bounds__(256) void k_kry_start_(const ProbDesc* __restrict__ probs, const double* src) {
  __shared__ double sh[4];
  const ProbDesc& P = *probs;
  const LevelDesc& L = P.lv[0];
  long long lo, hi;
  chunk_range(L, blockIdx.x, lo, hi);
  double* v = L.vec64;
  double a = 0.0;
#pragma unroll
  for (int q = 0; q < TG_VCHUNK / 256; ++q) {
    const long long i = lo + threadIdx.x + 256LL * q;
    if (i < hi) {
      const double x = src[i];
      if (v != src) v[i] = x;
      a += x * x;
    } else {
      v[i] = 0.0;
    }
  }
  a = block_sum256(a, sh);
  if (threadIdx.x == 0) P.part[blockIdx.x] = a;
}
// beta = ||V_0||, then the cycle start (k_cycle_start_) with no tolerance
__global__ __launch_bounds__(256) void k_kry_begin_(const ProbDesc* __restrict__ probs, SmallOffs o, double* rr,
                                                    double* status) {
  __shared__ double sh[4];
  const ProbDesc& P = *probs;
  const int nc = P.lv[0].n_chunks;
  double a = 0.0;
  for (int c = threadIdx.x; c < nc; c += 256) a += P.part[c];
  a = block_sum256(a, sh);
  double* S = P.small;
  for (int q = threadIdx.x; q <= o.mmax; q += 256)
    if (q) S[o.g + q] = 0.0;
  if (threadIdx.x != 0) return;
  double* sc = S + o.scal;
  const double beta = sqrt(a);
  const double st = !isfinite(beta) ? TG_NONFINITE : beta == 0.0 ? TG_PROJ_CONVERGED : TG_RUNNING;
  *rr = a;
  S[o.g] = beta;
  sc[SC_BNORM] = sc[SC_BETA] = sc[SC_RHO] = beta;
  sc[SC_INV] = beta > 0.0 ? 1.0 / beta : 0.0;
  sc[SC_ITERS] = sc[SC_JDONE] = 0.0;
  sc[SC_STATUS] = st;
  *status = st;
}
int krylov_start(const KrylovOne& K, const double* src, double* rr, hipStream_t s) {
  k_kry_start_<<<K.chunks, 256, 0, s>>>(K.desc, src);
  k_kry_begin_<<<1, 256, 0, s>>>(K.desc, offs(K.sl), rr, K.status);
  return check_launch("krylov start");
}
int krylov_step(const KrylovOne& K, int j, hipStream_t s) {
  const SmallOffs o = offs(K.sl);
  // (cap beyond the last column: its reorthogonalization follows in krylov_finish)
  k_dots2_<false><<<K.chunks, 256, 0, s>>>(K.desc, K.list, 0, j, j, K.q + 1);
  k_fin_a_<<<1, 256, 0, s>>>(K.desc, K.list, o, j, K.status);
  k_update2_<false><<<K.chunks, 256, 0, s>>>(K.desc, K.list, 0, j, j, K.q + 1, j + 1, o.tmp);
  k_fin_b_<<<1, 256, 0, s>>>(K.desc, K.list, o, j, K.q + 1, 0.0, 1e-14, K.status);
  return check_launch("krylov step");
}
// y = R^-1 g over the columns done, by columns on one wave: lane i holds
// entries i and i + 64 of the right-hand side
__global__ __launch_bounds__(64) void k_kry_lsq_(const ProbDesc* __restrict__ probs, SmallOffs o) {
  double* S = probs->small;
  const int jd = (int)S[o.scal + SC_JDONE], ldh = o.mmax + 1, lane = threadIdx.x;
  double v0 = lane < jd ? S[o.g + lane] : 0.0, v1 = lane + 64 < jd ? S[o.g + lane + 64] : 0.0;
  const auto* H = gp((const double*)S + o.H);
  auto col = [&](int c, double& r0, double& r1) {
    r0 = c >= 0 && lane <= c ? H[(long long)ldh * c + lane] : 1.0;
    r1 = c >= 0 && lane + 64 <= c ? H[(long long)ldh * c + lane + 64] : 1.0;
  };
  double r0, r1, n0, n1;
  col(jd - 1, r0, r1);
  for (int c = jd - 1; c >= 0; --c) {
    col(c - 1, n0, n1);   // the next column is read ahead
    const double y = __shfl((c < 64 ? v0 : v1) / (c < 64 ? r0 : r1), c & 63, 64);
    if (lane < c) v0 -= r0 * y;
    if (lane + 64 < c) v1 -= r1 * y;
    if (lane == 0) S[o.y + c] = y;
    r0 = n0;
    r1 = n1;
  }
}
// out = sum_{j < done} y_j Z_j
__global__ __launch_bounds__(256) void k_kry_combine_(const double* __restrict__ Z, long long stride,
                                                      const double* __restrict__ S, SmallOffs o, long long n,
                                                      double* __restrict__ out) {
  __shared__ double sy[TG_MAX_RESTART];
  const int jd = (int)S[o.scal + SC_JDONE];
  if ((int)threadIdx.x < jd) sy[threadIdx.x] = S[o.y + threadIdx.x];
  __syncthreads();
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  double a = 0.0;
#pragma unroll 4
  for (int j = 0; j < jd; ++j) a += sy[j] * Z[j * stride + i];
  out[i] = a;
}
int krylov_finish(const KrylovOne& K, double* out, hipStream_t s) {
  const SmallOffs o = offs(K.sl);
  // the last column's second pass (w is not needed: V_q itself)
  k_dots2_<false><<<K.chunks, 256, 0, s>>>(K.desc, K.list, 0, K.q, K.q, K.q);
  k_fin_a_<<<1, 256, 0, s>>>(K.desc, K.list, o, K.q, K.status);
  k_kry_lsq_<<<1, 64, 0, s>>>(K.desc, o);
  k_kry_combine_<<<(unsigned)((K.n + 255) / 256), 256, 0, s>>>(K.Z(0), K.stride, K.small, o, K.n, out);
  return check_launch("krylov finish");
}

}  // namespace tg
