// Split schedule: one time step n -> n+1 in two kernels.
//
//   h_step: c^n = sum_k h~^n_k (pull of H), mu^n, grad phi^n and the normal
//           from the phi^n stencil, phi^{n+1} = sum_k g~^{n+1}_k + S^n/2 (pull
//           of G), dphi/dt = phi^{n+1} - phi^n, anti-trapping current, h
//           collision  ->  H' = h~*^n, PHI' = phi^{n+1}
//   g_step: c^{n+1} (pull of H'), mu^{n+1}, grad phi^{n+1}, sources, g
//           collision of the pulled g~^{n+1}  ->  G' = g~*^{n+1}
//
// Each kernel reads both distributions once and writes one, so the step
// moves 6Q+3 values per node against the 4Q+2 of the fused schedule.  It has
// no tile halo and works for every boundary combination; it is the baseline
// the fused kernels are checked against.
//
// Also here: initialisation, field read-out and the diagnostics reduction,
// which all schedules share.
#pragma once

#include "geometry.h"
#include "node_math.h"
#include "tiles.h"

namespace gplbm {

template <class S>
struct StepBufs {
  const S* __restrict__ G;    // g~*^n
  const S* __restrict__ H;    // h~*^{n-1}
  const S* __restrict__ PHI;  // phi^n
  S* __restrict__ Hn;         // h~*^n
  S* __restrict__ PHIn;       // phi^{n+1}
  S* __restrict__ Gn;         // g~*^{n+1}
};

// Addressing of the per-node kernels.  AddrGeneral takes any grid, by the
// rules of geometry.h.  AddrPlane serves grids of up to kGridYZ planes whose
// population planes are shorter than 4 GiB: threads run over the nodes of a z
// plane (blockIdx.z), so a plane's base is a scalar and a neighbour a 32-bit
// offset wrapped once per node, with no division or branch per population; with
// walls a bounced population is a selected address.  Both give the same nodes.
constexpr int kNodeThreads = 256;
constexpr int kGridYZ = 65535;          // blocks of a launch along y and z
constexpr int64_t kGridX = 1 << 22;     // and along x (2^32 threads at most)

// The launch of AddrGeneral: blocks over the nodes of a plane along x, in runs
// of kGridX, planes along z, and along y the runs of a plane times the layers of
// kGridYZ planes.
__host__ __device__ inline int64_t general_runs(int64_t plane) {
  const int64_t per_run = kGridX * kNodeThreads;
  return (plane + per_run - 1) / per_run;
}
inline dim3 general_grid(int64_t plane, int nz) {
  const int64_t nb = (plane + kNodeThreads - 1) / kNodeThreads;
  const int64_t layers = ((int64_t)nz + kGridYZ - 1) / kGridYZ;
  return dim3((unsigned)(nb < kGridX ? nb : kGridX), (unsigned)(general_runs(plane) * layers),
              nz < kGridYZ ? nz : kGridYZ);
}

struct AddrGeneral {
  const Geo& g;
  bool in;
  int x, y, z;
  __device__ AddrGeneral(const Geo& g_) : g(g_) {
    const int64_t plane = (int64_t)g.nx * g.ny;
    const int runs = int(general_runs(plane));
    const int64_t i =
        ((int64_t)(blockIdx.y % runs) * kGridX + blockIdx.x) * kNodeThreads + threadIdx.x;
    const int64_t zz = (int64_t)(blockIdx.y / runs) * kGridYZ + blockIdx.z;
    in = i < plane && zz < g.nz;
    y = in ? int(i / g.nx) : 0;
    x = in ? int(i - (int64_t)y * g.nx) : 0;
    z = in ? int(zz) : 0;
  }
  __device__ AddrGeneral(const Geo& g_, int x_, int y_, int z_)
      : g(g_), in(true), x(x_), y(y_), z(z_) {}
  __device__ bool inside() const { return in; }
  __device__ int64_t node() const { return node_index(g, x, y, z); }
  // element of plane m among the q planes per z of a distribution
  __device__ int64_t slot(int m, int q) const {
    return ((int64_t)z * q + m) * ((int64_t)g.nx * g.ny) + (int64_t)y * g.nx + x;
  }
  template <class P>
  __device__ bool bounced(int k) const {
    int sx = x, sy = y, sz = z;
    return !(pull_axis(sx, P::ex[k], g.nx, g.bcx) && pull_axis(sy, P::ey[k], g.ny, g.bcy) &&
             pull_axis(sz, P::ez[k], g.nz, g.bcz));
  }
  template <class P, class S, class M>
  __device__ const S* source(const S* f, int k, int q, const M& m) const {
    int sx = x, sy = y, sz = z, kk = k;
    if (!(pull_axis(sx, P::ex[k], g.nx, g.bcx) && pull_axis(sy, P::ey[k], g.ny, g.bcy) &&
          pull_axis(sz, P::ez[k], g.nz, g.bcz)))
      sx = x, sy = y, sz = z, kk = P::opp[k];
    return f + ((int64_t)sz * q + m(kk)) * ((int64_t)g.nx * g.ny) + (int64_t)sy * g.nx + sx;
  }
  // address that pulls slot k of this node: population k at x + e_k, or
  // opp(k) at x when x + e_k lies beyond a wall
  template <class P, class S, class M>
  __device__ const S* dest(const S* f, int k, int q, const M& m) const {
    int dx = x, dy = y, dz = z, kk = k;
    if (!(pull_axis(dx, -P::ex[k], g.nx, g.bcx) && pull_axis(dy, -P::ey[k], g.ny, g.bcy) &&
          pull_axis(dz, -P::ez[k], g.nz, g.bcz)))
      dx = x, dy = y, dz = z, kk = P::opp[k];
    return f + ((int64_t)dz * q + m(kk)) * ((int64_t)g.nx * g.ny) + (int64_t)dy * g.nx + dx;
  }
  template <class P, class S>
  __device__ S pull_pop(const S* __restrict__ f, int k) const { return pull<P>(g, f, k, x, y, z); }
  // a wall lies next to the node
  __device__ bool edge() const { return true; }
  template <class S>
  __device__ S at(const S* __restrict__ f, int dx, int dy, int dz) const {
    return f[node_index(g, stencil_axis(x + dx, g.nx, g.bcx), stencil_axis(y + dy, g.ny, g.bcy),
                        stencil_axis(z + dz, g.nz, g.bcz))];
  }
};

template <bool kWalls>
struct AddrPlane {
  int64_t plane;
  bool in;
  int x, y, z;
  int zs[3], ps[3];    // planes z - 1, z, z + 1: wrapped, and with the mirror ghost
  uint32_t src[3][3];  // in-plane offset of (x, y) + (c - 1, a - 1), wrapped, [a][c]
  bool xm, xp, ym, yp, zm, zp;  // that neighbour lies beyond a wall

  __device__ AddrPlane(const Geo& g) : plane((int64_t)g.nx * g.ny) {
    const uint32_t i = plane_block() * blockDim.x + threadIdx.x;
    in = i < (uint32_t)plane;
    const int yy = in ? i / (uint32_t)g.nx : 0;
    set(g, in ? i - yy * g.nx : 0, yy, blockIdx.z);
  }
  __device__ AddrPlane(const Geo& g, int x_, int y_, int z_) : plane((int64_t)g.nx * g.ny), in(true) {
    set(g, x_, y_, z_);
  }
  // The block of 256 nodes of the plane that this block takes.  In bands
  // (gridDim.y > 1, gridDim.x = kNumXcd, the XCD of a block by the round-robin
  // order of dispatch) an XCD takes neighbouring blocks of the plane, and the
  // same ones over four planes; then the bands turn, so that the XCDs of a
  // plane's last, partly empty bands change.
  static __device__ uint32_t plane_block() {
    if (gridDim.y == 1) return blockIdx.x;
    const uint32_t band = (blockIdx.x + (blockIdx.z >> 2)) % kNumXcd;
    return band * gridDim.y + blockIdx.y;
  }
  __device__ void set(const Geo& g, int x_, int y_, int z_) {
    x = x_;
    y = y_;
    z = z_;
    const int xo[3] = {x == 0 ? g.nx - 1 : x - 1, x, x == g.nx - 1 ? 0 : x + 1};
    const int yo[3] = {y == 0 ? g.ny - 1 : y - 1, y, y == g.ny - 1 ? 0 : y + 1};
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) src[a][c] = (uint32_t)yo[a] * g.nx + xo[c];
    zs[0] = z == 0 ? g.nz - 1 : z - 1;
    zs[1] = z;
    zs[2] = z == g.nz - 1 ? 0 : z + 1;
    xm = kWalls && g.bcx && x == 0;
    xp = kWalls && g.bcx && x == g.nx - 1;
    ym = kWalls && g.bcy && y == 0;
    yp = kWalls && g.bcy && y == g.ny - 1;
    zm = kWalls && g.bcz && z == 0;
    zp = kWalls && g.bcz && z == g.nz - 1;
    ps[0] = zm ? z : zs[0];
    ps[1] = z;
    ps[2] = zp ? z : zs[2];
  }
  __device__ bool inside() const { return in; }
  __device__ uint32_t self() const { return src[1][1]; }
  __device__ int64_t node() const { return zs[1] * plane + self(); }
  __device__ int64_t slot(int m, int q) const { return ((int64_t)zs[1] * q + m) * plane + self(); }
  template <class P>
  __device__ bool bounced(int k) const {
    if (!kWalls) return false;
    return (P::ex[k] > 0 && xm) || (P::ex[k] < 0 && xp) || (P::ey[k] > 0 && ym) ||
           (P::ey[k] < 0 && yp) || (P::ez[k] > 0 && zm) || (P::ez[k] < 0 && zp);
  }
  // element of a plane at a 32-bit byte offset
  template <class S>
  __device__ static const S* elem(const S* base, uint32_t i) {
    return reinterpret_cast<const S*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(S));
  }
  // address of the value population k pulls, from a distribution of q planes
  // per z with population j in plane m(j)
  template <class P, class S, class M>
  __device__ const S* source(const S* f, int k, int q, const M& m) const {
    const S* p = elem(f + ((int64_t)zs[1 - P::ez[k]] * q + m(k)) * plane,
                      src[1 - P::ey[k]][1 - P::ex[k]]);
    if (kWalls && bounced<P>(k)) p = elem(f + ((int64_t)zs[1] * q + m(P::opp[k])) * plane, self());
    return p;
  }
  template <class P, class S, class M>
  __device__ const S* dest(const S* f, int k, int q, const M& m) const {
    const S* p = elem(f + ((int64_t)zs[1 + P::ez[k]] * q + m(k)) * plane,
                      src[1 + P::ey[k]][1 + P::ex[k]]);
    if (kWalls && bounced<P>(P::opp[k]))
      p = elem(f + ((int64_t)zs[1] * q + m(P::opp[k])) * plane, self());
    return p;
  }
  template <class P, class S>
  __device__ S pull_pop(const S* __restrict__ f, int k) const {
    return *source<P>(f, k, P::Q, [](int j) { return j; });
  }
  __device__ bool edge() const { return kWalls && (xm || xp || ym || yp || zm || zp); }
  // field at x + (dx, dy, dz), the mirror ghost at a wall
  template <class S>
  __device__ S at(const S* __restrict__ f, int dx, int dy, int dz) const {
    uint32_t i = src[1 + dy][1 + dx];
    if (kWalls) {
      const int ox = (dx < 0 && xm) || (dx > 0 && xp) ? 0 : dx;
      const int oy = (dy < 0 && ym) || (dy > 0 && yp) ? 0 : dy;
      const uint32_t row = oy < 0 ? src[0][1] : (oy > 0 ? src[2][1] : src[1][1]);
      const int step = ox < 0 ? (int)(src[1][0] - src[1][1]) : (ox > 0 ? (int)(src[1][2] - src[1][1]) : 0);
      i = row + step;
    }
    return *elem(f + ps[1 + dz] * plane, i);
  }
};

// Values of a field at the nodes the gradient stencil of lattice L reads, all
// loaded at once.
template <class L, class C>
struct Stencil {
  C v[3][3][3];
  template <class A, class S>
  __device__ Stencil(const A& a, const S* __restrict__ f) {
#pragma unroll
    for (int k = 0; k < L::Q; ++k)
      v[1 + L::ez[k]][1 + L::ey[k]][1 + L::ex[k]] = C(a.at(f, L::ex[k], L::ey[k], L::ez[k]));
  }
  __device__ C operator()(int dx, int dy, int dz) const { return v[1 + dz][1 + dy][1 + dx]; }
};

// The loads of a node stay one batch: the scheduler does not move arithmetic
// between them.
__device__ __forceinline__ void loads_issued() { __builtin_amdgcn_sched_barrier(0); }

template <class L, class LH, class S, class C, bool kGen, class Addr>
__global__ void __launch_bounds__(256) k_split_h(Geo g, Coef<C> Kin, StepBufs<S> b) {
  const Coef<C> K = variant<kGen>(Kin);
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();

  S h[LH::Q], gv[L::Q];
  const Stencil<L, C> st(ad, b.PHI);
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) h[k] = ad.template pull_pop<LH>(b.H, k);
#pragma unroll
  for (int k = 0; k < L::Q; ++k) gv[k] = ad.template pull_pop<L>(b.G, k);
  loads_issued();
  double c = 0.0;
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) c = k == 0 ? double(h[k]) : c + double(h[k]);
  const C phi = st(0, 0, 0);
  const double mu_d = closure(K.q, c, double(phi));
  const C mu = C(mu_d);
  C gr[3], n[3];
  gradient_normal<L, C>(st, K.eps2, gr, n);
  const C sbar = source_moment<C>(K, phi, mu);

  double sg = 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) sg = k == 0 ? double(gv[k]) : sg + double(gv[k]);
  const double phin = sg + 0.5 * double(sbar);
  const C dtphi = C(phin) - phi;

  C F[3];
  h_flux<L, C>(K, mu, gr, n, dtphi, K.anti_trapping != 0, F);
  const C lam = h_lambda<C>(K, phi, mu);
  const C cc = C(c);
  C hs[LH::Q];
  h_update<LH>(K, h, cc, lam, F, hs);
  balance_rest<LH, S, C>(hs, c);
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) b.Hn[ad.slot(k, LH::Q)] = S(hs[k]);
  b.PHIn[i] = S(phin);
}

template <class L, class LH, class S, class C, bool kGen, class Addr>
__global__ void __launch_bounds__(256) k_split_g(Geo g, Coef<C> Kin, StepBufs<S> b) {
  const Coef<C> K = variant<kGen>(Kin);
  const Addr ad(g);
  if (!ad.inside()) return;

  S hv[LH::Q], gv[L::Q];
  const Stencil<L, C> st(ad, (const S*)b.PHIn);
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) hv[k] = ad.template pull_pop<LH>((const S*)b.Hn, k);
#pragma unroll
  for (int k = 0; k < L::Q; ++k) gv[k] = ad.template pull_pop<L>(b.G, k);
  loads_issued();
  double c = 0.0;
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) c = k == 0 ? double(hv[k]) : c + double(hv[k]);
  const C phi = st(0, 0, 0);
  const C mu = C(closure(K.q, c, double(phi)));
  C gr[3], n[3];
  gradient_normal<L, C>(st, K.eps2, gr, n);
  C G[L::Q];
  phi_sources<L, C>(K, phi, mu, n, G);
  C gs[L::Q];
  double sg = 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    sg = k == 0 ? double(gv[k]) : sg + double(gv[k]);
    gs[k] = C(S(g_collide<L, C>(K, k, C(gv[k]), phi, G[k])));
  }
  balance_g_rest<L, S, C>(K, gs, sg, phi, source_moment<C>(K, phi, mu));
#pragma unroll
  for (int k = 0; k < L::Q; ++k) b.Gn[ad.slot(k, L::Q)] = S(gs[k]);
}

// ---------------------------------------------------------------------------
// Initialisation: g~^0 = w_k phi0 - G^0_k / 2, h~^0 = h^eq_k - H^0_k / 2
// (no anti-trapping current), then the collision of g at time 0 so that the
// state satisfies the invariant of geometry.h at n = 0.  h~^0 is stored
// "unstreamed": each value goes to the slot the pull of the first step reads
// it from (the inverse of the pull permutation).

// Bound by its writes (512^3 FP64 41.9 GB, at 4.6 TB/s): non-temporal, since
// the state of a large grid outlives no cache (512^3 FP64 9.7 -> 9.0 ms, 320^3
// FP32 with h on D3Q7 1.22 -> 0.87 ms; regular stores 10.3 and 1.13), and
// addressed as in the step (64^3 FP32 with walls 19.5 -> 13.2 us).
template <class L, class LH, class S, class C, class Addr>
__global__ void __launch_bounds__(256) k_init(Geo g, Coef<C> K, const double* __restrict__ phi0,
                                              const double* __restrict__ c0, S* __restrict__ G,
                                              S* __restrict__ H, S* __restrict__ PHI) {
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();

  // the stencil reads phi0 converted to the arithmetic type
  const Stencil<L, C> st(ad, phi0);
  const double cin = c0[i];
  loads_issued();
  const C phi = st(0, 0, 0);
  C gr[3], n[3];
  gradient_normal<L, C>(st, K.eps2, gr, n);

  // initial populations from (phi0, c0)
  const C mu0 = C(closure(K.q, cin, double(phi)));
  C G0[L::Q];
  phi_sources<L, C>(K, phi, mu0, n, G0);
  C F[3];
  h_flux<L, C>(K, mu0, gr, n, C(0), false, F);
  const C lam = h_lambda<C>(K, phi, mu0);
  S hs[LH::Q];
  double c = 0.0;
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) {
    hs[k] = S(h_initial<LH, C>(K, k, C(cin), lam, F));
    c = k == 0 ? double(hs[k]) : c + double(hs[k]);
  }
  // collision of g at time 0 with c^0 = sum_k h~^0_k
  const C mu = C(closure(K.q, c, double(phi)));
  C Gk[L::Q];
  phi_sources<L, C>(K, phi, mu, n, Gk);
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    C g0 = S(C(L::w[k]) * phi - C(0.5) * G0[k]);
    __builtin_nontemporal_store(S(g_collide<L, C>(K, k, g0, phi, Gk[k])), &G[ad.slot(k, L::Q)]);
  }
  // h~^0 into the slots the first pull reads
#pragma unroll
  for (int k = 0; k < LH::Q; ++k)
    __builtin_nontemporal_store(hs[k], const_cast<S*>(ad.template source<LH>(
                                           (const S*)H, k, LH::Q, [](int j) { return j; })));
  PHI[i] = S(phi);
}

// ---------------------------------------------------------------------------
// Read-out of phi^n, c^n, mu^n as doubles.

template <class L, class S, class Addr>
__global__ void __launch_bounds__(256) k_fields(Geo g, ClosureK q, const S* __restrict__ H,
                                                const S* __restrict__ PHI, double* phi_out,
                                                double* c_out, double* mu_out) {
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  S hv[L::Q];
#pragma unroll
  for (int k = 0; k < L::Q; ++k) hv[k] = ad.template pull_pop<L>(H, k);
  const double phi = double(PHI[i]);
  loads_issued();
  double c = 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) c = k == 0 ? double(hv[k]) : c + double(hv[k]);
  if (phi_out) phi_out[i] = phi;
  if (c_out) c_out[i] = c;
  if (mu_out) mu_out[i] = closure(q, c, phi);
}

// ---------------------------------------------------------------------------
// Diagnostics: fixed-shape two-pass reduction in double, wavefront shuffles
// inside each block (deterministic: the association of every sum depends
// only on the launch shape).

constexpr int kDiagThreads = 256;
constexpr int kDiagBlocks = 1024;
constexpr int kDiagVals = 8;  // mass, solid, count, sum phi, min, max, nonfinite, spare
constexpr int kDiagWaves = kDiagThreads / 64;

// Combination of two partial diagnostics (sums, min, max, flag).
__device__ __forceinline__ void diag_combine(double* v, const double* u) {
  v[0] = v[0] + u[0];
  v[1] = v[1] + u[1];
  v[2] = v[2] + u[2];
  v[3] = v[3] + u[3];
  v[4] = fmin(v[4], u[4]);
  v[5] = fmax(v[5], u[5]);
  v[6] = fmax(v[6], u[6]);
}

// Block reduction of the per-thread partials: within each wavefront by
// shuffles with halving offsets (lane l takes lane l + off), then the
// wavefront results in wave order.  The association depends only on the
// launch shape, so the result is deterministic.  Thread 0 returns the total.
__device__ __forceinline__ void diag_block_reduce(double* v) {
  __shared__ double wred[kDiagWaves][kDiagVals];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    double u[kDiagVals];
#pragma unroll
    for (int j = 0; j < kDiagVals; ++j) u[j] = __shfl_down(v[j], off, 64);
    diag_combine(v, u);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < kDiagVals; ++j) wred[wave][j] = v[j];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kDiagWaves; ++w) diag_combine(v, wred[w]);
  }
}

// Coordinates of the nodes i, i + stride, ... a thread of the reduction
// visits: the stride as (dx, dy, dz), added with carries, in place of two
// 64-bit divisions per node (with the pulls in one batch: 256^3 FP64 725 ->
// 459 us, 512^3 FP16 4.23 -> 1.72 ms).
struct NodeWalk {
  int x, y, z, dx, dy, dz;
  __device__ NodeWalk(const Geo& g, int64_t i, int64_t stride) {
    x = int(i % g.nx);
    y = int((i / g.nx) % g.ny);
    z = int(i / ((int64_t)g.nx * g.ny));
    dx = int(stride % g.nx);
    dy = int((stride / g.nx) % g.ny);
    dz = int(stride / ((int64_t)g.nx * g.ny));
  }
  __device__ void next(const Geo& g) {
    x += dx;
    y += dy;
    z += dz;
    if (x >= g.nx) x -= g.nx, ++y;
    if (y >= g.ny) y -= g.ny, ++z;
  }
};

// One node's c and phi into the partial diagnostics.
__device__ __forceinline__ void diag_add(double* v, double c, double phi) {
  v[0] = v[0] + c;
  v[1] = v[1] + (1.0 - phi);
  v[2] = v[2] + (phi < 0.5 ? 1.0 : 0.0);
  v[3] = v[3] + phi;
  v[4] = fmin(v[4], phi);
  v[5] = fmax(v[5], phi);
  if (!isfinite(c) || !isfinite(phi)) v[6] = 1.0;
}

template <class L, class S, class Addr>
__global__ void __launch_bounds__(kDiagThreads) k_diag_partial(Geo g, const S* __restrict__ H,
                                                               const S* __restrict__ PHI,
                                                               double* __restrict__ part) {
  double v[kDiagVals] = {0.0, 0.0, 0.0, 0.0, INFINITY, -INFINITY, 0.0, 0.0};
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  NodeWalk w(g, i, stride);
  for (; i < g.N; i += stride, w.next(g)) {
    const Addr ad(g, w.x, w.y, w.z);
    S hv[L::Q];
#pragma unroll
    for (int k = 0; k < L::Q; ++k) hv[k] = ad.template pull_pop<L>(H, k);
    const double phi = double(PHI[i]);
    loads_issued();
    double c = 0.0;
#pragma unroll
    for (int k = 0; k < L::Q; ++k) c = k == 0 ? double(hv[k]) : c + double(hv[k]);
    diag_add(v, c, phi);
  }
  diag_block_reduce(v);
  if (threadIdx.x == 0)
    for (int j = 0; j < kDiagVals; ++j) part[blockIdx.x * kDiagVals + j] = v[j];
}

__global__ void __launch_bounds__(kDiagThreads) k_diag_final(const double* __restrict__ part,
                                                             int nblocks, double* __restrict__ out) {
  double v[kDiagVals] = {0.0, 0.0, 0.0, 0.0, INFINITY, -INFINITY, 0.0, 0.0};
  for (int b = threadIdx.x; b < nblocks; b += kDiagThreads) {
    const double* p = part + b * kDiagVals;
    v[0] = v[0] + p[0];
    v[1] = v[1] + p[1];
    v[2] = v[2] + p[2];
    v[3] = v[3] + p[3];
    v[4] = fmin(v[4], p[4]);
    v[5] = fmax(v[5], p[5]);
    v[6] = fmax(v[6], p[6]);
  }
  diag_block_reduce(v);
  if (threadIdx.x == 0)
    for (int j = 0; j < kDiagVals; ++j) out[j] = v[j];
}

}  // namespace gplbm
