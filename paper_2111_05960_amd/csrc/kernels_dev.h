// Reduced-precision storage of the state on any lattice: the Q - 1 moving
// populations of each distribution are stored as FP16 or BF16 deviations from the local
// equilibrium of the node that wrote them, the rest populations, phi and
// Lambda = gamma D(phi) mu as FP32.  Collision arithmetic is FP32; the moments
// (c, phi) and the closure mu(c, phi) are FP64.
//
//   g: stored delta_k = S (g*_k - w_k phi(y))     (phi of the writing node y)
//   h: stored delta_k = S (h*_k - w_k Lambda(y))  (Lambda of the writing node)
// with S = 2^12 for FP16 (keeps the small deviations in the normal range) and
// S = 1 for BF16; rounding is round-to-nearest-even.  A reader decodes
// f = ref + delta / S with the reference of the source node, which is
// available to it (phi and Lambda are fields of the state).
//
// Solute mass: the writer sets the rest population of h so that the decoded
// populations it leaves behind sum exactly (in FP64, then one FP32 rounding)
// to the c it received - the collision conserves c exactly in arithmetic, so
// this only removes the rounding of the 16-bit encodings from the balance.
//
// Layout of one distribution: moving populations u16[z][m][y][x] (m = k
// before the rest vector, k - 1 after it), then the rest populations
// f32[z][y][x].  Every kernel takes the lattices of g and h as template
// arguments.
#pragma once

#include "kernels_fused3d.h"

namespace gplbm {

struct F16Codec {
  static constexpr float kScale = 4096.0f, kInv = 1.0f / 4096.0f;
  __device__ static uint16_t enc(float v, float ref) {
    return __builtin_bit_cast(uint16_t, (_Float16)((v - ref) * kScale));
  }
  // r (ref + delta / S), r a power of two: one mixed-precision multiply-add
  __device__ static float dec(uint16_t u, float ref, float r) {
    return __builtin_fmaf((float)__builtin_bit_cast(_Float16, u), kInv * r, ref);
  }
};
struct BF16Codec {
  static constexpr float kScale = 1.0f, kInv = 1.0f;
  __device__ static uint16_t enc(float v, float ref) {
    return __builtin_bit_cast(uint16_t, (__bf16)(v - ref));
  }
  __device__ static float dec(uint16_t u, float ref, float r) {
    return __builtin_fmaf((float)__builtin_bit_cast(__bf16, u), r, ref);
  }
};

// one distribution in the deviation format
struct DevDist {
  uint16_t* mov;
  float* rest;
};
struct DevState {
  DevDist G, H;
  float* PHI;
  float* LAM;
};
struct DevStep {
  DevState cur;  // G = g~*^n, H = h~*^{n-1}, PHI = phi^n, LAM = Lambda^{n-1}
  DevState nxt;  // written: G = g~*^{n+1}, H = h~*^n, PHI = phi^{n+1}, LAM = Lambda^n
};

constexpr int kMov = 18;  // the most moving populations per node (D3Q19)

// slot of moving population k among the Q - 1 of lattice L
template <class L>
__device__ __forceinline__ constexpr int mslot(int k) { return k < L::REST ? k : k - 1; }

// opposite populations share a weight (a bounced code decodes with w_k)
template <class L>
constexpr bool symmetric_weights() {
  for (int k = 0; k < L::Q; ++k)
    if (L::w[k] != L::w[L::opp[k]]) return false;
  return true;
}
static_assert(symmetric_weights<D3Q19>() && symmetric_weights<D3Q7>() &&
              symmetric_weights<D2Q9>() && symmetric_weights<D2Q5>(), "w_opp(k) = w_k");

// slot of plane q in a ring of four planes (q >= -8)
__device__ __forceinline__ int ring4(int q) { return (q + 8) & 3; }

template <class L>
__device__ __forceinline__ int64_t mov_index(const Geo& g, int k, int x, int y, int z) {
  const int64_t plane = (int64_t)g.nx * g.ny;
  return ((int64_t)z * (L::Q - 1) + mslot<L>(k)) * plane + (int64_t)y * g.nx + x;
}

template <class Codec>
__device__ __forceinline__ float dev_decode(uint16_t raw, float ref) {
  return Codec::dec(raw, ref, 1.0f);
}
template <class Codec>
__device__ __forceinline__ uint16_t dev_encode(float v, float ref) {
  return Codec::enc(v, ref);
}

// The moving weights of every lattice are powers of two apart, so a tile may
// hold the reference field times the smallest of them, w_min: the value of
// population k is then w_k / w_min times a sum with that one operand, exactly
// the sum with w_k ref (while w_min ref is a normal number; below 1.2e-38 the
// two may differ by a step of the subnormal numbers, 1.4e-45, which neither c
// nor a 16-bit code of normal size holds).
template <class L>
constexpr double min_weight() {
  double w = 1.0;
  for (int k = 0; k < L::Q; ++k)
    if (k != L::REST && L::w[k] < w) w = L::w[k];
  return w;
}
template <class L>
constexpr int weight_ratio(int k) {
  return int(L::w[k] / min_weight<L>() + 0.5);
}
template <class L>
constexpr bool weights_scale() {
  for (int k = 0; k < L::Q; ++k) {
    const int r = weight_ratio<L>(k);
    if (k != L::REST && ((r & (r - 1)) || float(L::w[k]) != r * float(min_weight<L>())))
      return false;
  }
  return true;
}
static_assert(weights_scale<D3Q19>() && weights_scale<D3Q7>() && weights_scale<D2Q9>() &&
              weights_scale<D2Q5>(), "moving weights are w_min times powers of two");

// Value of population k from its code and wref = w_min times the reference
// field of the node that wrote it.
template <class Codec, class L>
__device__ __forceinline__ float dev_decode_wmin(int k, uint16_t raw, float wref) {
  const int r = weight_ratio<L>(k);
  const float v = Codec::dec(raw, wref, 1.0f / r);
  return r == 1 ? v : r * v;
}

// Encode the post-collision h of one node with the mass balance of the rest
// population; hdec receives the decoded values (what readers will see).
template <class Codec, class L>
__device__ __forceinline__ void encode_h(const float hs[L::Q], float lam, double c_in,
                                         uint16_t enc[L::Q], float hdec[L::Q]) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    if (k == L::REST) continue;
    const float ref = float(L::w[k]) * lam;
    enc[k] = dev_encode<Codec>(hs[k], ref);
    hdec[k] = dev_decode<Codec>(enc[k], ref);
    s = s + double(hdec[k]);
  }
  hdec[L::REST] = float(c_in - s);
}

template <class Codec, class L>
__device__ __forceinline__ void encode_g(const float gs[L::Q], float phi, uint16_t enc[L::Q],
                                         float gdec[L::Q]) {
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    if (k == L::REST) {
      gdec[k] = gs[k];
      continue;
    }
    const float ref = float(L::w[k]) * phi;
    enc[k] = dev_encode<Codec>(gs[k], ref);
    gdec[k] = dev_decode<Codec>(enc[k], ref);
  }
}

// ---------------------------------------------------------------------------
// Initialisation: first Lambda^0 and phi^0 as FP32 fields, then the
// populations (h~^0 scattered to the slots the first pull reads, encoded with
// the reference of the slot's node).

__global__ void __launch_bounds__(256) k_dev_init_fields(Geo g, Coef<float> K,
                                                         const double* __restrict__ phi0,
                                                         const double* __restrict__ c0,
                                                         DevState s) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < g.N;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float phi = float(phi0[i]);
    const float mu0 = float(closure(K.q, c0[i], double(phi)));
    s.PHI[i] = phi;
    s.LAM[i] = h_lambda<float>(K, phi, mu0);
  }
}

// (Addressed as in the step: 250x230x190 with walls 726 -> 443 us, 512^3 8.5 ->
// 5.0 ms; the read-out 315 -> 169 us, 3.5 -> 1.9 ms.)
template <class Codec, class L, class LH, class Addr>
__global__ void __launch_bounds__(256) k_dev_init(Geo g, Coef<float> K,
                                                  const double* __restrict__ c0, DevState s) {
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  const Stencil<L, float> st(ad, (const float*)s.PHI);
  const Stencil<LH, float> sl(ad, (const float*)s.LAM);
  const double cin = c0[i];
  loads_issued();
  const float phi = st(0, 0, 0);
  float gr[3], n[3];
  gradient_normal<L, float>(st, K.eps2, gr, n);
  const float mu0 = float(closure(K.q, cin, double(phi)));
  float G0[L::Q];
  phi_sources<L, float>(K, phi, mu0, n, G0);
  float F[3];
  h_flux<L, float>(K, mu0, gr, n, 0.0f, false, F);
  const float lam = sl(0, 0, 0);
  // h~^0, encoded for the slot (x - e_k, k) or (x, opp k) at a wall
  double c = 0.0;
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) {
    const float hv = h_initial<LH, float>(K, k, float(cin), lam, F);
    float dec;
    if (k == LH::REST) {
      s.H.rest[i] = hv;
      dec = hv;
    } else {
      const float in = sl(-LH::ex[k], -LH::ey[k], -LH::ez[k]);
      const float ref = float(LH::w[k]) * (ad.template bounced<LH>(k) ? lam : in);
      const uint16_t e = dev_encode<Codec>(hv, ref);
      *const_cast<uint16_t*>(ad.template source<LH>((const uint16_t*)s.H.mov, k, LH::Q - 1,
                                                    [](int j) { return mslot<LH>(j); })) = e;
      dec = dev_decode<Codec>(e, ref);
    }
    c = k == 0 ? double(dec) : c + double(dec);
  }
  // collision of g at time 0 with c^0 = sum of the decoded h~^0
  const float mu = float(closure(K.q, c, double(phi)));
  float Gk[L::Q], gs[L::Q];
  phi_sources<L, float>(K, phi, mu, n, Gk);
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    const float g0 = float(L::w[k]) * phi - 0.5f * G0[k];
    gs[k] = g_collide<L, float>(K, k, g0, phi, Gk[k]);
  }
  uint16_t enc[L::Q];
  float gdec[L::Q];
  encode_g<Codec, L>(gs, phi, enc, gdec);
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    if (k == L::REST)
      s.G.rest[i] = gdec[k];
    else
      s.G.mov[ad.slot(mslot<L>(k), L::Q - 1)] = enc[k];
  }
}

// ---------------------------------------------------------------------------
// Split schedule in the deviation format (any boundaries).

// Codes of the moving populations a node pulls from a distribution, and the
// rest value, as one batch of loads; then the decoded values, given the
// reference field on the node's stencil (own value for a bounced population).
template <class L>
struct DevPulls {
  uint16_t code[L::Q];
  float rest;
  template <class A>
  __device__ DevPulls(const A& a, const DevDist& d) : rest(d.rest[a.node()]) {
#pragma unroll
    for (int k = 0; k < L::Q; ++k)
      code[k] = k == L::REST ? uint16_t(0)
                             : *a.template source<L>((const uint16_t*)d.mov, k, L::Q - 1,
                                                     [](int j) { return mslot<L>(j); });
  }
  template <class Codec, class A, class R>
  __device__ float value(const A& a, const R& ref, int k) const {
    if (k == L::REST) return rest;
    const float in = ref(-L::ex[k], -L::ey[k], -L::ez[k]);
    return dev_decode<Codec>(code[k],
                             float(L::w[k]) * (a.template bounced<L>(k) ? ref(0, 0, 0) : in));
  }
};

template <class Codec, class L, class LH, class Addr>
__global__ void __launch_bounds__(256) k_dev_split_h(Geo g, Coef<float> K, DevStep b) {
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  const Stencil<L, float> st(ad, (const float*)b.cur.PHI);
  const Stencil<LH, float> sl(ad, (const float*)b.cur.LAM);
  const DevPulls<LH> ph(ad, b.cur.H);
  const DevPulls<L> pg(ad, b.cur.G);
  loads_issued();
  float h[LH::Q];
  double c = 0.0;
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) {
    h[k] = ph.template value<Codec>(ad, sl, k);
    c = k == 0 ? double(h[k]) : c + double(h[k]);
  }
  const float phi = st(0, 0, 0);
  const float mu = float(closure(K.q, c, double(phi)));
  float gr[3], n[3];
  gradient_normal<L, float>(st, K.eps2, gr, n);
  const float sbar = source_moment<float>(K, phi, mu);
  double sg = 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    const double v = double(pg.template value<Codec>(ad, st, k));
    sg = k == 0 ? v : sg + v;
  }
  const float phin = float(sg + 0.5 * double(sbar));
  float F[3];
  h_flux<L, float>(K, mu, gr, n, phin - phi, K.anti_trapping != 0, F);
  const float lam = h_lambda<float>(K, phi, mu);
  const float cc = float(c);
  float hs[LH::Q];
  h_update<LH>(K, h, cc, lam, F, hs);
  uint16_t enc[LH::Q];
  float hdec[LH::Q];
  encode_h<Codec, LH>(hs, lam, c, enc, hdec);
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) {
    if (k == LH::REST)
      b.nxt.H.rest[i] = hdec[k];
    else
      b.nxt.H.mov[ad.slot(mslot<LH>(k), LH::Q - 1)] = enc[k];
  }
  b.nxt.LAM[i] = lam;
  b.nxt.PHI[i] = phin;
}

template <class Codec, class L, class LH, class Addr>
__global__ void __launch_bounds__(256) k_dev_split_g(Geo g, Coef<float> K, DevStep b) {
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  // g decodes with phi^n, the gradient is that of phi^{n+1}
  const Stencil<L, float> st(ad, (const float*)b.nxt.PHI), s0(ad, (const float*)b.cur.PHI);
  const Stencil<LH, float> sl(ad, (const float*)b.nxt.LAM);
  const DevPulls<LH> ph(ad, b.nxt.H);
  const DevPulls<L> pg(ad, b.cur.G);
  loads_issued();
  double c = 0.0;
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) {
    const double v = double(ph.template value<Codec>(ad, sl, k));
    c = k == 0 ? v : c + v;
  }
  const float phi = st(0, 0, 0);
  const float mu = float(closure(K.q, c, double(phi)));
  float gr[3], n[3];
  gradient_normal<L, float>(st, K.eps2, gr, n);
  float G[L::Q], gs[L::Q];
  phi_sources<L, float>(K, phi, mu, n, G);
  double sg = 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    const float gk = pg.template value<Codec>(ad, s0, k);
    sg = k == 0 ? double(gk) : sg + double(gk);
    gs[k] = g_collide<L, float>(K, k, gk, phi, G[k]);
  }
  uint16_t enc[L::Q];
  float gdec[L::Q];
  encode_g<Codec, L>(gs, phi, enc, gdec);
  balance_g_rest<L, float, float>(K, gdec, sg, phi, source_moment<float>(K, phi, mu));
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    if (k == L::REST)
      b.nxt.G.rest[i] = gdec[k];
    else
      b.nxt.G.mov[ad.slot(mslot<L>(k), L::Q - 1)] = enc[k];
  }
}

// read-out and diagnostics in the deviation format
template <class Codec, class L, class Addr>
__global__ void __launch_bounds__(256) k_dev_fields(Geo g, ClosureK q, DevState s,
                                                    double* phi_out, double* c_out,
                                                    double* mu_out) {
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  const Stencil<L, float> sl(ad, (const float*)s.LAM);
  const DevPulls<L> ph(ad, s.H);
  const double phi = double(s.PHI[i]);
  loads_issued();
  double c = 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    const double v = double(ph.template value<Codec>(ad, sl, k));
    c = k == 0 ? v : c + v;
  }
  if (phi_out) phi_out[i] = phi;
  if (c_out) c_out[i] = c;
  if (mu_out) mu_out[i] = closure(q, c, phi);
}

template <class Codec, class L, class Addr>
__global__ void __launch_bounds__(kDiagThreads) k_dev_diag_partial(Geo g, DevState s,
                                                                   double* __restrict__ part) {
  double v[kDiagVals] = {0.0, 0.0, 0.0, 0.0, INFINITY, -INFINITY, 0.0, 0.0};
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  NodeWalk w(g, i, stride);
  for (; i < g.N; i += stride, w.next(g)) {
    const Addr ad(g, w.x, w.y, w.z);
    const Stencil<L, float> sl(ad, (const float*)s.LAM);
    const DevPulls<L> ph(ad, s.H);
    const double phi = double(s.PHI[i]);
    loads_issued();
    double c = 0.0;
#pragma unroll
    for (int k = 0; k < L::Q; ++k) {
      const double hv = double(ph.template value<Codec>(ad, sl, k));
      c = k == 0 ? hv : c + hv;
    }
    diag_add(v, c, phi);
  }
  diag_block_reduce(v);
  if (threadIdx.x == 0)
    for (int j = 0; j < kDiagVals; ++j) part[blockIdx.x * kDiagVals + j] = v[j];
}

// ---------------------------------------------------------------------------
// output rows per tile of the fused deviation kernel (64 x 13 outputs, 1024
// threads at 4 waves per SIMD)
#ifndef GPLBM_DEV_TY
#define GPLBM_DEV_TY 13
#endif

// Fused z-marching schedule in the deviation format, periodic or with
// zero-flux walls.  Same structure as k_fused3d (x-aligned tiles, persistent
// grid, g carry in registers); in addition an LDS ring holds Lambda^{n-1} on
// T+2 for the h references, and the phi^n ring serves the g references.
//
// Walls (kWalls, any axis): a pull whose source lies beyond a wall reads the
// node's own opposite population, decoded with the node's own reference; the
// T+2 tiles are loaded with clamped coordinates (the mirror ghost of the
// gradient); the phi^{n+1} stencil of the g collision takes mirrored offsets;
// and the in-block h streaming keeps the index order of the pull sum: a node
// gathers the e_z = +1 layer of its c^{n+1} at its own plane, from the
// exchange of the plane below (kept one plane longer) or its own bounced
// values, takes the bounced e_z = -1 values from its own entries in that
// exchange, and a closing plane past a top wall finishes the last plane.

__device__ __forceinline__ uint16_t bload16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(uint16_t, __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0));
}
__device__ __forceinline__ void bstore16_nt(uint16_t v, __amdgpu_buffer_rsrc_t r, uint32_t voff,
                                            uint32_t soff) {
  using V = decltype(__builtin_amdgcn_raw_buffer_load_b16(r, 0, 0, 0));
  __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(V, v), r, voff, soff, 2);
}

template <int TX, int TY, class Codec, class LG, class LH, bool kGen, bool kWalls>
__global__ void __launch_bounds__((TileShape<TX, TY>::NT))
    k_dev_fused3d(Geo g, Coef<float> Kin, DevStep b, int tiles_x, int tiles_xy, int ntiles, int zc) {
  const Coef<float> K = variant<kGen>(Kin);
  using Shape = TileShape<TX, TY>;
  constexpr int Q = LG::Q;  // g lattice (D3Q19 or D3Q7)
  constexpr int BX = Shape::BX, BY = Shape::BY;
  constexpr int AX = BX + 2, AY = BY + 2;
  constexpr int NT = Shape::NT;
  constexpr int TILE_PER_THREAD = (AX * AY + NT - 1) / NT;
  // Rings of four planes and a double-buffered exchange, so that one barrier
  // per plane orders every LDS access: the tile of plane p + 2 is loaded, and
  // the next plane's exchange written, while other waves still read the
  // planes of p (see the hazards noted at the barrier).
  __shared__ float phiA[4][AY][AX];          // phi^n, planes p-1 .. p+2
  __shared__ float lamA[4][AY][AX];          // w_min Lambda^{n-1}, planes p-1 .. p+2
  __shared__ float phiB[4][BY][BX];          // phi^{n+1}, planes p-3 .. p
  constexpr int QH = LH::Q;  // h lattice (D3Q19 or D3Q7)
  constexpr float kWmin = float(min_weight<LH>());
  // e_z layers of the h lattice: +1 at [0, NU), 0 at [NU, NU + NM), -1 after
  constexpr int NU = count_ez<LH>(1), NM = count_ez<LH>(0);
  // Exchange of plane p: the 16-bit codes of the moving h*^n and w_min
  // Lambda^n, their reference.  Periodic: every moving population in hxe and Lambda in
  // hxl, by plane parity.  Walls: the e_z = +1 layer in hxu and Lambda in hxl
  // by plane modulo 3 (the plane above gathers that layer after its own
  // barrier, and a node's own entries there are the bounce of its e_z = -1
  // populations: with one barrier per plane a buffer is rewritten two planes
  // after it was read), the other moving populations in hxe by parity.
  static_assert(!kWalls || LH::REST == NU, "the rest vector opens the in-plane layer");
  constexpr int NXE = kWalls ? QH - 1 - NU : QH - 1;
  __shared__ uint16_t hxe[2][NXE][BY][BX];
  __shared__ uint16_t hxu[kWalls ? 3 : 1][kWalls ? NU : 1][kWalls ? BY : 1][kWalls ? BX : 1];
  __shared__ float hxl[kWalls ? 3 : 2][BY][BX];

  int tx, ty;
  bool valid;
  Shape::node(threadIdx.x, tx, ty, valid);
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int plane = nx * ny;
  const uint32_t planeB = uint32_t(plane) * 2u;            // one 16-bit population plane
  const int64_t groupB = int64_t(plane) * (Q - 1) * 2;        // one z group of moving g populations
  const int64_t groupBH = int64_t(plane) * (QH - 1) * 2;   // one z group of moving h populations
  const bool wz = kWalls && g.bcz;

  for (int tile = first_tile(); tile < ntiles; tile += gridDim.x) {
  const int chunk = tile / tiles_xy, txy = tile % tiles_xy;
  const int X0 = tile_column(txy, tiles_x, chunk, kWalls) * TX, Y0 = (txy / tiles_x) * TY;
  const int z0 = chunk * zc, z1 = min(z0 + zc, nz);
  const int ux = X0 - 1 + tx, uy = Y0 - 1 + ty;
  const bool out = valid && ux < nx && uy < ny && tx >= 1 && tx <= TX && ty >= 1 && ty <= TY;
  // region nodes beyond a wall take no part (with walls only)
  bool active = valid;
  if constexpr (kWalls)
    active = valid && (!g.bcx || (ux >= 0 && ux < nx)) && (!g.bcy || (uy >= 0 && uy < ny));
  const int x = kWalls ? tile_coord(ux, nx, g.bcx) : wrap_near(ux, nx);
  const int y = kWalls ? tile_coord(uy, ny, g.bcy) : wrap_near(uy, ny);
  // source offsets wrap also on wall axes: a source beyond a wall is never
  // read (its population bounces), the wrapped address only keeps it in range
  const int xo[3] = {x == 0 ? nx - 1 : x - 1, x, x == nx - 1 ? 0 : x + 1};
  const int yo[3] = {(y == 0 ? ny - 1 : y - 1) * nx, y * nx, (y == ny - 1 ? 0 : y + 1) * nx};
  uint32_t xyb[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) xyb[a][c] = uint32_t(yo[a] + xo[c]) * 2u;
  const uint32_t selfB = xyb[1][1];
  const int self_xy = y * nx + x;
  // populations arriving from beyond an x or y wall (bit k), and the mirror
  // offsets of the phi^{n+1} stencil
  uint32_t bmh = 0, bmg = 0;
  int xm = -1, xp = 1, ym = -1, yp = 1;
  if constexpr (kWalls) {
    bmh = xy_bounce_mask<LH>(g, ux, uy);
    bmg = xy_bounce_mask<LG>(g, ux, uy);
    xm = (g.bcx && ux == 0) ? 0 : -1;
    xp = (g.bcx && ux == nx - 1) ? 0 : 1;
    ym = (g.bcy && uy == 0) ? 0 : -1;
    yp = (g.bcy && uy == ny - 1) ? 0 : 1;
  }

  // tile positions this thread loads (T+2 in x-y; clamped along wall axes, the
  // mirror ghost): byte offset in a plane of PHI / LAM and slot in a ring plane
  uint32_t tile_off[TILE_PER_THREAD];
#pragma unroll
  for (int j = 0; j < TILE_PER_THREAD; ++j) {
    const int l = min((int)threadIdx.x + j * NT, AX * AY - 1);
    const int vx = X0 - 2 + l % AX, vy = Y0 - 2 + l / AX;
    const int gx = kWalls ? tile_coord(vx, nx, g.bcx) : wrap_near(vx, nx);
    const int gy = kWalls ? tile_coord(vy, ny, g.bcy) : wrap_near(vy, ny);
    tile_off[j] = uint32_t(gy * nx + gx) * 4u;
  }
  float tile_phi[TILE_PER_THREAD], tile_lam[TILE_PER_THREAD];
  auto fetch_tiles = [&](int p) {
    const int64_t zoff = (int64_t)(kWalls ? tile_coord(p, nz, g.bcz) : wrap_coord(p, nz)) * plane;
    const auto P = make_rsrc(b.cur.PHI + zoff, uint32_t(plane) * 4u);
    const auto Lm = make_rsrc(b.cur.LAM + zoff, uint32_t(plane) * 4u);
#pragma unroll
    for (int j = 0; j < TILE_PER_THREAD; ++j) {
      tile_phi[j] = bload<float>(P, tile_off[j], 0);
      tile_lam[j] = bload<float>(Lm, tile_off[j], 0);
    }
  };
  auto store_tiles = [&](int p) {
    float* const pa = &phiA[ring4(p)][0][0];
    float* const la = &lamA[ring4(p)][0][0];
#pragma unroll
    for (int j = 0; j < TILE_PER_THREAD; ++j) {
      const int l = threadIdx.x + j * NT;
      if ((j + 1) * NT <= AX * AY || l < AX * AY) {
        pa[l] = tile_phi[j];
        la[l] = kWmin * tile_lam[j];
      }
    }
  };
  auto load_tiles = [&](int p) {
    fetch_tiles(p);
    store_tiles(p);
  };
  // Fetching ahead (periodic D3Q7 h): the tiles of p + 3 and the h codes of p
  // + 1 are loaded behind the barrier of plane p, while g collides, instead of
  // right before their use.  512^3 FP16: D3Q7 3.21 -> 2.98 ms, D3Q19 g with
  // D3Q7 h 4.84 -> 4.72; 256^3: 0.434 -> 0.402 and 0.655 -> 0.638.  With 19 h
  // populations, or a general coupling on D3Q19, the registers are full, and
  // it costs more in spills than the latency it hides: 6.78 -> 7.15 ms.
  constexpr bool kAhead = QH == 7 && !kWalls && !(kGen && Q == 19);
  uint16_t h_ahead[kAhead ? QH : 1];
  auto fetch_h = [&](int p) {
    const int zp = wrap_coord(p, nz);
    const int zo[3] = {zp == 0 ? nz - 1 : zp - 1, zp, zp == nz - 1 ? 0 : zp + 1};
    __amdgpu_buffer_rsrc_t Hz[3];
#pragma unroll
    for (int j = 0; j < 3; ++j)
      Hz[j] = make_rsrc(reinterpret_cast<const char*>(b.cur.H.mov) + zo[j] * groupBH, uint32_t(groupBH));
#pragma unroll
    for (int k = 0; k < QH; ++k)
      h_ahead[kAhead ? k : 0] =
          k == LH::REST ? uint16_t(0)
                        : bload16(Hz[1 - LH::ez[k]], xyb[1 - LH::ey[k]][1 - LH::ex[k]],
                                  mslot<LH>(k) * planeB);
  };
  // first plane: the halo plane below the chunk, or the bottom plane at a z wall
  const int pfirst = (wz && z0 == 0) ? 0 : z0 - 1;
  load_tiles(pfirst - 1);
  load_tiles(pfirst);
  load_tiles(pfirst + 1);
  if constexpr (kAhead) {
    load_tiles(pfirst + 2);
    fetch_h(pfirst);
  }
  __syncthreads();

  float g_old[Q];
#pragma unroll
  for (int k = 0; k < Q; ++k) g_old[k] = 0.0f;
  // c^{n+1} of this thread's node on planes p - 1 and p, partly summed: the
  // e_z = +1 populations arrive one plane early, the e_z = -1 ones one plane
  // late, each group gathered in ascending k
  const bool inner = valid && tx >= 1 && tx <= TX && ty >= 1 && ty <= TY;
  double acc_dn = 0.0, acc_mid = 0.0, sg_old = 0.0;

  for (int p = pfirst; p <= z1; ++p) {
    // past a top wall: no plane, only the completion of plane nz - 1
    const bool closing = wz && p == nz;
    const int zp = wz ? min(p, nz - 1) : wrap_coord(p, nz);
    int zo[3];
    if (wz) {
      // a plane beyond the wall is never read (its populations bounce)
      zo[0] = max(zp - 1, 0);
      zo[1] = zp;
      zo[2] = min(zp + 1, nz - 1);
    } else {
      zo[0] = zp == 0 ? nz - 1 : zp - 1;
      zo[1] = zp;
      zo[2] = zp == nz - 1 ? 0 : zp + 1;
    }
    // all e_z = +1 (-1) sources of this plane lie beyond the bottom (top) wall
    const bool bz_up = wz && p == 0, bz_dn = wz && p == nz - 1;
    __amdgpu_buffer_rsrc_t Hz[3], Gz[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      Hz[j] = make_rsrc(reinterpret_cast<const char*>(b.cur.H.mov) + zo[j] * groupBH, uint32_t(groupBH));
      Gz[j] = make_rsrc(reinterpret_cast<const char*>(b.cur.G.mov) + zo[j] * groupB, uint32_t(groupB));
    }
    const int64_t selfnode = (int64_t)zp * plane + self_xy;
    const int sA = ring4(p);

    float g_new[Q];
    double sg = 0.0;
    float hdec[QH];
    float phin = 0.0f, lam = 0.0f;
    uint16_t enc[QH];
    if (!kWalls || (active && !closing)) {
      // pulls, decoded with the reference of the source node (LDS tiles), or
      // of the node itself for a population bounced back at a wall
      float h[QH];
      double c = 0.0;
      // populations bounced at a wall (bits k); a wavefront with none (all but
      // those of the tiles at a wall) takes the plain pulls
      uint32_t bh = 0u, bg = 0u;
      bool plain = true;
      if constexpr (kWalls) {
        bh = bmh | (bz_up ? ez_mask<LH>(1) : 0u) | (bz_dn ? ez_mask<LH>(-1) : 0u);
        bg = bmg | (bz_up ? ez_mask<LG>(1) : 0u) | (bz_dn ? ez_mask<LG>(-1) : 0u);
        plain = __builtin_amdgcn_ballot_w64((bh | bg) != 0u) == 0u;
      }
      if (!plain) {
        // Every pull first reads its neighbour (a wrapped address where x -
        // e_k lies beyond a wall: read, never used), then a lane with bounced
        // populations replaces those codes by its own opposite ones, and each
        // code decodes against the reference of the node that wrote it
        // (w_opp(k) = w_k): one batch of loads and no branch per population
        uint16_t ch[QH], cg[Q];
#pragma unroll
        for (int k = 0; k < QH; ++k)
          ch[k] = k == LH::REST ? uint16_t(0)
                                : bload16(Hz[1 - LH::ez[k]], xyb[1 - LH::ey[k]][1 - LH::ex[k]],
                                          mslot<LH>(k) * planeB);
#pragma unroll
        for (int k = 0; k < Q; ++k)
          cg[k] = k == LG::REST ? uint16_t(0)
                                : bload16(Gz[1 - LG::ez[k]], xyb[1 - LG::ey[k]][1 - LG::ex[k]],
                                          mslot<LG>(k) * planeB);
        if ((bh | bg) != 0u) {
#pragma unroll
          for (int k = 0; k < QH; ++k)
            if (k != LH::REST && ((bh >> k) & 1u))
              ch[k] = bload16(Hz[1], selfB, mslot<LH>(LH::opp[k]) * planeB);
#pragma unroll
          for (int k = 0; k < Q; ++k)
            if (k != LG::REST && ((bg >> k) & 1u))
              cg[k] = bload16(Gz[1], selfB, mslot<LG>(LG::opp[k]) * planeB);
        }
        const float lam_own = lamA[sA][ty + 1][tx + 1], phi_own = phiA[sA][ty + 1][tx + 1];
#pragma unroll
        for (int k = 0; k < QH; ++k) {
          float v;
          if (k == LH::REST) {
            v = b.cur.H.rest[selfnode];
          } else {
            const float src = lamA[ring4(p - LH::ez[k])][ty + 1 - LH::ey[k]][tx + 1 - LH::ex[k]];
            v = dev_decode_wmin<Codec, LH>(k, ch[k], ((bh >> k) & 1u) ? lam_own : src);
          }
          h[k] = v;
          c = k == 0 ? double(v) : c + double(v);
        }
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          float v;
          if (k == LG::REST) {
            v = b.cur.G.rest[selfnode];
          } else {
            const float src = phiA[ring4(p - LG::ez[k])][ty + 1 - LG::ey[k]][tx + 1 - LG::ex[k]];
            v = dev_decode<Codec>(cg[k], float(LG::w[k]) * (((bg >> k) & 1u) ? phi_own : src));
          }
          g_new[k] = v;
          sg = k == 0 ? double(v) : sg + double(v);
        }
      } else {
        // every pull in one batch before the first decode: left to itself the
        // scheduler may interleave loads and decodes, and the wave then waits
        // for memory once per population
        uint16_t ch[QH], cg[Q];
        const float h_rest = b.cur.H.rest[selfnode], g_rest = b.cur.G.rest[selfnode];
#pragma unroll
        for (int k = 0; k < QH; ++k) {
          if constexpr (kAhead)
            ch[k] = h_ahead[k];
          else
            ch[k] = k == LH::REST ? uint16_t(0)
                                  : bload16(Hz[1 - LH::ez[k]], xyb[1 - LH::ey[k]][1 - LH::ex[k]],
                                            mslot<LH>(k) * planeB);
        }
#pragma unroll
        for (int k = 0; k < Q; ++k)
          cg[k] = k == LG::REST ? uint16_t(0)
                                : bload16(Gz[1 - LG::ez[k]], xyb[1 - LG::ey[k]][1 - LG::ex[k]],
                                          mslot<LG>(k) * planeB);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < QH; ++k) {
          float v = h_rest;
          if (k != LH::REST)
            v = dev_decode_wmin<Codec, LH>(
                k, ch[k], lamA[ring4(p - LH::ez[k])][ty + 1 - LH::ey[k]][tx + 1 - LH::ex[k]]);
          h[k] = v;
          c = k == 0 ? double(v) : c + double(v);
        }
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          float v = g_rest;
          if (k != LG::REST)
            v = dev_decode<Codec>(cg[k], float(LG::w[k]) * phiA[ring4(p - LG::ez[k])]
                                                               [ty + 1 - LG::ey[k]][tx + 1 - LG::ex[k]]);
          g_new[k] = v;
          sg = k == 0 ? double(v) : sg + double(v);
        }
      }
      const float phi = phiA[sA][ty + 1][tx + 1];
      const float mu = float(closure(K.q, c, double(phi)));
      auto atA = [&](int dx, int dy, int dz) -> float {
        return phiA[ring4(p + dz)][ty + 1 + dy][tx + 1 + dx];
      };
      float gr[3], n[3];
      gradient_normal<LG, float>(atA, K.eps2, gr, n);
      const float sbar = source_moment<float>(K, phi, mu);
      phin = float(sg + 0.5 * double(sbar));
      float F[3];
      h_flux<LG, float>(K, mu, gr, n, phin - phi, K.anti_trapping != 0, F);
      lam = h_lambda<float>(K, phi, mu);
      const float cc = float(c);
      float hs[QH];
      h_update<LH>(K, h, cc, lam, F, hs);
      encode_h<Codec, LH>(hs, lam, c, enc, hdec);
    }
    if (active && !closing) phiB[sA][ty][tx] = phin;

    const bool own_p = p >= z0 && p < z1;
    if (out && own_p) {
      const auto Hw = make_rsrc(reinterpret_cast<char*>(b.nxt.H.mov) + zp * groupBH, uint32_t(groupBH));
#pragma unroll
      for (int k = 0; k < QH; ++k)
        if (k != LH::REST) bstore16_nt(enc[k], Hw, selfB, mslot<LH>(k) * planeB);
      __builtin_nontemporal_store(hdec[LH::REST], &b.nxt.H.rest[selfnode]);
      __builtin_nontemporal_store(lam, &b.nxt.LAM[selfnode]);
      __builtin_nontemporal_store(phin, &b.nxt.PHI[selfnode]);
    }

    // streaming of h* inside the block: every region node publishes its
    // codes and Lambda, then each inner node gathers from x - e_k and decodes
    // (the same arithmetic as the writer's, so the same values), keeping the
    // population order of a pull without ordered passes
    const int xb = p & 1;
    // walls: buffers of planes p and p - 1 modulo 3 (p >= -1)
    const int ub = (p + 3) % 3, pb = (p + 2) % 3;
    const int lb = kWalls ? ub : xb;
    if (active && !closing) {
#pragma unroll
      for (int k = 0; k < QH; ++k) {
        if (k == LH::REST) continue;
        if (kWalls && k < NU)
          hxu[kWalls ? ub : 0][kWalls ? k : 0][ty][tx] = enc[k];
        else
          hxe[xb][kWalls ? k - NU - 1 : mslot<LH>(k)][ty][tx] = enc[k];
      }
      hxl[lb][ty][tx] = kWmin * lam;
    }
    if constexpr (!kAhead) load_tiles(p + 2);
    // The one barrier of the plane.  Before it: reads of the phi / Lambda
    // planes p-1 .. p+1, writes of phi^{n+1}(p), of the exchange (p & 1) and
    // of the tile p+2.  After it: reads of the exchange (p & 1) and of
    // phi^{n+1}(p-2 .. p).  The slot of tile p+2 was last read before the
    // previous barrier, that of phi^{n+1}(p) after the barrier three planes
    // back, and the exchange buffer (p & 1) after the barrier two planes back
    // (with walls the buffers kept modulo 3, read also after the next
    // barrier, after the barrier three planes back).  Fetching ahead, the tile
    // of p + 3 is written after this barrier: its slot held plane p - 1, last
    // read before the barrier, and plane p + 3 is read after the next one.
    __syncthreads();
    if constexpr (kAhead) {
      fetch_tiles(p + 3);
      fetch_h(p + 1);
    }
    const bool dn_ok = p - 1 >= z0 && p - 1 < z1;
    // decoded h* that population k of this node receives from x - e_k in the
    // exchange of plane p (not the e_z = +1 layer with walls)
    auto xchg = [&](int k) -> double {
      const int sy = ty - LH::ey[k], sx = tx - LH::ex[k];
      return double(dev_decode_wmin<Codec, LH>(
          k, hxe[xb][kWalls ? k - NU - 1 : mslot<LH>(k)][sy][sx], hxl[lb][sy][sx]));
    };
    // walls: decoded e_z = +1 population k of plane p - 1 at region node
    // (sy, sx)
    auto xup = [&](int k, int sy, int sx) -> double {
      return double(dev_decode_wmin<Codec, LH>(k, hxu[kWalls ? pb : 0][kWalls ? k : 0][sy][sx],
                                               hxl[kWalls ? pb : 0][sy][sx]));
    };
    double acc_up = 0.0;
    if constexpr (!kWalls) {
      if (inner) {
#pragma unroll
        for (int k = 0; k < QH; ++k) {
          const double v = k == LH::REST ? double(hdec[k]) : xchg(k);
          if (LH::ez[k] > 0)
            acc_up = k == 0 ? v : acc_up + v;
          else if (LH::ez[k] == 0)
            acc_mid = acc_mid + v;
          else
            acc_dn = acc_dn + v;
        }
      }
    } else if (inner && active) {
      if (!closing) {
        // c^{n+1}(p) through its in-plane layer: the e_z = +1 layer gathered
        // at the plane below, or bounced (the node's own opposite values)
        double a = 0.0;
#pragma unroll
        for (int k = 0; k < NU; ++k) {
          const bool bnc = bz_up || ((bmh >> k) & 1u);
          const double v = bnc ? double(hdec[LH::opp[k]]) : xup(k, ty - LH::ey[k], tx - LH::ex[k]);
          a = k == 0 ? v : a + v;
        }
#pragma unroll
        for (int k = NU; k < NU + NM; ++k) {
          double v;
          if (k == LH::REST)
            v = double(hdec[k]);
          else if ((bmh >> k) & 1u)
            v = double(hdec[LH::opp[k]]);
          else
            v = xchg(k);
          a = a + v;
        }
        // c^{n+1}(p - 1): its e_z = -1 layer, from this plane or bounced
        // (this node's own e_z = +1 values of plane p - 1)
#pragma unroll
        for (int k = NU + NM; k < QH; ++k) {
          const double v = ((bmh >> k) & 1u) ? xup(LH::opp[k], ty, tx) : xchg(k);
          acc_dn = acc_dn + v;
        }
        acc_up = a;
      } else {
        // past the top wall every e_z = -1 population of plane nz - 1 bounces
#pragma unroll
        for (int k = NU + NM; k < QH; ++k) acc_dn = acc_dn + xup(LH::opp[k], ty, tx);
      }
    }

    if (out && dn_ok) {
      const int zq = wrap_coord(p - 1, nz);
      const double c1 = acc_dn;
      const float phi1 = phiB[ring4(p - 1)][ty][tx];
      const float mu1 = float(closure(K.q, c1, double(phi1)));
      const int zm = (wz && p - 1 == 0) ? 0 : -1, zpl = (wz && p - 1 == nz - 1) ? 0 : 1;
      auto atB = [&](int dx, int dy, int dz) -> float {
        const int ox = dx < 0 ? xm : (dx > 0 ? xp : 0);
        const int oy = dy < 0 ? ym : (dy > 0 ? yp : 0);
        const int oz = dz < 0 ? zm : (dz > 0 ? zpl : 0);
        return phiB[ring4(p - 1 + oz)][ty + oy][tx + ox];
      };
      float gr1[3], n1[3];
      gradient_normal<LG, float>(atB, K.eps2, gr1, n1);
      float G[Q], gs[Q];
      phi_sources<LG, float>(K, phi1, mu1, n1, G);
#pragma unroll
      for (int k = 0; k < Q; ++k) gs[k] = g_collide<LG, float>(K, k, g_old[k], phi1, G[k]);
      uint16_t genc[Q];
      float gdec[Q];
      encode_g<Codec, LG>(gs, phi1, genc, gdec);
      // sg_old: the double sum of these g, taken when they were pulled
      balance_g_rest<LG, float, float>(K, gdec, sg_old, phi1, source_moment<float>(K, phi1, mu1));
      const auto Gw = make_rsrc(reinterpret_cast<char*>(b.nxt.G.mov) + zq * groupB, uint32_t(groupB));
#pragma unroll
      for (int k = 0; k < Q; ++k)
        if (k != LG::REST) bstore16_nt(genc[k], Gw, selfB, mslot<LG>(k) * planeB);
      __builtin_nontemporal_store(gdec[LG::REST], &b.nxt.G.rest[(int64_t)zq * plane + self_xy]);
    }
    if constexpr (kAhead) store_tiles(p + 3);
#pragma unroll
    for (int k = 0; k < Q; ++k) g_old[k] = g_new[k];
    sg_old = sg;
    if constexpr (kWalls) {
      acc_dn = acc_up;
    } else {
      acc_dn = acc_mid;
      acc_mid = acc_up;
    }
  }
  __syncthreads();  // the LDS rings are refilled by the next tile
  }
}

// output rows per tile with walls: the wall bookkeeping (bounce masks,
// mirror offsets, the third exchange buffer) does not fit the 128 VGPRs of
// 16 waves per CU, so the walled z-march runs 64 x 9 tiles (12 waves, up to
// 168 VGPRs: no spill in the basic form, 3 VGPRs in the general one on D3Q19).
// Only an explicit request for the fused schedule takes it: AUTO steps walled
// deviation runs by the node pair.
#ifndef GPLBM_DEV_WALL_TY
#define GPLBM_DEV_WALL_TY 9
#endif

template <class Codec, class LG, class LH, bool kGen>
struct DevFused3D {
  template <bool kWalls>
  static int run(const Geo& g, const Coef<float>& K, const DevStep& b, hipStream_t st) {
    // z chunks of 128 planes on periodic grids (2 halo planes per 130; 1280
    // tiles at 512^3, 5 passes of the 256 resident blocks): FP16 6.98-7.01
    // against 7.10 ms with 64, which ran 7.37 against 7.52 with 32; 32 with
    // walls (64 x 9 tiles: 7296 at 512^3, 28.5 passes, against 14.25 with 64)
    constexpr int TX = 64, TY = kWalls ? GPLBM_DEV_WALL_TY : GPLBM_DEV_TY, ZC = kWalls ? 32 : 128;
    constexpr int NT = TileShape<TX, TY>::NT;
    auto kernel = k_dev_fused3d<TX, TY, Codec, LG, LH, kGen, kWalls>;
    const int tiles_x = (g.nx + TX - 1) / TX;
    const int tiles_y = (g.ny + TY - 1) / TY;
    const int tiles_xy = tiles_x * tiles_y;
    static int resident[64] = {0};
    const int slots = resident_slots(kernel, NT, resident);
    if (slots <= 0) return -1;
    const int zc = chunk_planes(tiles_xy, g.nz, ZC, slots);
    const int ntiles = tiles_xy * ((g.nz + zc - 1) / zc);
    hipLaunchKernelGGL(kernel, dim3(resident_grid(slots, ntiles)), dim3(NT), 0, st, g, K, b, tiles_x,
                       tiles_xy, ntiles, zc);
    return 0;
  }
  static int launch(const Geo& g, const Coef<float>& K, const DevStep& b, hipStream_t st) {
    return (g.bcx || g.bcy || g.bcz) ? run<true>(g, K, b, st) : run<false>(g, K, b, st);
  }
};

// ---------------------------------------------------------------------------
// Fused schedule in the deviation format on D2Q9 (any boundaries): one kernel
// per step, the 2-D tiling of the FP32 / FP64 fused kernel.  A block owns an
// output tile T (x-aligned, tiles.h) and computes T grown by one node (T+1):
//   - phi^n and Lambda^{n-1} of T+2 are staged in LDS; every pull decodes
//     with the reference (w_k phi or w_k Lambda) of its source node, or of the
//     node itself for a population bounced back at a wall;
//   - the threads of T+1 run the h collision of step n, write the 16-bit
//     codes (nodes of T) and publish the decoded h* to an LDS exchange;
//   - after one barrier each node of T gathers c^{n+1} from x - e_k in
//     population order (its own h*_{opp k} where x - e_k lies beyond a
//     wall), then runs the g collision of step n+1.
// The values and the order of every sum are those of the split kernels, so
// the two schedules give identical bits.
// Bound by instruction issue and load latency: one batch of loads with
// selected addresses in place of a branch and a 64-bit address computation per
// population, and two blocks of 8 rows per CU (68 VGPRs) in place of one of 13
// (114): 512^2 FP16 23.9 -> 10.5 us, 1024^2 55.5 -> 32.1 us, 2048^2 229 -> 147
// us; 128^2 12.6 -> 4.7 us.
template <int TX, int TY, class Codec, class L, class LH, bool kGen, bool kWalls, bool kStream>
__global__ void __launch_bounds__((TileShape<TX, TY>::NT))
    k_dev_fused2d(Geo g, Coef<float> Kin, DevStep b, int tiles_x, int ntiles) {
  const Coef<float> K = variant<kGen>(Kin);
  // g on L (D2Q9 or D2Q5), h on LH (L, or D2Q5 under D2Q9)
  constexpr int Q = L::Q, QH = LH::Q;
  using Shape = TileShape<TX, TY>;
  constexpr int BX = Shape::BX, BY = Shape::BY, NT = Shape::NT;
  constexpr int AX = BX + 2, AY = BY + 2;
  constexpr int TILE_PER_THREAD = (AX * AY + NT - 1) / NT;
  __shared__ float phiA[AY][AX];  // phi^n on T+2
  __shared__ float lamA[AY][AX];  // Lambda^{n-1} on T+2
  __shared__ float phiB[BY][BX];  // phi^{n+1} on T+1
  __shared__ float hx[QH][BY][BX];  // decoded h*^n of T+1 (moving populations)

  int tx, ty;
  bool valid;
  Shape::node(threadIdx.x, tx, ty, valid);

  for (int tile = first_tile(); tile < ntiles; tile += gridDim.x) {
    const int X0 = (tile % tiles_x) * TX, Y0 = (tile / tiles_x) * TY;
    const int ux = X0 - 1 + tx, uy = Y0 - 1 + ty;  // unwrapped node of this thread
    const bool active = valid && (!kWalls || ((!g.bcx || (ux >= 0 && ux < g.nx)) &&
                                              (!g.bcy || (uy >= 0 && uy < g.ny))));
    const bool out = valid && ux < g.nx && uy < g.ny && tx >= 1 && tx <= TX && ty >= 1 && ty <= TY;
    const Pull2D<kWalls> at(g, ux, uy);
    const int64_t i = at.self();
    auto mh = [](int k) { return mslot<LH>(k); };
    auto mg = [](int k) { return mslot<L>(k); };

    // every load of the tile in one batch before the first barrier: the codes
    // (of inactive nodes too, in range and not used) and the reference tiles
    float pv[TILE_PER_THREAD], lv[TILE_PER_THREAD];
    uint16_t ch[QH], cg[Q];
#pragma unroll
    for (int j = 0; j < TILE_PER_THREAD; ++j) {
      const int l = min((int)threadIdx.x + j * NT, AX * AY - 1);
      int vx = X0 - 2 + l % AX, vy = Y0 - 2 + l / AX;
      vx = kWalls && g.bcx ? min(max(vx, 0), g.nx - 1) : wrap_near(vx, g.nx);
      vy = kWalls && g.bcy ? min(max(vy, 0), g.ny - 1) : wrap_near(vy, g.ny);
      const int64_t q = (int64_t)vy * g.nx + vx;
      pv[j] = b.cur.PHI[q];
      lv[j] = b.cur.LAM[q];
    }
#pragma unroll
    for (int k = 0; k < QH; ++k)
      ch[k] = k == LH::REST ? uint16_t(0) : b.cur.H.mov[at.template slot<LH>(k, mh)];
#pragma unroll
    for (int k = 0; k < Q; ++k)
      cg[k] = k == L::REST ? uint16_t(0) : b.cur.G.mov[at.template slot<L>(k, mg)];
    const float h_rest = b.cur.H.rest[i], g_rest = b.cur.G.rest[i];
#pragma unroll
    for (int j = 0; j < TILE_PER_THREAD; ++j) {
      const int l = threadIdx.x + j * NT;
      if (l < AX * AY) {
        phiA[l / AX][l % AX] = pv[j];
        lamA[l / AX][l % AX] = lv[j];
      }
    }
    __syncthreads();

    // decoded with the reference of the source node, or of the node itself
    // for a bounced population (w_opp(k) = w_k)
    const float lam0 = lamA[ty + 1][tx + 1], phi = phiA[ty + 1][tx + 1];
    float gn[Q];     // g~^{n+1}
    float hdec[QH];  // h~*^n as readers decode it
    double sg = 0.0;
    {
      float h[QH];
      double c = 0.0;
#pragma unroll
      for (int k = 0; k < QH; ++k) {
        if (k == LH::REST) {
          h[k] = h_rest;
        } else {
          const float in = lamA[ty + 1 - LH::ey[k]][tx + 1 - LH::ex[k]];
          h[k] = dev_decode<Codec>(ch[k], float(LH::w[k]) * (at.template bounced<LH>(k) ? lam0 : in));
        }
        c = k == 0 ? double(h[k]) : c + double(h[k]);
      }
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        if (k == L::REST) {
          gn[k] = g_rest;
        } else {
          const float in = phiA[ty + 1 - L::ey[k]][tx + 1 - L::ex[k]];
          gn[k] = dev_decode<Codec>(cg[k], float(L::w[k]) * (at.template bounced<L>(k) ? phi : in));
        }
        sg = k == 0 ? double(gn[k]) : sg + double(gn[k]);
      }
      const float mu = float(closure(K.q, c, double(phi)));
      auto atA = [&](int dx, int dy, int) -> float {
        return phiA[ty + 1 + at.sy(dy)][tx + 1 + at.sx(dx)];
      };
      float gr[3], n[3];
      gradient_normal<L, float>(atA, K.eps2, gr, n);
      const float sbar = source_moment<float>(K, phi, mu);
      const float phin = float(sg + 0.5 * double(sbar));
      float F[3];
      h_flux<L, float>(K, mu, gr, n, phin - phi, K.anti_trapping != 0, F);
      const float lam = h_lambda<float>(K, phi, mu);
      const float cc = float(c);
      float hs[QH];
      h_update<LH>(K, h, cc, lam, F, hs);
      uint16_t enc[QH];
      encode_h<Codec, LH>(hs, lam, c, enc, hdec);
      if (active) {
        phiB[ty][tx] = phin;
#pragma unroll
        for (int k = 0; k < QH; ++k)
          if (k != LH::REST) hx[k][ty][tx] = hdec[k];
      }
      if (out) {
#pragma unroll
        for (int k = 0; k < QH; ++k)
          if (k != LH::REST) store_state<kStream>(enc[k], &b.nxt.H.mov[mh(k) * at.plane + i]);
        b.nxt.H.rest[i] = hdec[LH::REST];
        b.nxt.LAM[i] = lam;
        b.nxt.PHI[i] = phin;
      }
    }
    __syncthreads();

    if (out) {
      double c1 = 0.0;
#pragma unroll
      for (int k = 0; k < QH; ++k) {
        float v = hdec[k];
        if (k != LH::REST) {
          const float in = hx[k][ty - LH::ey[k]][tx - LH::ex[k]];
          v = at.template bounced<LH>(k) ? hdec[LH::opp[k]] : in;
        }
        c1 = k == 0 ? double(v) : c1 + double(v);
      }
      const float phi1 = phiB[ty][tx];
      const float mu1 = float(closure(K.q, c1, double(phi1)));
      auto atB = [&](int dx, int dy, int) -> float {
        return phiB[ty + at.sy(dy)][tx + at.sx(dx)];
      };
      float gr[3], n[3];
      gradient_normal<L, float>(atB, K.eps2, gr, n);
      float G[Q], gs[Q];
      phi_sources<L, float>(K, phi1, mu1, n, G);
#pragma unroll
      for (int k = 0; k < Q; ++k) gs[k] = g_collide<L, float>(K, k, gn[k], phi1, G[k]);
      uint16_t genc[Q];
      float gdec[Q];
      encode_g<Codec, L>(gs, phi1, genc, gdec);
      balance_g_rest<L, float, float>(K, gdec, sg, phi1, source_moment<float>(K, phi1, mu1));
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        if (k == L::REST)
          b.nxt.G.rest[i] = gdec[k];
        else
          store_state<kStream>(genc[k], &b.nxt.G.mov[mg(k) * at.plane + i]);
      }
    }
    __syncthreads();  // the LDS tiles are refilled by the next tile
  }
}

template <class Codec, class L, class LH, bool kGen>
struct DevFused2D {
  template <int TY, bool kWalls>
  static int run(const Geo& g, const Coef<float>& K, const DevStep& b, hipStream_t st) {
    if constexpr (TY >= 8)
      if (streams_out((int64_t)(2 * ((L::Q + LH::Q - 2) * 2 + 16)) * g.N))
        return run<TY, kWalls, true>(g, K, b, st);
    return run<TY, kWalls, false>(g, K, b, st);
  }
  template <int TY, bool kWalls, bool kStream>
  static int run(const Geo& g, const Coef<float>& K, const DevStep& b, hipStream_t st) {
    constexpr int TX = 64;
    constexpr int NT = TileShape<TX, TY>::NT;
    auto kernel = k_dev_fused2d<TX, TY, Codec, L, LH, kGen, kWalls, kStream>;
    const int tiles_x = (g.nx + TX - 1) / TX;
    const int tiles_y = (g.ny + TY - 1) / TY;
    const int ntiles = tiles_x * tiles_y;
    static int resident[64] = {0};
    const int slots = resident_slots(kernel, NT, resident);
    if (slots <= 0) return -1;
    hipLaunchKernelGGL(kernel, dim3(resident_grid(slots, ntiles)), dim3(NT), 0, st, g, K, b, tiles_x,
                       ntiles);
    return 0;
  }
  template <bool kWalls>
  static int by_rows(const Geo& g, const Coef<float>& K, const DevStep& b, hipStream_t st) {
    const int rows = tile_rows(g.nx, g.ny, 64, false);
    if (rows == 1) return run<1, kWalls>(g, K, b, st);
    if (rows == 4) return run<4, kWalls>(g, K, b, st);
    return run<8, kWalls>(g, K, b, st);
  }
  static int launch(const Geo& g, const Coef<float>& K, const DevStep& b, hipStream_t st) {
    return (g.bcx || g.bcy) ? by_rows<true>(g, K, b, st) : by_rows<false>(g, K, b, st);
  }
};

// 32-bit offsets inside a z plane group of moving populations; any boundary
inline bool dev_fused_supported(int nx, int ny, int nz, const int*) {
  return (int64_t)nx * ny * kMov * 2 < ((int64_t)1 << 31) &&
         (int64_t)nx * ny * nz < ((int64_t)1 << 31);
}

}  // namespace gplbm
