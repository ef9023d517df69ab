// Fused schedule in 3-D: one kernel per time step n -> n+1, marching in z.
// g runs on D3Q19 or D3Q7 (L), h on D3Q19 or D3Q7 (LH).
//
// A block owns an x-y output tile T of TX x TY nodes and a chunk of ZC planes,
// and computes the tile grown by one node in x and y (the region, BX x BY).
// It walks the planes p = z0-1 .. z1 (one halo plane below and above the
// chunk).  At plane p every thread
//   - pulls h~^n (-> c^n, mu^n) and g~^{n+1} (-> phi^{n+1}),
//   - takes phi^n of planes p-1, p, p+1 from a 3-plane LDS ring (T+2 in x-y)
//     for the gradient, writes phi^{n+1}(p) into a second ring,
//   - runs the h collision of step n.
// The post-collision h* are then streamed inside the block: they go to an LDS
// exchange, and after one barrier every node gathers its own contributions
// from x - e_k into three rolling partial sums (the e_z = +1 populations reach
// plane p+1, the in-plane ones plane p, the e_z = -1 ones plane p-1).  Because
// D3Q19 and D3Q7 are numbered by layers of e_z (+1, 0, -1), every node's
// c^{n+1} receives its populations in index order across the three planes, the
// order of a pull.
// After plane p, c^{n+1}(p-1) is complete and the threads of T run the g
// collision of step n+1 at plane p-1, on the g~^{n+1} pulled one plane
// earlier (kept in registers, or in the LDS, every thread in slots of its own).
//
// Tiles are x-aligned with the halo columns in extra lanes, and the grid is
// persistent with XCD-ordered passes (tiles.h): every output row is whole
// 128-byte lines (partial-line writes cost about a third of the write
// bandwidth), and neighbouring tiles march in step so that the lines of their
// shared halo are still in the L2 when the second tile reads them.
//
// Addressing: with the plane-major layout f[z][k][y][x] every population a
// thread pulls lies in one of three plane groups (z-1, z, z+1) of Q planes
// each (Qh for h).  Each group is a buffer resource in scalar registers; the
// population plane k*nx*ny is the uniform offset and the (x, y) source the
// per-lane offset, so a load costs no vector address arithmetic.
//
// Zero-flux walls (kWalls): a pull from beyond a wall reads the node's own
// opposite population; the phi^n tiles are loaded with clamped coordinates
// (the mirror ghost) and the phi^{n+1} stencil takes mirrored offsets.  A
// population that bounces at an x or y wall reaches its node from the node's
// own plane, not from the plane below or above, so the gather form keeps the
// index order of the pull sum by taking the e_z = +1 layer of a node's c^{n+1}
// at the node's own plane from a second, parity-buffered exchange of the
// plane below (or the node's own bounced values), and the bounced e_z = -1
// values from the node's own entries there; past a top wall a closing plane
// finishes the last one.
#pragma once

#include <type_traits>

#include "kernels_fused2d.h"
#include "tiles.h"

namespace gplbm {

__device__ __forceinline__ int ring3(int q) { return (q + 6) % 3; }

// Raw buffer access: a resource (base, byte range) held in scalar registers,
// a 32-bit per-lane offset and a 32-bit uniform offset.  Offsets outside the
// range read 0 and drop writes.
constexpr int kBufferFlags = 0x00020000;  // gfx9 buffer descriptor, dword 3

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                           kBufferFlags);
}

template <class S>
__device__ __forceinline__ S bload(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  if constexpr (sizeof(S) == 8)
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
  else
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

// non-temporal store (the written state is not read again in this step)
template <class S>
__device__ __forceinline__ void bstore_nt(S v, __amdgpu_buffer_rsrc_t r, uint32_t voff,
                                          uint32_t soff) {
  constexpr int kNT = 2;
  if constexpr (sizeof(S) == 8) {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, voff, soff, kNT);
  } else {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b32(r, 0, 0, 0));
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(V, v), r, voff, soff, kNT);
  }
}

// Pulls of the populations of lattice P at plane p: population k comes from
// plane group p - e_z and (x, y) - (e_x, e_y), whose byte offset inside a
// population plane is xyb[1 - e_y][1 - e_x].  With walls bounced populations
// (bits of `bounce` for the x and y walls, whole e_z layers at a z wall) are
// the node's own opposite ones.  kPlainWaves: a wavefront without any takes
// pulls of its own without the tests, which the forms that load ahead gain by
// (FP32 256^3 with z walls 1263 us against 1299, 160^3 357 against 374); the
// general FP64 form, which does not, is better off with one body (238^3 with
// walls 2292 us against 2453, 317^3 5523 against 5850).
template <class P, class S, bool kWalls, bool kPlainWaves>
__device__ __forceinline__ void fetch(const S* base, int p, int nz, bool wz, int plane,
                                      const uint32_t (&xyb)[3][3], uint32_t bounce, S (&v)[P::Q]) {
  const int64_t groupB = int64_t(plane) * P::Q * sizeof(S);
  const uint32_t planeB = uint32_t(plane) * sizeof(S);
  const int zp = wz ? min(p, nz - 1) : wrap_coord(p, nz);
  const int zs[3] = {wz ? max(zp - 1, 0) : (zp == 0 ? nz - 1 : zp - 1), zp,
                     wz ? min(zp + 1, nz - 1) : (zp == nz - 1 ? 0 : zp + 1)};
  __amdgpu_buffer_rsrc_t R[3];
#pragma unroll
  for (int j = 0; j < 3; ++j)
    R[j] = make_rsrc(reinterpret_cast<const char*>(base) + zs[j] * groupB, uint32_t(groupB));
  if constexpr (kWalls) {
    uint32_t m = bounce;
    if (wz && p == 0) m |= ez_mask<P>(1);
    if (wz && p == nz - 1) m |= ez_mask<P>(-1);
    if (!kPlainWaves || __builtin_amdgcn_ballot_w64(m != 0u) != 0u) {
#pragma unroll
      for (int k = 0; k < P::Q; ++k) {
        if ((m >> k) & 1u)
          v[k] = bload<S>(R[1], xyb[1][1], P::opp[k] * planeB);
        else
          v[k] = bload<S>(R[1 - P::ez[k]], xyb[1 - P::ey[k]][1 - P::ex[k]], k * planeB);
      }
      return;
    }
  }
#pragma unroll
  for (int k = 0; k < P::Q; ++k)
    v[k] = bload<S>(R[1 - P::ez[k]], xyb[1 - P::ey[k]][1 - P::ex[k]], k * planeB);
}

// Carry of the pulled g~^{n+1} from its plane to the collision one plane
// later: in registers, or in the LDS, in slots that only their own thread
// touches.  The pulls of plane p wait in registers until the collision of
// plane p - 1 has read the slots, so one buffer does.
enum class Carry { kRegisters, kLds };

// Zero-flux walls in the z-marching kernels.  A population whose source
// x - e_k lies beyond a wall is the node's own opposite population (halfway
// bounce-back); the gradient stencils use the mirror ghost, which the T+2
// tiles get by loading clamped coordinates along wall axes.
//
// Coordinate of a tile node along one axis: wrapped on a periodic axis,
// clamped (mirror ghost) on a wall axis.
__device__ __forceinline__ int tile_coord(int u, int n, int bc) {
  return bc ? min(max(u, 0), n - 1) : wrap_coord(u, n);
}

// Bit k set when population k of lattice P reaches the node at unwrapped
// coordinates (ux, uy) from beyond an x or a y wall.
template <class P>
__device__ __forceinline__ uint32_t xy_bounce_mask(const Geo& g, int ux, int uy) {
  uint32_t m = 0;
#pragma unroll
  for (int k = 0; k < P::Q; ++k) {
    const int sx = ux - P::ex[k], sy = uy - P::ey[k];
    const bool b = (g.bcx && (sx < 0 || sx >= g.nx)) || (g.bcy && (sy < 0 || sy >= g.ny));
    m |= b ? (1u << k) : 0u;
  }
  return m;
}


// Which pulls of the next plane are issued while a plane is computed (into
// registers; with any of them also the phi^n tile of the plane after next).
enum class Prefetch { kNone, kH, kBoth };

// Tile height, longest z chunk, carry and prefetch, measured on the 512^3 and
// 256^3 (or 320^3) steps in ms against the form before (g carried in two
// buffers by plane parity and h* pushed in ordered passes in FP64, else g
// carried in registers, no prefetch of the pulls):
//   D3Q19 FP64  18.5-19.0 against 19.8-20.1 (2.35 against 2.53); the LDS is
//               full (163392 of 163840 bytes) and so are the 168 VGPRs of 9
//               waves, of which 8 spill; a prefetch of h spills more and one
//               of both on 5 rows loses the neighbours' lines from the L2
//               (21.0 and 21.9); chunks of at most 64 planes 18.8, 32 19.0, 128
//               18.9
//   D3Q19 FP32  8.90 against 9.86 (1.17 against 1.29); both prefetched 9.25,
//               13 rows 10.4, 11 and 10 rows 8.96
//   h on D3Q7   320^3 FP64 2.94 on 8 rows against 3.62 on 6 (512^3 in chunks
//               of 128 planes 11.7, of 32 12.1); FP32 1.58 on 13 rows against
//               1.78 on 12
//   D3Q7 FP64   320^3 1.56 against 1.75; 512^3 6.72 against 6.91
//   D3Q7 FP32   320^3 0.863 on 12 rows, 0.895 on 8, against 1.00; 512^3 3.59
//               against 3.99
template <class L, class LH, class S>
struct Fused3DConfig;
template <>
struct Fused3DConfig<D3Q19, D3Q19, double> {
  static constexpr int TX = 64, TY = 6, ZC = 64;
  static constexpr Carry carry = Carry::kLds;
  static constexpr Prefetch prefetch = Prefetch::kNone;
};
template <>
struct Fused3DConfig<D3Q19, D3Q19, float> {
  static constexpr int TX = 64, TY = 12, ZC = 64;
  static constexpr Carry carry = Carry::kLds;
  static constexpr Prefetch prefetch = Prefetch::kH;
};
template <>
struct Fused3DConfig<D3Q19, D3Q7, double> {
  static constexpr int TX = 64, TY = 8, ZC = 128;
  static constexpr Carry carry = Carry::kLds;
  static constexpr Prefetch prefetch = Prefetch::kH;
};
template <>
struct Fused3DConfig<D3Q19, D3Q7, float> {
  static constexpr int TX = 64, TY = 13, ZC = 64;
  static constexpr Carry carry = Carry::kLds;
  static constexpr Prefetch prefetch = Prefetch::kH;
};
template <>
struct Fused3DConfig<D3Q7, D3Q7, double> {
  static constexpr int TX = 64, TY = 12, ZC = 32;
  static constexpr Carry carry = Carry::kRegisters;
  static constexpr Prefetch prefetch = Prefetch::kH;
};
template <>
struct Fused3DConfig<D3Q7, D3Q7, float> {
  static constexpr int TX = 64, TY = 12, ZC = 64;
  static constexpr Carry carry = Carry::kRegisters;
  static constexpr Prefetch prefetch = Prefetch::kH;
};

template <int TX, int TY, Carry kCarryMode, Prefetch kPF, class L, class LH, class S, class C,
          bool kGen, bool kWalls>
__global__ void __launch_bounds__((TileShape<TX, TY>::NT))
    k_fused3d(Geo g, Coef<C> Kin, StepBufs<S> b, int tiles_x, int tiles_xy, int ntiles, int zc) {
  const Coef<C> K = variant<kGen>(Kin);
  using Shape = TileShape<TX, TY>;
  constexpr int Q = L::Q, QH = LH::Q;
  // e_z layers of the h lattice: +1 at [0, NU), 0 at [NU, NU+NM), -1 after
  constexpr int NU = count_ez<LH>(1), NM = count_ez<LH>(0), ND = count_ez<LH>(-1);
  static_assert(NU + NM + ND == QH, "h lattice must be numbered by layers of e_z");
  static_assert(LH::REST == NU, "the rest vector opens the in-plane layer");
  constexpr int BX = Shape::BX, BY = Shape::BY;
  constexpr int AX = BX + 2, AY = BY + 2;
  constexpr int NT = Shape::NT;
  constexpr int PHI_PER_THREAD = (AX * AY + NT - 1) / NT;
  constexpr bool kRegs = kCarryMode == Carry::kRegisters;
  constexpr bool kPrefetch = kPF != Prefetch::kNone, kPrefetchG = kPF == Prefetch::kBoth;
  __shared__ C phiA[3][AY][AX];  // phi^n, planes p-1, p, p+1
  __shared__ C phiB[3][BY][BX];  // phi^{n+1}, planes p-2, p-1, p
  // Moving h* of plane p (the readers gather from x - e_k after one barrier):
  // slots 0 .. NX-1; with walls the e_z = +1 layer is in hxu instead, kept for
  // one more plane (by plane parity): the plane above gathers it after its own
  // barrier, and a node's own values in it are the bounce of its e_z = -1
  // populations.  The plane's two barriers order the reuse of a parity buffer.
  constexpr int NX = kWalls ? QH - 1 - NU : QH - 1;
  __shared__ C hx[NX][BY][BX];
  __shared__ C hxu[kWalls ? 2 : 1][kWalls ? NU : 1][kWalls ? BY : 1][kWalls ? BX : 1];
  // g~^{n+1} of the output nodes, pulled at plane p - 1 (LDS carry): every
  // thread reads and writes its own slots only, so no barrier orders them
  __shared__ C gkeep[kRegs ? 1 : Q][kRegs ? 1 : TY][kRegs ? 1 : TX];
  // slot of moving population k in hx
  auto xslot = [](int k) constexpr { return kWalls ? k - NU - 1 : (k < LH::REST ? k : k - 1); };

  int tx, ty;
  bool valid;
  Shape::node(threadIdx.x, tx, ty, valid);
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int plane = nx * ny;
  const uint32_t planeB = uint32_t(plane) * sizeof(S);     // one population plane
  const int64_t groupB = int64_t(plane) * Q * sizeof(S);   // one z plane group of g
  const int64_t groupH = int64_t(plane) * QH * sizeof(S);  // one z plane group of h
  const bool wz = kWalls && g.bcz;

  for (int tile = first_tile(); tile < ntiles; tile += gridDim.x) {
    const int chunk = tile / tiles_xy, txy = tile % tiles_xy;
    const int X0 = tile_column(txy, tiles_x, chunk, kWalls) * TX, Y0 = (txy / tiles_x) * TY;
    const int z0 = chunk * zc, z1 = min(z0 + zc, nz);

    const int ux = X0 - 1 + tx, uy = Y0 - 1 + ty;
    const bool inner = valid && tx >= 1 && tx <= TX && ty >= 1 && ty <= TY;
    const bool out = inner && ux < nx && uy < ny;
    // region nodes beyond a wall take no part (with walls only)
    bool active = valid;
    if constexpr (kWalls)
      active = valid && (!g.bcx || (ux >= 0 && ux < nx)) && (!g.bcy || (uy >= 0 && uy < ny));
    const int x = kWalls ? tile_coord(ux, nx, g.bcx) : wrap_near(ux, nx);
    const int y = kWalls ? tile_coord(uy, ny, g.bcy) : wrap_near(uy, ny);
    // source offsets wrap also on wall axes: a source beyond a wall is never
    // read (its population bounces), the wrapped address keeps it in range
    const int xo[3] = {x == 0 ? nx - 1 : x - 1, x, x == nx - 1 ? 0 : x + 1};
    const int yo[3] = {(y == 0 ? ny - 1 : y - 1) * nx, y * nx, (y == ny - 1 ? 0 : y + 1) * nx};
    // byte offset, inside a population plane, of the source x - e_k (by e_x, e_y)
    uint32_t xyb[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) xyb[a][c] = uint32_t(yo[a] + xo[c]) * sizeof(S);
    const uint32_t selfB = xyb[1][1];
    // populations arriving from beyond an x or y wall (bit k), and the mirror
    // offsets of the phi^{n+1} stencil
    uint32_t bmh = 0, bmg = 0;
    int xm = -1, xp = 1, ym = -1, yp = 1;
    if constexpr (kWalls) {
      bmh = xy_bounce_mask<LH>(g, ux, uy);
      bmg = xy_bounce_mask<L>(g, ux, uy);
      xm = (g.bcx && ux == 0) ? 0 : -1;
      xp = (g.bcx && ux == nx - 1) ? 0 : 1;
      ym = (g.bcy && uy == 0) ? 0 : -1;
      yp = (g.bcy && uy == ny - 1) ? 0 : 1;
    }
    // phi^n tile positions this thread loads (T+2 in x-y; clamped along wall
    // axes, the mirror ghost)
    uint32_t phi_off[PHI_PER_THREAD];
#pragma unroll
    for (int j = 0; j < PHI_PER_THREAD; ++j) {
      const int l = min((int)threadIdx.x + j * NT, AX * AY - 1);
      const int gx = kWalls ? tile_coord(X0 - 2 + l % AX, nx, g.bcx) : wrap_near(X0 - 2 + l % AX, nx);
      const int gy = kWalls ? tile_coord(Y0 - 2 + l / AX, ny, g.bcy) : wrap_near(Y0 - 2 + l / AX, ny);
      phi_off[j] = uint32_t(gy * nx + gx);
    }
    auto fetch_phi = [&](int p, S (&v)[PHI_PER_THREAD]) {
      const int pz = kWalls ? tile_coord(p, nz, g.bcz) : wrap_coord(p, nz);
      const S* src = b.PHI + (int64_t)pz * plane;
#pragma unroll
      for (int j = 0; j < PHI_PER_THREAD; ++j) v[j] = src[phi_off[j]];
    };
    auto put_phi = [&](int p, const S (&v)[PHI_PER_THREAD]) {
#pragma unroll
      for (int j = 0; j < PHI_PER_THREAD; ++j) {
        const int l = threadIdx.x + j * NT;
        if (l < AX * AY) phiA[ring3(p)][l / AX][l % AX] = C(v[j]);
      }
    };
    // pulls of plane p (h or g); a source beyond a wall gives the node's own
    // opposite population (bounce-back); a plane beyond a z wall is never read
    auto fetch_h = [&](int p, S (&v)[QH]) {
      fetch<LH, S, kWalls, kPrefetch>(b.H, p, nz, wz, plane, xyb, bmh, v);
    };
    auto fetch_g = [&](int p, S (&v)[Q]) {
      fetch<L, S, kWalls, kPrefetch>(b.G, p, nz, wz, plane, xyb, bmg, v);
    };
    // first plane: the halo plane below the chunk, or the bottom plane at a
    // z wall
    const int pfirst = (wz && z0 == 0) ? 0 : z0 - 1;
    S hv[QH], gv[Q], phi_next[PHI_PER_THREAD];
    {
      S v0[PHI_PER_THREAD], v1[PHI_PER_THREAD];
      fetch_phi(pfirst - 1, v0);
      fetch_phi(pfirst, v1);
      if constexpr (kPrefetch) {
        fetch_phi(pfirst + 1, phi_next);
        fetch_h(pfirst, hv);
        if constexpr (kPrefetchG) fetch_g(pfirst, gv);
      }
      put_phi(pfirst - 1, v0);
      put_phi(pfirst, v1);
    }
    C g_old[kRegs ? Q : 1];
#pragma unroll
    for (int k = 0; k < (kRegs ? Q : 1); ++k) g_old[k] = C(0);
    // c^{n+1} of this thread's node on planes p-1 and p, partly summed (the
    // e_z = +1 populations arrive one plane early, the e_z = -1 ones one plane
    // late, each layer in ascending k)
    double acc_dn = 0.0, acc_mid = 0.0;
    double sg_old = 0.0;

    for (int p = pfirst; p <= z1; ++p) {
      // past a top wall: no plane, only the completion of plane nz - 1
      const bool closing = wz && p == nz;
      const bool work = !kWalls || (active && !closing);
      // whether plane p + 1 pulls; past a top wall none does (with walls a flat
      // box would load a plane in six for nothing: 1000 x 1000 x 5 FP64 general
      // 1030 us, 920 without)
      const bool pulls_next = p < z1 && !(wz && p + 1 == nz);
      if constexpr (!kPrefetch) fetch_phi(p + 1, phi_next);
      put_phi(p + 1, phi_next);
      if constexpr (kPrefetch) {
        if (p < z1) fetch_phi(p + 2, phi_next);
      }
      __syncthreads();
      const int zp = wz ? min(p, nz - 1) : wrap_coord(p, nz);
      // all e_z = +1 sources of this plane lie beyond the bottom wall
      const bool bz_up = wz && p == 0;
      const int sA = ring3(p);
      const bool own_p = p >= z0 && p < z1;

      C hs[QH];
      double sg = 0.0;
      if (work) {
        if constexpr (!kPrefetch) fetch_h(p, hv);
        if constexpr (!kPrefetchG) fetch_g(p, gv);
        double c = 0.0;
#pragma unroll
        for (int k = 0; k < QH; ++k) c = k == 0 ? double(hv[k]) : c + double(hv[k]);
        const C phi = phiA[sA][ty + 1][tx + 1];
        const C mu = C(closure(K.q, c, double(phi)));
        auto atA = [&](int dx, int dy, int dz) -> C {
          return phiA[ring3(p + dz)][ty + 1 + dy][tx + 1 + dx];
        };
        C gr[3], n[3];
        gradient_normal<L, C>(atA, K.eps2, gr, n);
        const C sbar = source_moment<C>(K, phi, mu);
#pragma unroll
        for (int k = 0; k < Q; ++k) sg = k == 0 ? double(gv[k]) : sg + double(gv[k]);
        const double phin = sg + 0.5 * double(sbar);
        const C phin_c = C(phin);
        if (active) phiB[sA][ty][tx] = phin_c;
        const C dtphi = phin_c - phi;
        C F[3];
        h_flux<L, C>(K, mu, gr, n, dtphi, K.anti_trapping != 0, F);
        const C lam = h_lambda<C>(K, phi, mu);
        const C cc = C(c);
        h_update<LH>(K, hv, cc, lam, F, hs);
        balance_rest<LH, S, C>(hs, c);
        if (active) {
#pragma unroll
          for (int k = 0; k < QH; ++k) {
            if (k == LH::REST) continue;
            if (kWalls && k < NU)
              hxu[kWalls ? p & 1 : 0][kWalls ? k : 0][ty][tx] = hs[k];
            else
              hx[xslot(k)][ty][tx] = hs[k];
          }
        }
      }
      if (work && out && own_p) {
        const auto Hw = make_rsrc(reinterpret_cast<char*>(b.Hn) + zp * groupH, uint32_t(groupH));
#pragma unroll
        for (int k = 0; k < QH; ++k) bstore_nt<S>(S(hs[k]), Hw, selfB, k * planeB);
        __builtin_nontemporal_store(S(phiB[sA][ty][tx]), &b.PHIn[(int64_t)zp * plane + y * nx + x]);
      }
      // after the h stores: the wait for these pulls then waits for no store
      // issued later
      if constexpr (kPrefetch) {
        if (pulls_next) fetch_h(p + 1, hv);
      }

      __syncthreads();
      const bool dn_ok = p - 1 >= z0 && p - 1 < z1;
      double acc_up = 0.0;
      if constexpr (!kWalls) {
        if (inner) {
#pragma unroll
          for (int k = 0; k < QH; ++k) {
            const double v = k == LH::REST ? double(hs[k])
                                           : double(hx[xslot(k)][ty - LH::ey[k]][tx - LH::ex[k]]);
            if (LH::ez[k] > 0)
              acc_up = k == 0 ? v : acc_up + v;
            else if (LH::ez[k] == 0)
              acc_mid = acc_mid + v;
            else
              acc_dn = acc_dn + v;
          }
        }
      } else {
        // the node's c^{n+1}(p) through its in-plane layer (the e_z = +1 layer
        // from plane p - 1, or bounced) and the e_z = -1 layer of
        // c^{n+1}(p - 1) (from plane p, or bounced: the node's own e_z = +1
        // values of plane p - 1), each in population order
        const int pb = (p & 1) ^ 1;
        if (inner && active) {
          if (!closing) {
            double a = 0.0;
#pragma unroll
            for (int k = 0; k < NU; ++k) {
              const double v = (bz_up || ((bmh >> k) & 1u))
                                   ? double(hs[LH::opp[k]])
                                   : double(hxu[pb][k][ty - LH::ey[k]][tx - LH::ex[k]]);
              a = k == 0 ? v : a + v;
            }
#pragma unroll
            for (int k = NU; k < NU + NM; ++k) {
              double v;
              if (k == LH::REST)
                v = double(hs[k]);
              else if ((bmh >> k) & 1u)
                v = double(hs[LH::opp[k]]);
              else
                v = double(hx[xslot(k)][ty - LH::ey[k]][tx - LH::ex[k]]);
              a = a + v;
            }
#pragma unroll
            for (int k = NU + NM; k < QH; ++k) {
              const double v = ((bmh >> k) & 1u) ? double(hxu[pb][LH::opp[k]][ty][tx])
                                                 : double(hx[xslot(k)][ty - LH::ey[k]][tx - LH::ex[k]]);
              acc_dn = acc_dn + v;
            }
            acc_up = a;
          } else {
            // past the top wall every e_z = -1 population of plane nz - 1
            // bounces
#pragma unroll
            for (int k = NU + NM; k < QH; ++k) acc_dn = acc_dn + double(hxu[pb][LH::opp[k]][ty][tx]);
          }
        }
      }

      // g collision of step n+1 at plane p-1
      if (out && dn_ok) {
        const int zq = wrap_coord(p - 1, nz);
        const int sB = ring3(p - 1);
        const double c1 = acc_dn;
        const C phi1 = phiB[sB][ty][tx];
        const C mu1 = C(closure(K.q, c1, double(phi1)));
        const int zm = (wz && p - 1 == 0) ? 0 : -1, zpl = (wz && p - 1 == nz - 1) ? 0 : 1;
        auto atB = [&](int dx, int dy, int dz) -> C {
          if constexpr (kWalls) {
            const int ox = dx < 0 ? xm : (dx > 0 ? xp : 0);
            const int oy = dy < 0 ? ym : (dy > 0 ? yp : 0);
            const int oz = dz < 0 ? zm : (dz > 0 ? zpl : 0);
            return phiB[ring3(p - 1 + oz)][ty + oy][tx + ox];
          } else {
            return phiB[ring3(p - 1 + dz)][ty + dy][tx + dx];
          }
        };
        C gr1[3], n1[3];
        gradient_normal<L, C>(atB, K.eps2, gr1, n1);
        C G[Q];
        phi_sources<L, C>(K, phi1, mu1, n1, G);
        const auto Gw = make_rsrc(reinterpret_cast<char*>(b.Gn) + zq * groupB, uint32_t(groupB));
        // storage narrower than double: the zeroth moment of the stored g is
        // balanced through the rest population (balance_g_rest), each moving
        // population stored as soon as it is computed; sg_old is the double
        // sum of these g, taken when they were pulled
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          if (sizeof(S) < sizeof(double) && k == L::REST) continue;
          C gk;
          if constexpr (kRegs)
            gk = g_old[k];
          else
            gk = gkeep[k][ty - 1][tx - 1];
          const S v = S(g_collide<L, C>(K, k, gk, phi1, G[k]));
          bstore_nt<S>(v, Gw, selfB, k * planeB);
          if (sizeof(S) < sizeof(double)) s = s + double(v);
        }
        if constexpr (sizeof(S) < sizeof(double)) {
          const double wg = K.omega_g_d;
          const double m0 = ((1.0 - wg) * sg_old + wg * double(phi1)) +
                            (1.0 - 0.5 * wg) * double(source_moment<C>(K, phi1, mu1));
          bstore_nt<S>(S(m0 - s), Gw, selfB, L::REST * planeB);
        }
      }
      if constexpr (kRegs) {
#pragma unroll
        for (int k = 0; k < Q; ++k) g_old[k] = C(gv[k]);
      } else {
        if (inner) {
#pragma unroll
          for (int k = 0; k < Q; ++k) gkeep[k][ty - 1][tx - 1] = C(gv[k]);
        }
      }
      if constexpr (kPrefetchG) {
        if (pulls_next) fetch_g(p + 1, gv);
      }
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

// 32-bit offsets inside a z plane group: Q * nx * ny * 8 bytes must fit
// (checked for the larger lattice, 19 populations); any boundary.
inline bool fused3d_supported(int nx, int ny, int nz, const int*) {
  return (int64_t)nx * ny * 19 * 8 < ((int64_t)1 << 32) && (int64_t)nx * ny * nz < ((int64_t)1 << 31);
}

// With zero-flux walls the e_z = +1 layer of the exchange is kept twice, so
// D3Q19 carries g in registers: FP64 on 64 x 5 tiles (one 8-wave block per
// CU, 4 of 256 VGPRs spilled; 512^3 20.5 ms against 20.6 without the prefetch, 256^3 2.45 against
// 2.61; carry in the LDS 21.0, 2.56), FP32 on 64 x 9 (12 waves; 9.95 against
// 11.0 ms, 1.29 against 1.38; 8 rows 10.4; carry in the LDS 10.4), in
// 32-plane chunks.
template <class L, class LH, class S>
struct Fused3DWallConfig : Fused3DConfig<L, LH, S> {};
template <class LH>
struct Fused3DWallConfig<D3Q19, LH, double> {
  static constexpr int TX = 64, TY = 5, ZC = 32;
  static constexpr Carry carry = Carry::kRegisters;
  static constexpr Prefetch prefetch = Prefetch::kBoth;
};
template <class LH>
struct Fused3DWallConfig<D3Q19, LH, float> {
  static constexpr int TX = 64, TY = 9, ZC = 32;
  static constexpr Carry carry = Carry::kRegisters;
  static constexpr Prefetch prefetch = Prefetch::kBoth;
};

// The general instantiation in FP64 with h on D3Q19 needs the registers of 8
// waves (64 x 5 tiles, g carried in registers), and with walls those of the
// prefetch too.  Periodic, h fetched ahead, in us against no prefetch and
// against the basic form's tiles: 317^3 5020 (5500, 5900), 438 x 438 x 26 826
// (910, 900), 256^3 2280 (2590, 2800).  With walls, without / with h fetched
// ahead: 238^3 2290 / 2640.
template <bool kWalls>
struct Fused3DGeneralConfig {
  static constexpr int TX = 64, TY = 5, ZC = 32;
  static constexpr Carry carry = Carry::kRegisters;
  static constexpr Prefetch prefetch = kWalls ? Prefetch::kNone : Prefetch::kH;
};

template <class L, class LH, class S, class C, bool kGen>
struct Fused3D {
  static constexpr bool kGeneral = kGen && sizeof(S) == 8 && LH::Q == 19;
  using Walls = std::conditional_t<kGeneral, Fused3DGeneralConfig<true>, Fused3DWallConfig<L, LH, S>>;
  using Periodic = std::conditional_t<kGeneral, Fused3DGeneralConfig<false>, Fused3DConfig<L, LH, S>>;

  // Tiles, chunk and resident blocks of a launch; slots <= 0 on an error.
  struct Plan {
    int tiles_x, tiles_xy, zc, ntiles, slots;
  };
  template <class Cfg, bool kWalls>
  static Plan plan(const Geo& g) {
    static int resident[64] = {0};
    Plan p{};
    p.slots = resident_slots(k_fused3d<Cfg::TX, Cfg::TY, Cfg::carry, Cfg::prefetch, L, LH, S, C, kGen, kWalls>,
                             TileShape<Cfg::TX, Cfg::TY>::NT, resident);
    if (p.slots <= 0) return p;
    p.tiles_x = (g.nx + Cfg::TX - 1) / Cfg::TX;
    p.tiles_xy = p.tiles_x * ((g.ny + Cfg::TY - 1) / Cfg::TY);
    p.zc = chunk_planes(p.tiles_xy, g.nz, Cfg::ZC, p.slots);
    p.ntiles = p.tiles_xy * ((g.nz + p.zc - 1) / p.zc);
    return p;
  }
  template <class Cfg, bool kWalls>
  static int run(const Geo& g, const Coef<C>& K, const StepBufs<S>& b, hipStream_t st) {
    const Plan p = plan<Cfg, kWalls>(g);
    if (p.slots <= 0) return -1;
    hipLaunchKernelGGL((k_fused3d<Cfg::TX, Cfg::TY, Cfg::carry, Cfg::prefetch, L, LH, S, C, kGen, kWalls>),
                       dim3(resident_grid(p.slots, p.ntiles)), dim3(TileShape<Cfg::TX, Cfg::TY>::NT),
                       0, st, g, K, b, p.tiles_x, p.tiles_xy, p.ntiles, p.zc);
    return 0;
  }
  // Planes that a step takes one after the other: passes over the resident
  // blocks times the planes of a chunk with its halo and the filling of the
  // rings (chunk_planes), of which a chunk at a z wall has fewer.  -1 on an
  // error.
  static double planes(const Geo& g) {
    const Plan p = (g.bcx || g.bcy || g.bcz) ? plan<Walls, true>(g) : plan<Periodic, false>(g);
    if (p.slots <= 0) return -1.0;
    const int passes = (p.ntiles + p.slots - 1) / p.slots;
    return passes * (p.zc + 3 - (g.bcz ? 1.5 * p.zc / g.nz : 0.0));
  }
  static int launch(const Geo& g, const Coef<C>& K, const StepBufs<S>& b, hipStream_t st) {
    if (g.bcx || g.bcy || g.bcz) return run<Walls, true>(g, K, b, st);
    return run<Periodic, false>(g, K, b, st);
  }
};

template <class L, class LH, class S, class C, bool kGen>
struct FusedLaunch {
  static int launch(const Geo& g, const Coef<C>& K, const StepBufs<S>& b, hipStream_t st) {
    if constexpr (L::D == 2)
      return Fused2D<L, LH, S, C, kGen>::launch(g, K, b, st);
    else
      return Fused3D<L, LH, S, C, kGen>::launch(g, K, b, st);
  }
};

}  // namespace gplbm
