// Fused schedule in 2-D: one kernel per time step n -> n+1.  g runs on
// D2Q9 or D2Q5 (L), h on D2Q9 or D2Q5 (LH).
//
// A block owns an output tile T of TX x TY nodes (x-aligned, tiles.h) and
// computes T grown by one node on each side (T+1).  Every thread of T+1:
//   - pulls h~^n (sum -> c^n, mu^n) and g~^{n+1} (kept in registers),
//   - reads phi^n around itself from an LDS tile covering T+2 (gradient,
//     normal, source moment), forms phi^{n+1} and writes it to an LDS tile,
//   - runs the h collision of step n (anti-trapping current from
//     phi^{n+1} - phi^n).
// The post-collision h* of T+1 are then streamed inside the block: they go to
// an LDS exchange, and after one barrier every node of T gathers the
// population k arriving from x - e_k (its own h*_{opp k} where x - e_k lies
// beyond a wall) in index order, so that c^{n+1} is summed in the same order
// as a pull would sum it.  Finally the threads of T run the g
// collision of step n+1 (gradient of phi^{n+1} from the LDS tile) and write
// g~*^{n+1}, h~*^n and phi^{n+1}.
//
// HBM traffic per node and step is the minimum: Q + Qh reads, Q + Qh writes,
// one phi read and one phi write, plus the recomputed halo ring where the L2
// misses it.  The grid is persistent with XCD-ordered passes (tiles.h).
#pragma once

#include "kernels_split.h"
#include "tiles.h"

namespace gplbm {

// Store of a population of the next state: past the caches (kStream) where the
// two states are well beyond the 256 MB of the last-level cache, so that
// writes that no step reads back in time do not displace what the next one
// pulls.  In us, regular / past the caches: FP64 1024^2 (319 MB) 75.6 / 71.6,
// 2048^2 270 / 263, FP32 1536^2 (359 MB) 91.0 / 87.0, FP16 2048^2 (403 MB) 146
// / 139; but FP64 1000^2 (304 MB) 66.7 / 67.6, FP16 1700^2 (277 MB) 98.2 / 106
// and FP32 1024^2 (159 MB) 30 / 41.
template <bool kStream, class S>
__device__ __forceinline__ void store_state(S v, S* p) {
  if constexpr (kStream)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}
inline bool streams_out(int64_t bytes) { return bytes > ((int64_t)300 << 20); }

// Addresses of a node's pulls in 2-D: the sources x - e_k by (e_x, e_y), wrapped
// on every axis, and with walls the populations that bounce.
template <bool kWalls>
struct Pull2D {
  int64_t src[3][3];  // in-plane offset of (x, y) + (c - 1, a - 1), [a][c]
  int64_t plane;
  bool xm, xp, ym, yp;  // the neighbour x - 1, x + 1, y - 1, y + 1 lies beyond a wall

  __device__ Pull2D(const Geo& g, int ux, int uy) : plane(g.N) {
    const int x = wrap_near(ux, g.nx), y = wrap_near(uy, g.ny);
    const int xo[3] = {x == 0 ? g.nx - 1 : x - 1, x, x == g.nx - 1 ? 0 : x + 1};
    const int yo[3] = {y == 0 ? g.ny - 1 : y - 1, y, y == g.ny - 1 ? 0 : y + 1};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int64_t row = (int64_t)yo[a] * g.nx;
#pragma unroll
      for (int c = 0; c < 3; ++c) src[a][c] = row + xo[c];
    }
    xm = kWalls && g.bcx && ux == 0;
    xp = kWalls && g.bcx && ux == g.nx - 1;
    ym = kWalls && g.bcy && uy == 0;
    yp = kWalls && g.bcy && uy == g.ny - 1;
  }
  __device__ int64_t self() const { return src[1][1]; }
  // population k of lattice P arrives from beyond a wall
  template <class P>
  __device__ bool bounced(int k) const {
    if (!kWalls) return false;
    return (P::ex[k] > 0 && xm) || (P::ex[k] < 0 && xp) || (P::ey[k] > 0 && ym) ||
           (P::ey[k] < 0 && yp);
  }
  // offset of the value population k pulls, in a distribution that stores
  // population j in plane m(j): one selected address, so that a node's pulls
  // stay one batch of loads without branches
  template <class P, class M>
  __device__ int64_t slot(int k, const M& m) const {
    const int64_t in = m(k) * plane + src[1 - P::ey[k]][1 - P::ex[k]];
    return bounced<P>(k) ? m(P::opp[k]) * plane + self() : in;
  }
  template <class P>
  __device__ int64_t slot(int k) const {
    return slot<P>(k, [](int j) { return j; });
  }
  // the gradient stencil's neighbour offset (mirror ghost at a wall)
  __device__ int sx(int dx) const { return dx < 0 ? (xm ? 0 : -1) : (dx > 0 ? (xp ? 0 : 1) : 0); }
  __device__ int sy(int dy) const { return dy < 0 ? (ym ? 0 : -1) : (dy > 0 ? (yp ? 0 : 1) : 0); }
};

// Bound by the issue of vector instructions where the state sits in the last
// level cache (FP64 at 512^2: 11 waves x about 700 instructions per tile,
// 4 cycles each, on 4 SIMDs is half of a pass of 8.7 us) and by memory beyond
// it (1024^2 4.3 TB/s, 2048^2 4.6 TB/s of algorithmic bytes).  Hence addresses
// without divisions or branches, and every load of a tile in one batch before
// the first barrier: 1024^2 FP64 85.2 -> 74.0 us, FP32 47.1 -> 30.0 us; 512^2
// FP64 22.4 -> 17.4, FP32 15.1 -> 10.1 us; 512 x 8 with walls 10.5 -> 5.3 us (6.0
// on tiles of 8 rows).
template <int TX, int TY, class L, class LH, class S, class C, bool kGen, bool kWalls, bool kStream>
__global__ void __launch_bounds__((TileShape<TX, TY>::NT), (sizeof(S) == 4 ? 6 : 1))
    k_fused2d(Geo g, Coef<C> Kin, StepBufs<S> b, int tiles_x, int ntiles) {
  const Coef<C> K = variant<kGen>(Kin);
  using Shape = TileShape<TX, TY>;
  constexpr int BX = Shape::BX, BY = Shape::BY, NT = Shape::NT;
  constexpr int AX = BX + 2, AY = BY + 2;  // phi^n tile with a 2-node halo
  constexpr int PHI_PER_THREAD = (AX * AY + NT - 1) / NT;
  // FP64 runs one block per CU with registers to spare: the next tile's loads
  // are issued after the h collision and arrive during the g collision (512^2
  // 18.1 -> 17.4 us; FP32, with two blocks per CU at 6 waves per SIMD, would
  // lose one of them, 10.1 -> 11.7 us)
  constexpr bool kPrefetch = sizeof(S) == 8;
  __shared__ C phiA[AY][AX];
  __shared__ C phiB[BY][BX];
  __shared__ C hx[LH::Q][BY][BX];  // h*^n of T+1 (moving populations)

  int tx, ty;
  bool valid;
  Shape::node(threadIdx.x, tx, ty, valid);

  // Every load of a tile: the pulls (of inactive nodes too, in range and not
  // used) and phi^n on T+2 (periodic wrap, or clamp = mirror ghost at a wall).
  auto fetch = [&](int tile, S (&hv)[LH::Q], S (&gv)[L::Q], S (&pv)[PHI_PER_THREAD]) {
    const int X0 = (tile % tiles_x) * TX, Y0 = (tile / tiles_x) * TY;
#pragma unroll
    for (int j = 0; j < PHI_PER_THREAD; ++j) {
      const int l = min((int)threadIdx.x + j * NT, AX * AY - 1);
      int vx = X0 - 2 + l % AX, vy = Y0 - 2 + l / AX;
      vx = kWalls && g.bcx ? min(max(vx, 0), g.nx - 1) : wrap_near(vx, g.nx);
      vy = kWalls && g.bcy ? min(max(vy, 0), g.ny - 1) : wrap_near(vy, g.ny);
      pv[j] = b.PHI[(int64_t)vy * g.nx + vx];
    }
    const Pull2D<kWalls> at(g, X0 - 1 + tx, Y0 - 1 + ty);
#pragma unroll
    for (int k = 0; k < LH::Q; ++k) hv[k] = b.H[at.template slot<LH>(k)];
#pragma unroll
    for (int k = 0; k < L::Q; ++k) gv[k] = b.G[at.template slot<L>(k)];
  };
  S hv[LH::Q], gv[L::Q], pv[PHI_PER_THREAD];
  if (first_tile() < ntiles) fetch(first_tile(), hv, gv, pv);

  for (int tile = first_tile(); tile < ntiles; tile += gridDim.x) {
    const int X0 = (tile % tiles_x) * TX, Y0 = (tile / tiles_x) * TY;
    const int ux = X0 - 1 + tx, uy = Y0 - 1 + ty;  // unwrapped node of this thread
    // region nodes beyond a wall take no part
    const bool active = valid && (!kWalls || ((!g.bcx || (ux >= 0 && ux < g.nx)) &&
                                              (!g.bcy || (uy >= 0 && uy < g.ny))));
    const bool out = valid && ux < g.nx && uy < g.ny && tx >= 1 && tx <= TX && ty >= 1 && ty <= TY;
    const Pull2D<kWalls> at(g, ux, uy);
    const int64_t i = at.self();
#pragma unroll
    for (int j = 0; j < PHI_PER_THREAD; ++j) {
      const int l = threadIdx.x + j * NT;
      if (l < AX * AY) phiA[l / AX][l % AX] = C(pv[j]);
    }
    __syncthreads();

    C gn[L::Q];   // g~^{n+1}
    C hs[LH::Q];  // h~*^n
    C h[LH::Q];
    double c = 0.0;
#pragma unroll
    for (int k = 0; k < LH::Q; ++k) {
      h[k] = C(hv[k]);
      c = k == 0 ? double(hv[k]) : c + double(hv[k]);
    }
    double sg = 0.0;
#pragma unroll
    for (int k = 0; k < L::Q; ++k) {
      gn[k] = C(gv[k]);
      sg = k == 0 ? double(gv[k]) : sg + double(gv[k]);
    }
    {
      const C phi = phiA[ty + 1][tx + 1];
      const C mu = C(closure(K.q, c, double(phi)));
      auto atA = [&](int dx, int dy, int) -> C {
        return phiA[ty + 1 + at.sy(dy)][tx + 1 + at.sx(dx)];
      };
      C gr[3], n[3];
      gradient_normal<L, C>(atA, K.eps2, gr, n);
      const C sbar = source_moment<C>(K, phi, mu);
      const C phin = C(sg + 0.5 * double(sbar));
      C F[3];
      h_flux<L, C>(K, mu, gr, n, phin - phi, K.anti_trapping != 0, F);
      const C lam = h_lambda<C>(K, phi, mu);
      const C cc = C(c);
      h_update<LH>(K, h, cc, lam, F, hs);
      balance_rest<LH, S, C>(hs, c);
      if (active) {
        phiB[ty][tx] = phin;
#pragma unroll
        for (int k = 0; k < LH::Q; ++k)
          if (k != LH::REST) hx[k][ty][tx] = hs[k];
      }
      if (out) {
#pragma unroll
        for (int k = 0; k < LH::Q; ++k) store_state<kStream>(S(hs[k]), &b.Hn[k * at.plane + i]);
        b.PHIn[i] = S(phin);
      }
    }
    if (kPrefetch && tile + gridDim.x < ntiles) fetch(tile + gridDim.x, hv, gv, pv);
    __syncthreads();

    if (out) {
      // streaming of h* inside the tile: population k arrives from x - e_k, or
      // is this node's own h*_{opp k} bounced back where x - e_k is beyond a wall
      double c1 = 0.0;
#pragma unroll
      for (int k = 0; k < LH::Q; ++k) {
        C v = hs[k];
        if (k != LH::REST) {
          const C in = hx[k][ty - LH::ey[k]][tx - LH::ex[k]];
          v = at.template bounced<LH>(k) ? hs[LH::opp[k]] : in;
        }
        c1 = k == 0 ? double(v) : c1 + double(v);
      }
      const C phi1 = phiB[ty][tx];
      const C mu1 = C(closure(K.q, c1, double(phi1)));
      auto atB = [&](int dx, int dy, int) -> C { return phiB[ty + at.sy(dy)][tx + at.sx(dx)]; };
      C gr[3], n[3];
      gradient_normal<L, C>(atB, K.eps2, gr, n);
      C G[L::Q];
      phi_sources<L, C>(K, phi1, mu1, n, G);
      C gs[L::Q];
#pragma unroll
      for (int k = 0; k < L::Q; ++k) gs[k] = C(S(g_collide<L, C>(K, k, gn[k], phi1, G[k])));
      balance_g_rest<L, S, C>(K, gs, sg, phi1, source_moment<C>(K, phi1, mu1));
#pragma unroll
      for (int k = 0; k < L::Q; ++k) store_state<kStream>(S(gs[k]), &b.Gn[k * at.plane + i]);
    }
    if (!kPrefetch && tile + gridDim.x < ntiles) fetch(tile + gridDim.x, hv, gv, pv);
    __syncthreads();  // the LDS tiles are refilled by the next tile
  }
}

inline bool fused2d_supported(int, int) { return true; }

// Rows per tile of the 2-D kernels: of 1, 4, 8 and (where `tall`) 13 the
// height of least cost, passes over the CUs x rows of a tile with its halo.
// A small grid is then one pass of short blocks, a wave or two per SIMD (FP64
// 128^2 7.4 us with 8 rows, 6.3 with 4, 4.9 with 1; 256^2 8.1, 6.8 and 8.7;
// 512^2 16.9, 18.4 and 24.7), and a strip may fit one pass of tall ones (5000
// x 36 17.7 us with 8 rows, 13.8 with 13).  FP32 and the deviations run two
// blocks of 8 rows per CU, which 13 rows would not (FP32 512^2 10.1 and 14.6
// us, FP16 10.5 and 14.6 us).
inline int tile_rows(int nx, int ny, int tx, bool tall) {
  constexpr int kCus = 256;  // of an MI355X; on a part of one the choice is of another cost
  const int64_t columns = (nx + tx - 1) / tx;
  int best = 8;
  int64_t cost = INT64_MAX;
  for (int rows : {1, 4, 8, 13}) {
    if (rows > 8 && !tall) continue;
    const int64_t tiles = columns * ((ny + rows - 1) / rows);
    const int64_t c = (tiles + kCus - 1) / kCus * (rows + 2);
    if (c < cost) cost = c, best = rows;
  }
  return best;
}

template <class L, class LH, class S, class C, bool kGen>
struct Fused2D {
  template <int TY, bool kWalls>
  static int run(const Geo& g, const Coef<C>& K, const StepBufs<S>& b, hipStream_t st) {
    // for the tiles of 8 rows and more that large grids take; strips of a few
    // rows that are as large would gain 1-4% (300000 x 4 FP64 93 -> 89 us,
    // 2000000 x 4 565 -> 558), which is not worth two more sets of kernels
    if constexpr (TY >= 8)
      if (streams_out((int64_t)(2 * (L::Q + LH::Q + 1)) * g.N * sizeof(S)))
        return run<TY, kWalls, true>(g, K, b, st);
    return run<TY, kWalls, false>(g, K, b, st);
  }
  template <int TY, bool kWalls, bool kStream>
  static int run(const Geo& g, const Coef<C>& K, const StepBufs<S>& b, hipStream_t st) {
    constexpr int TX = 64;
    constexpr int NT = TileShape<TX, TY>::NT;
    auto kernel = k_fused2d<TX, TY, L, LH, S, C, kGen, kWalls, kStream>;
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
  static int by_rows(const Geo& g, const Coef<C>& K, const StepBufs<S>& b, hipStream_t st) {
    const int rows = tile_rows(g.nx, g.ny, 64, sizeof(S) == 8);
    if (rows == 1) return run<1, kWalls>(g, K, b, st);
    if (rows == 4) return run<4, kWalls>(g, K, b, st);
    if constexpr (sizeof(S) == 8)
      if (rows == 13) return run<13, kWalls>(g, K, b, st);
    return run<8, kWalls>(g, K, b, st);
  }
  static int launch(const Geo& g, const Coef<C>& K, const StepBufs<S>& b, hipStream_t st) {
    return (g.bcx || g.bcy) ? by_rows<true>(g, K, b, st) : by_rows<false>(g, K, b, st);
  }
};

}  // namespace gplbm
