// Hand-written adjoint (reverse mode) of the coupled step, FP64.
//
// The forward step maps the state S_n = (G = g~*^n, H = h~*^{n-1}, PHI = phi^n)
// to S_{n+1} (geometry.h).  Given the adjoint of S_{n+1} (Gb', Hb', Pb') and
// the forward states S_n and S_{n+1}, one reverse step produces the adjoint of
// S_n and accumulates the parameter adjoints (lambda, D_l) per node.  Every
// operation of the step is linear in the populations, so the reverse of a
// collision is a weighted copy; the nonlinear parts (closure products, p'(phi),
// the normal, mu D' grad phi, the anti-trapping product, D(phi) mu) are
// differentiated by hand at the forward values, which the reverse kernels
// recompute from S_n and S_{n+1}.
//
// Two kernels per reverse step (each node reads its neighbours only through
// the previous kernel's output):
//   ra: gathers the adjoint of G' from the previous reverse step, then the
//       reverse of the g collision of step n+1: adjoint of the pulled
//       g~^{n+1} (A1), of grad phi^{n+1} (A2, plus the previous step's B3),
//       of c^{n+1} (A3) and the local adjoint of phi^{n+1} (A4, plus the
//       previous step's B4);
//   rb: adjoint of h~*^n (gathered from the previous step, plus c^{n+1} from
//       the node it streams to), total adjoint of phi^{n+1} (A4 and the
//       stencil transpose of A2), reverse of the h collision of step n and of
//       phi^{n+1} = sum g~^{n+1} + S^n / 2: B1, B2, B3, B4.
// The transposes of the pulls and of the gradient stencil are done as gathers
// by the consumer, so the adjoint of a state is never written out.  Bound by
// memory on large grids (256^3 D3Q19: 19.2 GB of algorithmic bytes in 4.2 ms
// with threads over 64 x 4 tiles and 64-bit indices, 3.8 ms with threads over
// the nodes of a plane, scalar plane bases and every load issued first) and by
// latency and idle lanes on small ones (96^3 290 -> 217 us, with walls 485 ->
// 243 us).
// Parameters are held fixed except lambda and D_l (gamma, M_phi, W and a do
// not follow D_l).
#pragma once

#include <type_traits>

#include "kernels_dev.h"
#include "kernels_split.h"

namespace gplbm {

// Intermediates of one reverse step that the next one (or the reverse of the
// initialisation) gathers from; double-buffered by step parity.  The adjoint
// of the state S_n is never materialised: its G, H and PHI parts are the
// gathers  Gb(slot) = A1(dest) + B2(dest),  Hb(slot) = B1(dest),
// Pb = B4 + stencil transpose of B3  (dest = the node and population that
// pull the slot).
struct AdjSet {
  double* A1;  // Q*N: adjoint of the pulled g~^{n+1}
  double* B1;  // Q*N: adjoint of the pulled h~^n
  double* B2;  // N:   adjoint of phi^{n+1} (every pulled g adds to it)
  double* B3;  // 3*N: adjoint of grad phi^n
  double* B4;  // N:   local adjoint of phi^n
};

struct AdjWork {
  AdjSet set[2];
  double *A2, *A3, *A4;  // 3*N, N, N: adjoint of grad phi^{n+1}, c^{n+1}, local phi^{n+1}
  double *lamb, *dlb;    // per-node accumulators of dJ/dlambda, dJ/dD_l
  double* red;           // reduction scratch
};

// A forward state in the storage type S of the context (FP64 or FP32); the
// reverse kernels recompute the forward quantities from it in FP64.
template <class S>
struct FwdState {
  const S* G;
  const S* H;
  const S* PHI;
};

// A forward state in a deviation format (any lattices): the h populations decode
// with the Lambda field of the state, phi is FP32.  The reverse kernels take
// the decoded values as the state and differentiate the FP64 step there.
template <class Codec>
struct DevFwdState {
  DevDist H;
  const float* PHI;
  const float* LAM;
};

// Population planes of a distribution, and of a field.
struct PopPlane {
  __device__ int operator()(int k) const { return k; }
};
struct FieldPlane {
  __device__ int operator()(int) const { return 0; }
};

// Forward quantities at one node from a state: c, mu, phi, grad phi, normal.
template <class L>
struct NodeFwd {
  double c, mu, phi, g[3], n[3], s;  // s = sqrt(|grad|^2 + eps^2)
};

// c, phi and the stencil values to the forward quantities.
template <class L>
__device__ __forceinline__ NodeFwd<L> node_fwd_from(const Coef<double>& K, double c, double phi,
                                                    const Stencil<L, double>& st) {
  NodeFwd<L> f;
  f.c = c;
  f.phi = phi;
  f.mu = closure(K.q, c, phi);
  gradient_normal<L, double>(st, K.eps2, f.g, f.n);
  double nn = f.g[0] * f.g[0] + f.g[1] * f.g[1];
  if (L::D == 3) nn = nn + f.g[2] * f.g[2];
  f.s = sqrt(nn + K.eps2);
  return f;
}

// Loads of a node's forward quantities from a state, and their evaluation.
template <class L, class LH, class FS>
struct FwdLoads;
template <class L, class LH, class S>
struct FwdLoads<L, LH, FwdState<S>> {
  Stencil<L, double> st;
  S hv[LH::Q];
  template <class A>
  __device__ FwdLoads(const FwdState<S>& F, const A& a) : st(a, F.PHI) {
#pragma unroll
    for (int k = 0; k < LH::Q; ++k) hv[k] = a.template pull_pop<LH>(F.H, k);
  }
  template <class A>
  __device__ NodeFwd<L> eval(const Coef<double>& K, const A&) const {
    double c = 0.0;
#pragma unroll
    for (int k = 0; k < LH::Q; ++k) c = k == 0 ? double(hv[k]) : c + double(hv[k]);
    return node_fwd_from<L>(K, c, st(0, 0, 0), st);
  }
};
template <class L, class LH, class Codec>
struct FwdLoads<L, LH, DevFwdState<Codec>> {
  Stencil<L, double> st;
  Stencil<LH, float> sl;
  DevPulls<LH> ph;
  template <class A>
  __device__ FwdLoads(const DevFwdState<Codec>& F, const A& a) : st(a, F.PHI), sl(a, F.LAM), ph(a, F.H) {}
  template <class A>
  __device__ NodeFwd<L> eval(const Coef<double>& K, const A& a) const {
    double c = 0.0;
#pragma unroll
    for (int k = 0; k < LH::Q; ++k) {
      const double v = double(ph.template value<Codec>(a, sl, k));
      c = k == 0 ? v : c + v;
    }
    return node_fwd_from<L>(K, c, st(0, 0, 0), st);
  }
};

// The same where c is known: between the steps of a segment on a periodic grid,
// the second kernel of a reverse step n + 1 leaves the c^{n+1} that it summed
// for the first kernel of step n, which then reads one value instead of pulling
// LH::Q: 96^3 FP64 212 -> 197 us a step, FP32 178 -> 169, 256^3 FP64 3.77 ->
// 3.55 ms, 512^2 FP64 33.4 -> 31.2 us.  With walls it lost (80^3
// FP64 141 -> 146-151 us, 96^3 243 -> 250).
template <class Addr>
constexpr bool hands_c_on() {
  return std::is_same<Addr, AddrPlane<false>>::value;
}
template <class L>
struct FwdCarried {
  Stencil<L, double> st;
  double c;
  template <class S, class A>
  __device__ FwdCarried(const S* phi, const double* cf, const A& a) : st(a, phi), c(cf[a.node()]) {}
  template <class A>
  __device__ NodeFwd<L> eval(const Coef<double>& K, const A&) const {
    return node_fwd_from<L>(K, c, st(0, 0, 0), st);
  }
};

// Derivatives of the closure mu(c, phi): 1 and c_s - c_l for equal
// curvatures; for general quadratic free energies, with
// mu = fac (c - phi m_l - (1 - phi) m_s), fac = E / (eps_s phi + eps_l (1 - phi)):
// d mu / dc = fac, d mu / dphi = -fac (eps_s - eps_l) / den r + fac (m_s - m_l).
__device__ __forceinline__ void closure_grad(const Coef<double>& K, double c, double phi,
                                             double& dmu_dc, double& dmu_dphi) {
  if (K.q.quad) {
    const double den = (K.q.eps_s * phi) + (K.q.eps_l * (1.0 - phi));
    const double fac = K.q.efac / den;
    const double r = (c - phi * K.q.m_l) - (1.0 - phi) * K.q.m_s;
    dmu_dc = fac;
    dmu_dphi = -fac * (K.q.eps_s - K.q.eps_l) / den * r + fac * (K.q.m_s - K.q.m_l);
  } else {
    dmu_dc = 1.0;
    dmu_dphi = K.q.cs - K.q.cl;
  }
}

// Bracket B(mu) of S_phi = p'(phi) B and its slope B'(mu): dc (mu - mu_eq) and
// dc, or k2 mu^2 / 2 - (m_l - m_s) mu - df_min and k2 mu - (m_l - m_s).
__device__ __forceinline__ void bracket_and_slope(const Coef<double>& K, double mu, double& B,
                                                  double& Bp) {
  if (K.fe_quad) {
    B = ((K.k2 * (mu * mu)) * 0.5 - (K.dml * mu)) - K.dfm;
    Bp = K.k2 * mu - K.dml;
  } else {
    B = K.dc * (mu - K.mueq_c);
    Bp = K.dc;
  }
}

// Adjoint of the phi sources G_k (given their adjoints Gb_k) and of the
// extra adjoint sbar_b of their zeroth moment, at (phi, mu, n).  Adds to
// phi_b, mu_b, n_b and returns the lambda adjoint.
template <class L>
__device__ __forceinline__ double sources_adj(const Coef<double>& K, double lam_M_W2, double phi,
                                              double mu, const double n[3], const double* Gb,
                                              double sbar_b, double& phi_b, double& mu_b,
                                              double nb[3]) {
  const double pp = phi * (1.0 - phi);
  // p' of the coupling takes phi limited to [0, 1] (zero derivative outside)
  const double pl = limit01(phi);
  const double ppl = pl * (1.0 - pl);
  const bool in01 = phi >= 0.0 && phi <= 1.0;
  double Gst_b = sbar_b, kphi_b = 0.0, Gdw_b = 0.0;
  if (K.counter_term) {
#pragma unroll
    for (int k = 0; k < L::Q; ++k) {
      if (Gb == nullptr) break;
      const double wg = L::w[k] * Gb[k];
      Gst_b += wg;
      if (k != L::REST) {
        const double en = edot<L, double>(k, n[0], n[1], n[2]);
        kphi_b += en * wg;
        const double kphi = K.k4w * pp;
        if (L::ex[k]) nb[0] += (L::ex[k] > 0 ? 1.0 : -1.0) * kphi * wg;
        if (L::ey[k]) nb[1] += (L::ey[k] > 0 ? 1.0 : -1.0) * kphi * wg;
        if (L::D == 3 && L::ez[k]) nb[2] += (L::ez[k] > 0 ? 1.0 : -1.0) * kphi * wg;
      }
    }
  } else {
    double s = 0.0;
    if (Gb != nullptr) {
#pragma unroll
      for (int k = 0; k < L::Q; ++k) s += L::w[k] * Gb[k];
    }
    Gst_b += s;
    Gdw_b = s + sbar_b;
  }
  double B, Bp;
  bracket_and_slope(K, mu, B, Bp);
  const double Sphi = (6.0 * ppl) * B;
  const double ppl_b = (K.kst * 6.0 * B) * Gst_b;
  double pp_b = K.k4w * kphi_b;
  mu_b += (K.kst * 6.0 * ppl * Bp) * Gst_b;
  if (!K.counter_term) {
    pp_b += K.kdw * 2.0 * (1.0 - 2.0 * phi) * Gdw_b;
    phi_b += K.kdw * 2.0 * pp * (-2.0) * Gdw_b;
  }
  phi_b += (1.0 - 2.0 * phi) * pp_b;
  if (in01) phi_b += (1.0 - 2.0 * pl) * ppl_b;
  return -lam_M_W2 * Sphi * Gst_b;
}

// Adjoint of the normal n = g / s: adds the gradient adjoint to gb.
template <class L>
__device__ __forceinline__ void normal_adj(const NodeFwd<L>& f, const double nb[3], double gb[3]) {
  const double nd = f.n[0] * nb[0] + f.n[1] * nb[1] + (L::D == 3 ? f.n[2] * nb[2] : 0.0);
  for (int a = 0; a < L::D; ++a) gb[a] += (nb[a] - f.n[a] * nd) / f.s;
}

// Gather of the transposed gradient stencil at node (x, y, z):
// sum over k != rest and over the nodes q with stencil(q + e_k) = (x, y, z)
// of (1 / xi_s^2) w_k e_k . gb(q).
__device__ __forceinline__ int preimage(int z, int e, int n, int bc, int out[2]) {
  if (!bc) {
    int v = z - e;
    v = v < 0 ? v + n : (v >= n ? v - n : v);
    out[0] = v;
    return 1;
  }
  int m = 0;
  if (e == 0) {
    out[m++] = z;
  } else if (e > 0) {
    if (z - 1 >= 0) out[m++] = z - 1;
    if (z == n - 1) out[m++] = z;
  } else {
    if (z + 1 <= n - 1) out[m++] = z + 1;
    if (z == 0) out[m++] = z;
  }
  return m;
}

template <class L>
__device__ __forceinline__ double stencil_adj_gather(const Geo& g, const double* gb3, int x, int y,
                                                     int z) {
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    if (k == L::REST) continue;
    int px[2], py[2], pz[2];
    const int mx = preimage(x, L::ex[k], g.nx, g.bcx, px);
    const int my = preimage(y, L::ey[k], g.ny, g.bcy, py);
    const int mz = L::D == 3 ? preimage(z, L::ez[k], g.nz, g.bcz, pz) : (pz[0] = z, 1);
    for (int a = 0; a < mx; ++a)
      for (int b = 0; b < my; ++b)
        for (int c = 0; c < mz; ++c) {
          const int64_t q = node_index(g, px[a], py[b], pz[c]);
          const double e_g = edot<L, double>(k, gb3[q], gb3[g.N + q], L::D == 3 ? gb3[2 * g.N + q] : 0.0);
          acc += L::inv_cs2 * L::w[k] * e_g;
        }
  }
  return acc;
}

// --------------------------------------------------------------------------

// The same gather in the addressing of a node: away from walls there is one
// preimage per population, x - e_k; a wavefront with a node next to a wall
// takes the general form.
template <class L, class A>
__device__ __forceinline__ double stencil_adj_gather_at(const Geo& g, const double* gb3, const A& a) {
  if (__builtin_amdgcn_ballot_w64(a.edge()) != 0u)
    return stencil_adj_gather<L>(g, gb3, a.x, a.y, a.z);
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    if (k == L::REST) continue;
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int d = 0; d < L::D; ++d)
      if ((d == 0 && L::ex[k]) || (d == 1 && L::ey[k]) || (d == 2 && L::ez[k]))
        v[d] = a.at(gb3 + d * g.N, -L::ex[k], -L::ey[k], -L::ez[k]);
    acc += L::inv_cs2 * L::w[k] * edot<L, double>(k, v[0], v[1], v[2]);
  }
  return acc;
}

// Adjoint of G' in slot k of the node, gathered from the previous set.
template <class L, class A>
__device__ __forceinline__ double gather_Gb(const AdjSet& P, int k, const A& a) {
  return *a.template dest<L>((const double*)P.A1, k, L::Q, PopPlane{}) +
         *a.template dest<L>((const double*)P.B2, k, 1, FieldPlane{});
}

// kGen: the general instantiation keeps the scheme flags (h^eq,alt, general
// free energies) of the run; the basic one fixes them off at compile time.
// The two halves of a reverse step at one node (the two kernels below).
//
// reverse_g: the reverse of the g collision of step n+1.  Writes the adjoint
// of the node's pulled g~^{n+1} (C.A1), and returns the adjoint of grad
// phi^{n+1} with the previous step's B3 added (a2), of c^{n+1} (a3), the local
// adjoint of phi^{n+1} with the previous step's B4 added (a4), and the lambda
// adjoint (lb).  The h collision of step n+1 (previous reverse
// step) also used grad phi^{n+1} and phi^{n+1}: their adjoints are added here,
// so that the second half applies the transposed stencil once.
template <class L, class LH, class FS, bool kCarried, class Addr>
__device__ __forceinline__ void reverse_g(const Geo& g, const Coef<double>& K, double lam_M_W2,
                                          const FS& S1, const double* c1, const AdjSet& P,
                                          const AdjSet& C, const Addr& ad, double (&a2)[3],
                                          double& a3, double& a4, double& lb) {
  const int64_t i = ad.node();
  const auto fwd = [&] {
    if constexpr (kCarried)
      return FwdCarried<L>(S1.PHI, c1, ad);
    else
      return FwdLoads<L, LH, FS>(S1, ad);
  }();
  double a_in[L::Q];
#pragma unroll
  for (int k = 0; k < L::Q; ++k) a_in[k] = gather_Gb<L>(P, k, ad);
  double b3[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int a = 0; a < L::D; ++a) b3[a] = P.B3[a * g.N + i];
  const double b4 = P.B4[i];
  loads_issued();
  const NodeFwd<L> f = fwd.eval(K, ad);  // c^{n+1}, mu^{n+1}, ...
  const double om = K.omega_g;
  double Gb[L::Q];
  double phi_b = 0.0, mu_b = 0.0, nb[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    const double a = a_in[k];
    C.A1[ad.slot(k, L::Q)] = (1.0 - om) * a;
    Gb[k] = (1.0 - 0.5 * om) * a;
    phi_b += om * L::w[k] * a;
  }
  lb = sources_adj<L>(K, lam_M_W2, f.phi, f.mu, f.n, Gb, 0.0, phi_b, mu_b, nb);
  double gb[3] = {0.0, 0.0, 0.0};
  normal_adj<L>(f, nb, gb);
  for (int a = 0; a < 3; ++a) a2[a] = a < L::D ? gb[a] + b3[a] : 0.0;
  double dmu_dc, dmu_dphi;
  closure_grad(K, f.c, f.phi, dmu_dc, dmu_dphi);
  a3 = dmu_dc * mu_b;   // adjoint of c^{n+1}
  phi_b += dmu_dphi * mu_b;  // closure
  a4 = phi_b + b4;
}

// reverse_h: the reverse of the h collision of step n and of phi^{n+1} =
// sum g~^{n+1} + S^n / 2.  p1b: the adjoint of
// phi^{n+1} at this node gathered so far (a4 and the transposed stencil of
// a2).  Writes B1 .. B4 of the node into C, accumulates its parameter adjoints
// and with keep_c leaves c^n in A4.
template <class L, class LH, class FS, class Addr>
__device__ __forceinline__ void reverse_h(const Geo& g, const Coef<double>& K, double lam_M_W2,
                                          const FS& S0, const FS& S1, const AdjSet& P,
                                          const AdjSet& C, const AdjWork& w, const Addr& ad,
                                          double p1b, bool keep_c) {
  const int64_t i = ad.node();
  const FwdLoads<L, LH, FS> fwd(S0, ad);
  // total adjoint of h~*^n in this node's slots
  double Hb[LH::Q];
#pragma unroll
  for (int k = 0; k < LH::Q; ++k)
    Hb[k] = *ad.template dest<LH>((const double*)P.B1, k, LH::Q, PopPlane{}) +
            *ad.template dest<LH>((const double*)w.A3, k, 1, FieldPlane{});
  const double phi1 = double(S1.PHI[i]), lamb = w.lamb[i], dlb = w.dlb[i];
  loads_issued();
  // forward quantities of step n
  const NodeFwd<L> f = fwd.eval(K, ad);
  const double dtphi = phi1 - f.phi;
  const double oh = K.omega_h;
  const double Dp = K.Dp;
  // D = D_l q + D_s (1 - q), q = phi limited to [0, 1]
  const double qd = limit01(f.phi);
  const double D = (K.Dl * qd) + (K.Ds * (1.0 - qd));
  const bool q_in = f.phi >= 0.0 && f.phi <= 1.0;
  // reverse of h* = (1 - oh) h + oh heq + (1 - oh/2) H
  double hb[LH::Q];
  double c_b = 0.0, lam_b = 0.0, Fb[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) {
    hb[k] = (1.0 - oh) * Hb[k];
    const double heq_b = oh * Hb[k];
    if (k == LH::REST) {
      c_b += heq_b;
      lam_b += -(1.0 - LH::w[k]) * heq_b;
    } else {
      lam_b += LH::w[k] * heq_b;
      // the flux enters through H_k = gamma w_k e_k.F (source scheme) or
      // through h^eq,alt_k = w_k (Lambda + e_k.F / xi_s^2)
      const double HHb = K.h_alt ? heq_b * (LH::w[k] * LH::inv_cs2)
                                 : (1.0 - 0.5 * oh) * Hb[k] * (K.gamma * LH::w[k]);
      if (LH::ex[k]) Fb[0] += (LH::ex[k] > 0 ? HHb : -HHb);
      if (LH::ey[k]) Fb[1] += (LH::ey[k] > 0 ? HHb : -HHb);
      if (LH::D == 3 && LH::ez[k]) Fb[2] += (LH::ez[k] > 0 ? HHb : -HHb);
    }
  }
  double mu_b = 0.0, phi_b = 0.0, dl_b = 0.0, gb[3] = {0.0, 0.0, 0.0}, nb[3] = {0.0, 0.0, 0.0};
  // Lambda = gamma D mu
  mu_b += K.gamma * D * lam_b;
  const double D_b = K.gamma * f.mu * lam_b;
  if (q_in) phi_b += (K.Dl - K.Ds) * D_b;
  dl_b += qd * D_b;
  // F = mu D' grad + jfac dtphi n
  const double gF = f.g[0] * Fb[0] + f.g[1] * Fb[1] + (L::D == 3 ? f.g[2] * Fb[2] : 0.0);
  mu_b += Dp * gF;
  dl_b += f.mu * gF;
  for (int a = 0; a < L::D; ++a) gb[a] += f.mu * Dp * Fb[a];
  if (K.anti_trapping) {
    const double nF = f.n[0] * Fb[0] + f.n[1] * Fb[1] + (L::D == 3 ? f.n[2] * Fb[2] : 0.0);
    // j_at = jf dphi/dt n, jf = a W dc, or a W (ks mu + m_s - m_l)
    const double jf = K.fe_quad ? K.aW * ((K.ks * f.mu + K.ms) - K.ml) : K.jfac;
    const double dt_b = jf * nF;
    for (int a = 0; a < L::D; ++a) nb[a] += jf * dtphi * Fb[a];
    if (K.fe_quad) mu_b += K.aW * K.ks * dtphi * nF;
    p1b += dt_b;
    phi_b -= dt_b;
  }
  // phi^{n+1} = sum g~^{n+1} + sbar^n / 2
  const double lb = sources_adj<L>(K, lam_M_W2, f.phi, f.mu, f.n, nullptr, 0.5 * p1b, phi_b, mu_b, nb);
  normal_adj<L>(f, nb, gb);
  // closure and c^n = sum h~^n
  {
    double dmu_dc, dmu_dphi;
    closure_grad(K, f.c, f.phi, dmu_dc, dmu_dphi);
    c_b += dmu_dc * mu_b;
    phi_b += dmu_dphi * mu_b;
  }
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) C.B1[ad.slot(k, LH::Q)] = hb[k] + c_b;
  C.B2[i] = p1b;
  for (int a = 0; a < 3; ++a) C.B3[a * g.N + i] = gb[a];
  C.B4[i] = phi_b;
  if constexpr (hands_c_on<Addr>())
    if (keep_c) w.A4[i] = f.c;  // its reader is this thread, above
  w.lamb[i] = lamb + lb;
  w.dlb[i] = dlb + dl_b;
}

// kCarried: A4 holds c^{n+1}, left there by k_adj_rb of the step before.
template <class L, class LH, class FS, bool kGen, bool kCarried, class Addr>
__global__ void __launch_bounds__(256) k_adj_ra(Geo g, Coef<double> Kin, double lam_M_W2,
                                                FS S1, AdjSet P, AdjSet C, AdjWork w) {
  const Coef<double> K = variant<kGen>(Kin);
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  double a2[3], a3, a4, lb;
  const double lamb = w.lamb[i];
  reverse_g<L, LH, FS, kCarried>(g, K, lam_M_W2, S1, (const double*)w.A4, P, C, ad, a2, a3, a4, lb);
  for (int a = 0; a < L::D; ++a) w.A2[a * g.N + i] = a2[a];
  w.A3[i] = a3;
  w.A4[i] = a4;
  w.lamb[i] = lamb + lb;
}

template <class L, class LH, class FS, bool kGen, class Addr>
__global__ void __launch_bounds__(256) k_adj_rb(Geo g, Coef<double> Kin, double lam_M_W2,
                                                FS S0, FS S1, AdjSet P, AdjSet C, AdjWork w,
                                                bool keep_c) {
  const Coef<double> K = variant<kGen>(Kin);
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  // adjoint of phi^{n+1} at this node (A2, A4 hold both collisions' parts)
  const double p1b = w.A4[i] + stencil_adj_gather_at<L>(g, (const double*)w.A2, ad);
  reverse_h<L, LH>(g, K, lam_M_W2, S0, S1, P, C, w, ad, p1b, keep_c);
}

// Seed: the adjoint of S_K from dJ/dphi^K and dJ/dc^K (c^K = sum of the
// pulled H), written as a set the first reverse step gathers from:
// Gb = 0, Hb(slot) = dJ/dc^K(dest), Pb = dJ/dphi^K.
template <class L, class LH, class Addr>
__global__ void __launch_bounds__(256) k_adj_seed(Geo g, const double* __restrict__ phib,
                                                  const double* __restrict__ cb, AdjSet P, AdjWork w) {
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  const double cv = cb ? cb[i] : 0.0;
#pragma unroll
  for (int k = 0; k < L::Q; ++k) P.A1[ad.slot(k, L::Q)] = 0.0;
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) P.B1[ad.slot(k, LH::Q)] = cv;
  P.B2[i] = 0.0;
  for (int a = 0; a < 3; ++a) P.B3[a * g.N + i] = 0.0;
  P.B4[i] = phib ? phib[i] : 0.0;
  w.lamb[i] = 0.0;
  w.dlb[i] = 0.0;
}

// Adjoint of the initialisation (phi0, c0) -> S_0, local part: writes the
// adjoint of c0 and, in B4 / B3, the local part of the adjoint of phi0 and the
// adjoint of grad phi0.
template <class L, class LH, class Addr>
__global__ void __launch_bounds__(256) k_adj_init_a(Geo g, Coef<double> K, double lam_M_W2,
                                                    const double* __restrict__ phi0,
                                                    const double* __restrict__ c0, AdjSet P,
                                                    AdjSet C, AdjWork w, double* __restrict__ c0b) {
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  const Stencil<L, double> st(ad, phi0);
  const double phi = st(0, 0, 0), cin = c0[i];
  const NodeFwd<L> f = node_fwd_from<L>(K, cin, phi, st);
  const double mu0 = f.mu;
  // forward h~^0 and c^0
  double F[3];
  h_flux<L, double>(K, mu0, f.g, f.n, 0.0, false, F);
  const double lam = h_lambda<double>(K, phi, mu0);
  double c = 0.0;
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) {
    const double hv = h_initial<LH, double>(K, k, cin, lam, F);
    c = k == 0 ? hv : c + hv;
  }
  const double mu = closure(K.q, c, phi);
  // adjoints of the pulled h~^0 (from H of S_0) and of G of S_0
  double hb[LH::Q], Gb[L::Q], g0b[L::Q];
  double phi_b = P.B4[i] + stencil_adj_gather_at<L>(g, (const double*)P.B3, ad);
  double mu_b = 0.0, mu0_b = 0.0, nb[3] = {0.0, 0.0, 0.0};
  double lb = 0.0;
  const double om = K.omega_g;
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) hb[k] = P.B1[ad.slot(k, LH::Q)];  // gathered Hb
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    const double gsb = gather_Gb<L>(P, k, ad);
    g0b[k] = (1.0 - om) * gsb;
    Gb[k] = (1.0 - 0.5 * om) * gsb;
    phi_b += om * L::w[k] * gsb;
  }
  // g collision at time 0 (sources at phi, mu(c^0), n)
  lb += sources_adj<L>(K, lam_M_W2, phi, mu, f.n, Gb, 0.0, phi_b, mu_b, nb);
  double dmu_dc, dmu_dphi;
  closure_grad(K, c, phi, dmu_dc, dmu_dphi);
  const double c_b = dmu_dc * mu_b;  // c^0 = sum h~^0
  phi_b += dmu_dphi * mu_b;
  // g~^0 = w phi - G^0 / 2
  double G0b[L::Q];
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    phi_b += L::w[k] * g0b[k];
    G0b[k] = -0.5 * g0b[k];
  }
  lb += sources_adj<L>(K, lam_M_W2, phi, mu0, f.n, G0b, 0.0, phi_b, mu0_b, nb);
  // h~^0 = heq(c0, Lambda0) - H^0 / 2
  double cin_b = 0.0, lam_b = 0.0, Fb[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < LH::Q; ++k) {
    const double hk = hb[k] + c_b;
    if (k == LH::REST) {
      cin_b += hk;
      lam_b += -(1.0 - LH::w[k]) * hk;
    } else {
      lam_b += LH::w[k] * hk;
      // h~^0 = h^eq - H/2, or h^eq,alt
      const double HHb = K.h_alt ? hk * (LH::w[k] * LH::inv_cs2) : -0.5 * hk * (K.gamma * LH::w[k]);
      if (LH::ex[k]) Fb[0] += (LH::ex[k] > 0 ? HHb : -HHb);
      if (LH::ey[k]) Fb[1] += (LH::ey[k] > 0 ? HHb : -HHb);
      if (LH::D == 3 && LH::ez[k]) Fb[2] += (LH::ez[k] > 0 ? HHb : -HHb);
    }
  }
  const double qd = limit01(phi);
  const double D = (K.Dl * qd) + (K.Ds * (1.0 - qd));
  double dl_b = 0.0, gb[3] = {0.0, 0.0, 0.0};
  mu0_b += K.gamma * D * lam_b;
  const double D_b = K.gamma * mu0 * lam_b;
  if (phi >= 0.0 && phi <= 1.0) phi_b += (K.Dl - K.Ds) * D_b;
  dl_b += qd * D_b;
  const double gF = f.g[0] * Fb[0] + f.g[1] * Fb[1] + (L::D == 3 ? f.g[2] * Fb[2] : 0.0);
  mu0_b += K.Dp * gF;
  dl_b += mu0 * gF;
  for (int d = 0; d < L::D; ++d) gb[d] += mu0 * K.Dp * Fb[d];
  normal_adj<L>(f, nb, gb);
  // mu0 = closure(c0, phi0)
  closure_grad(K, cin, phi, dmu_dc, dmu_dphi);
  cin_b += dmu_dc * mu0_b;
  phi_b += dmu_dphi * mu0_b;
  c0b[i] = cin_b;
  C.B4[i] = phi_b;
  for (int d = 0; d < 3; ++d) C.B3[d * g.N + i] = gb[d];
  w.lamb[i] += lb;
  w.dlb[i] += dl_b;
}

template <class L, class Addr>
__global__ void __launch_bounds__(256) k_adj_init_b(Geo g, AdjSet C, double* __restrict__ phi0b) {
  const Addr ad(g);
  if (!ad.inside()) return;
  const int64_t i = ad.node();
  phi0b[i] = C.B4[i] + stencil_adj_gather_at<L>(g, (const double*)C.B3, ad);
}

// Deterministic sum of the two per-node accumulators (fixed launch shape).
__global__ void __launch_bounds__(kDiagThreads) k_adj_reduce(const double* __restrict__ a,
                                                             const double* __restrict__ b, int64_t n,
                                                             double* __restrict__ part) {
  __shared__ double ra[kDiagThreads], rb[kDiagThreads];
  double sa = 0.0, sb = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    sa = sa + a[i];
    sb = sb + b[i];
  }
  ra[threadIdx.x] = sa;
  rb[threadIdx.x] = sb;
  __syncthreads();
  for (int s = kDiagThreads / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      ra[threadIdx.x] = ra[threadIdx.x] + ra[threadIdx.x + s];
      rb[threadIdx.x] = rb[threadIdx.x] + rb[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = ra[0];
    part[2 * blockIdx.x + 1] = rb[0];
  }
}

// Sum of the block partials, in their order: loaded by all threads into the
// LDS, then added by one (begin and finish of a 512^2 sweep 146 -> 62 us; one
// thread reading global memory took 84 us, a wait per partial).
__global__ void __launch_bounds__(kDiagThreads) k_adj_reduce_final(const double* __restrict__ part,
                                                                   double* __restrict__ out) {
  __shared__ double p[2 * kDiagBlocks];
  for (int b = threadIdx.x; b < 2 * kDiagBlocks; b += blockDim.x) p[b] = part[b];
  __syncthreads();
  if (threadIdx.x < 2) {
    double s = 0.0;
#pragma unroll 16
    for (int b = 0; b < kDiagBlocks; ++b) s = s + p[2 * b + threadIdx.x];
    out[threadIdx.x] = s;
  }
}

}  // namespace gplbm
