// Adjoint (reverse-time) kernels of the pull update, FP64 storage.
//
// The paper defines no adjoint; this is the transpose of the update that
// hlb_kernels.hip computes.  With s_t the stored post-collision state at
// time t, g_t = G_t(s_{t-1}) the gathered pre-collision state (tables at
// t-1) and s_t = C(g_t) the BGK collision (eq. (3a), equilibrium eq. (4)),
// and the objective J = sum_{t in window} sum_x WSS(g_t(x)):
//   mu_t      = (dG_{t+1}/ds_t)^T nu_{t+1}
//   nu_t      = (dC/dg)^T mu_t + dJ_t/dg_t
//   dJ/dA_k(t-1) = sum over Ladd links of nu_t,i corr_i
//   dJ/dphi_x   += sum over wall links of nu_t,i (rest_i - back_i)
// where mu_t = dJ/ds_t.  The transpose of the pull gather is again a gather
// (the site at x + c_i is the pull entry of direction opp(i)), so nothing is
// scattered and no further table is needed, and mu need not be stored: a
// reverse step gathers nu_{t+1}, transposes the collision at once and writes
// nu_t to the other of two buffers (k_adj_step).  Only the iolet groups' mu,
// which depends on s_t through the ghost density's velocity, is formed one
// kernel earlier (k_adj_iolet, once nu_{t+1} is complete) and kept in the
// slots that the site's own nu_t will take.

#include "hlb_adjoint.h"
#include "hlb_device.h"

namespace hlb {
namespace {

using namespace dev;

struct AdjArgs {
  GatherArgs a;             // forward gather arguments, tables at t-1
  const double *S;          // s_{t-1}: post-collision state at t-1 (tiled, as the state)
  const double *next;       // nu_{t+1} (tiled)
  double *nu;               // nu_t (tiled); before that mu_t in the iolet groups' slots
  const int32_t *order;     // caller id per position (-1: padding)
  int64_t n0;               // sites of the bulk+wall group
  double omega, tau;
  int in_window;            // t lies in the objective window
  int n_io;                 // iolets
  int64_t n_steps;          // row length of dA
  int64_t step;             // column of this step in dA: t-1-t0
  double *J;                // objective: [0] total, [8, 8 + kAdjJSlots) partial sums
  double *dA;               // [n_io][n_steps]: iolet table-value derivatives
  double *dphi;             // [np], accumulated over the sweep
  int objective;            // HLB_OBJ_WSS or HLB_OBJ_IOLET_FLUX
  const double *w;          // [n_io] iolet-flux weights of the objective
  // [n_io] outflow weights of this reverse step, dJ/dQ_k(t-1): the
  // objective's inside its window plus a Windkessel outlet's model term
  double *wq;
  double *lamX;             // [n_io] adjoint of the Windkessel outlets' X
  const WkParams *wk;
};

// The wavefront's share s of the objective, added to its partial-sum slot
// (one atomic per wavefront, spread over kAdjJSlots addresses); lane 0 adds.
__device__ inline void add_objective(double *J, double s) {
  static_assert((kAdjJSlots & (kAdjJSlots - 1)) == 0, "slot count is a power of two");
  if ((threadIdx.x & 63) == 0 && s != 0.0) {
    const int64_t wave = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    atomicAdd(J + 8 + (wave & (kAdjJSlots - 1)), s);
  }
}

// (dM/dg)^T w for M(g) = f^eq(rho(g), u(g)):
//   sum_i w_i f^eq_i / rho + (sum_i w_i w8_i rho (3 c_i + 9 (c_i.u) c_i - 3 u)) . (c_j - u) / rho
// returned as the scalar a and the vector b with result_j = a + b.(c_j - u).
__device__ inline void eq_transpose(const double (&w)[Q], double rho, double ux, double uy, double uz,
                                    double &a, double &bx, double &by, double &bz) {
  const double usq = 1.5 * (ux * ux + uy * uy + uz * uz);
  a = 0.0;
  bx = by = bz = 0.0;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const double cu = cx(i) * ux + cy(i) * uy + cz(i) * uz;
    const double feq_over_rho = wgt<double>(i) * (1.0 + 3.0 * cu + 4.5 * cu * cu - usq);
    a += w[i] * feq_over_rho;
    const double s = w[i] * wgt<double>(i);  // times rho, divided by rho
    bx += s * (3.0 * cx(i) + 9.0 * cu * cx(i) - 3.0 * ux);
    by += s * (3.0 * cy(i) + 9.0 * cu * cy(i) - 3.0 * uy);
    bz += s * (3.0 * cz(i) + 9.0 * cu * cz(i) - 3.0 * uz);
  }
}

// Outflow weights of the reverse step of the update s -> s+1 (s = step):
// the objective's weight inside its window, plus, for a Windkessel outlet,
// dJ/dQ_k(s) from the adjoint of its model:
//   LX(s+1) = Lr(s+1) + kappa LX(s+2),  kappa = dX(s+2)/dX(s+1),
//   dJ/dQ_k(s) = R1 Lr(s+1) + dX(s+1)/dQ LX(s+1),
// Lr(s+1) = column s+1 of dA (the derivative with respect to the density of
// step s+1, written by the previous reverse step), zero past the last step.
// lamX holds LX(s+2) on entry and LX(s+1) on return.
__device__ inline void outflow_weight(const AdjArgs &A, int k) {
  double v = A.objective == HLB_OBJ_IOLET_FLUX && A.in_window ? A.w[k] : 0.0;
  if (A.wk && A.a.io[k].wk) {
    const WkParams P = A.wk[k];
    const double lr = A.step + 1 < A.n_steps ? A.dA[(int64_t)k * A.n_steps + A.step + 1] : 0.0;
    const double kappa = P.C > 0.0 ? 1.0 - (P.R2 > 0.0 ? 1.0 / (P.R2 * P.C) : 0.0) : 0.0;
    const double lx = lr + kappa * A.lamX[k];
    v += P.R1 * lr + (P.C > 0.0 ? 1.0 / P.C : P.R2) * lx;
    A.lamX[k] = lx;
  }
  A.wq[k] = v;
}

// Waves per SIMD, at least: the WSS form takes 131 registers at 3 waves and
// spills at 4 (2.95e6-site tree: 284 us a reverse step against 290); the other
// forms stay below 128 and run 4.
constexpr int kAdjWaves = 3;

// Density, velocity and (for the stress) second moments of a gathered state.
struct GatheredMoments {
  double rho, ux, uy, uz;
  double pxx = 0, pyy = 0, pzz = 0, pxy = 0, pxz = 0, pyz = 0;
  template <bool SECOND>
  __device__ void form(const double (&g)[Q]) {
    double dr;
    moments<false>(g, 0.0, dr, rho, ux, uy, uz);
    ux = ux / rho;
    uy = uy / rho;
    uz = uz / rho;
    if constexpr (SECOND) {
#pragma unroll
      for (int i = 1; i < Q; ++i) {
        if (cx(i)) pxx += g[i];
        if (cy(i)) pyy += g[i];
        if (cz(i)) pzz += g[i];
        if (cx(i) && cy(i)) pxy += cx(i) * cy(i) > 0 ? g[i] : -g[i];
        if (cx(i) && cz(i)) pxz += cx(i) * cz(i) > 0 ? g[i] : -g[i];
        if (cy(i) && cz(i)) pyz += cy(i) * cz(i) > 0 ? g[i] : -g[i];
      }
    }
  }
};

// One reverse step t for every site but the iolet groups' boundary terms:
//   mu_t = (dG_{t+1}/ds_t)^T nu_{t+1}: population i of p at t went to the site
//     at x + c_i -- the pull entry of direction opp(i), which names the site
//     that pulled it -- or was reflected back to p (wall: times 1 - phi); an
//     iolet site reads the mu_t that k_adj_iolet left in its slots;
//   nu_t = (dC/dg)^T mu_t + dWSS/dg_t.
// Bound by HBM: two gathers of 19 values and 19 non-temporal stores, 456 B
// per site and the pull table, where separate collide and stream kernels
// moved mu through memory in between (814 B).  Reverse step of the 2.95e6-site
// tree, k_adj_iolet included: 496 -> 261 us outside the objective window, 577
// -> 279 inside it; with porosity 643 -> 275 and 734 -> 285.
//
// The porosity derivative: at a wall link j the reflected value is
// s_{t-1}(p, opp(j)), so with h_j = w_j rho0 - s_{t-1}(p, opp(j)) and
// nu_j = (1 - omega) mu_j + omega (a + b.(c_j - u)) + d_j (d: the WSS term),
//   sum over wall links of nu_j h_j
//     = (1 - omega) sum mu_j h_j + omega (a H + b.(Hc - u H)) + sum d_j h_j,
//   H = sum h_j,  Hc = sum h_j c_j.
// Without porosity the gathered g_j is s_{t-1}(p, opp(j)) itself and outside
// the WSS window the sums are formed before g is dropped; else the few wall
// links read their slots again (cache hits).
//
// WSS (the WSS objective inside its window): J += WSS(g_t) and its
// gradient.  With n the wall normal, s the tangential traction, fac =
// -(1 - 1/(2 tau)) and e = s/|s|, the stress is fac (sum g c c - sum f^eq c
// c), sum f^eq c c = rho/3 I + rho u u (eq. (4) with the 1/2 factors), so
//   d_j = dWSS/dg_j = fac e.(c_j c_j - I/3 - c_j u - u c_j + u u) n
//       = ((c_j - u).n)((c_j - u).E),   E = fac e   (e.n = 0).
// Only the six second moments of g are formed while g is live.
template <bool POROUS, bool WSS, bool NARROW>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kAdjWaves, 8))) void k_adj_step(AdjArgs A, int64_t nb_io, int64_t nb_bulk, int xcd_chunk) {
  const GatherArgs &a = A.a;
  // blocks as in the forward step: the iolet groups' longer chains first, then
  // the bulk+wall blocks renumbered over the XCDs; before both one block for
  // the outflow weights that k_adj_iolet will use
  if (blockIdx.x == 0) {
    for (int k = threadIdx.x; k < A.n_io; k += kBlock) outflow_weight(A, k);
    return;
  }
  const int64_t b = (int64_t)blockIdx.x - 1;
  const bool bulk = b >= nb_io;
  const int64_t blk = bulk ? block_id(b - nb_io, nb_bulk, xcd_chunk) : a.io_begin / kBlock + b;
  const int64_t p = blk * kBlock + threadIdx.x;
  // bulk+wall blocks (block-uniform): the segment rows through LDS
  __shared__ int4 lrows[kSegBlock * (kSegRow / 4)];
  const int4 *lrow = bulk ? stage_rows<true>(a, blk, p, A.n0, lrows) : nullptr;
  double jsum = 0.0;
  if (!bulk || p < A.n0) {
    const int32_t p32 = (int32_t)p;
    // a padding position of the iolet groups goes through without waiting for
    // its order entry, and stores nothing
    const bool live = bulk || A.order[p] >= 0;
    constexpr bool kFromG = !POROUS && !WSS;  // a bulk+wall site's h from the gathered values
    GatheredMoments G;
    double m[Q];
    double hm = 0.0, h0 = 0.0, hx = 0.0, hy = 0.0, hz = 0.0;
    uint32_t walls = 0;  // bit i: the pull entry of direction i is a wall link
    if (bulk) {
      double g[Q];
      gather<POROUS, false, NARROW>(A.S, p, a, g, lrow);
      int32_t off[Q - 1];
      lds_offsets(lrow, off);
      if constexpr (NARROW) {
        // the addresses of gather(), with the pull entry of direction opp(i)
        using N = Narrow<double>;
        uint32_t pb = ((uint32_t)p << N::S) + N::D;
        asm("" : "+v"(pb));
        const uint32_t own = N::voff(pb);
        const uint32_t jb_wall = ((uint32_t)a.np << N::S) + N::D;
        m[0] = *N::at(A.next, 0, own);
#pragma unroll
        for (int i = 1; i < Q; ++i) {
          const uint32_t jb = ((uint32_t)off[opp(i) - 1] << N::S) + pb;
          uint32_t vj = N::voff(jb);
          asm("" : "+v"(vj));
          const bool wall = jb >= jb_wall;
          m[i] = *N::at(A.next, i, wall ? (opp(i) > i ? own + N::D : own - N::D) : vj);
          walls |= (uint32_t)wall << opp(i);
        }
      } else {
        m[0] = *at<NARROW>(A.next, p32, 0);
#pragma unroll
        for (int i = 1; i < Q; ++i) {
          const int32_t q = p32 + off[opp(i) - 1];
          const bool wall = (uint32_t)q >= (uint32_t)a.np;
          m[i] = *at<NARROW>(A.next, wall ? p32 : q, wall ? opp(i) : i);
          walls |= (uint32_t)wall << opp(i);
        }
      }
      // all 38 loads are in flight before any is used (to save registers the
      // compiler would fetch mu one value at a time behind the gather)
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (POROUS) {
        if (walls) {
          const double keep = 1.0 - a.phi[p];
#pragma unroll
          for (int i = 1; i < Q; ++i)
            if ((walls >> opp(i)) & 1u) m[i] *= keep;
        }
      }
      G.template form<WSS>(g);
      if constexpr (kFromG) {
#pragma unroll
        for (int j = 1; j < Q; ++j) {
          const double h = ((walls >> j) & 1u) ? wgt<double>(j) * a.rho0 - g[j] : 0.0;
          hm += m[j] * h;
          h0 += h;
          hx += h * cx(j);
          hy += h * cy(j);
          hz += h * cz(j);
        }
      }
    } else {
      double g[Q];
      gather_iolet<POROUS, false, NARROW>(A.S, p, a, g, nullptr);
      G.template form<WSS>(g);
      // g is consumed before mu is fetched (registers)
      asm volatile("" : "+v"(G.rho), "+v"(G.ux), "+v"(G.uy), "+v"(G.uz)::"memory");
      int32_t pm = p32;  // addresses formed here (not kept from gather_iolet's)
      asm volatile("" : "+v"(pm));
      int32_t code[Q];
      load_codes(a, (uint32_t)pm - (uint32_t)a.io_begin, code);
#pragma unroll
      for (int i = 1; i < Q; ++i) walls |= (uint32_t)(code[i] == HLB_LINK_WALL) << i;
#pragma unroll
      for (int i = 0; i < Q; ++i) m[i] = *at<NARROW>(A.nu, pm, i);
    }
    const double rho = G.rho, ux = G.ux, uy = G.uy, uz = G.uz;
    double pxx = G.pxx, pyy = G.pyy, pzz = G.pzz, pxy = G.pxy, pxz = G.pxz, pyz = G.pyz;
    // the WSS term's n and E (zero without a wall normal or traction)
    double nx = 0, ny = 0, nz = 0, Ex = 0, Ey = 0, Ez = 0;
    if constexpr (WSS) {
#pragma unroll
      for (int i = 1; i < Q; ++i)
        if ((walls >> i) & 1u) {
          nx -= cx(i);
          ny -= cy(i);
          nz -= cz(i);
        }
      const double nn = sqrt(nx * nx + ny * ny + nz * nz);
      if (nn > 0.0) {
        nx /= nn;
        ny /= nn;
        nz /= nn;
        const double fac = -(1.0 - 1.0 / (2.0 * A.tau));
        pxx -= rho * (1.0 / 3.0 + ux * ux);
        pyy -= rho * (1.0 / 3.0 + uy * uy);
        pzz -= rho * (1.0 / 3.0 + uz * uz);
        pxy -= rho * ux * uy;
        pxz -= rho * ux * uz;
        pyz -= rho * uy * uz;
        const double tx = fac * (pxx * nx + pxy * ny + pxz * nz);
        const double ty = fac * (pxy * nx + pyy * ny + pyz * nz);
        const double tz = fac * (pxz * nx + pyz * ny + pzz * nz);
        const double tn = tx * nx + ty * ny + tz * nz;
        const double sx = tx - tn * nx, sy = ty - tn * ny, sz = tz - tn * nz;
        const double w = sqrt(sx * sx + sy * sy + sz * sz);
        jsum = live ? w : 0.0;
        if (w > 0.0) {
          const double fw = fac / w;
          Ex = fw * sx;
          Ey = fw * sy;
          Ez = fw * sz;
        } else {
          nx = ny = nz = 0.0;
        }
      }
    }
    const double un = ux * nx + uy * ny + uz * nz, uE = ux * Ex + uy * Ey + uz * Ez;
    double dphi = 0.0;
    if (!kFromG || !bulk) {
      if (walls) {
        // one unconditional load per direction, all in flight together: a
        // link that is no wall reads the site's slot of direction 0 instead
        double back[Q];
        int32_t pw = p32;
        asm volatile("" : "+v"(pw));
#pragma unroll
        for (int j = 1; j < Q; ++j) back[j] = *at<NARROW>(A.S, pw, ((walls >> j) & 1u) ? opp(j) : 0);
#pragma unroll
        for (int j = 1; j < Q; ++j) {
          const double h = ((walls >> j) & 1u) ? wgt<double>(j) * a.rho0 - back[j] : 0.0;
          hm += m[j] * h;
          h0 += h;
          hx += h * cx(j);
          hy += h * cy(j);
          hz += h * cz(j);
          if constexpr (WSS)
            dphi += h * (cx(j) * nx + cy(j) * ny + cz(j) * nz - un) * (cx(j) * Ex + cy(j) * Ey + cz(j) * Ez - uE);
        }
      }
    }
    double ea, ebx, eby, ebz;
    eq_transpose(m, rho, ux, uy, uz, ea, ebx, eby, ebz);
    if (walls && live)
      A.dphi[p] += dphi + (1.0 - A.omega) * hm +
                   A.omega * (ea * h0 + ebx * (hx - ux * h0) + eby * (hy - uy * h0) + ebz * (hz - uz * h0));
    int32_t ps = p32;  // store addresses formed here (not kept from the loads)
    asm volatile("" : "+v"(ps));
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      double v = (1.0 - A.omega) * m[j] + A.omega * (ea + ebx * (cx(j) - ux) + eby * (cy(j) - uy) + ebz * (cz(j) - uz));
      if constexpr (WSS) v += (cx(j) * nx + cy(j) * ny + cz(j) * nz - un) * (cx(j) * Ex + cy(j) * Ey + cz(j) * Ez - uE);
      if (live) __builtin_nontemporal_store(v, at<NARROW>(A.nu, ps, j));
    }
  }
  if constexpr (WSS) add_objective(A.J, wave_sum(jsum));
}

// The iolet groups' part of the reverse step t, once nu_t is complete:
//   table values: dJ/dA_k(t-1) += sum over links of k of (nu_i - w_k)
//     d(fill_i)/dA_k, w_k = dJ/dQ_k(t-1) the step's outflow weight (a
//     population leaving through a pressure iolet adds w_k to its own
//     adjoint), and with the iolet-flux objective J += (its weight) (leaving
//     population - fill) per link;
//   mu_{t-1} = (dG_t/ds_{t-1})^T nu_t, into the slots of `out`: as in
//     k_adj_step, but at a Ladd link the reflected value (plus a constant)
//     and at a pressure link no direct path, while the fill depends on the
//     site's velocity at t-1 (moments of s_{t-1}).
// A few sites, so latency: codes, own nu and own s are fetched together,
// then the neighbours' nu, then each iolet's record once: 11 us on the
// 48,192-site tree, where the boundary and stream kernels it replaces took 23
// and 27.  That tree's 40-step outflow gradient: 2372 -> 2256 us with the sums
// of dA not waited for, -> 2235 with the leaving populations in flight together.
template <bool POROUS, bool NARROW>
__global__ __launch_bounds__(kBlock) void k_adj_iolet(AdjArgs A, double *out) {
  const GatherArgs &a = A.a;
  const int64_t p = a.io_begin + (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double jsum = 0.0;
  WkFlux dtab;  // this site's table-value derivative (one iolet per site, mostly)
  {
    const bool live = A.order[p] >= 0;  // a padding position has no iolet links and stores nothing
    const int32_t p32 = (int32_t)p;
    const uint32_t q = (uint32_t)(p - a.io_begin);
    int32_t code[Q];
    load_codes(a, q, code);
    double nu[Q], m[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) nu[i] = *at<NARROW>(A.nu, p32, i);
    double rho, ux, uy, uz;  // at t-1
    {
      double s[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) s[i] = *at<NARROW>(A.S, p32, i);
      double dr;
      moments<false>(s, 0.0, dr, rho, ux, uy, uz);
      ux = ux / rho;
      uy = uy / rho;
      uz = uz / rho;
    }
    const double keep = POROUS ? 1.0 - a.phi[p] : 1.0;
    m[0] = nu[0];
#pragma unroll
    for (int i = 1; i < Q; ++i) {
      const int32_t c = code[opp(i)];
      m[i] = *at<NARROW>(A.nu, c >= 0 ? c : p32, c >= 0 ? i : opp(i));
      if (POROUS && c == HLB_LINK_WALL) m[i] *= keep;
      if (c < HLB_LINK_WALL) m[i] = 0.0;  // filled below
    }
    const bool flux = A.objective == HLB_OBJ_IOLET_FLUX && A.in_window;
    NextIolet io(code, HLB_LINK_WALL);
    while (io.links) {
      uint32_t ql = q;  // the addresses of this turn are formed in it
      asm volatile("" : "+v"(ql));
      const int k = -io.code - 2;
      const IoletDev K = a.io[k];
      const double val = iolet_value(a, K, k, a.t);
      const double wk = A.wq[k];
      double d = 0.0, o = 0.0;  // derivative of the table value; outflow
      if (K.kind == HLB_IOLET_VELOCITY) {
        double corr[Q];
#pragma unroll
        for (int i = 1; i < Q; ++i) corr[i] = a.corr[(int64_t)(i - 1) * a.nio + ql];
#pragma unroll
        for (int i = 1; i < Q; ++i) {
          if (!((io.links >> i) & 1u)) continue;
          d += (nu[i] - wk) * corr[i];
          o -= corr[i] * val;
          m[opp(i)] += nu[i];
        }
      } else {
        const double un = ux * K.n[0] + uy * K.n[1] + uz * K.n[2];
        const double gx = un * K.n[0], gy = un * K.n[1], gz = un * K.n[2];
        const double usq = 1.5 * (gx * gx + gy * gy + gz * gz);
        double coef = 0.0;  // of the fills' dependence on u.n
        // the leaving populations, in flight together (inside the loop below
        // each was a round trip of its own)
        double leave[Q] = {};
        if (flux) {
          int32_t pl = p32;
          asm volatile("" : "+v"(pl));
#pragma unroll
          for (int i = 1; i < Q; ++i) leave[i] = *at<NARROW>(A.S, pl, ((io.links >> i) & 1u) ? opp(i) : 0);
        }
#pragma unroll
        for (int i = 1; i < Q; ++i) {
          if (!((io.links >> i) & 1u)) continue;
          const double feq = s_eq<false>(i, 0.0, 1.0, gx, gy, gz, usq);
          d += (nu[i] - wk) * feq;
          o += leave[i] - val * feq;
          const double cu = cx(i) * gx + cy(i) * gy + cz(i) * gz;
          const double cn = cx(i) * K.n[0] + cy(i) * K.n[1] + cz(i) * K.n[2];
          const double gn = gx * K.n[0] + gy * K.n[1] + gz * K.n[2];
          coef += (nu[i] - wk) * wgt<double>(i) * val * (3.0 * cn + 9.0 * cu * cn - 3.0 * gn);
          m[opp(i)] += wk;  // replaced by the ghost-density equilibrium
        }
        coef /= rho;
#pragma unroll
        for (int j = 0; j < Q; ++j)
          m[j] += coef * (K.n[0] * (cx(j) - ux) + K.n[1] * (cy(j) - uy) + K.n[2] * (cz(j) - uz));
      }
      dtab.add(A.dA + A.step, k, d, A.n_steps);
      if (flux) jsum += A.w[k] * o;
      if (!io.more) break;
      int32_t again[Q];
      load_codes(a, ql, again);
      io = NextIolet(again, io.code);
    }
#pragma unroll
    for (int i = 0; i < Q; ++i)
      if (live) *at<NARROW>(out, p32, i) = m[i];
  }
  add_objective(A.J, wave_sum(jsum));
  wave_add_grouped(A.dA + A.step, dtab, A.n_steps);  // one atomic per iolet per wavefront
}

// J[0] := sum of the kAdjJSlots partial sums (one workgroup of kBlock).
__global__ __launch_bounds__(kBlock) void k_adj_objective(double *J) {
  __shared__ double part[kBlock / 64];
  double v = 0.0;
  for (int64_t i = threadIdx.x; i < kAdjJSlots; i += kBlock) v += J[8 + i];
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) t += part[w];
    J[0] = t;
  }
}

inline unsigned blocks_of(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

hipError_t launch_adjoint_step(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, int src, int64_t t,
                               const AdjBuffers &b, int in_window, int64_t n_steps, int64_t step,
                               hipStream_t s) {
  if (cfg.storage != HLB_F64 || (b.n_io > 0 && (!b.wq || !b.lamX))) return hipErrorInvalidValue;
  AdjArgs A;
  A.a = make_args(cfg, L, d, t - 1);
  A.a.io_flux = nullptr;
  A.S = static_cast<const double *>(d.f[src]);
  A.next = b.nu[b.cur];
  A.nu = b.nu[1 - b.cur];
  A.order = d.order;
  A.n0 = L.gcnt[0];
  A.omega = 1.0 / cfg.tau;
  A.tau = cfg.tau;
  A.in_window = in_window;
  A.n_io = b.n_io;
  A.n_steps = n_steps;
  A.step = step;
  A.J = b.J;
  A.dA = b.dA;
  A.dphi = b.dphi;
  A.objective = b.objective;
  A.w = b.w;
  A.wq = b.wq;
  A.lamX = b.lamX;
  A.wk = d.wk;
  const bool wss = b.objective == HLB_OBJ_WSS && in_window;
  const int64_t nb_io = (L.gbeg[kGroups] - L.io_begin) / kBlock, nb_bulk = blocks_of(L.gcnt[0]);
  const unsigned grid = (unsigned)(1 + nb_io + nb_bulk);
  // 32-bit byte offsets when a population buffer fits in them, as in the
  // forward step
  const bool narrow = (uint64_t)Q * (uint64_t)L.np * sizeof(double) + Narrow<double>::BIAS <= (uint64_t(1) << 32);
  // k_adj_iolet writes mu_{t-1} over nu_{t+1}, which k_adj_step has consumed
  double *mu = b.nu[b.cur];
#define HLB_ADJ(P, N)                                                             \
  do {                                                                            \
    if (wss)                                                                      \
      k_adj_step<P, true, N><<<grid, kBlock, 0, s>>>(A, nb_io, nb_bulk, cfg.xcd_chunk); \
    else                                                                          \
      k_adj_step<P, false, N><<<grid, kBlock, 0, s>>>(A, nb_io, nb_bulk, cfg.xcd_chunk); \
    if (nb_io > 0) k_adj_iolet<P, N><<<(unsigned)nb_io, kBlock, 0, s>>>(A, mu);   \
  } while (0)
  if (cfg.porous) {
    if (narrow) HLB_ADJ(true, true);
    else HLB_ADJ(true, false);
  } else {
    if (narrow) HLB_ADJ(false, true);
    else HLB_ADJ(false, false);
  }
#undef HLB_ADJ
  return hipGetLastError();
}

hipError_t launch_adjoint_objective(double *J, hipStream_t s) {
  k_adj_objective<<<1, kBlock, 0, s>>>(J);
  return hipGetLastError();
}

}  // namespace hlb
