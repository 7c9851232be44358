// gfx950 kernels of the sparse D3Q19 LBGK update (pull scheme).
//
// One thread owns one fluid site.  Populations live in two buffers (f_old /
// f_new swapped by pointer, Sec. 3.2.3), each a structure of arrays per
// tile of 4096 positions, [np/4096][19][4096] of the storage type.  FP64
// stores f_i itself, as the paper does; the FP32 / FP16 forms store the
// deviation f_i - w_i rho0 from the rest state and collide in FP32.  A step gathers the 19
// post-collision populations that stream into the site (eq. (3b) read
// backwards: the pull order the paper proposes in its future-work section),
// substitutes the boundary rules for links that cross a wall or an iolet
// (Sec. 2.3), collides (eq. (3a) with eq. (4)) and stores the 19 results at
// the site's own, coalesced, slots.
//
// Sites are grouped by collision-streaming type (Sec. 3.2.2): positions
// [0, n0) hold the merged bulk+wall group, whose pull table encodes
// bounce-back as one load with a selected address; the four iolet groups follow, each
// starting on a 256-site boundary, with the boundary rules applied per link.
// k_step runs both code paths in one launch, one group per workgroup.
//
// The method is bound by HBM bandwidth (~0.7 flop per byte in FP64), so
// nothing here uses the matrix cores.

#include "hlb_device.h"

namespace hlb {
namespace {

using namespace dev;

// ---------------------------------------------------------------- step ----

// One launch per step covers every group (Sec. 3.2.2's per-type kernels as
// block-uniform code paths of a single launch): the first nb_io blocks take
// the iolet groups, so that their longer-latency work starts first and
// overlaps the bulk blocks; the remaining nb_bulk blocks take the bulk+wall
// group's 256-position blocks blk0, blk0+1, ...  (a split step launches the
// edge blocks and the rest separately).  Every block, hence every wavefront,
// runs one group's code path only.
// The minimum waves per SIMD the step kernel is compiled for, per storage
// type.  FP64: the natural 4 (5 and 6 slower by 0.5-1% on the 2e8-site tree, 5 by 1%
// on the 2e7-site tree).  FP16: 7 waves (20 bytes of scratch in the iolet path)
// 320.7 us on the 2.0e7-site tree, 6 323.1, 8 322.2, 5 334.  FP32: 6 (5 slower by
// 0.2-0.3% on the trees and 0.9-1.0% on the 6e8-site forest, 7 by 1%, 4 by 5%).
// Population addresses are 32-bit byte offsets where a buffer allows it (see
// at()).  FP32, which once was slower with them, runs faster in every size since the
// iolet path spills no more and the rows are in LDS: 7.1 to 6.7 us a step of the
// 125,400-site vessel, 91.5 to 89.3 at 2.95e6 sites, 223.3 to 220.6 at 7.8e6, 553 to 552 at
// 2.0e7.
// SPT = 2 (two bulk+wall sites per thread, see below) needs about twice the
// registers of the bulk path: 4 waves.
// The push step's iolet path keeps more values at once: FP16 takes 6 waves
// there (28 to 36 bytes of scratch; with 7, 68 to 84, and 10 steps of the
// 13,312-site pipe take 85.6 us instead of 77.5, of the 1.1e6-site tree 306 instead of 296).
template <typename T, int SPT = 1>
constexpr int kStepWaves = SPT == 2 ? 4 : (std::is_same<T, double>::value ? 4 : sizeof(T) == 2 ? 7 : 6);
template <typename T>
constexpr int kPushWaves = std::is_same<T, double>::value ? 4 : 6;
// The bulk path of a full step stages each block's segment rows through LDS
// (stage_rows): FP64 and FP32 +0.4% on the 2e7- and +0.5-1.3% on the 2e8-site
// tree against five row loads per lane, each of which touches a cache line per
// distinct segment of its wavefront; FP16 +1.7% and +2.1% on the 7.8e6- and
// 2.0e7-site trees with the short chain of loads (with the long one 3-5%
// slower).
template <typename T>
constexpr bool kStepShortRows = sizeof(T) == 2;

// SPT: bulk+wall sites per thread.  With SPT = 2 a workgroup takes two
// consecutive 256-position blocks and each thread one position of each (both
// coalesced); the two sites' table loads and 36 gathers are all issued
// before either collides, which doubles the bytes a wavefront has in flight.
// nb_bulk then counts block pairs.  Only the full step (blk0 = 0) uses it.
template <typename T, bool POROUS, bool NARROW, bool CACHED, int SPT = 1>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kStepWaves<T, SPT>, 8))) void k_step(
    const T *__restrict__ A, T *__restrict__ B, GatherArgs a, const int32_t *__restrict__ order, int64_t n0,
    int64_t nb_io, int64_t blk0, int64_t nb_bulk, int xcd_chunk, typename Acc<T>::type omega, double *flux_slots,
    uint32_t *done) {
  using C = typename Acc<T>::type;
  constexpr bool SH = kShifted<T>;
  const int64_t b = blockIdx.x;
  C flux = 0;
  if (b < nb_io) {
    const int64_t p = a.io_begin + b * kBlock + threadIdx.x;
    WkFlux wkf;
    // a padding position (wall links only, zero values) goes through the
    // gather too, so that it need not wait for its order entry, and stores
    // nothing
    const int32_t id = order[p];
    C g[Q];
    flux = gather_iolet<POROUS, SH, NARROW>(A, p, a, g, &wkf);
    if (id >= 0) {
      collide<SH>(g, omega, C(a.rho0));
      // store addresses formed here, not shared with the loads of the site's
      // own slots (they would be kept, and spilled, across the whole path)
      int32_t ps = (int32_t)p;
      asm volatile("" : "+v"(ps));
#pragma unroll
      for (int i = 0; i < Q; ++i) st_step<CACHED>(at<NARROW>(B, ps, i), g[i]);
    } else {
      flux = 0;
    }
    add_flux(flux_slots, double(flux));
    if (a.wk_n > 0) {
      wave_add_grouped(a.io_flux, wkf);
      finish_outlets(a, nb_io, done);
    }
  } else if constexpr (SPT == 1) {
    const int64_t blk = blk0 + block_id(b - nb_io, nb_bulk, xcd_chunk);
    const int64_t p = blk * kBlock + threadIdx.x;
    __shared__ int4 lrows[kSegBlock * (kSegRow / 4)];
    const int4 *lrow = stage_rows<kStepShortRows<T> || CACHED>(a, blk, p, n0, lrows);
    if (p < n0) {
      C g[Q];
      flux = gather<POROUS, SH, NARROW>(A, p, a, g, lrow);
      collide<SH>(g, omega, C(a.rho0));
      if constexpr (NARROW) {
        using N = Narrow<T>;
        const uint32_t own = N::voff(((uint32_t)p << N::S) + N::D);
#pragma unroll
        for (int i = 0; i < Q; ++i) st_step<CACHED>(N::at(B, i, own), g[i]);
      } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) st_step<CACHED>(at<NARROW>(B, (int32_t)p, i), g[i]);
      }
    }
    if constexpr (POROUS) add_flux(flux_slots, double(flux));
  } else {
    const int64_t blk = 2 * block_id(b - nb_io, nb_bulk, xcd_chunk);
    const int64_t p = blk * kBlock + threadIdx.x;
    if (p < n0) {
      // the second site; past the group's end (last pair only) it repeats
      // the first and stores the same values again (a conditional store
      // would let the compiler sink the second site's loads behind the
      // first site's stores)
      const bool has2 = p + kBlock < n0;
      const int64_t p2 = has2 ? p + kBlock : p, blk2 = has2 ? blk + 1 : blk;
      C g[Q], h[Q], flux2;
      gather_bulk2<POROUS, SH, NARROW>(A, p, blk, p2, blk2, a, g, h, flux, flux2);
      if (has2) flux += flux2;
      collide<SH>(g, omega, C(a.rho0));
      collide<SH>(h, omega, C(a.rho0));
#pragma unroll
      for (int i = 0; i < Q; ++i) st_step<CACHED>(at<NARROW>(B, (int32_t)p, i), g[i]);
#pragma unroll
      for (int i = 0; i < Q; ++i) st_step<CACHED>(at<NARROW>(B, (int32_t)p2, i), h[i]);
    }
    if constexpr (POROUS) add_flux(flux_slots, double(flux));
  }
}

// One step in push order (the paper's implementation; the A/B partner of
// k_step): buffers hold the pre-collision state f(t); every site reads its
// own 19 values (coalesced), collides and scatters (scatter()).  Same block
// layout, XCD remap and occupancy as k_step.
template <typename T, bool POROUS, bool NARROW>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kPushWaves<T>, 8))) void k_step_push(
    const T *__restrict__ A, T *__restrict__ B, GatherArgs a, const int32_t *__restrict__ order, int64_t n0,
    int64_t nb_io, int64_t blk0, int64_t nb_bulk, int xcd_chunk, typename Acc<T>::type omega, double *flux_slots,
    uint32_t *done) {
  using C = typename Acc<T>::type;
  constexpr bool SH = kShifted<T>;
  const int64_t b = blockIdx.x;
  C flux = 0;
  if (b < nb_io) {
    const int64_t p = a.io_begin + b * kBlock + threadIdx.x;
    WkFlux wkf;
    if (p < a.np && order[p] >= 0) {
      C f[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) f[i] = ld(at<NARROW>(A, (int32_t)p, i));
      C dr, rho, jx, jy, jz;
      moments<SH>(f, C(a.rho0), dr, rho, jx, jy, jz);
      collide<SH>(f, omega, C(a.rho0));
      flux = scatter<true, POROUS, SH, NARROW>(B, p, 0, a, f, jx / rho, jy / rho, jz / rho, rho, &wkf);
    }
    add_flux(flux_slots, double(flux));
    if (a.wk_n > 0) {
      wave_add_grouped(a.io_flux, wkf);
      finish_outlets(a, nb_io, done);
    }
  } else {
    const int64_t blk = blk0 + block_id(b - nb_io, nb_bulk, xcd_chunk);
    const int64_t p = blk * kBlock + threadIdx.x;
    if (p < n0) {
      C f[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) f[i] = ld(at<NARROW>(A, (int32_t)p, i));
      collide<SH>(f, omega, C(a.rho0));
      flux = scatter<false, POROUS, SH, NARROW>(B, p, blk, a, f, C(0), C(0), C(0), C(0));
    }
    if constexpr (POROUS) add_flux(flux_slots, double(flux));
  }
}

// ------------------------------------------------------- init / state ----

template <typename T>
__global__ __launch_bounds__(kBlock) void k_init_eq(T *__restrict__ A, T *__restrict__ B,
                                                    const int32_t *__restrict__ order, int64_t np,
                                                    const double *__restrict__ staging, double rho0) {
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= np) return;
  const int32_t id = order[p];
  constexpr bool SH = kShifted<T>;
  double g[Q];
  if (id < 0) {
#pragma unroll
    for (int i = 0; i < Q; ++i) g[i] = 0.0;
  } else if (staging == nullptr) {
#pragma unroll
    for (int i = 0; i < Q; ++i) g[i] = rest<SH>(i, rho0);
  } else {
    const double rho = staging[4 * (int64_t)id], ux = staging[4 * (int64_t)id + 1],
                 uy = staging[4 * (int64_t)id + 2], uz = staging[4 * (int64_t)id + 3];
    const double usq = 1.5 * (ux * ux + uy * uy + uz * uz);
#pragma unroll
    for (int i = 0; i < Q; ++i) g[i] = s_eq<SH>(i, rho - rho0, rho, ux, uy, uz, usq);
  }
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    st(A + pidx((int32_t)p, i), static_cast<typename Acc<T>::type>(g[i]));
    st(B + pidx((int32_t)p, i), static_cast<typename Acc<T>::type>(g[i]));
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_set_state(T *__restrict__ Pre, T *__restrict__ Post,
                                                      const int32_t *__restrict__ order, int64_t np,
                                                      const double *__restrict__ staging, double rho0,
                                                      typename Acc<T>::type omega) {
  using C = typename Acc<T>::type;
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= np) return;
  const int32_t id = order[p];
  constexpr bool SH = kShifted<T>;
  C g[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i)
    g[i] = id < 0 ? C(0) : C(staging[(int64_t)id * Q + i] - shift<SH>(i, rho0));
#pragma unroll
  for (int i = 0; i < Q; ++i) st(Pre + pidx((int32_t)p, i), g[i]);
  if (id < 0) return;
  collide<SH>(g, omega, C(rho0));
#pragma unroll
  for (int i = 0; i < Q; ++i) st(Post + pidx((int32_t)p, i), g[i]);
}

// --------------------------------------------------------------- macros ----

// Density, velocity, wall shear stress (STATE: the populations) of the
// pre-collision state at time t, in FP64, written per caller id.  Bound by HBM:
// the gather of a step, 40 bytes written per site and its caller id.  Blocks
// and addresses are the step kernel's (iolet groups first, XCD chunks,
// segment rows in LDS, 32-bit offsets where a buffer allows), and the stress
// is formed from six moments, only where a wavefront has wall sites, so that
// the kernel runs at 4 waves per SIMD instead of 2: 863 -> 792 us on the 2.0e7-site
// tree in FP64, 619 -> 528 in FP32, 250 -> 185 on the 7.8e6-site tree in FP16, 10.2 ->
// 5.5 on the 13,312-site pipe, calls back to back (5 waves spill: 917 us in FP64).
// SRC: whether A holds pre-collision values, read as they are, or the
// post-collision values that they are gathered from.
enum MacroSrc { kDirect, kPulled, kPulledPorous };
template <typename T, MacroSrc SRC, bool NARROW, bool STATE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_macros(
    const T *__restrict__ A, GatherArgs a, const int32_t *__restrict__ order, int64_t n0, int64_t nb_io, int64_t nb_bulk,
    int xcd_chunk, double tau, double *__restrict__ rho_o, double *__restrict__ u_o,
    double *__restrict__ wss_o, double *__restrict__ f_o) {
  const int64_t b = blockIdx.x;
  const bool bulk = b >= nb_io;
  const int64_t blk = bulk ? block_id(b - nb_io, nb_bulk, xcd_chunk) : a.io_begin / kBlock + b;
  const int64_t p = blk * kBlock + threadIdx.x;
  __shared__ int4 lrows[kSegBlock * (kSegRow / 4)];
  // values read as they are need the rows for the wall links of the stress alone
  const int4 *lrow =
      bulk && (SRC != kDirect || wss_o) ? stage_rows<kStepShortRows<T>>(a, blk, p, n0, lrows) : nullptr;
  if (bulk && p >= n0) return;
  const int32_t id = order[p];
  const int32_t p32 = (int32_t)p;
  constexpr bool SH = kShifted<T>, POROUS = SRC == kPulledPorous;
  double g[Q];
  if constexpr (SRC == kDirect) {
#pragma unroll
    for (int i = 0; i < Q; ++i) g[i] = ld(at<NARROW>(A, p32, i));
  } else if (bulk) {
    gather<POROUS, SH, NARROW>(A, p, a, g, lrow);
  } else {
    gather_iolet<POROUS, SH, NARROW>(A, p, a, g, nullptr);
  }
  if (id < 0) return;
  if constexpr (STATE) {
#pragma unroll
    for (int i = 0; i < Q; ++i) f_o[(int64_t)id * Q + i] = g[i] + shift<SH>(i, a.rho0);
    return;
  }
  double dr, rho, ux, uy, uz;
  moments<SH>(g, a.rho0, dr, rho, ux, uy, uz);
  ux = ux / rho;
  uy = uy / rho;
  uz = uz / rho;
  if (rho_o) rho_o[id] = rho;
  if (u_o) {
    // 24 bytes at 8-byte alignment in two stores
    typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));
    double *o = u_o + 3 * (int64_t)id;
    *reinterpret_cast<d2 *>(o) = d2{ux, uy};
    o[2] = uz;
  }
  if (!wss_o) return;
  // wall links (bit i: the pull entry of direction i, which describes the
  // link leaving along opp(i) = -c_i)
  uint32_t walls = 0;
  if (bulk) {
    int32_t off[Q - 1];
    lds_offsets(lrow, off);
#pragma unroll
    for (int i = 1; i < Q; ++i) walls |= (uint32_t)((uint32_t)(p32 + off[i - 1]) >= (uint32_t)a.np) << i;
  } else {
    int32_t code[Q];
    load_codes(a, (uint32_t)(p - a.io_begin), code);
#pragma unroll
    for (int i = 1; i < Q; ++i) walls |= (uint32_t)(code[i] == HLB_LINK_WALL) << i;
  }
  double w = 0.0;
  if (walls) {
    // wall normal: normalised sum of the directions whose links hit a wall
    int sx = 0, sy = 0, sz = 0;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
      const int on = (int)((walls >> i) & 1u);
      sx -= on * cx(i);
      sy -= on * cy(i);
      sz -= on * cz(i);
    }
    const double nn = sqrt((double)(sx * sx + sy * sy + sz * sz));
    if (nn > 0.0) {
      const double nx = sx / nn, ny = sy / nn, nz = sz / nn;
      // non-equilibrium second moment sum (f - f_eq) c c = sum (f - w rho) c c - rho u u
      double pxx = -rho * ux * ux, pyy = -rho * uy * uy, pzz = -rho * uz * uz;
      double pxy = -rho * ux * uy, pxz = -rho * ux * uz, pyz = -rho * uy * uz;
#pragma unroll
      for (int i = 1; i < Q; ++i) {
        const double d = g[i] - wgt<double>(i) * dr;  // dr = rho - rho0 (rho unshifted), g alike
        if (cx(i)) pxx += d;
        if (cy(i)) pyy += d;
        if (cz(i)) pzz += d;
        if (cx(i) && cy(i)) pxy += cx(i) * cy(i) > 0 ? d : -d;
        if (cx(i) && cz(i)) pxz += cx(i) * cz(i) > 0 ? d : -d;
        if (cy(i) && cz(i)) pyz += cy(i) * cz(i) > 0 ? d : -d;
      }
      const double fac = -(1.0 - 1.0 / (2.0 * tau));
      const double tx = fac * (pxx * nx + pxy * ny + pxz * nz);
      const double ty = fac * (pxy * nx + pyy * ny + pyz * nz);
      const double tz = fac * (pxz * nx + pyz * ny + pzz * nz);
      const double tn = tx * nx + ty * ny + tz * nz;
      const double vx = tx - tn * nx, vy = ty - tn * ny, vz = tz - tn * nz;
      w = sqrt(vx * vx + vy * vy + vz * vz);
    }
  }
  wss_o[id] = w;
}

// ----------------------------------------------------------------- mass ----

template <typename T>
__global__ __launch_bounds__(kBlock) void k_mass_partial(const T *__restrict__ A,
                                                         const int32_t *__restrict__ order, int64_t np,
                                                         double *partial) {
  __shared__ double red[kBlock / 64];
  double s = 0.0;
  for (int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x; p < np; p += (int64_t)gridDim.x * kBlock) {
    if (order[p] < 0) continue;
    double q = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) q += ld(A + pidx((int32_t)p, i));
    s += q;
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double b = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) b += red[w];
    partial[1 + blockIdx.x] = b;
  }
}

// partial[0] = the mass, acc[1] = the boundary flux.
__global__ __launch_bounds__(kBlock) void k_mass_final(double *partial, int64_t nparts, double *acc,
                                                       const double *flux) {
  __shared__ double red[2][kBlock / 64];
  const double share = flux_share(flux);
  double s = 0.0;
  for (int64_t k = threadIdx.x; k < nparts; k += kBlock) s += partial[1 + k];
  const double m = block_sum(s, red[0]);
  const double f = block_sum(share, red[1]);
  if (threadIdx.x == 0) {
    partial[0] = m;
    acc[1] = acc[0] + f;
  }
}

// The Windkessel outlets of a step without iolet blocks (one thread each).
__global__ void k_windkessel(GatherArgs a) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < a.wk_n) windkessel(a, k, step_time(a), a.io_flux[k]);
}

__global__ void k_set_time(int64_t *p, int64_t v) { *p = v; }
__global__ void k_add_time(int64_t *p, int64_t k) { *p += k; }

__global__ __launch_bounds__(kBlock) void k_total_flux(const double *acc, const double *flux, double *out) {
  __shared__ double red[kBlock / 64];
  const double f = block_sum(flux_share(flux), red);
  if (threadIdx.x == 0) *out = acc[0] + f;
}

__global__ __launch_bounds__(kBlock) void k_set_flux(double *acc, double *flux, const double *from, double v) {
  const int k = blockIdx.x * kBlock + threadIdx.x;
  flux[k] = 0.0;
  if (k < 4) acc[k] = k == 0 ? (from ? *from : v) : 0.0;
}

__global__ void k_zero(double *p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// Byte offsets fit in 32 bits when a whole population buffer does, with the
// bias of the bulk path's addressing (Narrow).
template <typename T>
bool use_narrow(const Layout &L) {
  return (uint64_t)Q * (uint64_t)L.np * sizeof(T) + Narrow<T>::BIAS <= (uint64_t(1) << 32);
}

template <typename T>
hipError_t step_impl(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, int src, int64_t t,
                     hipStream_t s, hipEvent_t e0, hipEvent_t e1, int part) {
  using C = typename Acc<T>::type;
  const T *A = static_cast<const T *>(d.f[src]);
  T *B = static_cast<T *>(d.f[1 - src]);
  const GatherArgs a = make_args(cfg, L, d, t);
  const C omega = C(1.0 / cfg.tau);
  const int64_t n0 = L.gcnt[0];
  const int64_t nb_all = (n0 + kBlock - 1) / kBlock;
  // part 0: the whole step; 1: iolet groups + the edge blocks of the
  // bulk+wall group; 2: its remaining blocks
  // the iolet groups' blocks, without the padding and the ghosts behind them
  const int64_t nb_io = part == 2 ? 0 : (L.gbeg[kGroups] - L.io_begin) / kBlock;
  const int64_t blk0 = part == 2 ? L.edge_blocks : 0;
  const int64_t nb_bulk = part == 0 ? nb_all : (part == 1 ? L.edge_blocks : nb_all - L.edge_blocks);
  // two bulk+wall sites per thread: full pull steps only
  const bool pair = cfg.sites_per_thread == 2 && part == 0 && cfg.scheme == HLB_SCHEME_PULL;
  const int64_t nb_launch = pair ? (nb_bulk + 1) / 2 : nb_bulk;
  const unsigned grid = (unsigned)(nb_io + nb_launch);
  hipError_t er;
  if (e0 && (er = hipEventRecord(e0, s)) != hipSuccess) return er;
  const bool narrow = use_narrow<T>(L), cached = in_cache(L.np, sizeof(T));
  uint32_t *done = reinterpret_cast<uint32_t *>(d.acc + 3);
  if (grid > 0) {
#define HLB_STEP(P, N)                                                                                    \
  do {                                                                                                  \
    if (cfg.scheme == HLB_SCHEME_PUSH)                                                                  \
      k_step_push<T, P, N><<<grid, kBlock, 0, s>>>(A, B, a, d.order, n0, nb_io, blk0, nb_bulk,          \
                                                   cfg.xcd_chunk, omega, d.flux, done);                        \
    else if (pair)                                                                                      \
      k_step<T, P, N, false, 2><<<grid, kBlock, 0, s>>>(A, B, a, d.order, n0, nb_io, 0, nb_launch,      \
                                                        cfg.xcd_chunk, omega, d.flux, done);            \
    else if (cached)                                                                                    \
      k_step<T, P, N, true><<<grid, kBlock, 0, s>>>(A, B, a, d.order, n0, nb_io, blk0, nb_bulk,         \
                                                    cfg.xcd_chunk, omega, d.flux, done);                \
    else                                                                                                \
      k_step<T, P, N, false><<<grid, kBlock, 0, s>>>(A, B, a, d.order, n0, nb_io, blk0, nb_bulk,        \
                                                     cfg.xcd_chunk, omega, d.flux, done);               \
  } while (0)
    if (cfg.porous) {
      if (narrow) HLB_STEP(true, true);
      else HLB_STEP(true, false);
    } else {
      if (narrow) HLB_STEP(false, true);
      else HLB_STEP(false, false);
    }
#undef HLB_STEP
  }
  if ((er = hipGetLastError()) != hipSuccess) return er;
  if (a.wk_n > 0 && part == 0 && nb_io == 0) k_windkessel<<<(a.wk_n + 63) / 64, 64, 0, s>>>(a);
  if ((er = hipGetLastError()) != hipSuccess) return er;
  if (e1 && (er = hipEventRecord(e1, s)) != hipSuccess) return er;
  return hipSuccess;
}

// Halo exchange (one-GPU emulation of the domain split; the same kernels
// serve a multi-GPU run): pack copies the listed (position, direction)
// values of a population buffer into a contiguous buffer, unpack writes a
// contiguous buffer into the listed slots.  Raw stored values, no rounding.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pack(const T *__restrict__ A, const int32_t *__restrict__ pos,
                                                 const int32_t *__restrict__ dir, int64_t n, T *__restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (k < n) out[k] = A[pidx(pos[k], dir[k])];
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_unpack(T *__restrict__ A, const int32_t *__restrict__ pos,
                                                   const int32_t *__restrict__ dir, int64_t n,
                                                   const T *__restrict__ in) {
  const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (k < n) A[pidx(pos[k], dir[k])] = in[k];
}

template <typename T>
hipError_t halo_impl(const DevPtrs &d, int buf, const int32_t *pos, const int32_t *dir, int64_t n, void *io,
                     bool pack, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (pack)
    k_pack<T><<<blocks_for(n), kBlock, 0, s>>>(static_cast<const T *>(d.f[buf]), pos, dir, n, static_cast<T *>(io));
  else
    k_unpack<T><<<blocks_for(n), kBlock, 0, s>>>(static_cast<T *>(d.f[buf]), pos, dir, n,
                                                 static_cast<const T *>(io));
  return hipGetLastError();
}

template <typename T>
hipError_t macros_impl(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, int src, bool direct,
                       int64_t t_prev, double *rho, double *u, double *wss, double *f_out,
                       hipStream_t s) {
  const T *A = static_cast<const T *>(d.f[src]);
  GatherArgs a = make_args(cfg, L, d, t_prev < 0 ? 0 : t_prev);
  a.io_flux = nullptr;  // the re-gather does not count towards the outflow
  const int64_t n0 = L.gcnt[0], nb_bulk = (n0 + kBlock - 1) / kBlock;
  const int64_t nb_io = (L.gbeg[kGroups] - L.io_begin) / kBlock;
  const unsigned grid = (unsigned)(nb_io + nb_bulk);
  const bool narrow = use_narrow<T>(L);
#define HLB_MACROS(SRC, N)                                                                                       \
  do {                                                                                                           \
    if (f_out)                                                                                                   \
      k_macros<T, SRC, N, true><<<grid, kBlock, 0, s>>>(A, a, d.order, n0, nb_io, nb_bulk, cfg.xcd_chunk,        \
                                                        cfg.tau, rho, u, wss, f_out);                            \
    else                                                                                                         \
      k_macros<T, SRC, N, false><<<grid, kBlock, 0, s>>>(A, a, d.order, n0, nb_io, nb_bulk, cfg.xcd_chunk,       \
                                                         cfg.tau, rho, u, wss, f_out);                           \
  } while (0)
  if (direct) {
    if (narrow) HLB_MACROS(kDirect, true);
    else HLB_MACROS(kDirect, false);
  } else if (cfg.porous) {
    if (narrow) HLB_MACROS(kPulledPorous, true);
    else HLB_MACROS(kPulledPorous, false);
  } else {
    if (narrow) HLB_MACROS(kPulled, true);
    else HLB_MACROS(kPulled, false);
  }
#undef HLB_MACROS
  return hipGetLastError();
}

template <typename T>
hipError_t init_impl(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, const double *staging,
                     hipStream_t s) {
  k_init_eq<T><<<blocks_for(L.np), kBlock, 0, s>>>(static_cast<T *>(d.f[0]), static_cast<T *>(d.f[1]),
                                                   d.order, L.np, staging, cfg.rho0);
  return hipGetLastError();
}

template <typename T>
hipError_t set_state_impl(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, int pre,
                          const double *staging, hipStream_t s) {
  using C = typename Acc<T>::type;
  k_set_state<T><<<blocks_for(L.np), kBlock, 0, s>>>(static_cast<T *>(d.f[pre]), static_cast<T *>(d.f[1 - pre]),
                                                     d.order, L.np, staging, cfg.rho0, C(1.0 / cfg.tau));
  return hipGetLastError();
}

template <typename T>
hipError_t mass_impl(const Layout &L, const DevPtrs &d, int src, hipStream_t s) {
  int64_t nb = blocks_for(L.np);
  if (nb > d.partial_len - 1) nb = d.partial_len - 1;
  k_mass_partial<T><<<(unsigned)nb, kBlock, 0, s>>>(static_cast<const T *>(d.f[src]), d.order, L.np, d.partial);
  k_mass_final<<<1, kBlock, 0, s>>>(d.partial, nb, d.acc, d.flux);
  return hipGetLastError();
}

}  // namespace

#define HLB_DISPATCH(storage, CALL)                       \
  switch (storage) {                                      \
    case HLB_F64: { using T = double; return CALL; }      \
    case HLB_F32_SHIFTED: { using T = float; return CALL; } \
    case HLB_F16_SHIFTED: { using T = _Float16; return CALL; } \
    default: return hipErrorInvalidValue;                 \
  }

int default_sites_per_thread(int storage) {
  (void)storage;
  return 1;
}

hipError_t launch_step(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, int src, int64_t t,
                       hipStream_t s, hipEvent_t e0, hipEvent_t e1, int part) {
  HLB_DISPATCH(cfg.storage, step_impl<T>(cfg, L, d, src, t, s, e0, e1, part));
}

hipError_t launch_halo(const LaunchCfg &cfg, const DevPtrs &d, int buf, const int32_t *pos, const int32_t *dir,
                       int64_t n, void *io, bool pack, hipStream_t s) {
  HLB_DISPATCH(cfg.storage, halo_impl<T>(d, buf, pos, dir, n, io, pack, s));
}

hipError_t launch_init_eq(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, const double *staging,
                          hipStream_t s) {
  HLB_DISPATCH(cfg.storage, init_impl<T>(cfg, L, d, staging, s));
}

hipError_t launch_macros(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, int src, bool direct,
                         int64_t t_prev, double *rho, double *u, double *wss, double *f_out, hipStream_t s) {
  HLB_DISPATCH(cfg.storage, macros_impl<T>(cfg, L, d, src, direct, t_prev, rho, u, wss, f_out, s));
}

hipError_t launch_set_state(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, int pre,
                            const double *staging, hipStream_t s) {
  HLB_DISPATCH(cfg.storage, set_state_impl<T>(cfg, L, d, pre, staging, s));
}

hipError_t launch_set_time(int64_t *p, int64_t v, hipStream_t s) {
  k_set_time<<<1, 1, 0, s>>>(p, v);
  return hipGetLastError();
}

hipError_t launch_add_time(int64_t *p, int64_t k, hipStream_t s) {
  k_add_time<<<1, 1, 0, s>>>(p, k);
  return hipGetLastError();
}

hipError_t launch_total_flux(const double *acc, const double *flux, double *out, hipStream_t s) {
  k_total_flux<<<1, kBlock, 0, s>>>(acc, flux, out);
  return hipGetLastError();
}

hipError_t launch_set_flux(double *acc, double *flux, const double *from, double v, hipStream_t s) {
  k_set_flux<<<kFluxSlots / kBlock, kBlock, 0, s>>>(acc, flux, from, v);
  return hipGetLastError();
}

hipError_t launch_zero(double *p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_zero<<<blocks_for(n), kBlock, 0, s>>>(p, n);
  return hipGetLastError();
}

hipError_t launch_mass(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, int src, hipStream_t s) {
  HLB_DISPATCH(cfg.storage, mass_impl<T>(L, d, src, s));
}

}  // namespace hlb
