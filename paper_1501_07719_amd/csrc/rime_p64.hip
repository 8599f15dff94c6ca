// Float64 engine of one sky over large arrays (gfx950).
//
//   p64_planes    a_ps = e_ps K_ps (and the beam-gradient factor k3) of every
//                 (timestep, channel, source, antenna), once per call, in HBM,
//                 for one pass over time after the other;
//   p64_forward   source sums, visibilities, chi^2 and residual of 16 x 16
//                 antenna sub-blocks;
//   p64_adjoint   the gradient sums of 64 sources over one sub-block;
//   p64_fin_items, p64_stokes_t, p64_finalize
//                 the sums of the adjoint's partials, the first two per pass.
//
// The per-baseline kernel (rime_main) forms every antenna's terms in each
// workgroup whose tile holds the antenna, which took half of its float64
// forward, and feeds both passes from LDS: 64 bytes per term and lane, as much
// LDS time as float64 instructions.  Here the terms are formed once and one
// wavefront owns a 16 x 16 sub-block, without workgroup barriers: in the
// forward a lane holds four baselines and a term costs 16 to 20 bytes of LDS,
// brightness and shape being SGPR operands; in the adjoint a lane is a source
// and holds eight antennas in registers, the residual coming as LDS
// broadcasts.
//
// Bound by float64 instruction issue (the chip holds 1.9 to 2.0 GHz under them).
// 64 antennas, 100 timesteps, 64 channels, 1000 points + 500 Gaussians, beam,
// sums over the passes of a call:
//   planes 2.1 ms (2.7 ms with k3), forward 18.4 ms (12 instructions per point
//   term and 37 per Gaussian term in the loops, 22.8 per term in all, 72 to 76 %
//   of the issue slots used), adjoint 17.8 ms for the points (28 in the loop,
//   33.7 in all, 75 %) and 17.3 ms for the Gaussians (61, 68.9, 77 %);
//   chi^2 + gradient 57.0 ms, chi^2 20.0 ms, against 88.7 and 28.0 ms on the
//   per-baseline kernel.
// Measured and not kept: point-source sums on v_mfma_f64_16x16x4_f64 (forward
// 9.4 ms for the points alone; float64 matrix and vector instructions have the
// same rate and do not overlap, and the matrix form takes 16 multiply-adds per
// term against 12); the residual through scalar loads (points 33 ms: each load
// waits about 2000 cycles); antenna-fastest planes (points 31.5 ms: every load
// of the adjoint touched 64 cache lines).
#include "rime_device.h"

namespace rime {

// ---------------------------------------------------------------------------
// Planes: thread = (antenna, source) of one timestep and one block of
// p.phase_nc channels; the phase argument and the beam radius are formed once
// per block.  The source is the fastest index (the adjoint's lanes are sources).
// ---------------------------------------------------------------------------
template <bool WITH_K3>
__global__ __launch_bounds__(256) void p64_planes(const KParams p) {
  const int tt = blockIdx.y;
  const int t = p.pme_t0 + tt;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t plane = static_cast<int64_t>(p.nap) * p.p64_ns;
  if (idx >= plane) return;
  const int cb = blockIdx.z * p.phase_nc;
  const int ce = min(p.nchan, cb + p.phase_nc);
  const int a = static_cast<int>(idx / p.p64_ns);
  const int s = static_cast<int>(idx - static_cast<int64_t>(a) * p.p64_ns);
  if (s >= p.total_src) return;  // row padding, never used
  const int64_t o = static_cast<int64_t>(tt) * p.nchan * plane + idx;
  double2 *pa = p.p64_a + o;
  double *pk = p.p64_k3 + o;
  if (a >= p.na) {
    for (int c = cb; c < ce; ++c) {
      pa[c * plane] = make_double2(0.0, 0.0);
      if (WITH_K3) pk[c * plane] = 0.0;
    }
    return;
  }
  const double4 g = p.src_geo[s];
  const double *x = p.uvw + (static_cast<int64_t>(t) * p.na + a) * 3;
  const PhaseArg<true> tau(x[0], x[1], x[2], g.x, g.y, g.z);
  double r2b = 0.0, rb = 0.0;
  if (p.beam) {
    const double *q = p.pointing + (static_cast<int64_t>(t) * p.na + a) * 2;
    r2b = sumsq_rn(g.x - q[0], g.y - q[1]);
    rb = sqrt(r2b);
  }
  for (int c = cb; c < ce; ++c) {
    double2 v;
    double k3;
    antenna_term<double, WITH_K3>(p, tau, r2b, rb, c, v, k3);
    pa[c * plane] = v;
    if (WITH_K3) pk[c * plane] = k3;
  }
}

// A wavefront's task in the forward: sub-block (si, sj) of an antenna-block
// pair.  Lane (j = lane % 16, g = lane / 16) holds the baselines (row 4 r + g,
// column j), r < NR; with fewer than four rows per lane, `part` says which
// quarter or half.  A folded task is a sub-block on the diagonal whose
// baselines all lie above it: rows 0..7 only, and a lane below the diagonal
// takes the baseline (j + 8, row + 8) of the lower right quarter instead, so
// that two rows per lane cover all 120 baselines.
struct Task {
  int pair, si, sj, fold, part;
};

__device__ inline Task task_of(int w) {
  return {w >> 6, (w >> 5) & 1, (w >> 4) & 1, (w >> 3) & 1, w & 7};
}

// Waits for every scalar load and LDS access of the wavefront.  Scalar loads
// return out of order and share their counter with LDS, so the first use of
// any of them waits for all that are in flight: the loops below wait once per
// step and only then start the next step's loads, which the step's arithmetic
// covers.
__device__ inline void wait_lgkm() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0); vmcnt and expcnt at their maximum
  __builtin_amdgcn_sched_barrier(0);
}

// Between LDS accesses of a wavefront's lanes to each other's data.  The
// hardware keeps a wavefront's LDS accesses in order; this keeps the compiler
// from reordering them.  No instruction.
__device__ inline void lane_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Source sums over [s0, s1) (one morphology) of this lane's NR baselines.  The
// antenna terms of four sources at a time go from the planes (one 16-byte load
// per lane and side) through the wavefront's own LDS buffers, two chunks ahead;
// brightness, shape and the lane's terms of the next source are loaded during
// the current one.
template <int SHAPE, bool ST, int NR, bool FOLD>
__device__ inline void p64_sweep(const KParams &p, const double2 *pp, const double2 *pq,
                                 double2 (*s_a)[4][32], int s0, int s1, int c, int t,
                                 const int (&ip)[NR], const int (&iq)[NR], const double (&du)[NR],
                                 const double (&dv)[NR], double gq, double (&aR)[NR][4],
                                 double (&aI)[NR][4]) {
  using N = Num<double>;
  constexpr int NQ = FOLD ? NR : 1;
  if (s0 >= s1) return;
  const int lane = threadIdx.x % kWave;
  const int ls = lane >> 4, la = lane & 15;
  const int nsrc = p.one.npsrc + p.one.ngsrc + p.one.nxsrc;
  double2 xp, xq;
  auto fetch = [&](int s) {
    // past the range: its last source again, never used
    const int o = la * p.p64_ns + min(s + ls, s1 - 1);
    xp = pp[o];
    xq = pq[o];
  };
  auto put = [&](int buf) {
    lane_exchange();
    s_a[buf][ls][la] = xp;
    s_a[buf][ls][16 + la] = xq;
    lane_exchange();
  };
  // brightness by (channel, source): the next source's lies in the same cache line
  const RIME_CONST Quad<double> *st =
      const_ptr<Quad<double>>(p.src_st) + static_cast<int64_t>(c) * p.p64_ns;
  const RIME_CONST Quad<double> *gs = const_ptr<Quad<double>>(p.src_gs);
  const RIME_CONST Quad<double> *stt =
      const_ptr<Quad<double>>(p.stokes_t) + static_cast<int64_t>(t) * nsrc;
  const RIME_CONST double *sf = const_ptr<double>(p.src_sf) + static_cast<int64_t>(c) * p.p64_ns;
  struct Op {
    Quad<double> b, g;  // brightness (ST: Stokes of the timestep), shape
    double f;           // ST: spectral factor
    double2 ap[NR], aq[NQ];
  };
  auto load = [&](Op &o, int s, int buf, int i) {
#pragma unroll
    for (int r = 0; r < NR; ++r) o.ap[r] = s_a[buf][i][ip[r]];
#pragma unroll
    for (int r = 0; r < NQ; ++r) o.aq[r] = s_a[buf][i][16 + iq[r]];
    s = min(s, s1 - 1);
    if (ST) {
      o.b = stt[s];
      o.f = sf[s];
    } else {
      o.b = st[s];
    }
    if (SHAPE != SHAPE_POINT) o.g = gs[s];
  };
  auto compute = [&](const Op &o) {
    double bk[4] = {o.b.x, o.b.y, o.b.z, o.b.w};
    if (ST) {
#pragma unroll
      for (int k = 0; k < 4; ++k) bk[k] *= o.f;
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const double2 ap = o.ap[r], aq = o.aq[FOLD ? r : 0];
      double cr = ap.x * aq.x + ap.y * aq.y;
      double ci = ap.y * aq.x - ap.x * aq.y;
      if (SHAPE != SHAPE_POINT) {
        const double A = du[r] * o.g.x + dv[r] * o.g.y;
        const double B = du[r] * o.g.z - dv[r] * o.g.w;
        const double Q = A * A + B * B;
        double S;
        if (SHAPE == SHAPE_GAUSS) {
          S = N::expb(gq * Q);
        } else {
          const double h = N::rsqrt_(1.0 + gq * Q);
          S = h * h * h;
        }
        cr *= S;
        ci *= S;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        aR[r][k] += cr * bk[k];
        aI[r][k] += ci * bk[k];
      }
    }
  };
  fetch(s0);
  put(0);
  fetch(s0 + 4);
  Op nxt;
  load(nxt, s0, 0, 0);
  int buf = 0;
  for (int s = s0; s < s1; s += 4) {
    put(buf ^ 1);
    fetch(s + 8);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (s + i >= s1) break;
      wait_lgkm();
      const Op cur = nxt;
      load(nxt, s + i + 1, i < 3 ? buf : buf ^ 1, (i + 1) & 3);
      __builtin_amdgcn_sched_barrier(0);
      compute(cur);
    }
    buf ^= 1;
  }
}

// One task over timesteps [t0, t1) at channel c; returns this lane's chi^2.
template <int MODE, bool TERMS, int NR, bool FOLD>
__device__ inline Comp p64_task(const KParams &p, const Task tk, int t0, int t1, int c,
                                double2 (*s_a)[4][32]) {
  constexpr bool PREDICT = MODE == MODE_PREDICT;
  constexpr bool RHO = MODE == MODE_GRAD || MODE == MODE_RESID;
  using DT = typename Pick<MODE == MODE_RESID, float, double>::T;
  const int lane = threadIdx.x % kWave;
  const int j = lane & 15, g = lane >> 4;
  const int2 blk = p.pair_blk[tk.pair];
  const int P0 = blk.x * kPmeBlk + tk.si * 16, Q0 = blk.y * kPmeBlk + tk.sj * 16;
  int ip[NR], iq[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int i = (tk.part * NR + r) * 4 + g;
    const bool low = FOLD && j < i && j < 8;
    ip[r] = low ? j + 8 : i;
    iq[r] = low ? i + 8 : j;
  }
  const int64_t plane = static_cast<int64_t>(p.nap) * p.p64_ns;
  const double nuc = p.nu_c[c];
  const double gg_ = -kGauss * kLog2e * nuc * nuc, gd = 4.0 * kPi * kPi * nuc * nuc;
  const int np = p.one.npsrc, ng = np + p.one.ngsrc, nx = ng + p.one.nxsrc;
  Comp chi;
  for (int t = t0; t < t1; ++t) {
    const int tt = t - p.pme_t0;
    const double2 *pl = p.p64_a + (static_cast<int64_t>(tt) * p.nchan + c) * plane;
    const double2 *pp = pl + static_cast<int64_t>(P0) * p.p64_ns;
    const double2 *pq = pl + static_cast<int64_t>(Q0) * p.p64_ns;
    double du[NR], dv[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      // antennas past the array (in the last sub-block) carry no baseline
      const int a = min(P0 + ip[r], p.na - 1), b = min(Q0 + iq[r], p.na - 1);
      const double *up = p.uvw + (static_cast<int64_t>(t) * p.na + a) * 3;
      const double *uq = p.uvw + (static_cast<int64_t>(t) * p.na + b) * 3;
      du[r] = up[0] - uq[0];
      dv[r] = up[1] - uq[1];
    }
    double aR[NR][4], aI[NR][4];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k) aR[r][k] = aI[r][k] = 0.0;
    const bool st = TERMS && p.stokes_t;
    if (st) {
      p64_sweep<SHAPE_POINT, TERMS, NR, FOLD>(p, pp, pq, s_a, 0, np, c, t, ip, iq, du,
                                              dv, gg_, aR, aI);
      p64_sweep<SHAPE_GAUSS, TERMS, NR, FOLD>(p, pp, pq, s_a, np, ng, c, t, ip, iq, du,
                                              dv, gg_, aR, aI);
      p64_sweep<SHAPE_DISK, TERMS, NR, FOLD>(p, pp, pq, s_a, ng, nx, c, t, ip, iq, du,
                                             dv, gd, aR, aI);
    } else {
      p64_sweep<SHAPE_POINT, false, NR, FOLD>(p, pp, pq, s_a, 0, np, c, t, ip, iq, du,
                                              dv, gg_, aR, aI);
      p64_sweep<SHAPE_GAUSS, false, NR, FOLD>(p, pp, pq, s_a, np, ng, c, t, ip, iq, du,
                                              dv, gg_, aR, aI);
      p64_sweep<SHAPE_DISK, false, NR, FOLD>(p, pp, pq, s_a, ng, nx, c, t, ip, iq, du,
                                             dv, gd, aR, aI);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int i = tk.si * 16 + ip[r], jj = tk.sj * 16 + iq[r];
      const int slot = (tk.pair * kPmeBlk + i) * kPmeBlk + jj;
      const int sb = p.slot_bl[slot];
      if (sb < 0) continue;
      // a baseline stored as (q, p) takes the conjugate sums
      const int bl = sb >> 1;
      const bool sw = sb & 1;
      const double cj = sw ? -1.0 : 1.0;
      const int gap = sw ? Q0 + iq[r] : P0 + ip[r], gaq = sw ? P0 + ip[r] : Q0 + iq[r];
      double2 gg[4];
      gain_products(p, gap, gaq, gg);
      double S[8];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        S[2 * k] = aR[r][k];
        S[2 * k + 1] = cj * aI[r][k];
      }
      const int64_t vidx = ((static_cast<int64_t>(t) * p.nbl + bl) * p.nchan + c) * 4;
      using A = DT;
      typename Num<A>::R2 rho[4];
      visibility<double, DT, A, PREDICT, RHO, TERMS>(p, true, t, gap, gaq, c, vidx, S, gg, chi,
                                                     rho);
      if constexpr (MODE == MODE_GRAD) {
        double2 *o = p.p64_rho +
                     ((static_cast<int64_t>(tt) * p.nchan + c) * p.npair * (kPmeBlk * kPmeBlk) +
                      slot) *
                         4;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = make_double2(rho[k].x, cj * rho[k].y);
      } else if constexpr (MODE == MODE_RESID) {
        if (p.rho_b) {
#pragma unroll
          for (int k = 0; k < 4; ++k) p.rho_b[vidx + k] = make_float2(rho[k].x, rho[k].y);
        }
        if (p.pme_adj) {
          const float cf = sw ? -1.0f : 1.0f;
          float2 *o = p.rho_t +
                      ((static_cast<int64_t>(t) * p.nchan + c) * p.npair + tk.pair) * 4 *
                          (kPmeBlk * kPmeBlk) +
                      i * kPmeBlk + jj;
#pragma unroll
          for (int k = 0; k < 4; ++k)
            o[k * kPmeBlk * kPmeBlk] = make_float2(rho[k].x, cf * rho[k].y);
        }
      }
    }
  }
  return chi;
}

// Forward: wavefront = (chunk of p.p64_tch timesteps, channel, task); the four
// wavefronts of a workgroup take four adjacent channels, whose data share
// cache lines.
template <int MODE, bool TERMS, int NR>
__global__ __launch_bounds__(256, 2) void p64_forward(const KParams p) {
  __shared__ __attribute__((aligned(16))) double2 s_a[4][2][4][32];
  const int ncq = (p.nchan + 3) / 4;
  const int ntch = (p.pme_nt + p.p64_tch - 1) / p.p64_tch;
  const int nwg = ntch * ncq * p.p64_ntask;
  const int wg = xcd_item(nwg);
  if (wg >= nwg) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int task = wg % p.p64_ntask;
  const int rest = wg / p.p64_ntask;
  const int c = (rest % ncq) * 4 + wave;
  const int tc = rest / ncq;
  if (c >= p.nchan) return;
  const Task tk = task_of(p.p64_task[task]);
  const int t0 = p.pme_t0 + tc * p.p64_tch;
  const int t1 = min(p.pme_t0 + p.pme_nt, t0 + p.p64_tch);
  Comp chi = tk.fold ? p64_task<MODE, TERMS, (NR > 2 ? 2 : NR), true>(p, tk, t0, t1, c, s_a[wave])
                     : p64_task<MODE, TERMS, NR, false>(p, tk, t0, t1, c, s_a[wave]);
  if (MODE != MODE_PREDICT) {
    chi = wave_reduce(chi);
    if (threadIdx.x % kWave == 0)
      p.chi2_part[p.p64_item0 + (static_cast<int64_t>(tc) * p.nchan + c) * p.p64_ntask + task] =
          make_double2(chi.s, chi.c);
  }
}

// ---------------------------------------------------------------------------
// Adjoint: wavefront = (64 sources of one morphology, timestep, p.p64_ncw
// channels, sub-block or, in small calls, an eighth of one); lane = source.
// The sub-block's columns are taken eight at a time: their antenna terms and
// their sums of Re P and Im P (P = c sum_k St'_k rho_k) stay in registers, the
// rows pass by, and the residual and baseline vector of a slot come as LDS
// broadcasts.  With the row and column sums of P the position gradient needs no
// per-baseline factor:
//   sum (u_p - u_q) Im P        = sum_p u_p row_p - sum_q u_q col_q
//                                 (u from an origin inside the sub-block),
//   sum (beta_p + beta_q) Re P  = sum_p beta_p row_p + sum_q beta_q col_q.
// The Stokes and shape sums are those of adjoint_loop (rime_kernels.hip).
// ---------------------------------------------------------------------------
// LDS of one wavefront of the adjoint: residual and baseline vectors of two
// rows of eight slots, double buffered; the sub-block's 32 antennas
// (u, v | w | pointing l, m); and the sums over the item's channels.
struct AdjLds {
  double2 rho[2][2][8][4];
  double2 geo[2][2][8];
  double2 ant[32][3];
  double grad[10][kWave];
};

// The value of x in one lane (wavefront-uniform index).
__device__ inline double lane_value(double x, int lane) {
  const int64_t b = __double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(b), lane);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), lane);
  return __longlong_as_double(static_cast<int64_t>(static_cast<uint64_t>(hi) << 32 | lo));
}

template <int SHAPE, bool ST>
__device__ inline void p64_adj_item(const KParams &p, int sub, int part, int t, int cg, int s,
                                    AdjLds &lds) {
  using N = Num<double>;
  constexpr int NQ = 8;
  const int lane = threadIdx.x % kWave;
  const int tt = t - p.pme_t0;
  const int pair = sub >> 2, si = (sub >> 1) & 1, sj = sub & 1;
  const int2 blk = p.pair_blk[pair];
  const int P0 = __builtin_amdgcn_readfirstlane(blk.x) * kPmeBlk + si * 16;
  const int Q0 = __builtin_amdgcn_readfirstlane(blk.y) * kPmeBlk + sj * 16;
  // row masks, one per lane.  The coordinates of the 16 + 16 antennas are taken
  // from the first row's antenna that holds a baseline here: only differences
  // enter, and an offset common to all antennas would otherwise cost digits in
  // the difference of the row and column sums.
  const uint32_t maskv = p.pair_mask[pair * kPmeBlk + si * 16 + (lane & 15)];
  {
    const int a = min((lane & 16 ? Q0 : P0) + (lane & 15), p.na - 1);
    const double *x = p.uvw + (static_cast<int64_t>(t) * p.na + a) * 3;
    const double *q = p.pointing + (static_cast<int64_t>(t) * p.na + a) * 2;
    const double u = x[0], v = x[1], w = x[2], ql = q[0], qm = q[1];
    const uint64_t rows = __ballot(((maskv >> (sj * 16)) & 0xffffu) != 0u);
    const int first = __builtin_ctzll(rows);
    const double u0 = lane_value(u, first), v0 = lane_value(v, first), w0 = lane_value(w, first);
    if (lane < 32) {
      lds.ant[lane][0] = make_double2(u - u0, v - v0);
      lds.ant[lane][1] = make_double2(w - w0, 0.0);
      lds.ant[lane][2] = make_double2(ql, qm);
    }
    lane_exchange();
  }
  const int64_t plane = static_cast<int64_t>(p.nap) * p.p64_ns;
  const int64_t slot0 = static_cast<int64_t>(pair) * (kPmeBlk * kPmeBlk) + si * 16 * kPmeBlk +
                        sj * 16;
  // this lane's part of two rows of eight slots: row, slot and Stokes parameter
  const int64_t lrho = ((lane >> 5) * kPmeBlk + ((lane >> 2) & 7)) * 4 + (lane & 3);
  const int64_t lgeo = ((lane >> 3) & 1) * kPmeBlk + (lane & 7);
  const double2 *geo = p.p64_geo +
                       static_cast<int64_t>(t) * p.npair * (kPmeBlk * kPmeBlk) + slot0 + lgeo;
  const double4 sg = p.src_geo[s];
  const double2 lo = p.src_lon[s];
  double4 e0 = make_double4(0.0, 0.0, 0.0, 0.0);
  double Rr = 0.0;
  if (SHAPE != SHAPE_POINT) {
    e0 = static_cast<const double4 *>(p.src_gs)[s];
    const int xi = s - p.one.npsrc;
    Rr = SHAPE == SHAPE_DISK ? p.one.xshape[3 * (xi - p.one.ngsrc) + 2] : p.one.gshape[3 * xi + 2];
  }
  // a split item: one half of the columns against a quarter of the rows
  const bool split = p.p64_split > 1;
  const int h0 = split ? part & 1 : 0, h1 = split ? h0 + 1 : 16 / NQ;
  const int r0 = split ? (part >> 1) * 4 : 0, r1 = split ? r0 + 4 : 16;
  const int c1 = min(p.nchan, (cg + 1) * p.p64_ncw);
  for (int c = cg * p.p64_ncw; c < c1; ++c) {
    const int64_t pc = static_cast<int64_t>(tt) * p.nchan + c;
    const int64_t ro = pc * plane + s;
    const double2 *col = p.p64_a + ro;  // this source's terms, p.p64_ns apart
    // without a beam the loads of k3 stay (a wait must not depend on a
    // branch), from the other plane, and what they read (padding that no
    // kernel writes among it) is replaced by zero, not multiplied by it
    const bool beam = p.p64_k3 != nullptr;
    const double *k3 = (beam ? p.p64_k3 : reinterpret_cast<const double *>(p.p64_a)) + ro;
    const double2 *rho = p.p64_rho + (pc * p.npair * (kPmeBlk * kPmeBlk) + slot0) * 4 + lrho;
    const int64_t cs = static_cast<int64_t>(c) * p.p64_ns + s;
    const double f = static_cast<const double *>(p.src_sf)[cs];
    double4 st = static_cast<const double4 *>(p.src_st)[cs];
    if (ST) {
      const double *q = p.stokes_t + (static_cast<int64_t>(t) * p.total_src + s) * 4;
      st = make_double4(f * q[0], f * q[1], f * q[2], f * q[3]);
    }
    const double nuc = p.nu_c[c];
    const double kap = (SHAPE == SHAPE_DISK ? 2.0 * kPi : sqrt(kGauss * N::kExpScale)) * nuc;
    const double ex = kap * e0.x, ey = kap * e0.y, ez = kap * e0.z, ew = kap * e0.w;
    double g0 = 0.0, g1 = 0.0, g2 = 0.0, g3 = 0.0;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0, s4 = 0.0;
    double o1 = 0.0, o2 = 0.0, o3 = 0.0, bl = 0.0, bm = 0.0;
    // a row or column sum of P at an antenna into the position sums
    auto fold = [&](int a, double k, double sR, double sI) {
      const double2 uv = lds.ant[a][0], w = lds.ant[a][1], pl = lds.ant[a][2];
      o1 += uv.x * sI;
      o2 += uv.y * sI;
      o3 += w.x * sI;
      const double kR = beam ? k * sR : 0.0;
      bl += kR * (sg.x - pl.x);
      bm += kR * (sg.y - pl.y);
    };
#pragma unroll 1
    for (int h = h0; h < h1; ++h) {
      double2 xr, xg = make_double2(0.0, 0.0);
      auto fetch = [&](int i) {
        // rows i and i + 1; past the sub-block its last two again, never used
        const int o = min(i, 14) * kPmeBlk + h * NQ;
        xr = rho[o * 4];
        if (SHAPE != SHAPE_POINT) xg = geo[o];
      };
      auto put = [&](int buf) {
        lane_exchange();
        (&lds.rho[buf][0][0][0])[lane] = xr;
        if (SHAPE != SHAPE_POINT && lane < 16) (&lds.geo[buf][0][0])[lane] = xg;
        lane_exchange();
      };
      double2 aq[NQ];
      double colR[NQ], colI[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        aq[q] = col[static_cast<int64_t>(Q0 + h * NQ + q) * p.p64_ns];
        colR[q] = colI[q] = 0.0;
      }
      fetch(r0);
      put(0);
      fetch(r0 + 2);
      double2 ap_n = col[static_cast<int64_t>(P0 + r0) * p.p64_ns];
      double kp_n = k3[static_cast<int64_t>(P0 + r0) * p.p64_ns];
      int buf = 0;
#pragma unroll 1
      for (int i2 = r0; i2 < r1; i2 += 2) {
        put(buf ^ 1);
        fetch(i2 + 4);
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int i = i2 + y, in = min(i + 1, 15);
          const double2 ap = ap_n;
          const double kp = kp_n;
          ap_n = col[static_cast<int64_t>(P0 + in) * p.p64_ns];
          kp_n = k3[static_cast<int64_t>(P0 + in) * p.p64_ns];
          const uint32_t m =
              (__builtin_amdgcn_readlane(maskv, i) >> (sj * 16 + h * NQ)) & ((1u << NQ) - 1u);
          if (m == 0u) continue;
          double rowR = 0.0, rowI = 0.0;
          struct Slot {
            double2 r0, r1, r2, r3, d;  // residual, baseline vector
          };
          auto slot = [&](int q) {
            Slot x;
            x.r0 = lds.rho[buf][y][q][0];
            x.r1 = lds.rho[buf][y][q][1];
            x.r2 = lds.rho[buf][y][q][2];
            x.r3 = lds.rho[buf][y][q][3];
            if (SHAPE != SHAPE_POINT) x.d = lds.geo[buf][y][q];
            return x;
          };
          auto term = [&](int q, const Slot &x) {
            const double2 r0 = x.r0, r1 = x.r1, r2 = x.r2, r3 = x.r3;
            double cr = ap.x * aq[q].x + ap.y * aq[q].y;
            double ci = ap.y * aq[q].x - ap.x * aq[q].y;
            double2 d = make_double2(0.0, 0.0);
            double A = 0.0, B = 0.0, hh = 1.0;
            if (SHAPE != SHAPE_POINT) {
              d = x.d;
              A = d.x * ex + d.y * ey;
              B = d.x * ez - d.y * ew;
              double S;
              if (SHAPE == SHAPE_GAUSS) {
                S = N::expb(-(A * A + B * B));
              } else {
                const double r = N::rsqrt_(1.0 + A * A + B * B);
                hh = r * r;
                S = hh * r;
              }
              cr *= S;
              ci *= S;
            }
            g0 += cr * r0.x;
            g0 -= ci * r0.y;
            g1 += cr * r1.x;
            g1 -= ci * r1.y;
            g2 += cr * r2.x;
            g2 -= ci * r2.y;
            g3 += cr * r3.x;
            g3 -= ci * r3.y;
            const double phr = st.x * r0.x + st.y * r1.x + st.z * r2.x + st.w * r3.x;
            const double phi = st.x * r0.y + st.y * r1.y + st.z * r2.y + st.w * r3.y;
            const double Pr = cr * phr - ci * phi;
            const double Pi = cr * phi + ci * phr;
            rowR += Pr;
            rowI += Pi;
            colR[q] += Pr;
            colI[q] += Pi;
            if (SHAPE != SHAPE_POINT) {
              const double hP = SHAPE == SHAPE_DISK ? hh * Pr : Pr;
              const double t1 = A * hP, t2 = B * hP;
              s0 += d.x * t1;
              s1 += d.y * t2;
              s2 += d.y * t1;
              s3 += d.x * t2;
              s4 += B * t2;
            }
          };
          // a full row reads each slot during the one before
          if (m == (1u << NQ) - 1u) {
            Slot nxt = slot(0);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              const Slot cur = nxt;
              if (q + 1 < NQ) nxt = slot(q + 1);
              __builtin_amdgcn_sched_barrier(0);
              term(q, cur);
              __builtin_amdgcn_sched_barrier(0);
            }
          } else {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
              if ((m >> q) & 1u) term(q, slot(q));
          }
          fold(i, kp, rowR, rowI);
        }
        buf ^= 1;
      }
      double kq[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) kq[q] = k3[static_cast<int64_t>(Q0 + h * NQ + q) * p.p64_ns];
#pragma unroll
      for (int q = 0; q < NQ; ++q) fold(16 + h * NQ + q, kq[q], colR[q], -colI[q]);
    }
    const double tpnc = 2.0 * kPi * nuc;
    lds.grad[0][lane] += bl + tpnc * (o1 - lo.x * o3);
    lds.grad[1][lane] += bm + tpnc * (o2 - lo.y * o3);
    lds.grad[2][lane] += g0 * f;
    lds.grad[3][lane] += g1 * f;
    lds.grad[4][lane] += g2 * f;
    lds.grad[5][lane] += g3 * f;
    lds.grad[6][lane] += (st.x * g0 + st.y * g1 + st.z * g2 + st.w * g3) * p.lnfr[c];
    if (SHAPE != SHAPE_POINT) {
      const double dsc = SHAPE == SHAPE_DISK ? -3.0 * kap : -2.0 * kap / N::kExpScale;
      lds.grad[7][lane] += dsc * (s0 - Rr * s1);
      lds.grad[8][lane] += dsc * (s2 + Rr * s3);
      if (Rr > 0.0) lds.grad[9][lane] += dsc * s4 / (kap * Rr);
    }
  }
}

// SHAPED: the groups of Gaussians and disks, else those of point sources (two
// kernels, since the point sources need fewer registers).  Consecutive
// wavefronts take the source groups of one (timestep, channel group,
// sub-block), whose residual they share in L2.
template <bool SHAPED, bool ST>
__global__ __launch_bounds__(256, 2) void p64_adjoint(const KParams p) {
  __shared__ AdjLds s_lds[4];
  const int npg = (p.one.npsrc + kWave - 1) / kWave;
  const int sg0 = SHAPED ? npg : 0, nsg = SHAPED ? p.p64_nsg - npg : npg;
  const int nit = p.nsub * p.p64_split;
  const int64_t nitems = static_cast<int64_t>(nsg) * p.pme_nt * p.p64_ncg * nit;
  const int nwg = static_cast<int>((nitems + 3) / 4);
  const int wg = xcd_item(nwg);
  if (wg >= nwg) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t item = static_cast<int64_t>(wg) * 4 + wave;
  if (item >= nitems) return;
  const int sgr = sg0 + static_cast<int>(item % nsg);
  int64_t rest = item / nsg;
  const int isub = static_cast<int>(rest % nit);
  rest /= nit;
  const int cg = static_cast<int>(rest % p.p64_ncg);
  const int t = p.pme_t0 + static_cast<int>(rest / p.p64_ncg);
  const SrcTile tl = src_tile(p.one, sgr, kWave, npg, (p.one.ngsrc + kWave - 1) / kWave);
  const int lane = threadIdx.x % kWave;
  const int s = tl.s0 + min(lane, tl.cnt - 1);  // lanes past the group repeat its last source
  const int sub = const_ptr<int32_t>(p.sub)[isub / p.p64_split];
  const int part = isub % p.p64_split;
#pragma unroll
  for (int i = 0; i < 10; ++i) s_lds[wave].grad[i][lane] = 0.0;
  if constexpr (SHAPED) {
    if (tl.shape == SHAPE_GAUSS)
      p64_adj_item<SHAPE_GAUSS, ST>(p, sub, part, t, cg, s, s_lds[wave]);
    else
      p64_adj_item<SHAPE_DISK, ST>(p, sub, part, t, cg, s, s_lds[wave]);
  } else {
    p64_adj_item<SHAPE_POINT, ST>(p, sub, part, t, cg, s, s_lds[wave]);
  }
  // partials [source group][timestep][channel group][sub-block part][10][64]
  double *dst = p.p64_part +
                (((static_cast<int64_t>(sgr) * p.pme_nt + t - p.pme_t0) * p.p64_ncg + cg) * nit +
                 isub) * (10 * kWave) +
                lane;
#pragma unroll
  for (int i = 0; i < 10; ++i) dst[i * kWave] = s_lds[wave].grad[i][lane];
}

// Gradient rows from the adjoint partials, with a fixed order: after each pass
// over time, thread = one column (parameter, source) of a chunk of the pass's
// items, added to what the earlier passes left; at the end thread = (source,
// parameter) over the chunks.  The first launch after the last pass also forms
// chi^2, in an extra row of workgroups.
__global__ __launch_bounds__(256) void p64_fin_items(const KParams p) {
  constexpr int kRow = 10 * kWave;
  __shared__ double2 scr[256 / kWave];
  const int sg = blockIdx.y, ch = blockIdx.z;
  if (sg == p.p64_nsg) {
    if (blockIdx.x == 0 && ch == 0) chi2_reduce(p, 0, scr);
    return;
  }
  const int col = blockIdx.x * 256 + threadIdx.x;
  if (col >= kRow) return;
  const int64_t nper = static_cast<int64_t>(p.pme_nt) * p.p64_ncg * p.nsub * p.p64_split;
  const int64_t cs = (nper + p.pme_fchunk - 1) / p.pme_fchunk;
  const int64_t i1 = min(nper, (ch + 1) * cs);
  const double *src = p.p64_part + static_cast<int64_t>(sg) * nper * kRow + col;
  double2 *sum = p.pfin + (static_cast<int64_t>(sg) * p.pme_fchunk + ch) * kRow + col;
  Comp acc;
  if (p.pme_t0 > 0) {
    const double2 v = *sum;
    acc.merge(v.x, v.y);
  }
  int64_t i = ch * cs;
  for (; i + 8 <= i1; i += 8) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = src[(i + k) * kRow];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc.add(v[k]);
  }
  for (; i < i1; ++i) acc.add(src[i * kRow]);
  *sum = make_double2(acc.s, acc.c);
}

__global__ __launch_bounds__(256) void p64_finalize(const KParams p) {
  constexpr int kRow = 10 * kWave;
  const SrcTile tl = src_tile(p.one, blockIdx.y, kWave, (p.one.npsrc + kWave - 1) / kWave,
                              (p.one.ngsrc + kWave - 1) / kWave);
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int s = idx / 10, j = idx - s * 10;
  if (s >= tl.cnt) return;
  const double2 *src =
      p.pfin + static_cast<int64_t>(blockIdx.y) * p.pme_fchunk * kRow + j * kWave + s;
  Comp r;
  int ch = 0;
  for (; ch + 8 <= p.pme_fchunk; ch += 8) {
    double2 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = src[(ch + k) * kRow];
#pragma unroll
    for (int k = 0; k < 8; ++k) r.merge(v[k].x, v[k].y);
  }
  for (; ch < p.pme_fchunk; ++ch) {
    const double2 v = src[ch * kRow];
    r.merge(v.x, v.y);
  }
  p.grad_out[static_cast<int64_t>(tl.s0 + s) * 10 + j] = 2.0 * (r.s + r.c);
}

// Gradient of the brightness per timestep of the pass from the same partials.
__global__ __launch_bounds__(256) void p64_stokes_t(const KParams p) {
  const SrcTile tl = src_tile(p.one, blockIdx.y, kWave, (p.one.npsrc + kWave - 1) / kWave,
                              (p.one.ngsrc + kWave - 1) / kWave);
  const int t = p.pme_t0 + blockIdx.x;
  const int k = threadIdx.x / kWave, s = threadIdx.x % kWave;
  if (s >= tl.cnt) return;
  const int nit = p.p64_ncg * p.nsub * p.p64_split;
  const double *src = p.p64_part +
                      (static_cast<int64_t>(blockIdx.y) * p.pme_nt + blockIdx.x) * nit *
                          (10 * kWave) +
                      (2 + k) * kWave + s;
  Comp acc;
  int i = 0;
  for (; i + 8 <= nit; i += 8) {
    double v[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) v[x] = src[static_cast<int64_t>(i + x) * (10 * kWave)];
#pragma unroll
    for (int x = 0; x < 8; ++x) acc.add(v[x]);
  }
  for (; i < nit; ++i) acc.add(src[static_cast<int64_t>(i) * (10 * kWave)]);
  const int nsrc = p.one.npsrc + p.one.ngsrc + p.one.nxsrc;
  p.grad_stokes_t[(static_cast<int64_t>(t) * nsrc + tl.s0 + s) * 4 + k] = 2.0 * (acc.s + acc.c);
}

// ---------------------------------------------------------------------------
// Launchers (timesteps [p.pme_t0, p.pme_t0 + p.pme_nt))
// ---------------------------------------------------------------------------
hipError_t launch_p64_planes(const KParams &p, hipStream_t stream) {
  const int64_t plane = static_cast<int64_t>(p.nap) * p.p64_ns;
  KParams q = p;
  q.phase_nc = plane * static_cast<int64_t>(sizeof(double2)) >= (int64_t(1) << 20) ? 4 : 16;
  const dim3 g(static_cast<unsigned>((plane + 255) / 256), static_cast<unsigned>(p.pme_nt),
               static_cast<unsigned>((p.nchan + q.phase_nc - 1) / q.phase_nc));
  if (p.p64_k3)
    hipLaunchKernelGGL(p64_planes<true>, g, dim3(256), 0, stream, q);
  else
    hipLaunchKernelGGL(p64_planes<false>, g, dim3(256), 0, stream, q);
  return hipGetLastError();
}

template <int MODE, int NR>
static void forward(const KParams &p, dim3 g, hipStream_t stream) {
  if (p.die || p.stokes_t)
    hipLaunchKernelGGL((p64_forward<MODE, true, NR>), g, dim3(256), 0, stream, p);
  else
    hipLaunchKernelGGL((p64_forward<MODE, false, NR>), g, dim3(256), 0, stream, p);
}

hipError_t launch_p64_forward(const KParams &p, int mode, hipStream_t stream) {
  const int64_t nwg = static_cast<int64_t>((p.pme_nt + p.p64_tch - 1) / p.p64_tch) *
                      ((p.nchan + 3) / 4) * p.p64_ntask;
  const dim3 g(static_cast<unsigned>(8 * ((nwg + 7) / 8)));
  const bool wide = p.p64_nr == 4;
  switch (mode) {
    case MODE_PREDICT:
      wide ? forward<MODE_PREDICT, 4>(p, g, stream) : forward<MODE_PREDICT, 1>(p, g, stream);
      break;
    case MODE_CHI2:
      wide ? forward<MODE_CHI2, 4>(p, g, stream) : forward<MODE_CHI2, 1>(p, g, stream);
      break;
    case MODE_GRAD:
      wide ? forward<MODE_GRAD, 4>(p, g, stream) : forward<MODE_GRAD, 1>(p, g, stream);
      break;
    default:
      wide ? forward<MODE_RESID, 4>(p, g, stream) : forward<MODE_RESID, 1>(p, g, stream);
  }
  return hipGetLastError();
}

template <bool SHAPED>
static void adjoint(const KParams &p, int64_t nsg, hipStream_t stream) {
  if (nsg <= 0) return;
  const int64_t n = (nsg * p.pme_nt * p.p64_ncg * p.nsub * p.p64_split + 3) / 4;
  const dim3 g(static_cast<unsigned>(8 * ((n + 7) / 8)));
  if (p.stokes_t)
    hipLaunchKernelGGL((p64_adjoint<SHAPED, true>), g, dim3(256), 0, stream, p);
  else
    hipLaunchKernelGGL((p64_adjoint<SHAPED, false>), g, dim3(256), 0, stream, p);
}

hipError_t launch_p64_adjoint(const KParams &p, hipStream_t stream) {
  const int64_t npg = (p.one.npsrc + kWave - 1) / kWave;
  adjoint<false>(p, npg, stream);
  adjoint<true>(p, p.p64_nsg - npg, stream);
  return hipGetLastError();
}

// Sums of the partials of the pass just done; last: chi^2 too.
hipError_t launch_p64_partials(const KParams &p, bool last, hipStream_t stream) {
  const dim3 g((10 * kWave + 255) / 256, static_cast<unsigned>(p.p64_nsg + (last ? 1 : 0)),
               static_cast<unsigned>(p.pme_fchunk));
  hipLaunchKernelGGL(p64_fin_items, g, dim3(256), 0, stream, p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !p.grad_stokes_t) return e;
  hipLaunchKernelGGL(p64_stokes_t,
                     dim3(static_cast<unsigned>(p.pme_nt), static_cast<unsigned>(p.p64_nsg)),
                     dim3(256), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_p64_finalize(const KParams &p, hipStream_t stream) {
  const dim3 g((10 * kWave + 255) / 256, static_cast<unsigned>(p.p64_nsg));
  hipLaunchKernelGGL(p64_finalize, g, dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace rime
