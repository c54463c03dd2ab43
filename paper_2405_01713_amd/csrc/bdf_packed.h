// bdf_packed.h -- several cells per wave for mechanisms of at most 21 species.
//
// k_integrate gives a cell the whole wave, of which a small mechanism uses S of
// 64 lanes, and computes every per-cell scalar of the step control (t, h, xi_i,
// l_j, gamma, norms, eta) at wave width.  Here a wave integrates G cells, one
// per group of 64 / G lanes (lane i of a group owns species i): the vector work
// of one step, and the scalar work that is bound to it, is issued once for G
// cells.  The kernels are bound by VALU issue (77 to 85 % busy at 4 or 5 waves per
// SIMD), so that is where the time goes.  One cell per wave -> packed, ms (the
// same build, 5-wave budget): 9 species, 131,072 cells 69.6 -> 43.3; 3 species,
// 65,536 cells 13.3 -> 8.3; 16 species, 65,536 cells 44.5 -> 37.5; 21 species
// FP32, 262,144 cells 275 -> 257.  What is left is above all the setups (42 % of
// the instructions at 9 species), which run a cell at a time.
//
// Two things make the groups worth their divergence.  The loop runs over step
// *attempts*, not over cells: a group whose cell is finished writes it and takes
// its next cell while the others go on, so no group waits for the longest cell
// of its wave.  And a setup is not run under a group's exec mask: the wave
// visits the groups that need one and forms and inverts that cell's Newton
// matrix with all 64 lanes (newton_matrix and invert of one cell per wave), so
// its cost per cell is the one of k_integrate.
//
// Every operation of a cell is the one k_integrate does, in its order (the
// reductions leave out only additions of zero; the scattered sums are issued in
// slot order over 64 reactions at a time, as there), so the results are equal to
// the ones of one cell per wave bit for bit.
#pragma once

#include "bdf_device.h"

namespace bdfx {

// Lane groups of a wave, one cell each.
template <int G>
struct Pack {
  static_assert(G == 2 || G == 4, "two or four cells per wave");
  static constexpr int kLanes = kWave / G;
  int lane, grp;
  __device__ explicit Pack(int li) : lane(li % kLanes), grp(li / kLanes) {}
  // a lane index the optimizer cannot trace (see local_lane)
  __device__ int local() const {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  }

  // Sum over the group, in every lane of it: lane 15 of each 16-lane row (the
  // lane that Grp<1>::sum reads; the other lanes may hold other roundings of
  // the same sum, since a product in v can be fused into the first addition of
  // its own lane), and the two rows of a 32-lane group added.
  __device__ double sum(double v) const {
    v += dpp<kQuadXor1>(v);
    v += dpp<kQuadXor2>(v);
    v += dpp<kHalfMirror>(v);
    v += dpp<kMirror>(v);
    v = row_bcast<15>(v);
    if constexpr (kLanes == 32) {
      double a, b;
      rows(v, a, b);
      v = a + b;
    }
    return v;
  }
  // max of non-negative values
  __device__ double max(double v) const {
    v = fmax(v, dpp<kQuadXor1>(v));
    v = fmax(v, dpp<kQuadXor2>(v));
    v = fmax(v, dpp<kHalfMirror>(v));
    v = fmax(v, dpp<kMirror>(v));
    if constexpr (kLanes == 32) {
      double a, b;
      rows(v, a, b);
      v = fmax(a, b);
    }
    return v;
  }
  // the values of the group's two 16-lane rows (same lane of each)
  __device__ void rows(double v, double &a, double &b) const {
    const int2 p = __builtin_bit_cast(int2, v);
    const auto x = __builtin_amdgcn_permlane16_swap(p.x, p.x, false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(p.y, p.y, false, false);
    a = __builtin_bit_cast(double, make_int2(static_cast<int>(x[0]), static_cast<int>(y[0])));
    b = __builtin_bit_cast(double, make_int2(static_cast<int>(x[1]), static_cast<int>(y[1])));
  }
  __device__ bool any(bool pred) const {
    const uint64_t b = __ballot(pred);
    constexpr uint64_t m = (1ull << kLanes) - 1ull;
    return ((b >> (grp * kLanes)) & m) != 0ull;
  }
  // the value of lane K of the own 16-lane row
  template <int K>
  __device__ double row_bcast(double v) const {
    return dpp<0x150 + K>(v);
  }
  // the value of lane 0 of the group
  __device__ int from_lane0(int v) const {
    return __builtin_amdgcn_ds_bpermute((grp * kLanes) << 2, v);
  }
};

// LDS of one group (doubles): state for gathers (entry kLanes is the 1.0 that
// empty reaction slots read), right-hand-side accumulator, control block, pivot
// order, rate constants, inverse Newton matrix.
template <int G>
struct PackLds {
  static constexpr int L = Pack<G>::kLanes;
  static constexpr int kYb = 0, kFb = L + 8, kC = kFb + L, kPerm = kC + Ctl::kSize, kKk = kPerm + L / 2;
  __host__ __device__ static constexpr int fac(int R) { return kKk + 2 * R; }
  // an even number: 16-byte aligned areas
  __host__ __device__ static constexpr int size(int S, int R, int lt_bytes) {
    return (fac(R) + (S * S * lt_bytes + 7) / 8 + 1) / 2 * 2;
  }
};

// Block header (doubles), shared by all cells of the launch: per-order constants
// of the order selection, then the reaction slot words.
struct PackHead {
  static constexpr int kTab = 0;  // [3][8]: (q-1)!/H_{q-1}, 1/((q+2) H_{q+1}), hold bound, by q
  static constexpr int kRx = 24;
  __host__ __device__ static constexpr int size(int R) { return (kRx + R + 1) / 2 * 2; }
};

template <int G>
__device__ __forceinline__ Lds pack_carve(double *base, int R, const double *head) {
  using A = PackLds<G>;
  Lds L;
  L.yb = base + A::kYb;
  L.fb = base + A::kFb;
  L.C = base + A::kC;
  L.perm = reinterpret_cast<int *>(base + A::kPerm);
  L.kk = base + A::kKk;
  L.rx = reinterpret_cast<const int2 *>(head + PackHead::kRx);
  L.fac = base + A::fac(R);
  L.kry = nullptr;
  L.uT = L.uj = nullptr;
  return L;
}

// f_i of rhs() for the group's cell: 64 reactions at a time, 64 / G lanes per
// pass, all passes of a chunk scattered slot by slot, so that every sum takes
// its terms in the order of one cell per wave (LDS atomics of one instruction
// land in lane order).
template <bool ABC, int G>
__device__ __forceinline__ double pack_rhs(int R, const Lds &L, const Pack<G> &W, double yi, double Fi) {
  constexpr int NL = Pack<G>::kLanes;
  const int lane = W.local();
  wave_lds_sync();
  L.yb[lane] = yi;
  L.fb[lane] = Fi;
  wave_lds_sync();
  for (int c0 = 0; c0 < R; c0 += kWave) {
    int2 w[G];
    double q[G];
#pragma unroll
    for (int p = 0; p < G; ++p) {
      const int r = c0 + p * NL + lane;
      q[p] = 0.0;
      w[p] = make_int2(0, 0);
      if (r < R) {
        w[p] = L.rx[r];
        const double kf = L.kk[2 * r], krn = L.kk[2 * r + 1];
        if constexpr (ABC) {
#pragma clang fp contract(off)
          const double pf = kf * L.yb[slot_species(w[p].x, 0)] * L.yb[slot_species(w[p].x, 1)];
          const double pr = krn * L.yb[slot_species(w[p].y, 0)];
          q[p] = pf + pr;
        } else {
          double pf = kf, pr = krn;
#pragma unroll
          for (int s = 0; s < 3; ++s) {
            pf *= L.yb[slot_species(w[p].x, s)];
            pr *= L.yb[slot_species(w[p].y, s)];
          }
          q[p] = pf + pr;
        }
      }
    }
    if constexpr (ABC) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int p = 0; p < G; ++p) {
          if (c0 + p * NL + lane < R) {
            const int a = k == 0 ? slot_species(w[p].x, 0)
                                 : k == 1 ? slot_species(w[p].y, 0) : slot_species(w[p].x, 1);
            atomicAdd(&L.fb[a], k == 1 ? q[p] : -q[p]);
          }
          lanes_meet();
        }
    } else {
#pragma unroll
      for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int side = 0; side < 2; ++side)
#pragma unroll
          for (int p = 0; p < G; ++p) {
            const int a = slot_species(side ? w[p].y : w[p].x, s);
            if (c0 + p * NL + lane < R && a != NL) atomicAdd(&L.fb[a], side ? q[p] : -q[p]);
            lanes_meet();
          }
    }
  }
  wave_lds_sync();
  return L.fb[lane];
}

// x = M^{-1} b, as inv_solve (lane i passes b_i and gets x_i).
template <int S, typename LT, bool SPLIT, int G>
__device__ __forceinline__ double pack_solve(const Lds &L, const Pack<G> &W, double b) {
  const int lane = W.local();
  const LT *inv = reinterpret_cast<const LT *>(L.fac);
  LT *bb = reinterpret_cast<LT *>(L.yb);
  wave_lds_sync();
  if (lane < S) bb[lane] = static_cast<LT>(b);
  wave_lds_sync();
  const int lr = lane < S ? lane : 0;
  if constexpr (SPLIT) {
    LT acc0 = 0, acc1 = 0, acc2 = 0;
#pragma unroll
    for (int c = 0; c < S; c += 3) {
      acc0 = fma(inv[c * S + lr], bb[c], acc0);
      if (c + 1 < S) acc1 = fma(inv[(c + 1) * S + lr], bb[c + 1], acc1);
      if (c + 2 < S) acc2 = fma(inv[(c + 2) * S + lr], bb[c + 2], acc2);
    }
    return lane < S ? static_cast<double>((acc0 + acc1) + acc2) : 0.0;
  } else {
    LT acc = 0;
#pragma unroll
    for (int c = 0; c < S; ++c) acc = fma(inv[c * S + lr], bb[c], acc);
    return lane < S ? static_cast<double>(acc) : 0.0;
  }
}

// Cells of the launch, G per wave (see the top of the file).  Isothermal
// mechanisms, direct solver with the analytic Jacobian, no lock-step, no
// checkpoints; full step records are kept.  Grid: persistent waves whose groups
// take their cells from the work queue, under every scheduler (the library's
// static one has no order of cells to keep, and every (groups of the grid)-th cell
// for a group leaves the groups with the long cells behind: 9 species, 20,011
// cells 9.9 ms against 9.0).  Blocks of at most 256 threads.
template <int S, typename LT, int MINW, int G, bool ABC>
__global__ void __launch_bounds__(256, MINW) k_integrate_packed(Params P) {
  static_assert(S <= Pack<G>::kLanes, "a group holds one lane per species");
  extern __shared__ double smem[];
  const int wib = uni(static_cast<int>(threadIdx.x / kWave));
  const int li = threadIdx.x & (kWave - 1);
  const Pack<G> W(li);
  const Grp<1> W1(li);
  constexpr int NL = Pack<G>::kLanes;
  const MechDev &m = P.mech;
  const int R = m.R;
  double *const head = smem;
  double *const wave_base = smem + PackHead::size(R) + static_cast<int64_t>(wib) * G * P.lds_doubles;
  const Lds L = pack_carve<G>(wave_base + W.grp * P.lds_doubles, R, head);
  double *const C = L.C;

  // block header: slot words with empty slots renamed to entry kLanes of yb
  {
    int2 *rx = reinterpret_cast<int2 *>(head + PackHead::kRx);
    auto rename = [](int w) {
      int o = 0;
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        const int a = slot_species(w, s);
        o |= (a == kEmptySlot ? NL : a) << (8 * s);
      }
      return o;
    };
    for (int r = threadIdx.x; r < R; r += blockDim.x) {
      const int2 w = reinterpret_cast<const int2 *>(m.rx)[r];
      rx[r] = make_int2(rename(w.x), rename(w.y));
    }
    if (threadIdx.x >= 1 && threadIdx.x <= kQmax) {
      const int q = threadIdx.x;
      head[q] = factorial(q - 1) / (q > 1 ? harmonic(q - 1) : 1.0);
      head[8 + q] = rcp((q + 2) * harmonic(q + 1));
      head[16 + q] = hold_bound(q + 1);
    }
    if (W.lane == 0) L.yb[NL] = 1.0;
    __syncthreads();
  }

  const int n = P.n_sp;
  const double inv_n = 1.0 / n;
  const bool own = W.lane < n;
  auto norm2 = [&](double v, double w) {
    const double t = v * w;  // w = 0 on lanes without a species
    return W.sum(t * t) * inv_n;
  };
  const double rtol = P.rtol, t0 = P.t0, tout = P.tout;
  const int qmax = P.max_order < 1 ? 1 : (P.max_order > kQmax ? kQmax : P.max_order);
  const double atol_i = own ? (P.atol_len == 1 ? P.atol[0] : P.atol[W.lane]) : 1.0;
  const bool keep = P.rec != nullptr;

  // the group's share of the list
  int64_t next = 0, stop = 0;
  bool drained = false;

  bool live = false;  // the group has a cell
  int64_t cell = 0;
  int status = kSuccess;
  int nst = 0, nfe = 0, nni = 0, nsetups = 0, netf = 0, ncfn = 0;
  int q = 1, qwait = 2, nst_setup = 0;
  int nef_step = 0, ncf_step = 0, nsf_step = 0;
  bool top = false, write_y = true;
  bool need_setup = true, have_eprev = false, rebuilt = false;
  double t = t0, h = 0.0, R2 = 1.0;
  double z[kQmax + 1];
#pragma unroll
  for (int j = 0; j <= kQmax; ++j) z[j] = 0.0;
  double eprev = 0.0, ewt = 0.0, Fi = 0.0;

  for (;;) {
    // ---- groups without a cell take one -------------------------------------
    if (!live && !drained) {
      if (next >= stop) {
        unsigned int base = 0;
        if (W.lane == 0) base = atomicAdd(P.queue, static_cast<unsigned int>(P.chunk));
        next = static_cast<unsigned int>(W.from_lane0(static_cast<int>(base)));
        stop = next + P.chunk;
      }
      if (next >= P.n_list) {
        drained = true;
      } else {
        cell = P.list ? P.list[next] : next;
        ++next;
        live = true;
        // rate constants (Arrhenius, frozen T)
        const double T = P.T ? P.T[cell] : 1.0;
        wave_lds_sync();
        for (int r = W.lane; r < R; r += NL) {
          double lk = m.lnA[r];
          lk -= m.EaR[r] / T;
          double kf = exp(lk);
          if (P.kscale) kf *= P.kscale[cell * P.ldk + r];
          L.kk[2 * r] = kf;
          L.kk[2 * r + 1] = m.reversible ? -(kf * exp(-m.lnK[r])) : -0.0;
        }
        Fi = (own && P.F) ? P.F[cell * P.ldy + W.lane] : 0.0;
        status = kSuccess;
        nst = nfe = nni = nsetups = netf = ncfn = 0;
        q = 1;
        qwait = 2;
        nst_setup = 0;
        t = t0;
        h = 0.0;
        R2 = 1.0;
        need_setup = true;
        have_eprev = rebuilt = false;
        write_y = true;
        eprev = 0.0;
        ewt = 0.0;
#pragma unroll
        for (int j = 0; j <= kQmax; ++j) z[j] = 0.0;
        const double yin = own ? P.y[cell * P.ldy + W.lane] : 0.0;
        if (keep && own) P.rec_y0[cell * P.rec_stride + W.lane] = yin;
        double f = 0.0;
        if (W.any(!isfinite(T) || (own && !isfinite(yin)))) {
          status = kNonfinite;
          write_y = false;
        }
        // the initial step's right-hand sides: it = -1 is f(y0), then at most
        // four refinements (one right-hand-side body)
        double hlb = 0.0, hub = 0.0, hg = 0.0, hnew = 0.0;
        if (status == kSuccess) {
          bool at_ub = false, small = false;
          for (int it = -1; it < 4; ++it) {
            const double ft = pack_rhs<ABC, G>(R, L, W, it < 0 ? yin : yin + hg * f, Fi);
            nfe++;
            if (it < 0) {
              f = ft;
              if (W.any(own && !isfinite(f))) {
                status = kNonfinite;
                write_y = false;
                z[0] = yin;
                break;
              }
              z[0] = yin;
              ewt = own ? 1.0 / (rtol * fabs(yin) + atol_i) : 0.0;
              const double tdist = fabs(tout - t0);
              hlb = 100.0 * kUround * fmax(fabs(t0), fabs(tout));
              hub = 0.1 * tdist;
              const double hub_inv = W.max(own ? fabs(f) / (0.1 * fabs(yin) + atol_i) : 0.0);
              if (hub * hub_inv > 1.0) hub = 1.0 / hub_inv;
              if (hub < hlb) {
                small = true;
                break;
              }
              hg = sqrt(hlb * hub);
              hnew = hg;
              continue;
            }
            const double ydd = (ft - f) / hg;
            const double yddnrm = sqrt(norm2(ydd, ewt));
            if (!(yddnrm > 0.0)) {
              at_ub = true;
              break;
            }
            hnew = sqrt(2.0 / yddnrm);
            const double ratio = hnew / hg;
            hg = hnew;
            if (ratio >= 0.5 && ratio <= 2.0) break;
          }
          if (status == kSuccess) {
            if (small || at_ub) {
              h = hub;
            } else {
              h = 0.5 * hnew;
              if (h < hlb) h = hlb;
              if (h > hub) h = hub;
            }
            z[1] = h * f;
          }
        }
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k <= kQmax; ++k) C[Ctl::kHist + k] = h;
        C[Ctl::kEtaMax] = 1.0e4;
        C[Ctl::kHprev] = h;
        C[Ctl::kGammaBar] = 0.0;
        if (keep && W.lane == 0) P.rec_hpad[cell] = h;
        top = true;
      }
    }
    if (!wany(live || !drained)) break;

    // ---- one attempt: predictor, coefficients ----------------------------------
    double gamma = 0.0, gamma_bar = 0.0, rl1 = 0.0, Cerr = 0.5;
    bool go = live && status == kSuccess, want = false, fresh = false;
    if (go) {
      if (top) {
        if (!(t < tout)) {
          go = false;  // (a finished integration: nothing to do)
        } else if (nst >= P.max_steps) {
          status = kTooMuchWork;
          go = false;
        } else if (keep && nst >= P.rec_cap) {
          status = kRecordFull;
          go = false;
        } else {
          ewt = own ? rcp(rtol * fabs(z[0]) + atol_i) : 0.0;  // from y^{n-1}, Eq. (3)
          nef_step = ncf_step = nsf_step = 0;
          top = false;
        }
      }
      if (go) {
        bool landing = false;
        if (plain_sum(t, h) >= tout * (1.0 - 4.0 * kUround)) {
          const double hnew = tout - t;
          nd_rescale(z, hnew / h);
          h = hnew;
          landing = true;
        }
        if (h <= 4.0 * kUround * fabs(t)) {
          status = kErrFailure;
          go = false;
        } else {
          nd_predict(z);
          // xi_i = (t_n - t_{n-i}) / h and the coefficients of this attempt
          double xi[kQmax + 2], l[kQmax + 2];
          double sum = h;
          const double rh = rcp(h);
          xi[0] = 0.0;
          xi[1] = 1.0;
#pragma unroll
          for (int i = 2; i <= kQmax + 1; ++i) {
            sum = plain_sum(sum, C[Ctl::kHist + i - 2]);
            xi[i] = i <= q + 1 ? sum * rh : 0.0;
          }
          bdf_coeffs(q, xi, l, Cerr);
          wave_lds_sync();
#pragma unroll
          for (int i = 0; i <= kQmax + 1; ++i) {
            C[Ctl::kXi + i] = xi[i];
            C[Ctl::kL + i] = l[i];
          }
          C[Ctl::kTn] = landing ? tout : plain_sum(t, h);
          rl1 = rcp(l[1]);
          gamma = h * rl1;
          gamma_bar = C[Ctl::kGammaBar];
          want = need_setup || nst >= nst_setup + 20 || fabs(gamma * rcp(gamma_bar) - 1.0) > 0.3;
          if (want) L.yb[W.lane] = z[0];  // the setup's state
        }
      }
    }

    // ---- setups, one cell at a time with the whole wave ---------------------
    if (const uint64_t wm = __ballot(want)) {
      int info_g = 0;
      uint64_t mask = wm;
      while (mask) {
        const int l0 = uni(static_cast<int>(__builtin_ctzll(mask))) / NL * NL;  // lane 0 of the group
        mask &= ~(((1ull << NL) - 1ull) << l0);
        const Lds Lg = pack_carve<G>(wave_base + (l0 / NL) * P.lds_doubles, R, head);
        Mat<S, LT, 1> a;
        newton_matrix<S, LT, ABC, 0, NL>(a, m, Lg, W1, 0.0, lane_bcast(gamma, l0), false);
        const int info = invert<S, LT>(a, W1, Lg, n);
        if (li / NL * NL == l0) info_g = info;
      }
      if (want) {
        nsetups++;
        nst_setup = nst;
        gamma_bar = gamma;
        C[Ctl::kGammaBar] = gamma;
        R2 = 1.0;
        need_setup = false;
        fresh = true;
        if (info_g != 0) {
          // singular Newton matrix: recoverable once per step by cutting h
          nd_unpredict(z);
          need_setup = true;
          go = false;
          if (++nsf_step >= 2) {
            status = kSetupFailure;
          } else {
            nd_rescale(z, 0.25);
            h = h * 0.25;
            C[Ctl::kEtaMax] = 1.0;
          }
        }
      }
    }

    // ---- Newton iteration, error test, acceptance ------------------------------
    if (go) {
      const double cfac = gamma != gamma_bar ? 2.0 * rcp(1.0 + gamma * rcp(gamma_bar)) : 1.0;
      bool conv = false;
      double dprev2 = 0.0, en2 = 0.0;
      // stopping test of Eq. (4) with eps = 1/Cerr, on squared norms
      const double tol2 = 0.01 * rcp(Cerr * Cerr);
      double e = 0.0;
      for (int mit = 0; mit < 3; ++mit) {
        const double f = pack_rhs<ABC, G>(R, L, W, z[0] + e, Fi);
        nfe++;
        nni++;
        const double Gi = e - gamma * f + z[1] * rl1;
        double delta = pack_solve<S, LT, sizeof(LT) == 4, G>(L, W, -Gi);
        if (cfac != 1.0) delta *= cfac;
        e = plain_sum(e, delta);
        const double d2 = norm2(delta, ewt);
        if (!isfinite(d2)) break;
        if (mit >= 1) {
          const double ratio2 = d2 * rcp(dprev2);
          R2 = 0.09 * R2 > ratio2 ? 0.09 * R2 : ratio2;
        }
        if ((R2 < 1.0 ? R2 : 1.0) * d2 <= tol2) {
          conv = true;
          // the squared norm of e, which is delta after one iteration
          en2 = mit == 0 ? d2 : norm2(e, ewt);
          break;
        }
        if (mit >= 1 && d2 > 4.0 * dprev2) break;
        dprev2 = d2;
      }
      double dsm2 = 0.0;
      bool accept = false;
      if (!conv) {
        ncfn++;
        nd_unpredict(z);
        if (++ncf_step >= P.max_ncf) {
          status = kConvFailure;
        } else {
          if (fresh) {
            nd_rescale(z, 0.25);
            h = h * 0.25;
            C[Ctl::kEtaMax] = 1.0;
          }
          need_setup = true;
        }
      } else {
        // local error test (Sec. 2)
        dsm2 = Cerr * Cerr * en2;
        accept = dsm2 <= 1.0;
        if (!accept) {
          netf++;
          nd_unpredict(z);
          if (++nef_step >= P.max_netf) {
            status = kErrFailure;
          } else {
            C[Ctl::kEtaMax] = 1.0;
            if (nef_step >= 3) {
              // restart at order 1 from the last accepted y
              const double hnew = 0.1 * h;
              q = 1;
              const double f0 = pack_rhs<ABC, G>(R, L, W, z[0], Fi);
              nfe++;
#pragma unroll
              for (int j = 2; j <= kQmax; ++j) z[j] = 0.0;
              z[1] = hnew * f0;
              h = hnew;
              qwait = 2;
              have_eprev = false;
              rebuilt = true;
            } else {
              double eta = eta_from2(6.0, dsm2, q + 1);
              if (eta < 0.1) eta = 0.1;
              if (nef_step >= 2 && eta > 0.2) eta = 0.2;
              nd_rescale(z, eta);
              h = h * eta;
            }
          }
        }
      }
      if (accept) {
        // correct the Nordsieck array (l_j = 0 for j > q)
        t = C[Ctl::kTn];
#pragma unroll
        for (int j = 0; j <= kQmax; ++j) z[j] = fma(C[Ctl::kL + j], e, z[j]);
        nst++;
        wave_lds_sync();
#pragma unroll
        for (int k = kQmax; k >= 1; --k) C[Ctl::kHist + k] = C[Ctl::kHist + k - 1];
        C[Ctl::kHist] = h;
        if (keep) {
          double *rp = P.rec + (static_cast<int64_t>(cell) * P.rec_cap + (nst - 1)) * P.rec_stride;
          if (own) rp[W.lane] = z[0];
          if (W.lane == 0) {
            rp[n] = h;
            rp[n + 1] = static_cast<double>(q + (rebuilt ? 256 : 0));
          }
        }
        rebuilt = false;
        top = true;
        const double hstep = h;
        qwait--;
        if (qwait == 1 && q < qmax) {
          eprev = e;
          C[Ctl::kHprev] = hstep;
          have_eprev = true;
        }
        const double eta_max = C[Ctl::kEtaMax];
        if (t < tout) {
          if (eta_max == 1.0) {
            if (qwait < 2) qwait = 2;  // right after a failure: hold h and q
          } else {
            // without an order decision this step, h changes only if eta >= 1.5
            double eta = 0.0;
            int qnew = q;
            const bool decide = qwait == 0;
            bool lower = false, higher = false;
            double lte2m = 0.0, lte2p = 0.0;
            if (decide) {
              qwait = 2;
              lower = q > 1;
              higher = q < qmax && have_eprev;
              if (lower) {
                const double lte = head[q];
                lte2m = lte * lte * norm2(nd_get(z, q), ewt);
              }
              if (higher) {
                const double r = ipow(hstep / C[Ctl::kHprev], q + 1);
                const double c = head[8 + q];
                lte2p = c * c * norm2(e - r * eprev, ewt);
              }
            }
            if (decide || 36.0 * dsm2 <= head[16 + q]) {
              // the candidates' roots in one evaluation: lane 0 of each 16-lane
              // row takes order q, lane 1 order q - 1, lane 2 order q + 1
              const int gl = W.lane & 15;
              const double et = eta_from2(gl == 2 ? 10.0 : 6.0,
                                          gl == 0 ? dsm2 : gl == 1 ? lte2m : lte2p,
                                          gl == 0 ? q + 1 : gl == 1 ? q : q + 2);
              eta = W.template row_bcast<0>(et);
              if (lower) {
                const double eta_qm1 = W.template row_bcast<1>(et);
                if (eta_qm1 > eta) {
                  eta = eta_qm1;
                  qnew = q - 1;
                }
              }
              if (higher) {
                const double eta_qp1 = W.template row_bcast<2>(et);
                if (eta_qp1 > eta) {
                  eta = eta_qp1;
                  qnew = q + 1;
                }
              }
            }
            if (eta >= 1.5) {
              if (eta > eta_max) eta = eta_max;
              if (qnew == q + 1) {
                // add (e / xi_{q+1}) x Lambda(x): keeps interpolation, raises the degree
                const double c = 1.0 / C[Ctl::kXi + q + 1];
#pragma unroll
                for (int j = 1; j <= kQmax; ++j) {
                  if (j == q + 1) z[j] = 0.0;
                  if (j <= q + 1) z[j] += c * C[Ctl::kL + j - 1] * e;
                }
              } else if (qnew == q - 1) {
                // subtract z_q x prod_{i<q} (x + xi_i)
                double c[kQmax + 2];
#pragma unroll
                for (int j = 0; j <= kQmax + 1; ++j) c[j] = 0.0;
                c[1] = 1.0;
#pragma unroll
                for (int i = 1; i <= kQmax - 1; ++i)
                  if (i <= q - 1) {
                    const double xi_i = C[Ctl::kXi + i];
#pragma unroll
                    for (int j = i + 1; j >= 1; --j) c[j] = c[j - 1] + xi_i * c[j];
                  }
                const double zq = nd_get(z, q);
#pragma unroll
                for (int j = 1; j <= kQmax; ++j) {
                  if (j < q) z[j] -= c[j] * zq;
                  if (j == q) z[j] = 0.0;
                }
              }
              if (qnew != q) {
                q = qnew;
                qwait = q + 1;
                have_eprev = false;
              }
              nd_rescale(z, eta);
              h = h * eta;
            }
          }
        }
        C[Ctl::kEtaMax] = 10.0;
      }
    }

    // ---- finished cells -----------------------------------------------------
    if (live && (status != kSuccess || (top && !(t < tout)))) {
      if (write_y && own) P.y[cell * P.ldy + W.lane] = z[0];
      if (W.lane == 0) {
        P.status[cell] = status;
        if (P.stats) {
          CellStats st;
          st.status = status;
          st.nst = nst;
          st.nfe = nfe;
          st.nni = nni;
          st.nsetups = nsetups;
          st.netf = netf;
          st.ncfn = ncfn;
          st.q_last = q;
          st.nli = 0;
          st.ncfl = 0;
          st.h_last = h;
          st.t_reached = t;
          P.stats[cell] = st;
        }
        if (keep) P.rec_n[cell] = nst < P.rec_cap ? nst : P.rec_cap;
      }
      live = false;
    }
  }
}

// Cells per wave of the packed kernel for a padded size (1: none is built).  At
// 32 species a cell's area is 10 KiB, so that two cells a wave leave fewer cells
// on a CU than one (16,384 cells of 30 species: 46.8 ms against 36.6).
__host__ __device__ constexpr int packed_cells(int S) { return S <= 16 ? 4 : S <= 21 ? 2 : 1; }

// Waves per SIMD the packed kernel's registers must allow.  (Up to 16 species five
// spilled 120 bytes per lane for no gain below 100,000 cells.)
constexpr int kPackedWaves = 4;

// nullptr: not built (17 to 21 species with the FP64 matrix, where one cell per
// wave is as fast, see packed_min_cells_per_cu)
template <int S>
const void *packed_kernel(bool fp32, bool abc) {
  constexpr int G = packed_cells(S), W = kPackedWaves;
  if (fp32)
    return abc ? (const void *)&k_integrate_packed<S, float, W, G, true>
               : (const void *)&k_integrate_packed<S, float, W, G, false>;
  if constexpr (S <= 16)
    return abc ? (const void *)&k_integrate_packed<S, double, W, G, true>
               : (const void *)&k_integrate_packed<S, double, W, G, false>;
  return nullptr;
}

}  // namespace bdfx

#define BDFX_DECLARE_PACKED(S)                                                                   \
  hipError_t bdfx_launch_packed_s##S(const bdfx::Params &P, bool fp32, bool abc,                 \
                                     const bdfx::LaunchCfg &c, hipStream_t s);                   \
  hipError_t bdfx_occupancy_packed_s##S(bool fp32, bool abc, int block, size_t lds, int *out);

#define BDFX_DEFINE_PACKED(S)                                                                    \
  hipError_t bdfx_launch_packed_s##S(const bdfx::Params &P, bool fp32, bool abc,                 \
                                     const bdfx::LaunchCfg &c, hipStream_t s) {                  \
    const void *f = bdfx::packed_kernel<S>(fp32, abc);                                           \
    if (!f) return hipErrorInvalidDeviceFunction;                                                \
    bdfx::Params arg = P;                                                                        \
    void *args[] = {&arg};                                                                       \
    return hipLaunchKernel(f, dim3(c.grid), dim3(c.block), args, c.lds_bytes, s);                \
  }                                                                                              \
  hipError_t bdfx_occupancy_packed_s##S(bool fp32, bool abc, int block, size_t lds, int *out) {  \
    const void *f = bdfx::packed_kernel<S>(fp32, abc);                                           \
    *out = 0;                                                                                    \
    return f ? hipOccupancyMaxActiveBlocksPerMultiprocessor(out, f, block, lds) : hipSuccess;    \
  }
