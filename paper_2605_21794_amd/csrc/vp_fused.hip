// The fused step kernel (k_fused) of the decorated-particle cycle, with its launch for one
// precision mode.  This unit is compiled once per mode (VP_FUSED_MODE = 0..3, the vpk::Mode
// values), so the modes' kernel instances build side by side.
#include "vp_device.h"

#ifndef VP_FUSED_MODE
#error "compile with -DVP_FUSED_MODE=<mode>"
#endif

namespace vpk {

// Wavefronts per SIMD the registers must leave room for: at six, the float32 state with float64
// sums and P1 elements keeps three workgroups of 512 threads on a CU (two at 82 registers).
template <int MODE, int TPB, bool GEN, bool P2>
constexpr int fused_waves() {
  return TPB <= 512 && MODE == kFP32Comp && !GEN && !P2 ? 6 : 1;
}

// DIP = false: every tile of the launch belongs to a monopole-only instance; p* and q* are
// neither read nor written (20 bytes of particle traffic per update instead of 36).
// GEN = false: no instance of the launch has general options (d.general) or the FFT solver, so
// the field on a particle is read straight from the mesh arrays.  P2 = true: the launch's instances have P2
// elements (separate instances keep the others' registers as they were).
// STREAM = false: plain accesses to the particle arrays.  (As a template parameter: chosen by a
// branch around the loads, the step of 2^20 float64 particles took 15.2 us instead of 14.1.)
template <int MODE, int TPB, bool DIP, bool GEN, bool P2, bool KM = false, bool STREAM = true>
__global__ __launch_bounds__(TPB, (fused_waves<MODE, TPB, GEN, P2>())) void k_fused(
                                               const InstDev* __restrict__ insts,
                                               const Tile* __restrict__ tiles, int tile0,
                                               int ppt_max, int phase) {
  extern __shared__ double smem[];
  __shared__ double red[4 * (TPB / 64)];
  __shared__ double sred[kSolveRed];
  using T = typename StateType<MODE>::T;
  constexpr int kGroup = group_of<MODE, TPB, KM>();
  const Tile tl = tiles[tile0 + blockIdx.x];
  const int ppt = min(ppt_max, (tl.count + TPB - 1) / TPB);  // tiles may be smaller
  const InstDev& d = insts[tl.inst];
  const int ng = d.ng;
  const int r0 = phase, r1 = ring_next(phase), r2 = ring_prev(phase);
  VPG T* __restrict__ Qp = gp<T>(d.Q);
  VPG T* __restrict__ Pp = gp<T>(d.P);
  VPG T* __restrict__ qsp = gp<T>(d.qs);
  VPG T* __restrict__ psp = gp<T>(d.ps);
  const VPG T* __restrict__ psip = gp<T>(d.psi);
  const int nacc = P2 ? d.nacc : ng;  // load-vector nodes (2 ng for P2)
  double* fE = smem;
  double* fG = smem + ng;
  double* sacc = smem + 2 * ng;
  double* bt = sacc + nacc;
  double* fft = bt + ng;
  VPG InstScal* sc = gp(d.scal);
  // An instance whose diagnostics went NaN / Inf is frozen: its state is no longer a
  // solution, and its particles would all land in element 0.  (Uniform per workgroup.)  The
  // flag is tested once the first loads are out, so its latency overlaps theirs.
  const int frozen = sc->nonfinite;
  const bool first = tl.local == 0;  // the instance's bookkeeping tile (uniform per workgroup)

  // one group of particles per thread: thread t takes tile.begin + k * TPB + t, k0 <= k < k0 + kGroup
  // KM: a launch of k = 3 instances (particles with second moments; P2, never kFP32), whose
  // moments travel with the group
  constexpr int kMG = KM ? kGroup : 1;
  struct Group {
    T q[kGroup], p[kGroup], a[kGroup], b[kGroup], w[kGroup];
    T m[3][kMG];
    long long idx[kGroup];
    bool v[kGroup];
  };
  VPG T* __restrict__ Mqp_ = gp<T>(d.Mqq);
  VPG T* __restrict__ Mqpp = gp<T>(d.Mqp);
  VPG T* __restrict__ Mppp = gp<T>(d.Mpp);
  const T zq = pad_position<T>(d);
  auto load_group = [&](int k0, Group& g) {
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      const int loc = (k0 + u) * TPB + (int)threadIdx.x;
      g.v[u] = (k0 + u < ppt) && (loc < tl.count);
      g.idx[u] = tl.begin + loc;
      // every lane loads (a lane past the end of the tile reads the tile's last particle, so
      // no load is under a branch); such a lane then holds an all-zero particle (run_group),
      // away from its neighbours' (pad_position)
      const long long li = tl.begin + (g.v[u] ? loc : tl.count - 1);
      const T z = T(0);
      const T lq = ntld<STREAM>(Qp + li), lp = ntld<STREAM>(Pp + li), lw = ntld<STREAM>(psip + li);
      g.q[u] = g.v[u] ? lq : zq;
      g.p[u] = g.v[u] ? lp : z;
      g.w[u] = g.v[u] ? lw : z;
      g.a[u] = g.b[u] = z;
      if constexpr (DIP) {
        const T la = ntld<STREAM>(qsp + li), lb = ntld<STREAM>(psp + li);
        g.a[u] = g.v[u] ? la : z;
        g.b[u] = g.v[u] ? lb : z;
      }
      if constexpr (KM) {
        const T l0 = ntld<STREAM>(Mqp_ + li), l1 = ntld<STREAM>(Mqpp + li), l2 = ntld<STREAM>(Mppp + li);
        g.m[0][u] = g.v[u] ? l0 : z;
        g.m[1][u] = g.v[u] ? l1 : z;
        g.m[2][u] = g.v[u] ? l2 : z;
      }
    }
  };

  // The solve's loads go out first and the first group's particle loads right behind them:
  // both latencies overlap, and the solve can start once its own loads are back (the loads
  // return in order) while the particle loads are still in flight.
  SolveIn sin_;
  solve_load<MODE, false, GEN, P2>(d, r0, first, sin_);
  Group g;
  load_group(0, g);
  if (frozen) return;
  for (int j = threadIdx.x; j < nacc; j += TPB) sacc[j] = 0.0;
  const int pend = sc->pend[r0];
  // the first tile records the previous step (if it was a fused step of this instance):
  // its inputs are read now and written after the solve
  long long step = 0;
  double rec[3] = {0.0, 0.0, 0.0};
  if (first) {
    step = sc->step;
    rec[0] = sc->W[r2];
    rec[1] = sc->e1r[r2];
    rec[2] = sc->e1i[r2];
  }
  double Ks = 0.0, Ms = 0.0, Cs = 0.0, Us = 0.0;
  {
    double sum[7];
    solve_compute<TPB, GEN, P2>(d, sin_, first, bt, fE, fG, sred, fft, nullptr, sum);
    if (first) {
      const int copies = d.acc_copies;
      for (int c = 0; c < copies; ++c)
        for (int j = threadIdx.x; j < nacc; j += TPB) {
          if constexpr (MODE == kFP32)
            gp<float>(d.acc)[acc_off(d, r2, c) + j] = 0.0f;
          else
            gp(d.acc)[acc_off(d, r2, c) + j] = 0.0;
        }
      if (threadIdx.x == 0) {
        if (pend && step >= 1)
          write_record(d, step - 1, sum[3], sum[4], sum[5], sum[6], rec[0], rec[1], rec[2]);
        sc->W[r0] = sum[0];
        sc->e1r[r0] = sum[1];
        sc->e1i[r0] = sum[2];
        if (!isfinite(sum[0])) sc->nonfinite = 1;
        sc->pend[r1] = 1;
        sc->step = step + 1;
      }
    }
  }

  // Every lane pushes all its particles without a branch: a weightless particle (a lane past
  // the end of the tile) deposits +0 and adds 0 to the kinetic sums, so the particles'
  // dependency chains interleave; only the stores test the lane.
  auto run_group = [&](Group& g) {
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      T Q = g.q[u], P = g.p[u], qs = g.a[u], ps = g.b[u];
      if constexpr (KM) {
        T Mv[3] = {g.m[0][u], g.m[1][u], g.m[2][u]};
        push_particle<MODE, T, DIP, GEN, P2, -1, false, true>(d, fE, fG, sacc, pend, Q, P, qs, ps,
                                                              g.w[u], Ks, Ms, Cs, Us, Mv);
        g.m[0][u] = Mv[0]; g.m[1][u] = Mv[1]; g.m[2][u] = Mv[2];
      } else {
        push_particle<MODE, T, DIP, GEN, P2>(d, fE, fG, sacc, pend, Q, P, qs, ps, g.w[u], Ks,
                                             Ms, Cs, Us);
      }
      g.q[u] = Q; g.p[u] = P; g.a[u] = qs; g.b[u] = ps;
    }
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      if (!g.v[u]) continue;
      ntst<STREAM>(Qp + g.idx[u], g.q[u]); ntst<STREAM>(Pp + g.idx[u], g.p[u]);
      if constexpr (DIP) { ntst<STREAM>(qsp + g.idx[u], g.a[u]); ntst<STREAM>(psp + g.idx[u], g.b[u]); }
      if constexpr (KM) {
        ntst<STREAM>(Mqp_ + g.idx[u], g.m[0][u]); ntst<STREAM>(Mqpp + g.idx[u], g.m[1][u]);
        ntst<STREAM>(Mppp + g.idx[u], g.m[2][u]);
      }
    }
  };

  run_group(g);
  for (int k0 = kGroup; k0 < ppt; k0 += kGroup) {
    load_group(k0, g);
    run_group(g);
  }

  // kinetic sums: one tree per wavefront for all of them, one barrier, one thread per sum
  // stores the workgroup total in this tile's slot while the flush is under way (the next
  // pass's first tile adds the slots in tile order)
  constexpr int kSums = GEN ? kKinFields : 3;  // U stays zero (no potential in this instance)
  double sums[kSums] = {Ks, Ms, Cs};
  if constexpr (GEN) sums[3] = Us;
  wave_totals_to(sums, red + kSums * (threadIdx.x >> 6), 1);
  __syncthreads();  // also completes every LDS deposit of the workgroup
  flush<MODE, TPB>(d, sacc, r1, tl.local % d.acc_copies);
  if (threadIdx.x < kSums) {
    double t = 0.0;
    for (int w = 0; w < TPB / 64; ++w) t += red[kSums * w + threadIdx.x];
    gp(d.kin)[((size_t)r0 * d.kin_cap + tl.local) * kKinFields + threadIdx.x] = t;
  }
}



template <int MODE>
hipError_t launch_fused_mode(int tpb, const InstDev* d_inst, const Tile* d_tiles, int tile0,
                        int ntiles, int ppt, int max_ng, bool lds_fft, int phase, bool dipoles,
                        bool general, bool p2, bool moments, bool stream, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  if (moments && (MODE == kFP32 || !dipoles || !p2)) return hipErrorInvalidValue;
  const size_t lds = fused_lds_bytes(lds_fft, max_ng);
#define VP_FUSED_K(M, TB, ...)                                                               \
  hipLaunchKernelGGL((k_fused<M, TB, __VA_ARGS__>), dim3(ntiles), dim3(TB), lds, s, d_inst,  \
                     d_tiles, tile0, ppt, phase)
// plain accesses: the default 512 threads, without general options
#define VP_FUSED_S(M, TB, D, P, KM)                                                          \
  do {                                                                                       \
    if constexpr (TB == 512) {                                                               \
      if (!stream) {                                                                         \
        VP_FUSED_K(M, TB, D, false, P, KM, false);                                           \
        break;                                                                               \
      }                                                                                      \
    }                                                                                        \
    VP_FUSED_K(M, TB, D, false, P, KM);                                                      \
  } while (0)
#define VP_FUSED(M, TB)                                                                      \
  do {                                                                                       \
    if constexpr (M != kFP32) {                                                              \
      if (moments) {                                                                         \
        if (general) VP_FUSED_K(M, TB, true, true, true, true);                              \
        else VP_FUSED_S(M, TB, true, true, true);                                            \
        break;                                                                               \
      }                                                                                      \
    }                                                                                        \
    if (dipoles) {                                                                           \
      if (p2) {                                                                              \
        if (general) VP_FUSED_K(M, TB, true, true, true);                                    \
        else VP_FUSED_S(M, TB, true, true, false);                                           \
      } else {                                                                               \
        if (general) VP_FUSED_K(M, TB, true, true, false);                                   \
        else VP_FUSED_S(M, TB, true, false, false);                                          \
      }                                                                                      \
    } else {                                                                                 \
      if (p2) {                                                                              \
        if (general) VP_FUSED_K(M, TB, false, true, true);                                   \
        else VP_FUSED_S(M, TB, false, true, false);                                          \
      } else {                                                                               \
        if (general) VP_FUSED_K(M, TB, false, true, false);                                  \
        else VP_FUSED_S(M, TB, false, false, false);                                         \
      }                                                                                      \
    }                                                                                        \
  } while (0)
#define VP_FUSED_TPB(M)                                                                      \
  do {                                                                                       \
    if (tpb == 1024) VP_FUSED(M, 1024);                                                      \
    else if (tpb == 512) VP_FUSED(M, 512);                                                   \
    else VP_FUSED(M, 256);                                                                   \
  } while (0)
  VP_FUSED_TPB(MODE);
#undef VP_FUSED_TPB
#undef VP_FUSED
#undef VP_FUSED_S
#undef VP_FUSED_K
  return hipGetLastError();
}

template hipError_t launch_fused_mode<VP_FUSED_MODE>(int tpb, const InstDev* d_inst,
                                                     const Tile* d_tiles, int tile0, int ntiles,
                                                     int ppt, int max_ng, bool lds_fft, int phase,
                                                     bool dipoles, bool general, bool p2,
                                                     bool moments, bool stream, hipStream_t s);

}  // namespace vpk
