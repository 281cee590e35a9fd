// Many steps of small instances in one launch (k_resident): an instance that fits one workgroup
// needs no other's results, so its particles stay in registers and its load vector in LDS.
#include "vp_device.h"

namespace vpk {

// Value of node j of the LDS deposit grid, as the flush would add it to a cleared accumulator.
template <int MODE>
__device__ __forceinline__ double grid_value(const double* sacc, int j) {
  if constexpr (MODE == kFP32) {
    return (double)reinterpret_cast<const float*>(sacc)[j];
  } else if constexpr (MODE == kFP32TwoSum) {
    const unsigned long long w = reinterpret_cast<const unsigned long long*>(sacc)[j];
    return (double)__uint_as_float((unsigned)(w & 0xffffffffull)) +
           (double)__uint_as_float((unsigned)(w >> 32));
  } else {
    return sacc[j];
  }
}

// nsteps steps of the instances `slots`, one workgroup each (n <= 1024 PPT).  The steps, their
// order and their arithmetic are those of k_fused on one tile; at the end the ring entry of the
// next phase, the per-tile sums and the scalars are left as a fused pass leaves them, so the two
// can follow one another.  The record of a step is written in that step (its field summary and
// kinetic sums are both here), by the last wavefront while the others go on to the next solve.
// An instance that turns non-finite stops where the fused steps would have frozen it: before the
// next pass when W (or E) did, after it when K or U did, which is then flagged (in the last pass
// it is left to whoever takes the owed record).  W is known after its pass only; waiting for it
// in every pass took 0.12 to 0.2 us a step, so a pass whose field is near overflow waits, others
// do not.
// GEN, P2: as for k_persist.
//
// Bound by the push's float64 issue (4096 particles on one CU) and the solve's barriers, with no
// launch, flush or accumulator load in the step.  4096 float64 particles, Ng 64: 3.7 us a step
// (4.2 before a wavefront's sums shared one tree, wave_totals), against 9.4 us with one launch
// per step of one tile, 7.5 us in tiles of 512 x 4.  Up to 1024 particles a step takes 2.25 us,
// the solve's and the sums' chain for the most part; each 1024 more add 0.47.
template <int MODE, int PPT, bool GEN, bool P2>
__global__ __launch_bounds__(kResidentThreads) void k_resident(
    const InstDev* __restrict__ insts, const int* __restrict__ slots, int phase0, int nsteps) {
  constexpr int TPB = kResidentThreads, kWaves = TPB / 64;
  constexpr int kSums = 7;  // K, momentum, charge, U, W, Re E1, Im E1
  extern __shared__ double smem[];
  __shared__ double red[kSums * kWaves];
  __shared__ double sred[kSolveRed];
  // of the last pass: nonfinite: 1 its kinetic sums came out NaN or Inf, 2 its W; huge: 4 its field
  // was near overflow
  __shared__ int nonfinite, huge;
  using T = typename StateType<MODE>::T;
  const InstDev& d = insts[slots[blockIdx.x]];
  const int ng = d.ng, n = (int)d.n, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int nacc = P2 ? d.nacc : ng;
  double* fE = smem;
  double* fG = smem + ng;
  double* sacc = smem + 2 * ng;
  double* bt = sacc + nacc;
  double* fft = bt + ng;
  VPG InstScal* sc = gp(d.scal);
  if (sc->nonfinite) return;  // frozen (uniform)

  // A lane past the end holds a weightless particle (pad_position).
  T q[PPT], p[PPT], a[PPT], b[PPT], w[PPT];
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int i = u * TPB + tid;
    p[u] = a[u] = b[u] = w[u] = T(0);
    q[u] = pad_position<T>(d);
    if (i < n) {
      q[u] = gp<T>(d.Q)[i]; p[u] = gp<T>(d.P)[i]; a[u] = gp<T>(d.qs)[i];
      b[u] = gp<T>(d.ps)[i]; w[u] = gp<T>(d.psi)[i];
    }
  }
  constexpr bool kCell = !GEN && !P2 && MODE != kFP32;
  int cell[PPT];
#pragma unroll
  for (int u = 0; u < PPT; ++u) cell[u] = kCell ? cell_of((double)q[u] * d.inv_h, ng) : 0;
  // Fourier weights of node tid (ng <= 1024 threads)
  double c1 = 0.0, s1 = 0.0;
  if (tid < ng) {
    const int half = ng >> 1, t = tid & (half - 1);
    const double sg = tid < half ? 1.0 : -1.0;  // cos / sin of theta + pi
    c1 = sg * gp(d.tw)[2 * t];
    s1 = sg * gp(d.tw)[2 * t + 1];
  }
  const long long step0 = sc->step;
  int pend = sc->pend[phase0];
  if (tid == 0) nonfinite = huge = 0;
  __syncthreads();
  if (tid == TPB - 64 && pend && step0 >= 1) {  // the record the previous pass still owes
    const int r2 = ring_prev(phase0);
    double s[kKinFields] = {0.0, 0.0, 0.0, 0.0};
    const VPG double* kin = gp(d.kin) + (size_t)r2 * d.kin_cap * kKinFields;
    for (int t = 0; t < d.ntiles; ++t)
      for (int f = 0; f < kKinFields; ++f) s[f] += kin[t * kKinFields + f];
    write_record(d, step0 - 1, s[0], s[1], s[2], s[3], sc->W[r2], sc->e1r[r2], sc->e1i[r2]);
    if (!isfinite(s[0]) || !isfinite(s[3])) nonfinite = 1;
  }

  const int per = solve_per(ng), j0 = tid * per;
  const bool owner = tid < kSolveThreads && j0 < ng;  // of nodes j0 .. j0 + per - 1
  double tot = 0.0;  // last wavefront, lane f: sum f of the last pass
  int done = 0;
  int stop = 0;
  for (;;) {
    while (done < nsteps && !stop) {
      // nothing is hoisted out of the step loop: keeps the step's registers per step
      __asm__ __volatile__("" ::: "memory");
      SolveIn in;
      if (done == 0) {
        solve_load<MODE, false, GEN, P2>(d, phase0, false, in);
        for (int j = tid; j < nacc; j += TPB) sacc[j] = 0.0;
      } else {
#pragma unroll
        for (int k = 0; k < kSolvePer; ++k) {
          in.b[k] = in.bm[k] = 0.0;
          if (owner && k < per) {
            in.b[k] = grid_value<MODE>(sacc, j0 + k);
            if (P2 && d.order == 2) in.bm[k] = grid_value<MODE>(sacc, ng + j0 + k);
          }
        }
        if constexpr (MODE == kFP32) __syncthreads();  // floats: nodes share a 64-bit word
        if (owner)
#pragma unroll
          for (int k = 0; k < kSolvePer; ++k)
            if (k < per) {
              sacc[j0 + k] = 0.0;
              if (P2 && d.order == 2) sacc[ng + j0 + k] = 0.0;
            }
      }
      double unused[7];
      solve_compute<TPB, GEN, P2>(d, in, false, bt, fE, fG, sred, fft, nullptr, unused,
                                  nullptr, &huge);
      // a non-finite load makes every E NaN through its mean
      stop = (isfinite(fE[0]) ? 0 : 1) | nonfinite | huge;
      double v[kSums] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      if (tid < ng) {
        const double Ee = fE[tid];
        v[4] = Ee * Ee;
        v[5] = Ee * c1;
        v[6] = -(Ee * s1);
        if (P2 && d.order == 2) {  // the midpoint load's part (see solve_compute): h g = -3 b~_m / 2
          const double hg = d.h * fG[tid];
          v[4] += 0.1875 * (4.0 / 9.0) * (hg * hg);
        }
      }
#pragma unroll
      for (int u = 0; u < PPT; ++u)
        push_particle<MODE, T, true, GEN, P2, -1, kCell>(d, fE, fG, sacc, pend, q[u], p[u], a[u],
                                                         b[u], w[u], v[0], v[1], v[2], v[3],
                                                         nullptr, &cell[u]);
      pend = 1;
      wave_totals_to(v, red + wid, kWaves);
      __syncthreads();  // also completes every LDS deposit
      if (wid == kWaves - 1) {
        tot = 0.0;
        if (lane < kSums)
          for (int x = 0; x < kWaves; ++x) tot += red[lane * kWaves + x];
        if (lane == 4) tot = 0.5 * d.h * tot;
        if (lane == 5 || lane == 6) tot = tot * inv_pow2(d.log2ng);
        const double K = __shfl(tot, 0), mom = __shfl(tot, 1), chg = __shfl(tot, 2);
        const double U = __shfl(tot, 3), W = __shfl(tot, 4), er = __shfl(tot, 5), ei = __shfl(tot, 6);
        if (lane == 0) {
          store_record_at(d, (int)((step0 + done) % d.hist_cap), step0 + done, K, mom, chg,
                          GEN ? U : 0.0, W, er, ei);
          nonfinite = (!isfinite(K) || (GEN && !isfinite(U)) ? 1 : 0) | (!isfinite(W) ? 2 : 0);
        }
      }
      ++done;
    }
    if (stop != 4 || done == nsteps) break;
    __syncthreads();  // the last wavefront's verdict on the pass near overflow
    if (nonfinite & 2) break;
    if (tid == 0) huge = 0;
    stop = 0;
  }

  const int rf = (phase0 + done) % kRing, rl = ring_prev(rf);  // next phase, last pass's
  const int copies = d.acc_copies;
  for (int c = 0; c < copies; ++c)
    for (int j = tid; j < nacc; j += TPB) {
      const double x = c == 0 ? grid_value<MODE>(sacc, j) : 0.0;
      if constexpr (MODE == kFP32) {
        gp<float>(d.acc)[acc_off(d, rf, c) + j] = (float)x;
        gp<float>(d.acc)[acc_off(d, ring_next(rf), c) + j] = 0.0f;
      } else {
        gp(d.acc)[acc_off(d, rf, c) + j] = x;
        gp(d.acc)[acc_off(d, ring_next(rf), c) + j] = 0.0;
      }
    }
  __syncthreads();  // the last wavefront's verdict
  if ((stop & 3) || (nonfinite & 2)) {
    // Frozen, while the engine's phase goes on: a read-back may come at the entry that the last
    // pass solved, so its load is put back there (from b~, and for P2 from g: see solve_compute).
    const double mean = solve_total(sred, 0) * inv_pow2(d.log2ng);
    for (int c = 0; c < copies; ++c)
      for (int j = tid; j < nacc; j += TPB) {
        double x = 0.0;
        if (c == 0) {
          auto mid = [&](int e) { return (2.0 / 3.0) * mean - fG[e & (ng - 1)] / (1.5 * d.inv_h); };
          if (!(P2 && d.order == 2)) x = bt[j] + mean;
          else x = j >= ng ? mid(j) : (bt[j] + mean) - 0.5 * (mid(j - 1) + mid(j));
        }
        if constexpr (MODE == kFP32) gp<float>(d.acc)[acc_off(d, rl, c) + j] = (float)x;
        else gp(d.acc)[acc_off(d, rl, c) + j] = x;
      }
  }
  if (wid == kWaves - 1) {
    VPG double* kin = gp(d.kin) + (size_t)rl * d.kin_cap * kKinFields;
    for (int t = lane; t < d.ntiles * kKinFields; t += 64)
      if (t >= kKinFields) kin[t] = 0.0;
    if (lane < kKinFields) kin[lane] = lane < 3 || GEN ? tot : 0.0;
    if (lane == 4) {
      sc->W[rl] = tot;
      sc->step = step0 + done;
      sc->pend[rf] = 1;  // and those of the passes before, as each pass sets its next
      if (done > 1) sc->pend[rl] = 1;
      if (done > 2) sc->pend[ring_next(rf)] = 1;
      if (!isfinite(tot) || (stop & 3)) sc->nonfinite = 1;
    }
    if (lane == 5) sc->e1r[rl] = tot;
    if (lane == 6) sc->e1i[rl] = tot;
  }
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int i = u * TPB + tid;
    if (i < n) {
      gp<T>(d.Q)[i] = q[u]; gp<T>(d.P)[i] = p[u]; gp<T>(d.qs)[i] = a[u]; gp<T>(d.ps)[i] = b[u];
    }
  }
}

// Largest instance per workgroup: where one launch per step takes over (us a step, Ng 64,
// resident against 512 x 4 fused): float64 4096 particles 4.2 / 7.5, which is also what the
// registers hold; float32 state with float64 sums 8192 6.6 / 7.1, but with general options or P2
// elements (which then spill) 4096 6.1 / 8.1 and 8192 10.9 / 8.2; the (hi, lo) pairs 2048 11.9 /
// 14.7 and 4096 18.4 / 14.7, the naive mode 1024 4.7 / 10.3 and 2048 12.5 / 10.5 (their LDS
// updates are slow and one CU takes them all).  (Measured before wave_totals, which since took
// 0.5 us off the resident steps and 0.2 off the fused.)
// One workgroup of 1024 threads fills a CU's registers, so more than 256 instances are taken in
// rounds, where the fused step spreads its tiles.  256, 512, 1024 instances, resident against
// 512 x 4 fused: float64 4096 particles 4.4 / 15.8, 8.7 / 29.6, 17 / 53; 200 particles 2.6 / 7.2,
// 5.0 / 10, 9.8 / 17; with a prescribed potential 4096 10 / 19, 20 / 36, 38 / 64; float32 state
// with float64 sums 8192 7.5 / 21, 15 / 36, 28 / 61; naive mode 1024 4.8 / 11, 9.6 / 17, 19 / 31.
// Only the pairs turn, above 1024 particles: 2048 11 / 16, 22 / 20, 43 / 36 (300 instances 21 /
// 18), 1500 9.1 / 14, 18 / 17, 36 / 31; 1024 6.8 / 12, 14 / 15, 27 / 26.
long long resident_capacity(int mode, bool general, bool p2, int nslots) {
  switch (mode) {
    case kFP64: return 4LL * kResidentThreads;
    case kFP32Comp: return (general || p2 ? 4LL : 8LL) * kResidentThreads;
    case kFP32TwoSum: return (nslots > 256 ? 1LL : 2LL) * kResidentThreads;
    default: return kResidentThreads;
  }
}

int resident_ppt(long long nmax) {
  return nmax <= kResidentThreads ? 1 : nmax <= 2 * kResidentThreads ? 2
         : nmax <= 4 * kResidentThreads ? 4 : 8;
}

template <int MODE, int PPT>
static void launch_resident_ppt(const InstDev* d_inst, const int* d_slots, int nslots, size_t lds,
                                bool general, bool p2, int phase, int nsteps, hipStream_t s) {
#define VP_RES(G, P)                                                                              \
  hipLaunchKernelGGL((k_resident<MODE, PPT, G, P>), dim3(nslots), dim3(kResidentThreads), lds, s, \
                     d_inst, d_slots, phase, nsteps)
  if constexpr (PPT <= 4) {
    if constexpr (MODE != kFP32) {
      if (p2 && general) { VP_RES(true, true); return; }
      if (p2) { VP_RES(false, true); return; }
    }
    if (general) { VP_RES(true, false); return; }
  }
  VP_RES(false, false);
#undef VP_RES
}

hipError_t launch_resident(int mode, long long nmax, const InstDev* d_inst, const int* d_slots,
                           int nslots, int max_ng, bool lds_fft, bool general, bool p2, int phase,
                           int nsteps, hipStream_t s) {
  if (nslots <= 0 || nsteps <= 0) return hipSuccess;
  if (nmax > resident_capacity(mode, general, p2, nslots) || (p2 && mode == kFP32))
    return hipErrorInvalidValue;
  const size_t lds = fused_lds_bytes(lds_fft, max_ng);
  const int ppt = resident_ppt(nmax);
#define VP_RES_CASE(M, PP)                                                                   \
  if (mode == M && ppt == PP) {                                                              \
    launch_resident_ppt<M, PP>(d_inst, d_slots, nslots, lds, general, p2, phase, nsteps, s); \
    return hipGetLastError();                                                                \
  }
  VP_RES_CASE(kFP64, 1) VP_RES_CASE(kFP64, 2) VP_RES_CASE(kFP64, 4)
  VP_RES_CASE(kFP32Comp, 1) VP_RES_CASE(kFP32Comp, 2) VP_RES_CASE(kFP32Comp, 4)
  VP_RES_CASE(kFP32Comp, 8)
  VP_RES_CASE(kFP32TwoSum, 1) VP_RES_CASE(kFP32TwoSum, 2)
  VP_RES_CASE(kFP32, 1)
#undef VP_RES_CASE
  return hipErrorInvalidValue;
}

}  // namespace vpk
