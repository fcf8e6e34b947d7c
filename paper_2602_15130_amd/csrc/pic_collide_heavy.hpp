// Collision calls where cells hold hundreds of particles and every outcome
// has tens of candidate pairs (the paper's refinement ladder: N_avg up to
// thousands, Table 1).  One workgroup per cell; a wave holds as many whole
// outcomes of Algorithm 1 as fit into its 64 lanes, one candidate pair per lane:
//   - N_pairs of all outcomes of the cell are tabulated first (one random block
//     per four outcomes, on all lanes);
//   - every lane draws its pair's two random blocks (partners, accept uniform,
//     scattering direction), none of which depends on a velocity;
//   - a pair must see the velocities left by the last earlier pair of its
//     outcome that held one of its particles: each lane finds that pair, and
//     the pairs run in rounds, a pair as soon as those it follows have run.  The
//     chains are short (a cell has many more particles than an outcome
//     pairs), so two or three rounds finish a wave's pairs;
//   - an accepted pair adds the changes it makes to the cell's accumulators.
// The accumulators are fixed point (int64, velocity minus pre-collision
// velocity times 2^scale_bits, added as new value minus value before the
// pair, so the sum over an outcome's pairs is exactly the particle's final
// change): integer sums do not depend on the order in which pairs finish, so the
// result is reproducible however a cell's outcomes are shared out, and the quantum 2^-scale_bits (chosen from N_avg and
// g_max so the sums cannot overflow) sits far below the FP64 state's rounding.
// <dv> = sum / N_avg (eq. avg_outcome).
//
// Bound: vector ALU work, about 1,500 instructions per 64-pair batch (two
// Philox4x64-10 blocks a pair, whose multiply-adds run at a quarter of the
// rate, then sqrt, division and sums in FP64) on ~52 of 64 lanes.  16^3 cells,
// 1,310,720 particles, N_avg 1,024, ~15 pairs per outcome (65 million pairs a
// call): 92 ms with one lane per wave applying an outcome's pairs in order,
// 8.8 ms with a lane per pair, 7 ms with several workgroups per cell and the
// changes added after the rounds.  12^3 cells, 174,960 particles, N_avg 243:
// 4.4 -> 0.28 ms.
#pragma once

#include "pic_kernels.hpp"

namespace pic {

constexpr int kHeavyWaves = 4;
constexpr int kHeavyThreads = 64 * kHeavyWaves;
// 64-pair batches that a wave gets of a mean cell.  12^3 cells as above: 1.9 ms a
// step with one workgroup per cell, 1.5 with two to four, 1.8 with eight; 16^3:
// 19, 16.5 (two), 16 (four to eight).
constexpr int kHeavyBatches = 6;
constexpr int kHeavySeg = 2048;   // outcomes whose pair counts are tabulated at a time
// Particles of the largest cell whose accumulators live in LDS (dynamic, 24 B a
// particle, chosen per launch within 64 KB a workgroup); denser cells
// accumulate in D itself.
constexpr int kHeavyMaxLdsN = 1920;

// LDS of a workgroup: per pair the velocities of its two particles after it,
// and their slots.  A wave's pairs sit at its share of the arrays: 64 entries of
// each of the four waves, or 128 of two, or all of one (outcomes of more pairs).
struct HeavyLds {
  double res[6][kHeavyThreads];
  unsigned pq[kHeavyThreads];     // p | q << 16
  unsigned char more[kHeavySeg];  // N_pairs above the cell's floor(n (n - 1) P_max / 2)
};

// Orders a wave's LDS accesses among its lanes.
__device__ inline void wave_lds_sync() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// Pre-collision velocities of the cell: v[d * NP + s + j].  lds_n: particles of
// a cell whose accumulators the launch's dynamic LDS holds.  u, w, hpq: idle
// per-particle scratch (three doubles each, and one word); a cell uses its
// own slots.
//
// FULL: the instance with the angle and pair logs, the anisotropic samplers and
// the coding errors (compiled apart: they would spill the plain one's registers).
// Four waves per SIMD with 44 spilled registers beat three with two (16^3 as
// above: 31.8 against 33.8 ms for two steps).
template <int SIG, bool FULL>
__global__ void __launch_bounds__(kHeavyThreads, 4)
    k_collide_heavy(SimConst K, int call, int64_t step, const double* v, const int* cstart,
                    double* D, double* u, double* w, unsigned* hpq, int lds_n, int scale_bits,
                    long long* pairlog, int64_t cap, unsigned long long* counters,
                    unsigned long long* spread, int* flags) {
  extern __shared__ unsigned long long heavy_acc[];
  __shared__ HeavyLds W;
  const int64_t NP = K.np;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int c = blockIdx.x;
  const int s = cstart[c], n = cstart[c + 1] - s;
  if (heavy_big_cell(K, n)) return;  // run by k_collide_big
  const double xbase = (double)n * (double)(n - 1) * K.pmax / 2.0;
  // N_pairs = floor(xbase + U), U at most 1 - 2^-53
  const int floor_pairs = (int)floor(xbase), smax = (int)floor(xbase + (1.0 - 0x1.0p-53));
  const int split = blockIdx.y, nsplit = gridDim.y;
  if (n < 2 || smax == 0) {  // (with several workgroups per cell D is already clear)
    if (nsplit == 1)
      for (int d = 0; d < 3; ++d)
        for (int j = tid; j < n; j += kHeavyThreads) D[d * NP + s + j] = 0.0;
    return;
  }
  // An outcome's earlier pairs in the scratch: entry e of row (particle side,
  // component) and of the slots.
  auto hist = [&](int row, int e) -> double& {
    return (row < 3 ? u : w)[(row < 3 ? row : row - 3) * NP + e];
  };
  // Waves at work: an outcome's earlier pairs stay in LDS (all four waves up to
  // 64 pairs, then two, then one) or in the cell's scratch (n entries), whichever
  // keeps more waves.
  const int by_lds = smax <= 64 ? 4 : (smax <= 128 ? 2 : (smax <= kHeavyMaxPairs ? 1 : 0));
  const int by_scratch = min(kHeavyWaves, n / (smax * nsplit));
  const bool LH = by_lds > 0 && by_lds >= by_scratch;
  const bool whole = !LH && by_scratch == 0;  // scratch for one wave only: the first workgroup's
  if (whole && split > 0) return;
  const int nw = LH ? by_lds : (whole ? min(kHeavyWaves, n / smax) : by_scratch);
  const int h0 = s + (split * nw + wave) * smax;  // the wave's scratch entries
  // this workgroup's outcomes [k_lo, k_hi), whole random blocks of four
  const int per = whole ? K.navg : 4 * ((K.navg + 4 * nsplit - 1) / (4 * nsplit));
  const int k_lo = min(split * per, K.navg), k_hi = min(k_lo + per, K.navg);
  const double scale = ldexp(1.0, scale_bits);
  const double dv_max = 8.0 * K.g_max;
  // accumulators: [3][n] in LDS (added to D's words at the end when the cell
  // has several workgroups), or D's own words
  const bool lds_acc = n <= lds_n;
  unsigned long long* gacc = (unsigned long long*)D + s;
  for (int d = 0; d < 3; ++d)
    for (int j = tid; j < n; j += kHeavyThreads) {
      if (lds_acc) heavy_acc[d * n + j] = 0ull;
      else if (nsplit == 1) gacc[d * NP + j] = 0ull;
    }
  if (!lds_acc) __threadfence();
  auto acc_add = [&](int d, int j, unsigned long long x) {
    if (lds_acc) atomicAdd(&heavy_acc[d * n + j], x);
    else atomicAdd(&gacc[d * NP + j], x);
  };

  const int entries = LH ? 64 * (kHeavyWaves / nw) : 64;  // LDS entries of a wave
  const int e0 = wave * entries;
  const int G = smax <= 64 ? 64 / smax : 1;  // outcomes per batch
  const int g = smax <= 64 ? lane / smax : 0;
  unsigned long long nacc = 0, ngmx = 0;
  for (int seg = k_lo; seg < k_hi; seg += kHeavySeg) {
    const int ns = min(kHeavySeg, k_hi - seg);
    __syncthreads();  // the accumulators are clear, the last segment's counts consumed
    for (int b = tid; 4 * b < ns; b += kHeavyThreads) {
      const U64x4 w = stream_block(K, (uint64_t)c, (uint64_t)step, kTagNpairs, (uint64_t)call,
                                   (uint64_t)((seg >> 2) + b), 0);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        if (4 * b + kk < ns)
          W.more[4 * b + kk] = (unsigned char)((int)floor(xbase + unif(w.w[kk])) - floor_pairs);
    }
    __syncthreads();
    if (wave >= nw) continue;
    for (int batch = wave; batch * G < ns; batch += nw) {
      const int ko = batch * G + g, k = seg + ko;
      const int npairs = g < G && ko < ns ? floor_pairs + (int)W.more[ko] : 0;
      // (one outcome per batch: npairs is the same on every lane)
      for (int base = 0; base < (smax <= 64 ? 1 : npairs); base += 64) {
        const int m0 = smax <= 64 ? lane - g * smax : lane;  // place among the outcome's pairs here
        const int m = base + m0;
        const bool valid = m < npairs;
        const int le = e0 + (LH && smax > 64 ? base : 0);    // this chunk's LDS entries
        int p = -1, q = -1;
        double uacc = 0.0, uchi = 0.0, nv[3] = {0.0, 0.0, 0.0}, v0p[3], v0q[3];
        if (valid) {
          const U64x4 wa = stream_block(K, (uint64_t)c, (uint64_t)step, kTagColl, (uint64_t)call,
                                        (uint64_t)k, (uint64_t)(1 + 2 * (int64_t)m));
          const U64x4 wb = stream_block(K, (uint64_t)c, (uint64_t)step, kTagColl, (uint64_t)call,
                                        (uint64_t)k, (uint64_t)(2 + 2 * (int64_t)m));
          p = index_below(wa.w[0], n);
          q = pick_partner(K, c, step, call, k, m, wa, wb, p, n);
          for (int d = 0; d < 3; ++d) {
            v0p[d] = v[d * NP + s + p];
            v0q[d] = v[d * NP + s + q];
          }
          uacc = unif(wa.w[2]);
          uchi = unif(wb.w[0]);
          double seps, ceps;  // eps = 2 pi U_eps, as sin(pi 2 U) and cos(pi 2 U)
          sincospi(2.0 * unif(wa.w[3]), &seps, &ceps);
          const double cchi = cos_chi<double, FULL>(K, uchi);  // eq. chi
          const double schi = sqrt(fmax(0.0, (1.0 - cchi) * (1.0 + cchi)));
          nv[0] = ceps * schi;  // eq. n
          nv[1] = seps * schi;
          nv[2] = cchi;
        }
        const unsigned pq = valid ? (unsigned)p | (unsigned)q << 16 : ~0u;
        W.pq[le + lane] = pq;
        wave_lds_sync();
        // The last earlier pair of the outcome that held p (q): its place and
        // which of its two particles, 2 place + side, or -1.
        int lp = -1, lq = -1;
        auto match = [&](int place, unsigned o) {
          const int pj = (int)(o & 0xffffu), qj = (int)(o >> 16);
          if (lp < 0) lp = pj == p ? 2 * place : (qj == p ? 2 * place + 1 : -1);
          if (lq < 0) lq = pj == q ? 2 * place : (qj == q ? 2 * place + 1 : -1);
        };
        const int reach = smax <= 64 ? smax - 1 : 63;
#pragma unroll 4
        for (int d = 1; d <= reach; ++d) {
          const unsigned o = W.pq[le + max(lane - d, 0)];
          if (d <= m0) match(m - d, o);
        }
#pragma unroll 4
        for (int j = base - 1; j >= 0; --j)  // earlier chunks (the same entry on every lane)
          match(j, LH ? W.pq[e0 + j] : hpq[h0 + j]);
        // a particle's velocity after the pair at place l / 2, side l mod 2
        auto after = [&](int l, int d) {
          const int e = l >> 1, row = 3 * (l & 1) + d;
          if (e >= base) return W.res[row][le + lane - (m - e)];
          return LH ? W.res[row][e0 + e] : hist(row, h0 + e);
        };
        // Rounds: a pair runs once those it follows have.  The first pair
        // still to run follows only pairs that have run, so every round
        // advances.
        const unsigned long long all = __ballot(valid);
        unsigned long long done = 0;
        bool ok = false;
        while (done != all) {
          auto ready = [&](int l) {
            return l < 0 || (l >> 1) < base || ((done >> (lane - (m - (l >> 1)))) & 1ull);
          };
          const bool now = valid && !((done >> lane) & 1ull) && ready(lp) && ready(lq);
          if (now) {
            double up[3], uq[3];
            for (int d = 0; d < 3; ++d) {
              up[d] = lp >= 0 ? after(lp, d) : v0p[d];
              uq[d] = lq >= 0 ? after(lq, d) : v0q[d];
            }
            const double dx = up[0] - uq[0], dy = up[1] - uq[1], dz = up[2] - uq[2];
            const double gr = sqrt(dx * dx + dy * dy + dz * dz);
            if (gr > K.g_max) ++ngmx;
            ok = uacc < sigma_g_t<SIG>(K, gr) / K.sgmax;
            if (ok) {
              ++nacc;
              double pn[3], qn[3];
              post_collision<double, FULL>(K, up, uq, gr, nv, uchi, pn, qn);
              if constexpr (FULL) record_angles<double>(pn, qn, gr, K.anglog, K.angcap, counters);
              for (int d = 0; d < 3; ++d) {
                up[d] = pn[d];
                uq[d] = qn[d];
              }
            }
            for (int d = 0; d < 3; ++d) {
              W.res[d][le + lane] = up[d];
              W.res[3 + d][le + lane] = uq[d];
            }
            if (FULL && pairlog) {
              const unsigned long long slot = atomicAdd(&counters[kCntPairLog], 1ull);
              if ((int64_t)slot < cap) {
                long long* r = pairlog + 7 * slot;
                r[0] = c; r[1] = call; r[2] = k; r[3] = m; r[4] = p; r[5] = q; r[6] = ok;
              }
            }
          }
          done |= __ballot(now);
          wave_lds_sync();
        }
        // The changes, once for all rounds (integer sums: any order): from the
        // value the pair found to the value it left, both as fixed-point
        // changes from the pre-collision velocity.
        if (ok) {
          auto fix = [&](double x, double x0) {
            double dv = x - x0;
            if (!(fabs(dv) <= dv_max)) {
              atomicOr(&flags[kFlagCapacity], 1);
              dv = dv > 0.0 ? dv_max : -dv_max;
            }
            return (unsigned long long)llrint(dv * scale);
          };
          auto add = [&](int slot, int l, const double v0[3], int side) {
            for (int d = 0; d < 3; ++d) {
              unsigned long long x = fix(W.res[3 * side + d][le + lane], v0[d]);
              if (l >= 0) x -= fix(after(l, d), v0[d]);
              acc_add(d, slot, x);
            }
          };
          add(p, lp, v0p, 0);
          add(q, lq, v0q, 1);
        }
        if (!LH && base + 64 < npairs) {  // later chunks of the outcome read these pairs
          const int e = h0 + m;
          hpq[e] = pq;
          for (int d = 0; d < 6; ++d) hist(d, e) = W.res[d][le + lane];
          __threadfence_block();
        }
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    nacc += __shfl_xor(nacc, off);
    ngmx += __shfl_xor(ngmx, off);
  }
  if (lane == 0) {
    count_pairs(spread, nacc, ngmx);
  }
  if (!lds_acc) __threadfence();
  __syncthreads();
  const double inv = 1.0 / (scale * (double)K.navg);
  for (int d = 0; d < 3; ++d)
    for (int j = tid; j < n; j += kHeavyThreads) {
      if (nsplit > 1) {  // k_heavy_finish turns the sums into <dv>
        if (lds_acc) atomicAdd(&gacc[d * NP + j], heavy_acc[d * n + j]);
        continue;
      }
      const unsigned long long a =
          lds_acc ? heavy_acc[d * n + j]
                  : __hip_atomic_load(&gacc[d * NP + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      D[d * NP + s + j] = (double)(long long)a * inv;
    }
}

// <dv> from the fixed-point sums of cells run by several workgroups.
__global__ void __launch_bounds__(kBlock) k_heavy_finish(SimConst K, double* D, int scale_bits) {
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= 3 * K.np) return;
  const double inv = 1.0 / (ldexp(1.0, scale_bits) * (double)K.navg);
  D[i] = (double)((const long long*)D)[i] * inv;
}

// Bits of the fixed-point scale for N_avg outcomes: the sum of N_avg changes of
// magnitude at most 8 g_max stays below 2^62.
inline int heavy_scale_bits(double g_max, int navg) {
  const double bound = 8.0 * g_max * (double)navg;
  int e = 0;
  std::frexp(bound, &e);  // bound < 2^e
  return 62 - e;
}

}  // namespace pic
