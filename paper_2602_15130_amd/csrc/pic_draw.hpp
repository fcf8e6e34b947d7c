// The candidate pairs of a pass's collision calls, drawn before the pass.
//
// N_pairs, the partners, the accept uniforms and the scattering directions of
// Algorithm 1 depend on the cell counts and the random stream only, not on a
// velocity.  Inside the pass they kept one wave of four busy, with a lane per
// outcome that has pairs (~8 of 64 at 32 particles per cell and ~0.06 pairs per
// outcome), for about half of all instructions the pass issued.  Here a wave
// takes several consecutive tiles: lanes draw N_pairs of (cell, four outcomes)
// items, append the pairs they find to a queue in LDS, and whenever 64 are
// queued every lane draws one.  A pair's record goes to its place in its
// tile's list, in increasing (cell, outcome, place), where the pass picks it up.
//
// Bound: integer multiplies of the random blocks.  64^3, 8,388,608 particles, 16
// outcomes, both calls: 65 us (mixed) for 2.1 million N_pairs blocks and 0.5 million
// pairs; the pass then takes 275 us instead of 557 (FP64 92 + 644 instead of 928),
// together with the spread pair counters.
#pragma once

#include "pic_particle.hpp"

namespace pic {

constexpr int kDrawWaves = 4;
// Tiles of a wave: four fill its lanes at the usual loads, one keeps the chain short
// where there are too few tiles to give every SIMD a wave anyway (per_wave).
constexpr int kDrawTiles = 4;
inline int draw_tiles_per_wave(int64_t tiles) { return tiles >= 8192 ? kDrawTiles : 1; }

struct DrawLds {
  // queued pairs: tile of the wave << 29 | call << 28 | place in the list << 20 |
  // N_pairs << 17 | pair << 14 | cell of the tile, and the outcome
  unsigned item[128];
  int k[128];
};

template <class R>
__global__ void __launch_bounds__(64 * kDrawWaves) k_draw_pairs(SimConst K, PartArgs a, int per_wave) {
  a = member_view(K, a);
  if (a.step_dev) {  // a captured step: its step index from the device
    a.nb = *K.stepc;
    a.na = a.nb + 1;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) a.defer[0] = 0;  // for the pass that follows
  __shared__ DrawLds lds[kDrawWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  DrawLds& Q = lds[wave];
  const int t0 = (blockIdx.x * kDrawWaves + wave) * per_wave;
  // (a collide-only call stands in call A's place)
  const int lo = (a.mode & kDoB) ? 0 : 1, hi = (a.mode & (kDoA | kCollideOnly)) ? 2 : 1;
  const int navg = K.navg, ngroups = (navg + 3) >> 2;
  auto sync = [] { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); };
  int queued = 0;
  // the first n queued pairs, one per lane
  auto draw = [&](int n) {
    sync();
    if (lane < n) {
      const unsigned it = Q.item[lane];
      const int b = t0 + (int)(it >> 29), li = (int)(it >> 28 & 1u), place = (int)(it >> 20 & 0xffu);
      const int ci = (int)(it & 0x3fffu), c = a.tile_c0[b] + ci, s = a.cstart[c];
      PairRec<R>* list = (PairRec<R>*)(li ? a.recA : a.recB) + (int64_t)b * kRecCap;
      list[place] = draw_pair<R>(K, c, ci, s - a.tile_s0[b], a.cstart[c + 1] - s, li ? a.na : a.nb,
                                 li ? a.callA : a.callB, Q.k[lane], (int)(it >> 14 & 7u),
                                 (int)(it >> 17 & 7u));
    }
    const unsigned it = Q.item[lane + 64 < 128 ? lane + 64 : lane];
    const int k = Q.k[lane + 64 < 128 ? lane + 64 : lane];
    sync();
    Q.item[lane] = it;
    Q.k[lane] = k;
    sync();
    queued -= n;
  };
  for (int ti = 0; ti < per_wave && t0 + ti < a.ntiles; ++ti) {
    const int b = t0 + ti;
    const int c0 = min(a.tile_c0[b], K.nn), ncells = max(min(a.tile_c0[b + 1], K.nn) - c0, 0);
    const int ns = a.tile_s0[b + 1] - a.tile_s0[b];
    // (true: the tile goes to the general instance)
    bool bad = ncells > 0x3fff || (int64_t)ncells * ngroups > (1 << 29);
    int run[2] = {0, 0};
    if (ns > 0 && ns <= kLdsSlots && !bad) {
      const int items = ncells * ngroups;
      for (int base = 0; base < (hi - lo) * items && !bad; base += 64) {
        const int l = base + lane;
        // (lanes past a single call's items stay on its list)
        const int li = l >= items ? 1 : lo, r = l - (li - lo) * items;
        const int ci = r / ngroups, g = r - ci * ngroups;
        int np[4] = {0, 0, 0, 0}, cnt = 0, most = 0;
        if (l < (hi - lo) * items) {
          const int n = a.cstart[c0 + ci + 1] - a.cstart[c0 + ci];
          if (n >= 2) {
            const U64x4 w = npairs_block(K, c0 + ci, li ? a.na : a.nb, li ? a.callA : a.callB, g);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
              if (4 * g + kk < navg) np[kk] = (int)npairs_from(K, n, w.w[kk], a.flags);
              cnt += np[kk];
              most = max(most, np[kk]);
            }
          }
        }
        if (__ballot(most > kSmallPairs)) {
          bad = true;
          break;
        }
        // places in the two lists (counts of both packed: at most 64 x 16 each)
        int incl = li ? cnt << 16 : cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int o = __shfl_up(incl, off);
          if (lane >= off) incl += o;
        }
        const int all = __shfl(incl, 63);
        int place = run[li] + (li ? incl >> 16 : incl & 0xffff) - cnt;
        run[0] += all & 0xffff;
        run[1] += all >> 16;
        if (max(run[0], run[1]) > kRecCap) {
          bad = true;
          break;
        }
        for (int kk = 0; kk < 4; ++kk) {
          const int mine = kk < 2 ? (kk == 0 ? np[0] : np[1]) : (kk == 2 ? np[2] : np[3]);
          for (int m = 0;; ++m) {
            const unsigned long long have = __ballot(mine > m);
            if (!have) break;
            if (mine > m) {
              const int at = queued + __popcll(have & ((1ull << lane) - 1ull));
              Q.item[at] = (unsigned)ti << 29 | (unsigned)li << 28 | (unsigned)(place + m) << 20 |
                           (unsigned)mine << 17 | (unsigned)m << 14 | (unsigned)ci;
              Q.k[at] = 4 * g + kk;
            }
            queued += __popcll(have);
            if (queued >= 64) draw(64);
          }
          place += mine;
        }
      }
    }
    if (lane < 2) a.nrec[2 * b + lane] = bad ? -1 : (lane ? run[1] : run[0]);
  }
  if (queued > 0) draw(queued);
}

}  // namespace pic
