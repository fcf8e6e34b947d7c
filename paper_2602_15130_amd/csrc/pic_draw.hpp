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
// Where tiles are few and have many items (N_avg of hundreds on a small mesh) a
// wave's chain of items is the call's time, and a workgroup takes one tile, each
// of its waves a quarter of the items (k_draw_tile).
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
// where there are too few tiles to give every SIMD a wave anyway (per_wave).  Steps
// with one and four (us; mixed, 16 outcomes, 0.06 pairs each): 64 tiles 104 / 117, 1,728
// tiles 141 / 152, 8,000 tiles 246 / 247, 13,824 tiles 363 / 359, 64,000 tiles 1,334 / 1,291.
constexpr int kDrawTiles = 4;
inline int draw_tiles_per_wave(int64_t tiles) { return tiles >= 8192 ? kDrawTiles : 1; }
// Whether a workgroup takes a tile: with tiles of all members and items of a tile
// and call.  Steps by waves against by tiles (us; mixed, 32 particles a cell, so
// two items to an outcome): 8^3 cells, 64 tiles: 109 / 104 (64 items), 139 / 111
// (512), 592 / 203 (8,192); 24^3, 1,728 tiles: 148 / 146, 194 / 164, 936 / 468;
// 32^3, 4,096 tiles: 192 / 196, 256 / 231, 1,327 / 838, 222 / 211 at 256 items; 48^3,
// 13,824 tiles: 404 / 419, 611 / 523, 4,046 / 2,337, 492 / 460.
inline bool draw_by_tile(int64_t tiles, int64_t items) { return items >= (tiles < 2048 ? 64 : 256); }

// A tile's (cell, four outcomes) items: cells c0 .. c0 + ncells, both lists
// lo .. hi (a collide-only call stands in call A's place).
struct DrawTile {
  int c0, ncells, ngroups, lo, hi;
  bool bad;  // the tile goes to the general instance
  __device__ DrawTile(const SimConst& K, const PartArgs& a, int b) {
    c0 = min(a.tile_c0[b], K.nn);
    ncells = max(min(a.tile_c0[b + 1], K.nn) - c0, 0);
    ngroups = (K.navg + 3) >> 2;
    lo = (a.mode & kDoB) ? 0 : 1;
    hi = (a.mode & (kDoA | kCollideOnly)) ? 2 : 1;
    bad = ncells > 0x3fff || (int64_t)ncells * ngroups > (1 << 29);
  }
  __device__ int items() const { return ncells * ngroups; }
};

// A lane's item: its list, cell of the tile, first outcome, the four N_pairs and
// the place of the first pair in the list.
struct DrawItem {
  int li, ci, k0, np[4], place;
};

// The wave's items [base, base + 64) of the n items from r0 on in each list, run:
// pairs in the lists so far; false where the tile has to go to the general instance.
__device__ __attribute__((always_inline)) inline bool draw_items(const SimConst& K, const PartArgs& a, const DrawTile& T, int r0,
                                                                 int n, int base, int run[2], DrawItem& it) {
  const int lane = threadIdx.x & 63, l = base + lane;
  // (lanes past a single call's items stay on its list)
  const int li = l >= n ? 1 : T.lo, r = r0 + l - (li - T.lo) * n;
  const int ci = r / T.ngroups, g = r - ci * T.ngroups;
  int cnt = 0, most = 0;
  it.np[0] = it.np[1] = it.np[2] = it.np[3] = 0;
  if (l < (T.hi - T.lo) * n) {
    const int np = a.cstart[T.c0 + ci + 1] - a.cstart[T.c0 + ci];
    if (np >= 2) {
      const U64x4 w = npairs_block(K, T.c0 + ci, li ? a.na : a.nb, li ? a.callA : a.callB, g);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (4 * g + kk < K.navg) it.np[kk] = (int)npairs_from(K, np, w.w[kk], a.flags);
        cnt += it.np[kk];
        most = max(most, it.np[kk]);
      }
    }
  }
  if (__ballot(most > kSmallPairs)) return false;
  // places in the two lists (counts of both packed: at most 64 x 16 each)
  int incl = li ? cnt << 16 : cnt;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  const int all = __shfl(incl, 63);
  it.li = li;
  it.ci = ci;
  it.k0 = 4 * g;
  it.place = run[li] + (li ? incl >> 16 : incl & 0xffff) - cnt;
  run[0] += all & 0xffff;
  run[1] += all >> 16;
  return max(run[0], run[1]) <= kRecCap;
}

// Draws pair m (of np) of outcome k on cell ci of tile b into its place.
template <class R>
__device__ __attribute__((always_inline)) inline void draw_record(const SimConst& K, const PartArgs& a, int b, int li, int place,
                                                                  int ci, int k, int m, int np) {
  const int c = a.tile_c0[b] + ci, s = a.cstart[c];
  PairRec<R>* list = (PairRec<R>*)(li ? a.recA : a.recB) + (int64_t)b * kRecCap;
  list[place] = draw_pair<R>(K, c, ci, s - a.tile_s0[b], a.cstart[c + 1] - s, li ? a.na : a.nb,
                             li ? a.callA : a.callB, k, m, np);
}

// The view of a launch: the member's arrays, a captured step's index, and an empty
// list of deferred tiles for the pass that follows.
__device__ inline PartArgs draw_view(const SimConst& K, PartArgs a) {
  a = member_view(K, a);
  if (a.step_dev) {  // a captured step: its step index from the device
    a.nb = *K.stepc;
    a.na = a.nb + 1;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) a.defer[0] = 0;
  return a;
}

struct DrawLds {
  // queued pairs: tile of the wave << 29 | call << 28 | place in the list << 20 |
  // N_pairs << 17 | pair << 14 | cell of the tile, and the outcome
  unsigned item[128];
  int k[128];
};

template <class R>
__global__ void __launch_bounds__(64 * kDrawWaves) k_draw_pairs(SimConst K, PartArgs a, int per_wave) {
  a = draw_view(K, a);
  __shared__ DrawLds lds[kDrawWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  DrawLds& Q = lds[wave];
  const int t0 = (blockIdx.x * kDrawWaves + wave) * per_wave;
  auto sync = [] { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); };
  int queued = 0;
  // the first n queued pairs, one per lane
  auto draw = [&](int n) {
    sync();
    if (lane < n) {
      const unsigned it = Q.item[lane];
      draw_record<R>(K, a, t0 + (int)(it >> 29), (int)(it >> 28 & 1u), (int)(it >> 20 & 0xffu),
                     (int)(it & 0x3fffu), Q.k[lane], (int)(it >> 14 & 7u), (int)(it >> 17 & 7u));
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
    DrawTile T(K, a, b);
    const int ns = a.tile_s0[b + 1] - a.tile_s0[b];
    int run[2] = {0, 0};
    if (ns > 0 && ns <= kLdsSlots && !T.bad) {
      const int items = T.items();
      for (int base = 0; base < (T.hi - T.lo) * items; base += 64) {
        DrawItem it;
        if (!draw_items(K, a, T, 0, items, base, run, it)) {
          T.bad = true;
          break;
        }
        int place = it.place;
        for (int kk = 0; kk < 4; ++kk) {
          const int mine = kk < 2 ? (kk == 0 ? it.np[0] : it.np[1]) : (kk == 2 ? it.np[2] : it.np[3]);
          for (int m = 0;; ++m) {
            const unsigned long long have = __ballot(mine > m);
            if (!have) break;
            if (mine > m) {
              const int at = queued + __popcll(have & ((1ull << lane) - 1ull));
              Q.item[at] = (unsigned)ti << 29 | (unsigned)it.li << 28 | (unsigned)(place + m) << 20 |
                           (unsigned)mine << 17 | (unsigned)m << 14 | (unsigned)it.ci;
              Q.k[at] = it.k0 + kk;
            }
            queued += __popcll(have);
            if (queued >= 64) draw(64);
          }
          place += mine;
        }
      }
    }
    if (lane < 2) a.nrec[2 * b + lane] = T.bad ? -1 : (lane ? run[1] : run[0]);
  }
  if (queued > 0) draw(queued);
}

// A workgroup per tile.  Its waves find the pairs of a quarter of the items each,
// in order; then every thread draws one pair of one of the two lists.
struct DrawTileLds {
  unsigned item[kDrawWaves][2][kRecCap];  // N_pairs << 17 | pair << 14 | cell of the tile
  int k[kDrawWaves][2][kRecCap];
  int n[kDrawWaves][2];                   // a wave's pairs (-1: not in this tile's lists)
};

template <class R>
__global__ void __launch_bounds__(64 * kDrawWaves) k_draw_tile(SimConst K, PartArgs a) {
  static_assert(64 * kDrawWaves == 2 * kRecCap, "a thread per place of both lists");
  a = draw_view(K, a);
  __shared__ DrawTileLds Q;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x;
  DrawTile T(K, a, b);
  const int ns = a.tile_s0[b + 1] - a.tile_s0[b];
  int run[2] = {0, 0};
  if (ns > 0 && ns <= kLdsSlots && !T.bad) {
    const int items = T.items();
    const int r0 = (int)((int64_t)items * wave / kDrawWaves);
    const int n = (int)((int64_t)items * (wave + 1) / kDrawWaves) - r0;
    for (int base = 0; base < (T.hi - T.lo) * n; base += 64) {
      DrawItem it;
      if (!draw_items(K, a, T, r0, n, base, run, it)) {
        T.bad = true;
        break;
      }
      int place = it.place;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        for (int m = 0; m < it.np[kk]; ++m, ++place) {
          Q.item[wave][it.li][place] = (unsigned)it.np[kk] << 17 | (unsigned)m << 14 | (unsigned)it.ci;
          Q.k[wave][it.li][place] = it.k0 + kk;
        }
    }
  }
  if (lane < 2) Q.n[wave][lane] = T.bad ? -1 : (lane ? run[1] : run[0]);
  __syncthreads();
  const int li = tid / kRecCap, place = tid % kRecCap;
  int total[2] = {0, 0}, w = 0, at = place;
  bool bad = false;
  for (int i = 0; i < kDrawWaves; ++i) {
    for (int j = 0; j < 2; ++j) {
      bad |= Q.n[i][j] < 0;
      total[j] += Q.n[i][j];
    }
    // (the wave whose pairs hold this place)
    const int mine = li ? Q.n[i][1] : Q.n[i][0];
    if (w == i && at >= mine) at -= mine, ++w;
  }
  bad |= max(total[0], total[1]) > kRecCap;
  if (tid < 2) a.nrec[2 * b + tid] = bad ? -1 : (tid ? total[1] : total[0]);
  if (bad || w >= kDrawWaves) return;
  const unsigned it = Q.item[w][li][at];
  draw_record<R>(K, a, b, li, place, (int)(it & 0x3fffu), Q.k[w][li][at], (int)(it >> 14 & 7u),
                 (int)(it >> 17 & 7u));
}

}  // namespace pic
