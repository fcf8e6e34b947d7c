// Test harness: the kernels that the library launches for the collisions of a
// pass, run on the CPU under the workgroup emulator (emu.hpp): k_draw_pairs or
// k_draw_tile and the instance that takes their lists, the instance that draws its pairs in chunks,
// each followed by the general instance over the tiles it left, the general
// instance alone, and k_collide_heavy beside the serial k_collide_f64.
// A fence of one wave is a barrier of that wave here: on the GPU its lanes run in
// step, in the emulator they do not.
//
// usage: pair_sources IN OUT
// IN  : pic_problem, pic_discretization, the header below, v[3][np], cs[nn + 1],
//       key[np], x[3][np], id[np], E[3][nn]
// OUT : state (or the call's dv_avg and dv_src) as 6 np FP64 values, key[np] and
//       count[nn] (int32), counters[4] (uint64), flags[4] (int32), tiles left to
//       the general instance (int32)
#include <cstdio>
#include <cstdlib>
#include <type_traits>
#include <vector>

#include "hip/hip_runtime.h"

#undef __builtin_amdgcn_fence
inline void emu_fence(const char* scope) {
  if (!std::strcmp(scope, "wavefront")) emu::wave_barrier(emu::my_wave());
}
#define __builtin_amdgcn_fence(order, scope) emu_fence(scope)
inline void __threadfence_block() {}
template <class T>
inline T __shfl_up(T v, int d) {
  const int lane = __lane_id();
  return emu::wave_shfl(v, lane >= d ? lane - d : lane);
}

#include "pic_host.hpp"
#include "pic_collide_heavy.hpp"
#include "pic_draw.hpp"

namespace pic {
unsigned long long heavy_acc[3 * kHeavyMaxLdsN];  // the launch's dynamic LDS
}
using namespace pic;

enum Source { kGeneral = 0, kDrawn = 1, kChunks = 2, kHeavy = 3, kSerial = 4, kDrawnByTile = 5 };

struct Header {
  uint64_t seed, rng_seed;
  int64_t step;
  int32_t precision, order, source, mode;  // mode: of PartArgs
  int32_t heavy_lds_n, heavy_split;
  int32_t scan_events, unused;
};

template <class T>
static void rd(FILE* f, T* p, size_t n) {
  if (std::fread(p, sizeof(T), n, f) != n) std::exit(2);
}
template <class T>
static void wr(FILE* f, const T* p, size_t n) {
  if (std::fwrite(p, sizeof(T), n, f) != n) std::exit(3);
}

// Workgroups along x and y.
static void run_grid2(unsigned nx, unsigned ny, unsigned nthreads, const std::function<void()>& k,
                      int order, std::mt19937_64& rng) {
  emu::g_griddim = emu::Dim{nx, ny, 1};
  std::vector<unsigned> b(nx * ny);
  std::iota(b.begin(), b.end(), 0u);
  if (order == emu::kReverse) std::reverse(b.begin(), b.end());
  if (order == emu::kShuffle) std::shuffle(b.begin(), b.end(), rng);
  for (unsigned i : b) {
    emu::g_block = emu::Dim{i % nx, i / nx, 0};
    emu::run_block(nthreads, k, order, rng);
  }
}

template <class R, int FAM, int SIG, class F>
static void run_pass(const SimConst& K, PartArgs a, const Header& h, std::mt19937_64& rng, F&& pass) {
  std::vector<PairRec<R>> recB((size_t)a.ntiles * kRecCap), recA(recB.size());
  std::vector<int> nrec(2 * a.ntiles, 12345);
  a.recB = recB.data();
  a.recA = recA.data();
  a.nrec = nrec.data();
  auto sweep = [&](int which, unsigned grid, const PartArgs& args) {
    run_grid2(grid, 1, kTileThreads, [&] { pass(which, args); }, h.order, rng);
  };
  if (h.source == kGeneral) return sweep(0, (unsigned)a.ntiles, a);
  a.defer[0] = 0;
  const bool drawn = h.source != kChunks;
  if (drawn) a.defer[0] = 99;  // (the draw empties the list)
  if (h.source == kDrawnByTile)
    run_grid2((unsigned)a.ntiles, 1, 64 * kDrawWaves, [&] { k_draw_tile<R>(K, a); }, h.order, rng);
  if (h.source == kDrawn) {
    const int per = h.order == emu::kForward ? 1 : kDrawTiles;
    run_grid2((unsigned)((a.ntiles + kDrawWaves * per - 1) / (kDrawWaves * per)), 1, 64 * kDrawWaves,
              [&] { k_draw_pairs<R>(K, a, per); }, h.order, rng);
  }
  sweep(drawn ? 1 : 2, (unsigned)a.ntiles, a);
  a.defer_list = 1;
  sweep(0, (unsigned)std::min(a.ntiles, 7), a);
}

template <int FAM, int SIG>
static int run(const SimConst& K, PartArgs a, const Header& h, std::vector<double>& out,
               const std::vector<double>& x, const std::vector<double>& v,
               const std::vector<double>& ash, const std::vector<double>& E) {
  const int64_t np = K.np;
  const int nn = K.nn;
  std::mt19937_64 rng(h.rng_seed);
  if (h.precision == 0) {
    run_pass<double, FAM, SIG>(K, a, h, rng, [&](int which, const PartArgs& args) {
      if (which == 0) k_particles_f64<FAM, SIG, false, false>(K, args);
      else if (which == 1) k_particles_f64<FAM, SIG, false, true, kPairsDrawn>(K, args);
      else k_particles_f64<FAM, SIG, false, true, kPairsChunks>(K, args);
    });
    if (!(a.mode & kCollideOnly)) {
      std::copy(a.x, a.x + 3 * np, out.begin());
      std::copy(a.v, a.v + 3 * np, out.begin() + 3 * np);
    }
    return 0;
  }
  std::vector<float> off(3 * np), vf(3 * np), ashf(3 * np), E32(3 * (size_t)nn);
  for (int64_t i = 0; i < np; ++i) {
    const double xp[3] = {x[i], x[np + i], x[2 * np + i]};
    int c[3];
    double o[3];
    locate(K, xp, c, o);
    for (int d = 0; d < 3; ++d) {
      off[d * np + i] = std::min((float)o[d], kOneBelow);
      vf[d * np + i] = (float)v[d * np + i];
      ashf[d * np + i] = (float)ash[d * np + i];
    }
  }
  for (int n = 0; n < nn; ++n)
    for (int d = 0; d < 3; ++d) E32[3 * n + d] = (float)E[(size_t)d * nn + n];
  const MixConst M = mix_const(K, a);
  run_pass<float, FAM, SIG>(K, a, h, rng, [&](int which, const PartArgs& args) {
    auto go = [&](auto fn) { fn(K, M, args, off.data(), vf.data(), ashf.data(), E32.data()); };
    if (which == 0) go(k_particles_mixed<FAM, SIG, false, false>);
    else if (which == 1) go(k_particles_mixed<FAM, SIG, false, true, false, kPairsDrawn>);
    else go(k_particles_mixed<FAM, SIG, false, true, false, kPairsChunks>);
  });
  if (!(a.mode & kCollideOnly))
    for (int64_t i = 0; i < 3 * np; ++i) {
      out[i] = off[i];
      out[3 * np + i] = vf[i];
    }
  return 0;
}

int main(int argc, char** argv) {
  if (argc != 3) return 1;
  FILE* in = std::fopen(argv[1], "rb");
  if (!in) return 1;
  pic_problem prob;
  pic_discretization disc;
  Header h;
  rd(in, &prob, 1);
  rd(in, &disc, 1);
  rd(in, &h, 1);
  const SimConst K = derive(&prob, &disc, h.seed, 0);
  const int64_t np = K.np;
  const int nn = K.nn;
  // all arrays sized exactly: an access out of range faults under the sanitizer
  std::vector<double> v(3 * np), x(3 * np), E(3 * (size_t)nn), ash(3 * np), out(6 * np, 0.0);
  std::vector<int> cs(nn + 1), key(np), id(np), slot(np), count(nn, 0);
  rd(in, v.data(), v.size());
  rd(in, cs.data(), cs.size());
  rd(in, key.data(), key.size());
  rd(in, x.data(), x.size());
  rd(in, id.data(), id.size());
  rd(in, E.data(), E.size());
  std::fclose(in);
  for (int64_t i = 0; i < np; ++i) {
    double xv[3], s[3];
    velocity_uniforms(K, id[i], xv);
    velocity_shape(K, xv, s);
    for (int d = 0; d < 3; ++d) ash[d * np + i] = s[d];
  }
  const int ntiles = (int)((np + kTileB - 1) / kTileB);
  std::vector<int> tile_c0(ntiles + 1, nn), tile_s0(ntiles + 1, (int)np), defer(ntiles + 1, 0);
  for (int t = 0; t <= ntiles; ++t) {
    const int64_t want = (int64_t)t * kTileB;
    if (want > np) continue;
    const int c = (int)(std::lower_bound(cs.begin(), cs.end(), (int)want) - cs.begin());
    tile_c0[t] = c;
    tile_s0[t] = cs[c];
  }
  std::vector<double> gv0(3 * np), gu(3 * np), gD(3 * np);
  std::vector<int> gmark(np), gtl(np), flags(kFlagCount, 0);
  std::vector<unsigned long long> counters(kCntCount, 0), spread(kCntSpread * kCntStride, 0);
  MembersAny any{};
  const int iters = 3;
  const double relres = 0.5;
  std::mt19937_64 rng(h.rng_seed);
  int left = 0, rc = 0;
  if (h.source == kHeavy || h.source == kSerial) {  // one FP64 collision call
    if (h.source == kSerial) {
      emu::run_grid((unsigned)((nn + kBlock - 1) / kBlock), kBlock, [&] {
        k_collide_f64(K, 0, h.step, v.data(), cs.data(), out.data(), gu.data(), nullptr, 0,
                      counters.data(), flags.data());
      }, h.order, rng);
    } else {
      if (K.sigma_model != 1 || K.omega != 0.5) return 4;
      const int bits = heavy_scale_bits(K.g_max, K.navg);
      std::vector<unsigned> hpq(np);
      run_grid2((unsigned)nn, (unsigned)h.heavy_split, kHeavyThreads, [&] {
        k_collide_heavy<kSigHS, false>(K, 0, h.step, v.data(), cs.data(), out.data(), gu.data(),
                                       gv0.data(), hpq.data(), h.heavy_lds_n, bits, nullptr, 0,
                                       counters.data(), spread.data(), flags.data());
      }, h.order, rng);
      if (h.heavy_split > 1)
        emu::run_grid((unsigned)((3 * np + kBlock - 1) / kBlock), kBlock,
                      [&] { k_heavy_finish(K, out.data(), bits); }, h.order, rng);
    }
  } else {
    PartArgs a;
    std::memset(&a, 0, sizeof(a));
    a.x = x.data();
    a.v = v.data();
    a.ash = ash.data();
    a.id = id.data();
    a.key = key.data();
    a.slot = slot.data();
    a.count = count.data();
    a.cstart = cs.data();
    a.tile_c0 = tile_c0.data();
    a.tile_s0 = tile_s0.data();
    a.E = E.data();
    a.gv0 = gv0.data();
    a.gu = gu.data();
    a.gD = gD.data();
    a.gmark = gmark.data();
    a.gtl = gtl.data();
    a.Dout = out.data();
    a.Sout = out.data() + 3 * np;
    a.counters = counters.data();
    a.spread = spread.data();
    a.flags = flags.data();
    a.defer = defer.data();
    a.ntiles = ntiles;
    a.mode = h.mode;
    a.nb = h.step;
    a.na = (h.mode & kDoB) ? h.step + 1 : h.step;
    a.callB = 1;
    a.scan_events = h.scan_events;
    const int sig = K.sigma_model == 0 ? kSigPoly : (K.omega == 1.0 ? kSigMaxwell : kSigHS);
    rc = K.family == 1 && sig == kSigHS ? run<1, kSigHS>(K, a, h, out, x, v, ash, E) : 4;
    left = h.source == kGeneral ? 0 : defer[0];
  }
  if (rc) return rc;
  emu::run_grid(1, kCntSpread, [&] {
    k_fold_counters(counters.data(), spread.data(), flags.data(), &iters, &relres, &any, 0);
  }, h.order, rng);
  if (any.gmax != counters[kCntGmax] || any.accepted != counters[kCntAccepted] || any.iters != iters ||
      any.relres != relres)
    return 6;
  FILE* f = std::fopen(argv[2], "wb");
  if (!f) return 1;
  wr(f, out.data(), out.size());
  wr(f, key.data(), key.size());
  wr(f, count.data(), count.size());
  wr(f, counters.data(), counters.size());
  wr(f, flags.data(), flags.size());
  wr(f, &left, 1);
  std::fclose(f);
  return 0;
}
