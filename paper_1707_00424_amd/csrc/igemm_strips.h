// Backward-weight kernels whose operands go from memory straight into MFMA fragments, a lane holding one channel (or one
// pair of channels) of eight neighbouring pixels: how they walk the images and how the work is split.
//
// A wavefront walks down strips eight output columns wide, one per lane half, so that images of any width fill the 16-deep
// contraction.  Strips go in pairs at the same height of the image, so that their rows are addressed by one scalar:
// neighbours of one image where it has an even number of them, else from a group of two images; pairs are numbered image
// by image, so that a split reads memory in order.
#pragma once
#include <algorithm>

#include "igemm_dev.h"

namespace igemm_dev {

struct StripGeom {
  int segs, images;        // strips per image row; images per replica
  int gi, pph, ppg;        // images per group; pairs per height and per group
  int PC, heights, pairs;  // rows of a strip; strips on top of each other; pairs in all
  int pps, splits;         // pairs per split
  int nt, ct, sg, units;   // tiles of dy and x channels; groups of taps per window row; wavefronts per split
  FastDiv dSegs, dPph, dPpg;
};

// Blocks of a launch: one per unit and split, a multiple of 8.
inline int strip_blocks(const StripGeom &wg) { return (wg.splits * wg.units + 7) / 8 * 8; }
// A wavefront's place in the launch.  Blocks are single wavefronts, in order of (split, unit); each XCD (ids that differ by
// 8) takes an eighth of that order, so that its L2 reads the dy and x of a split once for many units, and all XCDs have the
// same number whatever the number of splits.  With a split's units on one XCD, three splits ran on three of the eight: 3 x 3,
// 256 -> 256 channels, 7 x 7, 3 x 16 images, 68.8 -> 35.4 us;
// one replica of 128 images, ten splits, 85.4 -> 62.6.
struct StripUnit {
  int split, r, s0, ntile, ctile;
  bool live, first_taps;
};
__device__ __forceinline__ StripUnit strip_unit(const StripGeom &wg, int taps_per_unit) {
  StripUnit u;
  const int place = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int unit = place % wg.units;
  u.split = place / wg.units, u.live = u.split < wg.splits;
  const int ct_r = unit / wg.nt, taps = ct_r / wg.ct;
  u.ntile = unit % wg.nt, u.ctile = ct_r % wg.ct;
  u.r = taps / wg.sg, u.s0 = (taps - u.r * wg.sg) * taps_per_unit;
  u.first_taps = taps == 0;
  return u;
}

// S taps of a window row, stride SP, elements of ES bytes.  Tap s reads value i + s/SP of sequence s%SP, which holds the
// columns sp*q + s%SP - pad of the strip.
template <int S, int SP, int ES>
struct StripWalk {
  static constexpr int L0 = 8 + (S - 1) / SP, L1 = SP == 2 && S > 1 ? 8 + (S - 2) / 2 : 0, NX = L0 + L1;
  const ConvGeom &g;
  const StripGeom &wg;
  const int r, s0, h, c, n;  // window row, first tap, lane half, first channel of this lane in x and dy
  int first, last;           // pairs of this split
  void *x_ptr;
  int x_bytes;
  __amdgpu_buffer_rsrc_t d_rsrc;
  // what is loaded next: output row `p` (below `end`) of pair `pair`; beyond the last pair everything is out of range,
  // that is zero
  int pair, p, end;
  uint32_t xoff[NX], doff[8];

  __device__ __forceinline__ StripWalk(const ConvGeom &g_, const StripGeom &wg_, const WgradIO &io, int rep, const StripUnit &u,
                                       int h_, int c_, int n_)
      : g(g_), wg(wg_), r(u.r), s0(u.s0), h(h_), c(c_), n(n_) {
    first = u.split * wg.pps, last = min(wg.pairs, first + wg.pps);
    x_ptr = (void *)((const char *)io.x + rep * io.x_rs * ES);
    x_bytes = (int)((long long)wg.images * g.Hin * g.Win * g.Cc * ES);
    d_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)io.dy + rep * io.dy_rs * ES), 0,
                                               (int)((long long)g.M * g.N * ES), 0x00020000);
    restart();
  }
  __device__ __forceinline__ void restart() {
    pair = first;
    set_strip();
  }
  // output columns of this lane's strip, which is loaded next, inside the image row: where it is less than 8, dy is zero
  // for the others, but the x values beside them may belong to other taps of the row
  __device__ __forceinline__ int live_columns() const {
    const int in_group = pair - (int)fdiv((uint32_t)pair, wg.dPpg) * wg.ppg;
    const int strip = 2 * (in_group - (int)fdiv((uint32_t)in_group, wg.dPph) * wg.pph) + h;
    return g.Q - (strip - (int)fdiv((uint32_t)strip, wg.dSegs) * wg.segs) * 8;
  }
  __device__ __forceinline__ void set_strip() {
    const int group = (int)fdiv((uint32_t)pair, wg.dPpg), in_group = pair - group * wg.ppg;
    const int height = (int)fdiv((uint32_t)in_group, wg.dPph);
    p = height * wg.PC, end = min(g.P, p + wg.PC);
    const int strip = 2 * (in_group - height * wg.pph) + h;
    const int img = (int)fdiv((uint32_t)strip, wg.dSegs), q0 = (strip - img * wg.segs) * 8, b = group * wg.gi + img;
    const int live = (pair < last) & (b < wg.images), x_live = live & (c < g.Cc), d_live = live & (n < g.N);
    const int col0 = SP * q0 + s0 + g.off;
    const uint32_t xo = (uint32_t)((b * g.Hin * g.Win + col0) * g.Cc + c) * ES;
    const uint32_t dof = (uint32_t)((b * g.P * g.Q + q0) * g.N + n) * ES;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int j = i < L0 ? SP * i : SP * (i - L0) + 1;  // column relative to the strip's first
      xoff[i] = x_live & (int)((unsigned)(col0 + j) < (unsigned)g.Win) ? xo + (uint32_t)(j * g.Cc * ES) : kOobOffset;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) doff[i] = d_live & (int)(q0 + i < g.Q) ? dof + (uint32_t)(i * g.N * ES) : kOobOffset;
  }
  // loads the next row (XW, DW: 4 bytes per lane or 2) and moves on
  template <int XW, int DW>
  __device__ __forceinline__ void load(uint32_t (&xv)[NX], uint32_t (&dv)[8]) {
    const int row = p * SP + g.off + r;
    const bool row_ok = (unsigned)row < (unsigned)g.Hin;  // a row of the padding: a buffer of no bytes gives zeros
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(x_ptr, 0, row_ok ? x_bytes : 0, 0x00020000);
    const int xs = row_ok ? row * g.Win * g.Cc * ES : 0, ds = p * g.Q * g.N * ES;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      if constexpr (XW == 4)
        xv[i] = __builtin_amdgcn_raw_buffer_load_b32(x_rsrc, xoff[i], xs, 0);
      else
        xv[i] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(x_rsrc, xoff[i], xs, 0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (DW == 4)
        dv[i] = __builtin_amdgcn_raw_buffer_load_b32(d_rsrc, doff[i], ds, 0);
      else
        dv[i] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(d_rsrc, doff[i], ds, 0);
    }
    if (++p == end) {
      asm volatile("" ::: "memory");  // a branch: executed for every row, these address sums would rival the rest
      ++pair;
      set_strip();
    }
  }
  // rows of this split: whole strips, of which those at the last height of an image may be shorter
  __device__ __forceinline__ int rows() const {
    auto at_last_height = [&](int pairs) {
      const int group = (int)fdiv((uint32_t)pairs, wg.dPpg);
      return group * wg.pph + max(0, pairs - group * wg.ppg - (wg.heights - 1) * wg.pph);
    };
    return (last - first) * wg.PC - (at_last_height(last) - at_last_height(first)) * (wg.heights * wg.PC - g.P);
  }
};

// The walk of a layer: tiles of `tn` x `tc` channels and `taps` taps of a window row per wavefront, `slots` wavefronts on the
// chip.  False where the layer is none for these kernels.
inline bool strip_geom(const ConvGeom &g, int replicas, int es, int tn, int tc, int taps, int slots, StripGeom &wg) {
  if (g.dshift != 0 || g.sr != 1 || g.R != g.S || g.S < 3 || (g.sp != 1 && g.sp != 2) || g.M % (g.P * g.Q) != 0) return false;
  const int images = g.M / (g.P * g.Q);
  const long long lim = 1LL << 31;
  if ((long long)images * g.Hin * g.Win * g.Cc * es >= lim || (long long)g.M * g.N * es >= lim) return false;
  wg.segs = (g.Q + 7) / 8, wg.images = images, wg.gi = wg.segs % 2 == 0 ? 1 : 2;
  wg.nt = (g.N + tn - 1) / tn, wg.ct = (g.Cc + tc - 1) / tc, wg.sg = (g.S + taps - 1) / taps;
  wg.units = wg.nt * wg.ct * wg.sg * g.R;
  // strips as high as the image (a strip costs about one row in addresses), lower where that leaves fewer than four per
  // wavefront slot
  const long long columns = (long long)images * wg.segs / 2 * wg.units * replicas;
  wg.heights = 1;
  while (columns * wg.heights < 4 * slots && g.P / (wg.heights + 1) >= 4) ++wg.heights;
  wg.PC = (g.P + wg.heights - 1) / wg.heights, wg.heights = (g.P + wg.PC - 1) / wg.PC;
  wg.pph = wg.gi * wg.segs / 2, wg.ppg = wg.pph * wg.heights;
  if ((long long)(images + 1) * wg.ppg >= lim) return false;
  wg.pairs = (images + wg.gi - 1) / wg.gi * wg.ppg;
  wg.dSegs = make_fastdiv(wg.segs), wg.dPph = make_fastdiv(wg.pph), wg.dPpg = make_fastdiv(wg.ppg);
  return true;
}

// Splits the pairs by estimated time in ns: rows on the busiest slot (about `row_ns` with a full chip), writing and reading
// the partial sums (3 TB/s), adding them up.  Split counts that leave the same number of pairs to a split are one plan; the
// search visits each plan once (a few tens, under a microsecond).  Returns the estimate.
inline long long split_strips(const ConvGeom &g, int replicas, int slots, int row_ns, StripGeom &wg) {
  const long long per_split = (long long)wg.units * replicas;
  long long best = -1;
  const int max_splits = (int)std::min<long long>(std::min<long long>(wg.pairs, 65535 / replicas), slots / per_split + 1);
  for (int s = 1; s <= max_splits;) {
    const int pps = (wg.pairs + s - 1) / s, real = (wg.pairs + pps - 1) / pps;
    const long long rounds = (per_split * real + slots - 1) / slots;
    const long long cost = rounds * pps * wg.PC * row_ns + real * 60 + (long long)real * replicas * g.N * g.K * 4 / 3000;
    if (best < 0 || cost < best) best = cost, wg.pps = pps, wg.splits = real;
    if (pps == 1) break;
    s = (wg.pairs + pps - 2) / (pps - 1);  // the first with fewer pairs to a split
  }
  return best;
}

// The generic weight gradient's plan for tiles of tn x tk outputs: rows in steps of 32 to a workgroup, and workgroups.
struct GenericSplit {
  long long tiles, groups;
  int steps, splits;
};
inline GenericSplit generic_split(const ConvGeom &g, int replicas, int tn, int tk) {
  GenericSplit s;
  s.tiles = (long long)((g.K + tk - 1) / tk) * ((g.N + tn - 1) / tn) * replicas;
  const int all = (g.M + 31) / 32;
  const int want = (int)std::max<long long>(1, std::min<long long>(512 / s.tiles, all / 4));
  s.steps = (all + want - 1) / want, s.splits = (all + s.steps - 1) / s.steps;
  s.groups = s.tiles * s.splits;
  return s;
}

}  // namespace igemm_dev
