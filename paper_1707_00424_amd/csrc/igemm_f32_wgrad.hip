// fp32 weight gradients on the bf16 matrix units, at fp32 accuracy (the split of igemm_f32.hip: x = x0 + x1 + x2 in bf16,
// six products per pair, the five corrections in an accumulator of their own).
//
//   dW[n][r][s][c] = sum over pixels (b, p, q) of dy[b, p, q, n] * x[b, sp*p + r - pad, sp*q + s - pad, c]
//
// The contraction runs over pixels, the slow index of both operands in memory, and an MFMA fragment wants it contiguous.
// Here that transpose costs nothing, because the operands are converted on their way in anyway: a lane loads one channel
// of eight neighbouring pixels (dwords, 32 lanes on consecutive channels) and the conversion packs two pixels per
// instruction.  The fragments of the S horizontal taps are the same packed words shifted by one value each, so a row of x
// is loaded and split once for all of them.  No LDS, no barrier: a wavefront owns 32 output channels, 32 input channels
// and up to three taps of one row of the window (an accumulator pair each), and walks down strips eight output columns
// wide and about eight rows high, one strip per lane half, so that images of any size fill the 16-deep contraction; the
// loads of the next two rows are in flight while one is multiplied.
// Workgroups are single wavefronts; those of one pixel range and replica get ids that differ by 8, the same XCD, whose L2
// then reads dy and x once for all of them.
// 3 x 3, 96 -> 96 channels, 32 x 32, batch 3 x 128: 1680 us in the generic kernel (39 TFLOP/s, bound by its per-element
// gather), 375 us here (174 TFLOP/s; matrix units busy half of the time, the conversions the other half: an in-register
// split of one row serves 18 MFMAs.  Keeping three rows for all nine taps, 54 MFMAs per split, needs 450 registers, which
// the compiler spilled: 1600 us).  LeNet's 5 x 5 layer, six replicas: 62 -> 43 us.
// BIAS: the wavefronts of the first input-channel tile and window row also add up dy.
#include <algorithm>

#include "igemm_dev.h"
#include "igemm_split.h"

namespace {

using namespace igemm_dev;

struct WgF32Geom {
  // Strips go in pairs at the same height of the image, so that their rows are addressed by one scalar: neighbours of one
  // image where it has an even number of them, else from a group of two images; pairs are numbered image by image.
  int segs, images;         // strips per image row; images per replica
  int gi, pph, ppg;         // images per group; pairs per height and per group
  int PC, heights, pairs;   // rows of a strip; strips on top of each other; pairs in all
  int pps, splits;          // pairs per split
  int nt, ct, sg, units;    // 32-channel tiles of dy and x; groups of three taps per window row; wavefronts per split
  FastDiv dSegs, dPph, dPpg;
};

// S: taps per window row and wavefront, SP: stride, OCC: wavefronts per SIMD.
template <int S, int SP, int OCC, bool BIAS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(OCC))) void k_wgrad_f32x3(const ConvGeom g, const WgradIO io,
                                                                                             const WgF32Geom wg) {
  // tap s reads value (column) i + s/SP of sequence s%SP, which holds the columns sp*q + s%SP - pad
  constexpr int L0 = 8 + (S - 1) / SP, L1 = SP == 2 && S > 1 ? 8 + (S - 2) / 2 : 0, NX = L0 + L1;
  constexpr int W0 = (L0 + 1) / 2, W1 = (L1 + 1) / 2, WX = W0 + W1;
  const int xcd = blockIdx.x & 7, rest = blockIdx.x >> 3;
  const int unit = rest % wg.units, split = rest / wg.units * 8 + xcd;
  if (split >= wg.splits) return;
  const int rep = blockIdx.z;
  const int ntile = unit % wg.nt, ct_r = unit / wg.nt, ctile = ct_r % wg.ct, taps = ct_r / wg.ct;
  const int r = taps / wg.sg, s0 = (taps - r * wg.sg) * S;
  const int lane = threadIdx.x, ch = lane & 31, h = lane >> 5;
  const int n = ntile * 32 + ch, c = ctile * 32 + ch;
  void *const x_ptr = (void *)((const float *)io.x + rep * io.x_rs);
  const int x_bytes = (int)((long long)wg.images * g.Hin * g.Win * g.Cc * 4);
  const __amdgpu_buffer_rsrc_t d_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((const float *)io.dy + rep * io.dy_rs), 0, (int)((long long)g.M * g.N * 4), 0x00020000);

  const int first = split * wg.pps, last = min(wg.pairs, first + wg.pps);
  // what is loaded next: output row `ld_p` (below `ld_end`) of pair `ld_pair`; beyond the last pair everything is out of
  // range, that is zero
  int ld_pair = first, ld_p = 0, ld_end = 0;
  uint32_t xoff[NX], doff[8];
  auto set_strip = [&]() {
    const int group = (int)fdiv((uint32_t)ld_pair, wg.dPpg), in_group = ld_pair - group * wg.ppg;
    const int height = (int)fdiv((uint32_t)in_group, wg.dPph);
    ld_p = height * wg.PC, ld_end = min(g.P, ld_p + wg.PC);
    const int strip = 2 * (in_group - height * wg.pph) + h;
    const int img = (int)fdiv((uint32_t)strip, wg.dSegs), q0 = (strip - img * wg.segs) * 8, b = group * wg.gi + img;
    const int live = (ld_pair < last) & (b < wg.images), x_live = live & (c < g.Cc), d_live = live & (n < g.N);
    const int col0 = SP * q0 + s0 + g.off;
    const uint32_t xo = (uint32_t)((b * g.Hin * g.Win + col0) * g.Cc + c) * 4u, dof = (uint32_t)((b * g.P * g.Q + q0) * g.N + n) * 4u;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int j = i < L0 ? SP * i : SP * (i - L0) + 1;  // column relative to the strip's first
      xoff[i] = x_live & (int)((unsigned)(col0 + j) < (unsigned)g.Win) ? xo + (uint32_t)(j * g.Cc * 4) : kOobOffset;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) doff[i] = d_live & (int)(q0 + i < g.Q) ? dof + (uint32_t)(i * g.N * 4) : kOobOffset;
  };
  set_strip();
  auto load_row = [&](float (&xv)[NX], float (&dv)[8]) {
    const int row = ld_p * SP + g.off + r;
    const bool row_ok = (unsigned)row < (unsigned)g.Hin;  // a row of the padding: a buffer of no bytes gives zeros
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(x_ptr, 0, row_ok ? x_bytes : 0, 0x00020000);
    const int xs = row_ok ? row * g.Win * g.Cc * 4 : 0, ds = ld_p * g.Q * g.N * 4;
#pragma unroll
    for (int i = 0; i < NX; ++i) xv[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x_rsrc, xoff[i], xs, 0));
#pragma unroll
    for (int i = 0; i < 8; ++i) dv[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(d_rsrc, doff[i], ds, 0));
    if (++ld_p == ld_end) {
      asm volatile("" ::: "memory");  // a branch: executed for every row, these address sums would rival the conversions
      ++ld_pair;
      set_strip();
    }
  };

  f16v hi[S], lo[S];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int v = 0; v < 16; ++v) hi[s][v] = 0.f, lo[s][v] = 0.f;
  float bsum = 0.f, blow = 0.f;  // compensated sum of dy
  const bool tally = BIAS && ctile == 0 && taps == 0;

  // a row of x (and of dy) as packed words of its three parts
  auto split_x = [&](const float (&xv)[NX], uint32_t (&xw)[3][WX]) {
    uint32_t w0[3][W0];
    split_words<L0>(xv, w0);
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int i = 0; i < W0; ++i) xw[k][i] = w0[k][i];
    if constexpr (L1 > 0) {
      uint32_t w1[3][W1];
      split_words<L1>(xv + L0, w1);
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < W1; ++i) xw[k][W0 + i] = w1[k][i];
    }
  };
  auto split_d = [&](const float (&dv)[8], uint32_t (&dw)[3][4]) {
    split_words<8>(dv, dw);
    if (tally) {
      const float t = (((dv[0] + dv[1]) + (dv[2] + dv[3])) + ((dv[4] + dv[5]) + (dv[6] + dv[7]))) - blow, u = bsum + t;
      blow = (u - bsum) - t, bsum = u;
    }
  };
  auto row_product = [&](const uint32_t (&dw)[3][4], const uint32_t (&xw)[3][WX]) {
    u4 a[3], b[3][S];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      a[k] = u4{dw[k][0], dw[k][1], dw[k][2], dw[k][3]};
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int sh = s / SP, base = s % SP == 0 ? 0 : W0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int w = base + sh / 2 + e;
          b[k][s][e] = sh & 1 ? __builtin_amdgcn_alignbit(xw[k][w + 1 < WX ? w + 1 : w], xw[k][w], 16) : xw[k][w];
        }
      }
    }
    // tap by tap inside a product: no MFMA waits for the accumulator of the one in front of it
#pragma unroll
    for (int s = 0; s < S; ++s) mma<bf16_t>(a[0], b[0][s], hi[s]);
#pragma unroll
    for (int s = 0; s < S; ++s) mma<bf16_t>(a[0], b[1][s], lo[s]);
#pragma unroll
    for (int s = 0; s < S; ++s) mma<bf16_t>(a[1], b[0][s], lo[s]);
#pragma unroll
    for (int s = 0; s < S; ++s) mma<bf16_t>(a[1], b[1][s], lo[s]);
#pragma unroll
    for (int s = 0; s < S; ++s) mma<bf16_t>(a[0], b[2][s], lo[s]);
#pragma unroll
    for (int s = 0; s < S; ++s) mma<bf16_t>(a[2], b[0][s], lo[s]);
  };

  // rows of this split: whole strips, of which those at the last height of an image may be shorter
  auto at_last_height = [&](int pairs) {
    const int group = (int)fdiv((uint32_t)pairs, wg.dPpg);
    return group * wg.pph + max(0, pairs - group * wg.ppg - (wg.heights - 1) * wg.pph);
  };
  const int rows = (last - first) * wg.PC - (at_last_height(last) - at_last_height(first)) * (wg.heights * wg.PC - g.P);
  constexpr int D = SP == 1 ? 2 : 1;  // rows in flight, as registers allow
  float xr[D][NX], dr[D][8];
#pragma unroll
  for (int i = 0; i < D; ++i) load_row(xr[i], dr[i]);
  for (int t = 0; t < rows; t += D) {  // an odd last row is followed by one of zeros
#pragma unroll
    for (int i = 0; i < D; ++i) {
      uint32_t dw[3][4], xw[3][WX];
      split_d(dr[i], dw);
      split_x(xr[i], xw);
      __builtin_amdgcn_sched_barrier(0);
      load_row(xr[i], dr[i]);
      row_product(dw, xw);
    }
  }

  // register v of a lane: output channel 8*(v/4) + 4*h + v%4 of the tile, input channel `ch`
  float *out = io.out + rep * io.out_rs + split * io.split_stride;
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int nn = ntile * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
      const float hv = hi[s][v], t = hv + lo[s][v];
      if (nn < g.N && c < g.Cc && s0 + s < g.S) out[(long long)nn * g.K + (r * g.S + s0 + s) * g.Cc + c] = t == t ? t : hv;
    }
  if (tally) {
    bsum += __shfl_xor(bsum, 32, 64);
    if (h == 0 && n < g.N) out[(long long)g.N * g.K + n] = bsum;
  }
}

bool make_wgf32(const ConvGeom &g, int replicas, WgF32Geom &wg) {
  if (g.dshift != 0 || g.sr != 1 || g.R != g.S || g.M % (g.P * g.Q) != 0) return false;
  if (g.S < 3 || g.Cc < 12) return false;
  const int images = g.M / (g.P * g.Q);
  const long long lim = 1LL << 31;
  if ((long long)images * g.Hin * g.Win * g.Cc * 4 >= lim || (long long)g.M * g.N * 4 >= lim) return false;
  wg.segs = (g.Q + 7) / 8, wg.images = images, wg.gi = wg.segs % 2 == 0 ? 1 : 2;
  const bool five = g.sp == 1 && g.S == 5;
  wg.nt = (g.N + 31) / 32, wg.ct = (g.Cc + 31) / 32, wg.sg = five ? 1 : (g.S + 2) / 3, wg.units = wg.nt * wg.ct * wg.sg * g.R;
  // strips as high as the image (a strip costs about one row in addresses), lower where that leaves fewer than four per
  // wavefront slot
  const int slots = five ? 1024 : 2048;
  const long long columns = (long long)images * wg.segs / 2 * wg.units * replicas;
  wg.heights = 1;
  while (columns * wg.heights < 4 * slots && g.P / (wg.heights + 1) >= 4) ++wg.heights;
  wg.PC = (g.P + wg.heights - 1) / wg.heights, wg.heights = (g.P + wg.PC - 1) / wg.PC;
  wg.pph = wg.gi * wg.segs / 2, wg.ppg = wg.pph * wg.heights;
  if ((long long)(images + 1) * wg.ppg >= lim) return false;
  wg.pairs = (images + wg.gi - 1) / wg.gi * wg.ppg;
  wg.dSegs = make_fastdiv(wg.segs), wg.dPph = make_fastdiv(wg.pph), wg.dPpg = make_fastdiv(wg.ppg);
  // splits, by estimated time (units of 10 ns): rows on the busiest slot (about 0.9 us each with a full chip), writing and
  // reading the partial sums (3 TB/s) and adding them up
  const long long per_split = (long long)wg.units * replicas;
  long long best = -1;
  const int max_splits = (int)std::min<long long>(std::min<long long>(wg.pairs, 65535 / replicas), slots / per_split + 1);
  for (int s = 1; s <= max_splits; ++s) {
    const int pps = (wg.pairs + s - 1) / s, real = (wg.pairs + pps - 1) / pps;
    const long long rounds = (per_split * real + slots - 1) / slots;
    const long long cost = rounds * pps * wg.PC * 90 + real * 6 + (long long)real * replicas * g.N * g.K * 4 / 30000;
    if (best < 0 || cost < best) best = cost, wg.pps = pps, wg.splits = real;
  }
  return true;
}

}  // namespace

bool wgrad_f32x3_applicable(int dtype, int replicas, const ConvGeom &g) {
  WgF32Geom wg;
  return dtype == 0 && make_wgf32(g, replicas, wg);
}

int wgrad_f32x3_plan(int replicas, const ConvGeom &g, int *chunk_out) {
  WgF32Geom wg;
  make_wgf32(g, replicas, wg);
  if (chunk_out) *chunk_out = wg.pps * 32;
  return wg.splits;
}

hipError_t launch_wgrad_f32x3(hipStream_t st, int replicas, const ConvGeom &g, const WgradIO &io) {
  WgF32Geom wg;
  if (!make_wgf32(g, replicas, wg)) return hipErrorInvalidValue;
  wg.pps = io.chunk / 32, wg.splits = io.splits;
  if (wg.pps < 1 || (long long)wg.pps * wg.splits < wg.pairs) return hipErrorInvalidValue;
  const dim3 grid((wg.splits + 7) / 8 * 8 * wg.units, 1, replicas);
#define WGF32_LAUNCH(SV, SPV, OCCV)                                                                       \
  do {                                                                                                    \
    if (io.with_bias)                                                                                     \
      hipLaunchKernelGGL((k_wgrad_f32x3<SV, SPV, OCCV, true>), grid, dim3(64), 0, st, g, io, wg);         \
    else                                                                                                  \
      hipLaunchKernelGGL((k_wgrad_f32x3<SV, SPV, OCCV, false>), grid, dim3(64), 0, st, g, io, wg);        \
  } while (0)
  if (g.sp == 2)
    WGF32_LAUNCH(3, 2, 2);
  else if (g.S == 5)
    WGF32_LAUNCH(5, 1, 1);  // ten accumulators: one wavefront per SIMD
  else
    WGF32_LAUNCH(3, 1, 2);
#undef WGF32_LAUNCH
  return hipGetLastError();
}
