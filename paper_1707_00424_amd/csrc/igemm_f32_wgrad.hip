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
// wide and as high as the image (lower where that would leave wavefront slots without strips), one strip per lane half,
// so that images of any size fill the 16-deep contraction; the loads of the next two rows are in flight while one is
// multiplied.
// 3 x 3, 96 -> 96 channels, 32 x 32, batch 3 x 128: 1680 us in the generic kernel (39 TFLOP/s, bound by its per-element
// gather), 375 us here (174 TFLOP/s; matrix units busy half of the time).  Bound by its load instructions: a load takes
// 16 cycles of the compute unit whatever its width, and the 18 that a wavefront issues for every two rows make 2304 of
// the 2314 cycles that eight wavefronts take for them.  Keeping three rows for all nine taps, 54 MFMAs per split, needs 450 registers, which
// the compiler spilled: 1600 us.  LeNet's 5 x 5 layer, six replicas: 62 -> 43 us.
// BIAS: the wavefronts of the first input-channel tile and window row also add up dy.
// A wavefront with a result that is not finite, or too small to be sure of (igemm_split.h), walks its strips a second time
// in plain fp32.  Infinities and NaN leave NaN in the corrections (and in the compensation of the sum of dy), and operands
// beyond the largest bf16 value (3.39e38) have an infinite x0.  Where the width is no multiple of 8 there is a third
// source: the last columns of a strip lie beyond the row, their dy is zero, and the x values beside them belong to other
// taps; an infinity there would make 0 * inf of it.  The second walk sets them to zero, which the first need not do: 0 * x
// adds nothing while x is finite.
#include "igemm_dev.h"
#include "igemm_split.h"
#include "igemm_strips.h"

namespace {

using namespace igemm_dev;

// S: taps per window row and wavefront, SP: stride, OCC: wavefronts per SIMD.
template <int S, int SP, int OCC, bool BIAS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(OCC))) void k_wgrad_f32x3(const ConvGeom g, const WgradIO io,
                                                                                             const StripGeom wg) {
  typedef StripWalk<S, SP, 4> Walk;
  constexpr int L0 = Walk::L0, L1 = Walk::L1, NX = Walk::NX;
  constexpr int W0 = (L0 + 1) / 2, W1 = (L1 + 1) / 2, WX = W0 + W1;
  const StripUnit un = strip_unit(wg, S);
  if (!un.live) return;
  const int rep = blockIdx.z, r = un.r, s0 = un.s0;
  const int lane = threadIdx.x, ch = lane & 31, h = lane >> 5;
  const int n = un.ntile * 32 + ch, c = un.ctile * 32 + ch;
  Walk walk(g, wg, io, rep, un, h, c, n);

  f16v hi[S], lo[S];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int v = 0; v < 16; ++v) hi[s][v] = 0.f, lo[s][v] = 0.f;
  float bsum = 0.f, blow = 0.f;  // compensated sum of dy
  const bool tally = BIAS && un.ctile == 0 && un.first_taps;

  // a row of x (and of dy) as packed words of its three parts
  auto split_x = [&](const uint32_t (&xb)[NX], uint32_t (&xw)[3][WX]) {
    float xv[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) xv[i] = __uint_as_float(xb[i]);
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
  auto split_d = [&](const uint32_t (&db)[8], uint32_t (&dw)[3][4]) {
    float dv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) dv[i] = __uint_as_float(db[i]);
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

  const int rows = walk.rows();
  constexpr int D = SP == 1 ? 2 : 1;  // rows in flight, as registers allow
  uint32_t xr[D][NX], dr[D][8];
#pragma unroll
  for (int i = 0; i < D; ++i) walk.template load<4, 4>(xr[i], dr[i]);
  for (int t = 0; t < rows; t += D) {  // an odd last row is followed by one of zeros
#pragma unroll
    for (int i = 0; i < D; ++i) {
      uint32_t dw[3][4], xw[3][WX];
      split_d(dr[i], dw);
      split_x(xr[i], xw);
      __builtin_amdgcn_sched_barrier(0);
      walk.template load<4, 4>(xr[i], dr[i]);
      row_product(dw, xw);
    }
  }
  SplitRange range;
  range.add(bsum);
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int v = 0; v < 16; ++v) hi[s][v] += lo[s][v], range.add(hi[s][v]);
  bool left = false;
  if (range.in_doubt()) {
    left = out_of_split_range(bsum);
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) left |= out_of_split_range(hi[s][v]);
  }
  if (__builtin_expect(__any(left), 0)) {  // see above: the same sums on fp32 matrix instructions, a pixel of either strip at a time
    bsum = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) hi[s][v] = 0.f;
    walk.restart();
    for (int t = 0; t < rows; ++t) {
      const int live = walk.live_columns();
      walk.template load<4, 4>(xr[0], dr[0]);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float dv = __uint_as_float(dr[0][e]);
        bsum += dv;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float xv = __uint_as_float(xr[0][(s % SP == 0 ? 0 : L0) + s / SP + e]);
          hi[s] = __builtin_amdgcn_mfma_f32_32x32x2f32(dv, e < live ? xv : 0.f, hi[s], 0, 0, 0);
        }
      }
    }
  }

  // register v of a lane: output channel 8*(v/4) + 4*h + v%4 of the tile, input channel `ch`
  float *out = io.out + rep * io.out_rs + un.split * io.split_stride;
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int nn = un.ntile * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
      if (nn < g.N && c < g.Cc && s0 + s < g.S) out[(long long)nn * g.K + (r * g.S + s0 + s) * g.Cc + c] = hi[s][v];
    }
  if (tally) {
    bsum += __shfl_xor(bsum, 32, 64);
    if (h == 0 && n < g.N) out[(long long)g.N * g.K + n] = bsum;
  }
}

// the 5 x 5 kernel takes all five taps of a window row: one wavefront per SIMD
bool five_taps(const ConvGeom &g) { return g.sp == 1 && g.S == 5; }
int wgf32_slots(const ConvGeom &g) { return five_taps(g) ? 1024 : 2048; }

bool make_wgf32(const ConvGeom &g, int replicas, StripGeom &wg) {
  return g.Cc >= 12 && strip_geom(g, replicas, 4, 32, 32, five_taps(g) ? 5 : 3, wgf32_slots(g), wg);
}

// Layers of few pixels whose channels fill the generic kernel's tiles of 64: that kernel has no dead columns (half of a strip
// at a width of 4) and fewer partial sums to write, which is most of the time here.  Both by estimate, in ns: the generic
// kernel takes 2.5 us and per step of 32 rows 1.6, or 2.5 where two workgroups share a compute unit; splits cost either
// 4.5 us and their partial sums.  us, estimates in parentheses, generic / here: 256 -> 256 channels, 16 images of 4 x 4
// 16.7 (18.6) / 21.9 (21.2), of 6 x 6 23.5 (24.4) / 23.7 (23.0), three replicas of 16 images of 4 x 4 24.7 (22.5) / 28.6
// (29.6), one of 128 61 (64) / 45 (45); 128 -> 128, three of 128 images of 3 x 3 30.5 (31.9) / 36.7 (34.1).
bool generic_is_faster(const ConvGeom &g, int replicas, StripGeom &wg) {
  if (g.M > 2048 || g.N < 64 || g.Cc < 64) return false;
  const GenericSplit s = generic_split(g, replicas, 64, 64);
  const long long partial = (long long)replicas * g.N * g.K * 4 / 3000;
  const long long strips = split_strips(g, replicas, wgf32_slots(g), 900, wg) + 4500 + wg.splits * partial;
  return 2500 + s.steps * (s.groups > 256 ? 2500 : 1600) + (s.splits > 1 ? 4500 + s.splits * partial : 0) < strips;
}

}  // namespace

bool wgrad_f32x3_applicable(int dtype, int replicas, const ConvGeom &g) {
  StripGeom wg;
  return dtype == 0 && make_wgf32(g, replicas, wg) && !generic_is_faster(g, replicas, wg);
}

int wgrad_f32x3_plan(int replicas, const ConvGeom &g, int *chunk_out) {
  StripGeom wg;
  make_wgf32(g, replicas, wg);
  split_strips(g, replicas, wgf32_slots(g), 900, wg);
  if (chunk_out) *chunk_out = wg.pps * 32;
  return wg.splits;
}

hipError_t launch_wgrad_f32x3(hipStream_t st, int replicas, const ConvGeom &g, const WgradIO &io) {
  StripGeom wg;
  if (!make_wgf32(g, replicas, wg)) return hipErrorInvalidValue;
  wg.pps = io.chunk / 32, wg.splits = io.splits;
  if (wg.pps < 1 || (long long)wg.pps * wg.splits < wg.pairs) return hipErrorInvalidValue;
  const dim3 grid(strip_blocks(wg), 1, replicas);
#define WGF32_LAUNCH(SV, SPV, OCCV)                                                                       \
  do {                                                                                                    \
    if (io.with_bias)                                                                                     \
      hipLaunchKernelGGL((k_wgrad_f32x3<SV, SPV, OCCV, true>), grid, dim3(64), 0, st, g, io, wg);         \
    else                                                                                                  \
      hipLaunchKernelGGL((k_wgrad_f32x3<SV, SPV, OCCV, false>), grid, dim3(64), 0, st, g, io, wg);        \
  } while (0)
  if (g.sp == 2)
    WGF32_LAUNCH(3, 2, 2);
  else if (five_taps(g))
    WGF32_LAUNCH(5, 1, 1);  // ten accumulators: one wavefront per SIMD
  else
    WGF32_LAUNCH(3, 1, 2);
#undef WGF32_LAUNCH
  return hipGetLastError();
}
