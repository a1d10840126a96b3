// bf16 weight gradients without LDS: the operands go from memory into MFMA fragments in registers.
//
//   dW[n][r][s][c] = sum over pixels (b, p, q) of dy[b, p, q, n] * x[b, sp*p + r - pad, sp*q + s - pad, c]
//
// The contraction runs over pixels, the slow index of both operands in memory, and an MFMA fragment wants eight of them in
// one lane.  A lane loads a pair of channels (one dword; 32 lanes on 128 consecutive bytes) of eight neighbouring pixels,
// and one v_perm per two pixels and channel makes the fragments: lane l of the even (odd) fragment holds channel 2l
// (2l + 1) of a tile of 64.  A wavefront owns such a tile of dy, one of x and three taps of one row of the window: twelve
// accumulators, 26 permutes and 18 loads per 12 MFMAs (384 cycles).  The fragments of the three taps are the same loaded
// values paired one pixel further on.  No LDS, no barrier, no halo, any image size; a few rows of loads in flight cover
// the latency with one wavefront per SIMD.
// What bounds it is the number of load instructions, sixteen cycles each for a compute unit whatever their width: 320 -> 320
// channels on 16 x 16 take 380 us against 207 us in the kernel that stages blocks in LDS (k_wgrad9), 96 -> 96 on 32 x 32
// 235 against 97.  It runs the layers no vector kernel takes, channel counts that are no multiple of 8, where the
// generic kernel gathers element by element: 50 -> 64 channels on 16 x 16, batch 6 x 50, layer pass 187 -> 149 us; 20 -> 50
// on 28 x 28, 2 x 100, 265 -> 220 us.
// P: channels per lane, 1 where a count is odd.
// Where the width is no multiple of 8, the last columns of a strip lie beyond the row: dy is zero there, and the x values
// beside it belong to other taps.  0 * x adds nothing while x is finite; a wavefront with a result that is not finite
// walks its strips a second time with those values set to zero.
#include "igemm_dev.h"
#include "igemm_strips.h"

namespace {

using namespace igemm_dev;

template <int P, int S, int SP>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(P == 2 ? 1 : 2))) void k_wgrad_strips(const ConvGeom g,
                                                                                                       const WgradIO io,
                                                                                                       const StripGeom wg) {
  typedef StripWalk<S, SP, 2> Walk;
  constexpr int NX = Walk::NX, L0 = Walk::L0;
  const StripUnit un = strip_unit(wg, S);
  if (!un.live) return;
  const int rep = blockIdx.z;
  const int lane = threadIdx.x, ch = lane & 31, h = lane >> 5;
  const int n = (un.ntile * 32 + ch) * P, c = (un.ctile * 32 + ch) * P;
  Walk walk(g, wg, io, rep, un, h, c, n);

  f16v acc[P][P][S];
  auto each_acc = [&](auto f) {
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
      for (int j = 0; j < P; ++j)
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float a = acc[i][j][s][v];
            f(a);
            acc[i][j][s][v] = a;
          }
  };
  each_acc([](float &a) { a = 0.f; });

  // channel `par` of values a (low half of the result) and b
  auto pair = [](uint32_t a, uint32_t b, int par) {
    return __builtin_amdgcn_perm(b, a, par ? 0x07060302u : 0x05040100u);
  };
  // MASKED: only the first `live` columns of x
  auto multiply = [&](auto masked, int live, const uint32_t (&xv)[NX], const uint32_t (&dv)[8]) {
    u4 a[P], b[P][S];
#pragma unroll
    for (int i = 0; i < P; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[i][e] = pair(dv[2 * e], dv[2 * e + 1], i);
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const int v = (s % SP ? L0 : 0) + s / SP + 2 * e;
          b[i][s][e] = pair(xv[v], xv[v + 1], i);
          if (decltype(masked)::value) b[i][s][e] &= live > 2 * e + 1 ? ~0u : live > 2 * e ? 0xffffu : 0u;
        }
      }
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int i = 0; i < P; ++i)
#pragma unroll
        for (int j = 0; j < P; ++j) mma<bf16_t>(a[i], b[j][s], acc[i][j][s]);
  };
  constexpr int D = 3;  // rows in flight
  uint32_t xr[D][NX], dr[D][8];
#pragma unroll
  for (int i = 0; i < D; ++i) walk.template load<2 * P, 2 * P>(xr[i], dr[i]);
  const int rows = walk.rows();
  for (int t = 0; t < rows; t += D) {  // rows beyond the last are zeros
#pragma unroll
    for (int i = 0; i < D; ++i) {
      multiply(std::false_type{}, 8, xr[i], dr[i]);
      walk.template load<2 * P, 2 * P>(xr[i], dr[i]);
    }
  }
  if (g.Q % 8 != 0) {
    NonFinite odd;
    each_acc([&](float &a) { odd.add(a); });
    if (odd.any()) {
      each_acc([](float &a) { a = 0.f; });
      walk.restart();
      for (int t = 0; t < rows; ++t) {
        const int live = walk.live_columns();
        walk.template load<2 * P, 2 * P>(xr[0], dr[0]);
        multiply(std::true_type{}, live, xr[0], dr[0]);
      }
    }
  }

  // register v of a lane: row 8*(v/4) + 4*h + v%4 of the tile of dy, column `ch` of the tile of x
  float *out = io.out + rep * io.out_rs + un.split * io.split_stride;
  typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
#pragma unroll
  for (int i = 0; i < P; ++i)
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int nn = (un.ntile * 32 + 8 * (v >> 2) + 4 * h + (v & 3)) * P + i;
        if (nn < g.N && c < g.Cc && un.s0 + s < g.S) {
          float *dst = out + (long long)nn * g.K + (un.r * g.S + un.s0 + s) * g.Cc + c;
          if constexpr (P == 2)
            *(f2u *)dst = f2u{acc[i][0][s][v], acc[i][1][s][v]};
          else
            *dst = acc[i][0][s][v];
        }
      }
}

// channels per lane
int strips_pair(const ConvGeom &g) { return g.N % 2 == 0 && g.Cc % 2 == 0 ? 2 : 1; }

int strips_slots(const ConvGeom &g) { return strips_pair(g) == 2 ? 1024 : 2048; }

bool make_strips(const ConvGeom &g, int replicas, StripGeom &wg) {
  const int p = strips_pair(g);
  return strip_geom(g, replicas, 2, 32 * p, 32 * p, 3, strips_slots(g), wg);
}

}  // namespace

// Layers with so little to do that the generic kernel is at its shortest (four or five steps to a workgroup, 17 to 20 us with
// the sums of its splits), and a wavefront here walks eight rows or more, at half a microsecond each with nothing beside it
// to cover the loads.  Even channel counts only: odd ones cost the generic kernel 1.6 times as much.  us, generic / here, 20
// -> 20 channels, 128 images: 7 x 7 19.1 / 20.2, 10 x 10 19.7 / 22.2, 20 x 20 with stride 2 19.8 / 24.0; 4 x 32 images, 50 -> 50,
// 7 x 7 with stride 2 17.6 / 20.4; but 16 images of 20 channels, 7 x 7, seven rows 19.2 / 16.0, and more workgroups, 64 images
// of 7 x 7, 250 -> 130, 52.3 / 33.6.
bool generic_is_shorter(const ConvGeom &g, int replicas, StripGeom &wg) {
  if (strips_pair(g) != 2) return false;
  const int tn = g.N <= 32 ? 32 : g.N <= 64 ? 64 : g.N % 96 == 0 || g.N <= 96 ? 96 : 128;
  // 128 x 128 tiles are no shorter at stride 1 (32 -> 250 on 8 x 8, 3 x 29 images, 25.2 / 19.2), nor several of them (50 -> 320 on
  // 12 x 12 with stride 2, 31.3 / 26.1; 250 -> 130 on 7 x 7 with stride 2, 16 images, 19.0 / 22.0)
  if (tn > 64 && (g.sp == 1 || g.N > 256)) return false;
  const GenericSplit s = generic_split(g, replicas, tn, 128);
  if (s.steps > 5 || s.groups > (tn == 32 ? 512 : 256)) return false;
  split_strips(g, replicas, strips_slots(g), 260, wg);
  return wg.pps * wg.PC >= 8;
}

bool wgrad_strips_applicable(int dtype, int replicas, const ConvGeom &g) {
  StripGeom wg;
  return dtype == 1 && g.Cc >= 16 && g.N >= 16 && make_strips(g, replicas, wg) && !generic_is_shorter(g, replicas, wg);
}

int wgrad_strips_plan(int replicas, const ConvGeom &g, int *chunk_out) {
  StripGeom wg;
  make_strips(g, replicas, wg);
  split_strips(g, replicas, strips_slots(g), strips_pair(g) == 2 ? 260 : 200, wg);
  if (chunk_out) *chunk_out = wg.pps * 32;
  return wg.splits;
}

hipError_t launch_wgrad_strips(hipStream_t st, int replicas, const ConvGeom &g, const WgradIO &io) {
  StripGeom wg;
  if (io.with_bias || !make_strips(g, replicas, wg)) return hipErrorInvalidValue;
  if (strips_pair(g) == 2 && !(io.pairA && io.pairB)) return hipErrorInvalidValue;  // loads pairs of channels
  wg.pps = io.chunk / 32, wg.splits = io.splits;
  if (wg.pps < 1 || (long long)wg.pps * wg.splits < wg.pairs) return hipErrorInvalidValue;
  const dim3 grid(strip_blocks(wg), 1, replicas);
#define STRIPS_LAUNCH(PV, SPV) hipLaunchKernelGGL((k_wgrad_strips<PV, 3, SPV>), grid, dim3(64), 0, st, g, io, wg)
  if (strips_pair(g) == 2) {
    if (g.sp == 2)
      STRIPS_LAUNCH(2, 2);
    else
      STRIPS_LAUNCH(2, 1);
  } else {
    if (g.sp == 2)
      STRIPS_LAUNCH(1, 2);
    else
      STRIPS_LAUNCH(1, 1);
  }
#undef STRIPS_LAUNCH
  return hipGetLastError();
}
