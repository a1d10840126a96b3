// Backward-data of a stride-1 convolution with few input channels under a wide window, fp32 (LeNet's second
// convolution: 20 channels, 5 x 5 taps, 8 x 8 outputs), one image per workgroup, in ONE kernel:
//
//   col[m][(r, s, ci)] = sum_n dy[m][n] * w[n][r][s][ci]          a plain matrix product over the output channels
//   dx[h][w][ci]       = sum_{r, s} col[(h + pad - r, w + pad - s)][(r, s, ci)]
//
// As a direct implicit GEMM the pass has Cin = 20 of 32 MFMA columns in use and a contraction of R*S*Cout (the row
// kernel of igemm_f32.hip: LeNet's step 365 us against 314 here); as two kernels (the product, then the gather over the
// window) every entry of col travels to memory and back, 100 MB for the layer above.  Here col of ONE image never
// leaves LDS, 128 columns at a time: four pairs of wavefronts multiply 32 columns each (a row tile per wavefront) with
// the weights read straight from memory into MFMA fragments - as they lie, [Cout][R*S*Cin], they are the [K][N]
// operand, so the 32 lanes of a fragment half read 32 consecutive floats - park the product in LDS, and every thread
// adds the taps that lie in those columns to its elements of dx, which stay in LDS until the last columns are through.
// A chunk's weights travel while the one before is gathered.  With 34 KB for the columns and dx beside them (11 KB for
// that layer) two workgroups share a compute unit, one's products over the other's gather.  The product is the six
// products of bf16 parts of igemm_f32.hip; dy is split once, into registers, and serves every column.
// Bound by the vector work of the gather and of the splits, and by an image's chain of phases.  The layer above, against
// the whole of col at once in 125 KB, one workgroup per compute unit, fp32 MFMA: 128 / 384 / 768 images 17.7 / 35.7 /
// 56.7 -> 17.3 / 26.7 / 42.2 us, error against 64 bits 1.5e-7 -> 0.9e-7.  Four wavefronts with both row tiles each
// split the weights once instead of twice, but an image then takes longer: 1 us more at 128 and at 768 images.
#include "igemm_dev.h"
#include "igemm_split.h"

namespace {

using namespace igemm_dev;

constexpr int kWinThreads = 512;
constexpr int kWinMaxPix = 64;    // output pixels of an image: two 32-row MFMA tiles
constexpr int kWinMaxCout = 64;   // contraction length
constexpr int kWinLdsBytes = 160 * 1024;
constexpr int kDxCols = 128;              // columns of col in LDS: 32 per wavefront
constexpr int kDxPitch = kDxCols + 4;     // floats; the spare four of row 0 hold zeros for taps outside the image
constexpr int kDxDyPitch = kWinMaxCout + 4;  // of the dy tile, which lies there first

struct WinGeom {
  int B, H, W, Cin, Cout, R, pad, P, Q;  // dx [B][H][W][Cin], dy [B][P][Q][Cout]
  int NC;                                // R*R*Cin: columns of col
  int vec;                               // channels the gather takes at a time: 4, 2 or 1
  FastDiv dCin, dW, dCv, dR;             // no integer division on the device (dCv: vectors of a pixel)
};

// V elements of dx in plain fp32, a tap's products added up first as in the kernel: for results that split products do not
// give (see igemm_split.h).
template <int V>
__device__ __forceinline__ void plain_dx(const WinGeom &g, const float *dy, const float *w, int hh, int ww, int c, float (&sum)[V]) {
  typedef float fu __attribute__((ext_vector_type(V), aligned(4)));
  for (int r = 0; r < g.R; ++r)
    for (int s = 0; s < g.R; ++s) {
      const int p = hh + g.pad - r, q = ww + g.pad - s;
      if ((unsigned)p >= (unsigned)g.P || (unsigned)q >= (unsigned)g.Q) continue;
      const float *wt = w + (r * g.R + s) * g.Cin + c, *dt = dy + (p * g.Q + q) * g.Cout;
      float tap[V] = {};
#pragma unroll 8
      for (int n = 0; n < g.Cout; ++n) {
        const fu wv = *(const fu *)(wt + n * g.NC);  // Cout * NC < 2^22
        const float d = dt[n];
#pragma unroll
        for (int e = 0; e < V; ++e) tap[e] = fmaf(d, wv[e], tap[e]);
      }
#pragma unroll
      for (int e = 0; e < V; ++e) sum[e] += tap[e];
    }
}

// V: consecutive channels a thread gathers at a time (4, 2 or 1)
template <int V>
__global__ __launch_bounds__(kWinThreads, 4) void k_dgrad_window(const WinGeom g, const float *__restrict__ dy, long long dy_rs,
                                                             const float *__restrict__ w, long long w_rs,
                                                             const float *__restrict__ mask, long long mask_rs,
                                                             int accumulate, float *__restrict__ dx, long long dx_rs) {
  typedef float fv __attribute__((ext_vector_type(V)));
  constexpr int KS = kWinMaxCout / 16, NW = kWinThreads / 64, DI = kWinMaxPix / NW;
  extern __shared__ __attribute__((aligned(16))) float win_lds[];
  float *colS = win_lds;                        // [64][kDxPitch]; the dy tile before that
  float *dxS = win_lds + kWinMaxPix * kDxPitch;  // [H*W*Cin]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wc = wave & 3;
  const int b = blockIdx.x, rep = blockIdx.y;
  const int PQ = g.P * g.Q, ks_n = (g.Cout + 15) / 16;
  const int row0 = wave >> 2 << 5;  // this wavefront's rows of col; none of them may be in use
  const bool rows = row0 < PQ;
  const int r32 = lane & 31, h = lane >> 5;
  const float *dyp = dy + rep * dy_rs + (long long)b * PQ * g.Cout;
  const __amdgpu_buffer_rsrc_t w_rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void *)(w + rep * w_rs), 0, g.Cout * g.NC * 4, 0x00020000);

  // weights of one chunk: rows (output channels) 16 ks + 8 h + j of column c0 + 32 wc + r32; zero beyond either end
  float wraw[KS][8];
  auto load_w = [&](int c0) {
    const int col = c0 + wc * 32 + r32;
    const uint32_t first = col < g.NC ? (uint32_t)((8 * h * g.NC + col) * 4) : kOobOffset;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      if (ks < ks_n) {
#pragma unroll
        for (int j = 0; j < 8; ++j)  // a row beyond Cout lies beyond the buffer
          wraw[ks][j] = __uint_as_float(
              __builtin_amdgcn_raw_buffer_load_b32(w_rsrc, first + (uint32_t)((16 * ks + j) * g.NC * 4), 0, 0));
      }
  };
  {
    float t[DI];
#pragma unroll
    for (int i = 0; i < DI; ++i) {
      const int m = wave + NW * i;
      t[i] = lane < g.Cout && m < PQ ? dyp[m * g.Cout + lane] : 0.f;
    }
    load_w(0);
#pragma unroll
    for (int i = 0; i < DI; ++i) colS[(wave + NW * i) * kDxDyPitch + lane] = t[i];
  }
  __syncthreads();
  u4 a[KS][3];  // dy's parts: row row0 + r32, output channels 16 ks + 8 h ..
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    if (ks < ks_n) {
      const float *src = colS + (row0 + r32) * kDxDyPitch + 16 * ks + 8 * h;
      const f4 v0 = *(const f4 *)src, v1 = *(const f4 *)(src + 4);
      const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
      uint32_t p[3][4];
      split_words<8>(v, p);
#pragma unroll
      for (int q = 0; q < 3; ++q) a[ks][q] = u4{p[q][0], p[q][1], p[q][2], p[q][3]};
    }
  __syncthreads();  // the dy tile is dead
  if (tid < 4) colS[kDxCols + tid] = 0.f;

  const int total = g.H * g.W * g.Cin;
  const long long img = (long long)b * total;
  const float *mp = mask ? mask + rep * mask_rs + img : nullptr;
  float *op = dx + rep * dx_rs + img;
  auto finish = [&](int i, fv sum) {
    if (mp) {
      const fv mv = *(const fv *)&mp[i * V];
#pragma unroll
      for (int e = 0; e < V; ++e) sum[e] = mv[e] > 0.f ? sum[e] : 0.f;
    }
    if (accumulate) sum += *(const fv *)&op[i * V];
    *(fv *)&op[i * V] = sum;
  };
  bool left = false;
  const int taps = g.R * g.R;
  for (int c0 = 0; c0 < g.NC; c0 += kDxCols) {
    if (rows) {
      f16v hi, lo;
#pragma unroll
      for (int v = 0; v < 16; ++v) hi[v] = 0.f, lo[v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        if (ks < ks_n) {
          uint32_t p[3][4];
          split_words<8>(wraw[ks], p);
          u4 bw[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) bw[q] = u4{p[q][0], p[q][1], p[q][2], p[q][3]};
          mma<bf16_t>(a[ks][0], bw[2], lo);
          mma<bf16_t>(a[ks][2], bw[0], lo);
          mma<bf16_t>(a[ks][1], bw[1], lo);
          mma<bf16_t>(a[ks][0], bw[1], lo);
          mma<bf16_t>(a[ks][1], bw[0], lo);
          mma<bf16_t>(a[ks][0], bw[0], hi);
        }
      // accumulator v of a lane: row 8*(v/4) + 4*h + v%4 of its row tile, column r32 of the wavefront's columns
#pragma unroll
      for (int v = 0; v < 16; ++v)
        colS[(row0 + 8 * (v >> 2) + 4 * h + (v & 3)) * kDxPitch + wc * 32 + r32] = hi[v] + lo[v];
    }
    __syncthreads();
    const bool last = c0 + kDxCols >= g.NC;
    if (!last) load_w(c0 + kDxCols);

    // gather over the taps of these columns, in order
    for (int i = tid; i < total / V; i += kWinThreads) {
      const int pix = (int)fdiv((uint32_t)i, g.dCv), c = i * V - pix * g.Cin;
      const int hh = (int)fdiv((uint32_t)pix, g.dW), ww = pix - hh * g.W;
      const int t0 = (int)fdiv((uint32_t)max(c0 - c + g.Cin - 1, 0), g.dCin);
      const int t1 = min(taps, (int)fdiv((uint32_t)max(c0 + kDxCols - c + g.Cin - 1, 0), g.dCin));
      int p = (int)fdiv((uint32_t)t0, g.dR), q = t0 - p * g.R;
      p = hh + g.pad - p, q = ww + g.pad - q;
      const int q_lo = ww + g.pad - g.R;  // where a window row's taps end
      int col = t0 * g.Cin + c - c0;
      fv sum = {};
      if (c0) sum = *(const fv *)&dxS[i * V];
      for (int t = t0; t < t1; t += 4) {
        fv part[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bool ok = t + u < t1 && (unsigned)p < (unsigned)g.P && (unsigned)q < (unsigned)g.Q;
          part[u] = *(const fv *)&colS[ok ? (p * g.Q + q) * kDxPitch + col : kDxCols];
          col += g.Cin;
          if (--q == q_lo) q += g.R, --p;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) sum += part[u];
      }
      if (!last) {
        *(fv *)&dxS[i * V] = sum;
        continue;
      }
      bool odd = false;
#pragma unroll
      for (int e = 0; e < V; ++e) odd |= out_of_split_range(sum[e]);
      dxS[i * V] = odd ? 1.f : 0.f;  // left for plain fp32, after the loop: here it would cost the loop registers
      left |= odd;
      if (!odd) finish(i, sum);
    }
    if (!last) __syncthreads();  // the next columns replace these
  }
  if (__builtin_expect(!left, 1)) return;
  for (int i = tid; i < total / V; i += kWinThreads) {
    if (dxS[i * V] == 0.f) continue;
    const int pix = i * V / g.Cin, c = i * V - pix * g.Cin, hh = pix / g.W, ww = pix - hh * g.W;
    float sum[V] = {};
    plain_dx<V>(g, dyp, w + rep * w_rs, hh, ww, c, sum);
    fv out;
#pragma unroll
    for (int e = 0; e < V; ++e) out[e] = sum[e];
    finish(i, out);
  }
}

size_t dx_lds_bytes(const WinGeom &g) { return ((size_t)kWinMaxPix * kDxPitch + (size_t)g.H * g.W * g.Cin) * sizeof(float); }

// an image of at most 64 output pixels and 64 output channels, whose col would fit LDS (beyond, the window is so wide or the
// channels so many that a direct contraction has full columns to work on) and whose dx fits beside a chunk
bool make_win_geom(int B, int H, int W, int Cin, int Cout, int R, int pad, WinGeom &g) {
  g.B = B, g.H = H, g.W = W, g.Cin = Cin, g.Cout = Cout, g.R = R, g.pad = pad;
  g.P = H + 2 * pad - R + 1, g.Q = W + 2 * pad - R + 1;
  if (g.P < 1 || g.Q < 1 || g.P * g.Q > kWinMaxPix || Cout > kWinMaxCout || Cout < 1) return false;
  if ((long long)B * H * W * Cin >= (1LL << 31) || (long long)R * R * Cin > kWinLdsBytes / 4) return false;
  g.NC = R * R * Cin;
  g.vec = Cin % 4 == 0 ? 4 : Cin % 2 == 0 ? 2 : 1;
  g.dCin = make_fastdiv(Cin), g.dW = make_fastdiv(W), g.dR = make_fastdiv(R);
  g.dCv = make_fastdiv(Cin / g.vec);
  const long long col = ((long long)kWinMaxPix * ((Cout + 7) / 8 * 8 + 4) + (long long)g.P * g.Q * (g.NC + (g.vec == 4 ? 4 : 1))) * 4;
  return col <= kWinLdsBytes && dx_lds_bytes(g) <= kWinLdsBytes;
}

}  // namespace

bool dgrad_window_applicable(int dtype, int B, int H, int W, int Cin, int Cout, int R, int stride, int pad) {
  // A tap of 56 channels or more under a 3 x 3 window leaves two taps to a chunk of columns, and with few output channels the
  // products are short beside what the gather spends on each chunk: the row kernel of igemm_f32.hip is ahead.  us, this / row
  // kernel with its weight transpose, 7 x 7: 64 -> 16 channels, 16 images 12.6 / 9.5, 1000 32 / 17.9; 64 -> 32 14.7 / 13.0 and
  // 40 / 24; but 64 -> 50 18.5 / 21.5, 32 -> 32 8.3 / 12.9.
  if (R == 3 && Cin >= 56 && Cout >= 8 && Cout <= 32) return false;
  WinGeom g;
  return dtype == 0 && stride == 1 && R > 1 && B >= 1 && B <= 65535 && make_win_geom(B, H, W, Cin, Cout, R, pad, g);
}

hipError_t launch_dgrad_window(hipStream_t st, int n, int B, int H, int W, int Cin, int Cout, int R, int pad,
                               const float *dy, long long dy_rs, const float *w, long long w_rs,
                               const float *mask, long long mask_rs, int accumulate, float *dx, long long dx_rs) {
  WinGeom g;
  if (!make_win_geom(B, H, W, Cin, Cout, R, pad, g) || n < 1 || n > 65535 || B > 65535) return hipErrorInvalidValue;
  if (!aligned_to(dy, 16)) return hipErrorInvalidValue;
  const size_t lds = dx_lds_bytes(g);
  static bool raised = false;   // more than 64 KB of dynamic LDS has to be asked for once
  if (!raised) {
    for (const void *f : {(const void *)k_dgrad_window<4>, (const void *)k_dgrad_window<2>, (const void *)k_dgrad_window<1>}) {
      const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kWinLdsBytes);
      if (e != hipSuccess) return e;
    }
    raised = true;
  }
  const auto kernel = g.vec == 4 ? k_dgrad_window<4> : g.vec == 2 ? k_dgrad_window<2> : k_dgrad_window<1>;
  hipLaunchKernelGGL(kernel, dim3(B, n), dim3(kWinThreads), lds, st, g, dy, dy_rs, w, w_rs, mask, mask_rs, accumulate, dx,
                     dx_rs);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Backward-weight of the same kind of layer (fp32, stride 1, images of at most 64 output pixels) with fewer than 12 input
// channels or a 2 x 2 window (the register kernel of igemm_f32_wgrad.hip takes the others), the window gather done in LDS:
//   dW[n][(r, s, ci)] = sum over images and output pixels m of dy[m][n] * x[m + (r, s)][ci].
// A workgroup takes a few images one after the other; per image the input patch (12 x 12 x 8 floats, say) and the dy
// tile lie in LDS, and both MFMA operands are read from there element by element: the (tap, channel) column of a lane
// is a fixed offset into the patch, the pixel a wavefront-uniform base.  In the generic kernel the same gather runs
// against global memory, once per tap and input element.  Eight wavefronts own
// the 2 x 16 tiles of 32 x 32 outputs (two column tiles and both row tiles each); the partial sums of the
// workgroups are added by the fixed-order reduction every split backward-weight kernel uses.
// ---------------------------------------------------------------------------------------------
namespace {

constexpr int kWgwMaxPatch = 6144;  // floats of one padded input patch

struct WgWinGeom {
  int B, H, W, Cin, Cout, R, pad, P, Q, NC;
  int Hp, Wp;       // padded patch
  int ipw;          // images per workgroup
  int lda;          // pitch of the dy tile
  FastDiv dQ, dCin, dR, dW, dCout;
};

__global__ __launch_bounds__(kWinThreads) void k_wgrad_window(const WgWinGeom g, const float *__restrict__ dy,
                                                              long long dy_rs, const float *__restrict__ x,
                                                              long long x_rs, float *__restrict__ out, long long out_rs,
                                                              long long split_stride) {
  __shared__ __attribute__((aligned(16))) float xS[kWgwMaxPatch];
  __shared__ __attribute__((aligned(16))) float dyS[kWinMaxPix * (kWinMaxCout + 4)];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int split = blockIdx.x, rep = blockIdx.y;
  const int PQ = g.P * g.Q, patch = g.Hp * g.Wp * g.Cin, img_x = g.H * g.W * g.Cin;
  const int b_begin = split * g.ipw, b_end = min(g.B, b_begin + g.ipw);
  const float *xp = x + rep * x_rs, *dyp = dy + rep * dy_rs;
  const int r = lane & 31, h = lane >> 5;

  // this lane's two columns (tap, channel): offset into the patch from the pixel's window origin
  int off[2];
  bool ok[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int col = (2 * wave + t) * 32 + r;
    ok[t] = col < g.NC;
    const int tapi = (int)fdiv((uint32_t)(ok[t] ? col : 0), g.dCin), ci = (ok[t] ? col : 0) - tapi * g.Cin;
    const int dr = (int)fdiv((uint32_t)tapi, g.dR), ds = tapi - dr * g.R;
    off[t] = (dr * g.Wp + ds) * g.Cin + ci;
  }
  f16v acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][t][v] = 0.f;

  // zero once: the patch border (padding) and the rows / columns of the dy tile beyond the image stay zero
  for (int i = tid; i < patch; i += kWinThreads) xS[i] = 0.f;
  for (int i = tid; i < kWinMaxPix * g.lda; i += kWinThreads) dyS[i] = 0.f;

  constexpr int XI = (kWgwMaxPatch + kWinThreads - 1) / kWinThreads, DI = (kWinMaxPix * kWinMaxCout) / kWinThreads;
  float xr[XI], dr_[DI];
  auto load_img = [&](int b) {   // global -> registers (both tensors are contiguous per image)
    const float *xi = xp + (long long)b * img_x, *di = dyp + (long long)b * PQ * g.Cout;
#pragma unroll
    for (int u = 0; u < XI; ++u) {
      const int i = u * kWinThreads + tid;
      xr[u] = (b < b_end && i < img_x) ? xi[i] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < DI; ++u) {
      const int i = u * kWinThreads + tid;
      dr_[u] = (b < b_end && i < PQ * g.Cout) ? di[i] : 0.f;
    }
  };
  auto store_img = [&]() {
#pragma unroll
    for (int u = 0; u < XI; ++u) {
      const int i = u * kWinThreads + tid;
      if (i < img_x) {
        const int pix = (int)fdiv((uint32_t)i, g.dCin), ci = i - pix * g.Cin;
        const int hh = (int)fdiv((uint32_t)pix, g.dW), ww = pix - hh * g.W;
        xS[((hh + g.pad) * g.Wp + ww + g.pad) * g.Cin + ci] = xr[u];
      }
    }
#pragma unroll
    for (int u = 0; u < DI; ++u) {
      const int i = u * kWinThreads + tid;
      if (i < PQ * g.Cout) {
        const int m = (int)fdiv((uint32_t)i, g.dCout), k = i - m * g.Cout;
        dyS[m * g.lda + k] = dr_[u];
      }
    }
  };

  load_img(b_begin);
  for (int b = b_begin; b < b_end; ++b) {
    __syncthreads();  // the previous image has been multiplied (first trip: the zeros are in place)
    store_img();
    __syncthreads();
    load_img(b + 1);
    for (int q = 0; q < (PQ + 7) / 8; ++q) {
      // fragment element j of half h: pixel m = 8q + 4h + j (pixels beyond the image meet zero rows of dy)
      u4 af[2], bf[2];
      float av[2][4], bv[2][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int m = 8 * q + 4 * h + j, mc = m < PQ ? m : PQ - 1;
        const int p = (int)fdiv((uint32_t)mc, g.dQ), qq = mc - p * g.Q;
        const int base = (p * g.Wp + qq) * g.Cin;
#pragma unroll
        for (int a = 0; a < 2; ++a) av[a][j] = dyS[m * g.lda + a * 32 + r];
#pragma unroll
        for (int t = 0; t < 2; ++t) bv[t][j] = ok[t] ? xS[base + off[t]] : 0.f;
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
        af[a] = u4{__float_as_uint(av[a][0]), __float_as_uint(av[a][1]), __float_as_uint(av[a][2]), __float_as_uint(av[a][3])};
#pragma unroll
      for (int t = 0; t < 2; ++t)
        bf[t] = u4{__float_as_uint(bv[t][0]), __float_as_uint(bv[t][1]), __float_as_uint(bv[t][2]), __float_as_uint(bv[t][3])};
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int t = 0; t < 2; ++t) mma<float>(af[a], bf[t], acc[a][t]);
    }
  }
  // accumulator v of a lane: row (output channel) 8*(v/4) + 4*h + v%4 of its row tile, column r of its column tile
  float *op = out + rep * out_rs + split * split_stride;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int col = (2 * wave + t) * 32 + r;
      if (col >= g.NC) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int n = a * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
        if (n < g.Cout) op[(long long)n * g.NC + col] = acc[a][t][v];
      }
    }
}

bool make_wgwin_geom(const ConvGeom &cg, WgWinGeom &g) {
  if (cg.sp != 1 || cg.sr != 1 || cg.dshift != 0 || cg.R != cg.S || cg.R < 2) return false;
  const int PQ = cg.P * cg.Q;
  if (PQ > kWinMaxPix || PQ % 8 != 0 || cg.N > kWinMaxCout || cg.M % PQ != 0) return false;
  g.B = cg.M / PQ, g.H = cg.Hin, g.W = cg.Win, g.Cin = cg.Cc, g.Cout = cg.N, g.R = cg.R, g.pad = -cg.off;
  g.P = cg.P, g.Q = cg.Q, g.NC = cg.K;
  if (g.pad < 0 || g.NC > 512 || g.NC < 128) return false;
  g.Hp = g.H + 2 * g.pad, g.Wp = g.W + 2 * g.pad;
  if ((long long)g.Hp * g.Wp * g.Cin > kWgwMaxPatch) return false;
  g.lda = kWinMaxCout + 4;
  g.dQ = make_fastdiv(g.Q), g.dCin = make_fastdiv(g.Cin), g.dR = make_fastdiv(g.R), g.dW = make_fastdiv(g.W);
  g.dCout = make_fastdiv(g.Cout);
  return true;
}

// images per workgroup: about one workgroup per compute unit, rows per split a multiple of 32
int wgwin_images_per_wg(const WgWinGeom &g, int replicas) {
  int ipw = (int)(((long long)g.B * replicas + 255) / 256);
  if (ipw < 1) ipw = 1;
  while ((ipw * g.P * g.Q) % 32 != 0) ++ipw;
  return ipw;
}

}  // namespace

bool wgrad_window_applicable(int dtype, const ConvGeom &g) {
  WgWinGeom wg;
  return dtype == 0 && make_wgwin_geom(g, wg);
}

int wgrad_window_plan(int replicas, const ConvGeom &g, int *chunk_out) {
  WgWinGeom wg;
  make_wgwin_geom(g, wg);
  const int ipw = wgwin_images_per_wg(wg, replicas);
  if (chunk_out) *chunk_out = ipw * wg.P * wg.Q;
  return (wg.B + ipw - 1) / ipw;
}

hipError_t launch_wgrad_window(hipStream_t st, int replicas, const ConvGeom &g, const WgradIO &io) {
  WgWinGeom wg;
  if (!make_wgwin_geom(g, wg)) return hipErrorInvalidValue;
  const int PQ = wg.P * wg.Q;
  if (io.chunk % PQ != 0 || io.chunk < PQ) return hipErrorInvalidValue;
  wg.ipw = io.chunk / PQ;
  if ((long long)wg.ipw * io.splits < wg.B) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_wgrad_window, dim3(io.splits, replicas), dim3(kWinThreads), 0, st, wg, (const float *)io.dy, io.dy_rs,
                     (const float *)io.x, io.x_rs, io.out, io.out_rs, io.split_stride);
  return hipGetLastError();
}
