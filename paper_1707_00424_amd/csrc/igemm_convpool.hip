// A first layer (fp32, window of at most 31 values, at most 32 output channels) with bias, ReLU and the 2 x 2 max-pool behind it in
// one kernel, and its weight gradient from the pooled gradient (LeNet's first convolution: 5 x 5 on 28 x 28 x 1 to 20 channels).
//
// As three operations such a block is bound by what it writes and reads again: six replicas of 128 images make 35 MB of
// convolution outputs, which the pool reads (forward 26 + 9.7 us), whose gradient the pool's backward pass writes and the weight
// gradient reads (25 to 31 + 29.6 us); the images are 2.4 MB and the pooled outputs 8.8.  Here an image lies in LDS (3 KB), a
// wavefront takes eight windows of four outputs at a time, and the maximum of a window is taken between the four lanes that
// hold it.  What is kept for the backward pass is one byte per pooled value: which of the four it was, or that it has no
// gradient.  A matrix instruction (32 x 32 x 2) reads one value of LDS per lane, weights stay in registers.  us, before -> now:
// forward 36 -> 18, backward 55 -> 19 (alone), LeNet's step 313 -> 265.  Matrix work is 5 us in each direction; the rest goes on
// vector work (45 instructions per four windows' maxima and 32 channels' group) and on a workgroup's start and end.
#include "igemm_dev.h"

namespace {

using namespace igemm_dev;

constexpr int kTaps = 32;      // window values of a matrix tile
constexpr int kNoGrad = 4;     // code of a window whose maximum the ReLU cut off
constexpr int kBatch = 4;      // values per thread requested at a time on their way to LDS

struct PoolGeom {
  int H, W, C, S;   // image, window side
  int N, K;         // output channels, window values
  int Q2, windows;  // pooled columns, pooled outputs of an image
  int image;        // values of an image
  int parts;        // workgroups that share an image: gridDim.z
  FastDiv dQ2;
  int off[kTaps];   // of a window value from the window's first pixel; 0 beyond the last
};

template <int CTRL>
__device__ __forceinline__ float quad(float v) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
constexpr int kXor1 = 0xb1, kXor2 = 0x4e;  // quad permutations [1 0 3 2] and [2 3 0 1]

constexpr int step_value(int i) { return 8 * (i / 4) + i % 4; }

// One workgroup per image, or several (blockIdx.z) that share its windows.  out, code: [window][N].
__global__ __launch_bounds__(kThreads) void k_convpool(const PoolGeom g, const float *__restrict__ x, long long x_rs, const float *__restrict__ w,
                                                       long long w_rs, const float *__restrict__ bias, long long bias_rs,
                                                       float *__restrict__ out, long long out_rs, unsigned char *__restrict__ code) {
  extern __shared__ __attribute__((aligned(16))) float img[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, n = lane & 31;
  const int b = blockIdx.x, rep = blockIdx.y;
  const float *xp = x + rep * x_rs + (long long)b * g.image;
  float *ws = img + g.image;
  // all loads of a batch are on their way before the first is waited for (a workgroup works for about 3 us, and each round of
  // requests costs it most of one; LeNet's step, here and in the weight gradient, 269.4 -> 265.0 us against one load at a time)
  for (int base = tid; base < max(g.image, g.N * g.K); base += kBatch * kThreads) {
    float xv[kBatch], wv[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = base + u * kThreads;
      xv[u] = i < g.image ? xp[i] : 0.f;
      wv[u] = i < g.N * g.K ? w[rep * w_rs + i] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = base + u * kThreads;
      if (i < g.image) img[i] = xv[u];
      if (i < g.N * g.K) ws[i] = wv[u];
    }
  }
  const int pos = lane & 3, chan = 8 * pos + 4 * h;
  float bv[4];  // of the channels that this lane stores
#pragma unroll
  for (int e = 0; e < 4; ++e) bv[e] = chan < g.N ? bias[rep * bias_rs + chan + e] : 0.f;
  __syncthreads();
  // Step i multiplies window values step_value(i) + 4 h: the order of sums of the convolution without a pool (k_conv_smallk), so
  // that the output of a window that is the largest there, be it by the last bit, is the largest here.
  float wr[kTaps / 2];
  int off[kTaps / 2];
#pragma unroll
  for (int i = 0; i < kTaps / 2; ++i) {
    const int k = step_value(i) + 4 * h;
    wr[i] = n < g.N && k < g.K ? ws[n * g.K + k] : 0.f;
    off[i] = h ? g.off[step_value(i) + 4] : g.off[step_value(i)];
  }
  float *op = out + rep * out_rs + (long long)b * g.windows * g.N;
  unsigned char *cp = code ? code + rep * out_rs + (long long)b * g.windows * g.N : nullptr;
  for (int first = (blockIdx.z * 4 + wave) * 8; first < g.windows; first += g.parts * 4 * 8) {
    const int win = first + (n >> 2), wc = min(win, g.windows - 1);
    const int ph = (int)fdiv((uint32_t)wc, g.dQ2), qw = wc - ph * g.Q2;
    const float *px = img + ((2 * ph + (pos >> 1)) * g.W + 2 * qw + (pos & 1)) * g.C;
    f16v acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int i = 0; i < kTaps / 2; ++i)
      if (step_value(i) < g.K) {
        float t = px[off[i]];
        if (step_value(i) + 4 >= g.K) t = h ? 0.f : t;  // that half of the step lies beyond the window
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[i], t, acc, 0, 0, 0);
      }
    // Lane: one output pixel, channels 8 * (v / 4) + 4 h + v % 4.  The four lanes of a window exchange registers until each has
    // all four pixels of the channel group that its position names, and takes the maximum, the first one of equals.
    float best[4];
    uint32_t codes = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float t[4] = {acc[e], acc[4 + e], acc[8 + e], acc[12 + e]};
      // groups 2 and 3 go to the lower pixels' lanes, groups 0 and 1 to the upper ones'; then odd and even likewise
      const bool hi = pos & 2, odd = pos & 1;
      const float s0 = quad<kXor2>(hi ? t[0] : t[2]), s1 = quad<kXor2>(hi ? t[1] : t[3]);
      const float k0 = hi ? t[2] : t[0], k1 = hi ? t[3] : t[1];  // own pixel, groups 2 * hi and + 1
      // pixels (own, two away): of the group that is kept, and of its neighbour, which goes to the lane beside
      const float p0 = odd ? k1 : k0, q0 = odd ? s1 : s0;
      const float p1 = quad<kXor1>(odd ? k0 : k1), q1 = quad<kXor1>(odd ? s0 : s1);
      // in order of position: own = pos, p1 = pos ^ 1, q0 = pos ^ 2, q1 = pos ^ 3
      const float u0 = odd ? p1 : p0, u1 = odd ? p0 : p1, u2 = odd ? q1 : q0, u3 = odd ? q0 : q1;
      // (the larger of NaN and 0 is 0, as it is behind the ReLU of a convolution)
      const float w0 = fmaxf((hi ? u2 : u0) + bv[e], 0.f), w1 = fmaxf((hi ? u3 : u1) + bv[e], 0.f), w2 = fmaxf((hi ? u0 : u2) + bv[e], 0.f),
                  w3 = fmaxf((hi ? u1 : u3) + bv[e], 0.f);
      const float m01 = fmaxf(w0, w1), m23 = fmaxf(w2, w3), m = fmaxf(m01, m23);
      const uint32_t at = m23 > m01 ? (w3 > w2 ? 3u : 2u) : (w1 > w0 ? 1u : 0u);
      best[e] = m;
      codes |= (m > 0.f ? at : (uint32_t)kNoGrad) << (8 * e);
    }
    if (win < g.windows && chan < g.N) {
      *(f4 *)&op[win * g.N + chan] = f4{best[0], best[1], best[2], best[3]};
      if (cp) *(uint32_t *)&cp[win * g.N + chan] = codes;
    }
  }
}

// Weight gradient, and the bias gradient behind it: dy is the gradient of the pooled output where it came from, zero elsewhere.
// A workgroup takes `per` images of a replica, its wavefronts every fourth row of windows, or several (blockIdx.z) share the rows
// of one image; a matrix instruction contracts two of a window's four pixels.  The window value behind the last is 1: its column is
// the sum of dy.
__global__ __launch_bounds__(kThreads) void k_convpool_wgrad(const PoolGeom g, int B, int per, const float *__restrict__ x, long long x_rs,
                                                             const float *__restrict__ dp, long long dp_rs, const unsigned char *__restrict__ code,
                                                             float *__restrict__ out, long long out_rs, long long split_stride) {
  extern __shared__ __attribute__((aligned(16))) float img[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, n = lane & 31;
  const int rep = blockIdx.y, first = blockIdx.x * per;
  const int pooled = g.windows * g.N;
  float *gr = img + (g.image + 3) / 4 * 4;
  unsigned char *cd = (unsigned char *)(gr + pooled);
  const int off = g.off[n], P2 = g.windows / g.Q2;
  const int nc = min(n, g.N - 1);  // rows of the result beyond the channels are not stored
  const float edge = n == g.K ? 1.f : 0.f;
  f16v acc, acc2;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f, acc2[v] = 0.f;
  const int b1 = min(B, first + per);
  for (int b = first; b < b1; ++b) {
    const float *xp = x + rep * x_rs + (long long)b * g.image, *dpp = dp + rep * dp_rs + (long long)b * pooled;
    const unsigned char *cp = code + rep * dp_rs + (long long)b * pooled;
    __syncthreads();  // the image before has been read
    for (int base = tid; base < max(g.image, pooled / 4); base += kBatch * kThreads) {
      float xv[kBatch];
      f4 gv[kBatch];
      uint32_t cv[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int i = base + u * kThreads;
        xv[u] = i < g.image ? xp[i] : 0.f;
        gv[u] = i < pooled / 4 ? ((const f4 *)dpp)[i] : f4{0.f, 0.f, 0.f, 0.f};
        cv[u] = i < pooled / 4 ? ((const uint32_t *)cp)[i] : 0u;
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int i = base + u * kThreads;
        if (i < g.image) img[i] = xv[u];
        if (i < pooled / 4) ((f4 *)gr)[i] = gv[u], ((uint32_t *)cd)[i] = cv[u];
      }
    }
    __syncthreads();
    for (int ph = blockIdx.z * 4 + wave; ph < P2; ph += g.parts * 4) {
      const float *px = img + (2 * ph * g.W + h) * g.C + off, *gp = gr + ph * g.Q2 * g.N + nc;
      const unsigned char *kp = cd + ph * g.Q2 * g.N + nc;
#pragma unroll 4
      for (int qw = 0; qw < g.Q2; ++qw) {
        const float v = gp[qw * g.N];
        const int c = kp[qw * g.N];
        const float x0 = n < g.K ? px[2 * qw * g.C] : edge, x1 = n < g.K ? px[(g.W + 2 * qw) * g.C] : edge;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(c == h ? v : 0.f, x0, acc, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(c == 2 + h ? v : 0.f, x1, acc2, 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] += acc2[v];
  // the wavefronts' sums are added in their order
  __syncthreads();
  float *sums = img;  // [3][64][16]
  if (wave) {
#pragma unroll
    for (int q = 0; q < 4; ++q) *(f4 *)&sums[((wave - 1) * 64 + lane) * 16 + q * 4] = f4{acc[q * 4], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]};
  }
  __syncthreads();
  if (wave) return;
#pragma unroll
  for (int w = 0; w < 3; ++w)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f4 t = *(const f4 *)&sums[(w * 64 + lane) * 16 + q * 4];
      acc[q * 4] += t.x, acc[q * 4 + 1] += t.y, acc[q * 4 + 2] += t.z, acc[q * 4 + 3] += t.w;
    }
  float *o = out + rep * out_rs + (blockIdx.x * g.parts + blockIdx.z) * split_stride;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int c = 8 * (v >> 2) + 4 * h + (v & 3);
    if (c >= g.N) continue;
    if (n < g.K) o[(long long)c * g.K + n] = acc[v];
    if (n == g.K) o[(long long)g.N * g.K + c] = acc[v];
  }
}

PoolGeom pool_geom(const ConvShape &c) {
  PoolGeom g{};
  g.H = c.H, g.W = c.W, g.C = c.Cin, g.S = c.R;
  g.N = c.Cout, g.K = c.R * c.R * c.Cin;
  g.Q2 = c.Wo() / 2, g.windows = (c.Ho() / 2) * g.Q2;
  g.image = c.H * c.W * c.Cin;
  g.dQ2 = make_fastdiv(g.Q2 > 0 ? g.Q2 : 1);
  for (int k = 0; k < kTaps && k < g.K; ++k) {
    const int rs = k / c.Cin, r = rs / c.R;
    g.off[k] = (r * c.W + rs - r * c.R) * c.Cin + k - rs * c.Cin;
  }
  return g;
}
size_t wgrad_lds(const PoolGeom &g) {
  const size_t operands = (size_t)((g.image + 3) / 4 * 4 + g.windows * g.N) * 4 + (size_t)g.windows * g.N, part = 3 * 64 * 16 * 4;
  return operands > part ? operands : part;
}

}  // namespace

bool convpool_applicable(int dtype, const ConvShape &c) {
  if (dtype != 0 || c.stride != 1 || c.pad != 0 || c.Cout > 32 || c.Cout % 4 != 0 || c.R * c.R * c.Cin >= kTaps || c.H < c.R || c.W < c.R) return false;
  const PoolGeom g = pool_geom(c);
  // three workgroups in the LDS of a compute unit, each under the limit that needs no attribute
  return g.windows >= 8 && c.B <= 65535 * 16 && wgrad_lds(g) <= 48 * 1024;
}

namespace {
constexpr int kResident = 768;  // three workgroups per compute unit

// Workgroups per image, where images alone are too few to fill the chip; the four wavefronts of one keep at least six of the
// `units` (groups of windows, rows) that they share.  us per LeNet step, one workgroup per image / this / three separate kernels:
// 32 images of 28 x 28, 5 x 5 window, 98 / 94 / 108; 4 images of 48 x 48, 3 x 3, 108 / 83 / 93; 32 of 64 x 64, 5 x 5, 179 / 117 / 136; 128 of
// 56 x 56, 231 / 200 / 222; an evaluation of 16 of 64 x 64 112 / 78 / 80.
int image_parts(int n, const ConvShape &c, int units) {
  const long long room = kResident / ((long long)n * c.B);
  const int most = units / 6;
  return (int)(room < 1 || most < 1 ? 1 : room < most ? room : most);
}
struct WgradSplits {
  int per, parts, splits;
};
WgradSplits wgrad_splits(int n, const ConvShape &c) {
  const int per = (int)(((long long)n * c.B + kResident - 1) / kResident), parts = per > 1 ? 1 : image_parts(n, c, c.Ho() / 2);
  return {per, parts, (c.B + per - 1) / per * parts};
}
}  // namespace

hipError_t launch_convpool(hipStream_t st, int n, const ConvShape &c, const float *x, long long x_rs, const float *w, long long w_rs, const float *bias,
                           long long bias_rs, float *out, unsigned char *code) {
  PoolGeom g = pool_geom(c);
  g.parts = image_parts(n, c, (g.windows + 7) / 8);
  hipLaunchKernelGGL(k_convpool, dim3(c.B, n, g.parts), dim3(kThreads), (size_t)(g.image + g.N * g.K) * 4, st, g, x, x_rs, w, w_rs, bias, bias_rs, out,
                     (long long)c.B * g.windows * g.N, code);
  return hipGetLastError();
}

int convpool_wgrad_splits(int n, const ConvShape &c) { return wgrad_splits(n, c).splits; }
hipError_t launch_convpool_wgrad(hipStream_t st, int n, const ConvShape &c, const float *x, long long x_rs, const float *dpooled, const unsigned char *code,
                                 float *out, long long out_rs, long long split_stride) {
  PoolGeom g = pool_geom(c);
  const WgradSplits s = wgrad_splits(n, c);
  g.parts = s.parts;
  hipLaunchKernelGGL(k_convpool_wgrad, dim3(s.splits / s.parts, n, s.parts), dim3(kThreads), wgrad_lds(g), st, g, c.B, s.per, x, x_rs, dpooled,
                     (long long)c.B * g.windows * g.N, code, out, out_rs, split_stride);
  return hipGetLastError();
}
