// fp32 plain products (fully connected layers and small 1 x 1 convolutions) with few output tiles: forward, input
// gradient and weight gradient from one kernel, without transposed weights.
//
//   out[i][j] = sum_k A(i, k) * B(k, j)
//     forward          i = row m of the batch, j = output channel,  k = input value;   A = x [i][k],   B = w  [j][k]
//     input gradient   i = row m,              j = input value,     k = output channel; A = dy [i][k],  B = w  [k][j]
//     weight gradient  i = output channel,     j = input value,     k = row m;          A = dy [k][i],  B = x  [k][j]
//
// What bounds such a layer is latency: 0.6 GFLOP and 12 MB for LeNet's 800 x 500 with six replicas, 4 us of fp32 MFMA
// on the whole chip, and a handful of tiles with a long contraction.  So a tile (32 x 32, or 16 x 16 where those
// would leave compute units empty) belongs to one workgroup whose wavefronts split the contraction, each with a
// batch of loads in flight ahead of the one it multiplies and no barrier.  An operand passes through a strip of LDS that
// is private to its wavefront and is fetched in whole cache lines: as fragments, 32 rows at 32 bytes each, an
// instruction touches 32 lines for a quarter of their bytes.  The strip keeps the layout of memory, and an operand whose
// contraction index is the slow one is read from it by columns, so no layout needs a transpose.
// The partial tiles meet in LDS and are added in wavefront order (fixed: results are reproducible), four columns per
// thread.  Six replicas of 128 x 800 x 500, forward + input gradient + weight gradient: 80 -> 50 us (the three kernels 21 +
// 36 with its weight transpose + 19 -> 13.5 + 17.5 + 14); three of 128 x 784 x 128 forward 14.7 -> 4.6 us, weight
// gradient 10.7 -> 4.6 us.
#include <algorithm>

#include "igemm_dev.h"

namespace {

using namespace igemm_dev;

struct FcArgs {
  const float *a, *b;
  float *out;
  const float *bias, *resid, *mask;
  float *bias_out;  // weight gradient: sum over k of A(i, k) goes here, or NULL
  long long a_rs, b_rs, o_rs, bias_rs, resid_rs, mask_rs, bias_out_rs;  // replica strides, elements
  int lda, ldb, ldo;
  int I, J, K;
  int a_bytes, b_bytes;      // one replica's operand: range of the buffer loads
  int relu, accumulate;
  int vec_a, vec_b, vec_out;  // 16-byte operand loads (rows of whole vectors) / result accesses allowed
  int small;                  // a part of a group: tiles of 16 x 16
  long long p_off;            // ... where `out` begins in a parameter row
};

constexpr int kFcBatch = 32;  // contraction values per batch of loads: 128 bytes of a row

template <int TS>
struct Mfma32;
template <>
struct Mfma32<32> {
  typedef f16v Acc;
  static constexpr int kVals = 16;
  static __device__ __forceinline__ Acc mma1(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }
};
template <>
struct Mfma32<16> {
  typedef f4 Acc;
  static constexpr int kVals = 4;
  static __device__ __forceinline__ Acc mma1(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};

// A staged batch: [row][k] of an operand whose k is contiguous, [k][column] of one whose k is the slow index.  Pitches:
// 16-byte reads of consecutive rows hit distinct banks; dword reads of two groups four rows apart do too.
template <int TS, bool SLOW>
constexpr int kFcPitch = SLOW ? TS + 8 : kFcBatch + 4;
template <int TS, bool SLOW>
constexpr int kFcStaged = (SLOW ? kFcBatch : TS) * kFcPitch<TS, SLOW>;
// LDS of a workgroup in floats: a staged batch of both operands per wavefront, sums over k of A
template <int TS, bool A_SLOW, bool B_SLOW, int KS, int NJ>
constexpr int kFcLds = NJ * KS * (kFcStaged<TS, A_SLOW> + kFcStaged<TS, B_SLOW>)+KS * TS;

// TS: tile side.  KS wavefronts split the contraction of a tile, NJ tiles side by side per workgroup, which is number bx of
// row by of tiles of replica `rep`.
// UPDATE: the parameters that the result is the gradient of are updated as well.
template <int TS, bool A_SLOW, bool B_SLOW, int KS, int NJ, bool UPDATE = false>
__device__ __forceinline__ void fc_tile(const FcArgs &g, float *smem, const int bx, const int by, const int rep, const InnerState *st = nullptr) {
  typedef Mfma32<TS> M;
  constexpr int KG = 64 / TS;        // lanes that share a row hold KG groups of four consecutive k
  constexpr int STEP = 4 * KG;       // contraction values per step (four MFMAs)
  constexpr int U = kFcBatch / STEP;  // steps per batch of loads
  constexpr int V = TS / 8;           // 16-byte vectors per lane, operand and batch
  constexpr int LDC = kFcPitch<TS, false>, LDS = kFcPitch<TS, true>;
  constexpr int kStagedA = kFcStaged<TS, A_SLOW>, kStagedB = kFcStaged<TS, B_SLOW>;
  constexpr int LD = TS + 4;          // pitch of a partial tile, which takes the place of the staged operands
  static_assert(kStagedA + kStagedB >= TS * LD, "a partial tile has to fit");
  float(*lds)[KS][kStagedA + kStagedB] = reinterpret_cast<float(*)[KS][kStagedA + kStagedB]>(smem);
  float(*bpart)[TS] = reinterpret_cast<float(*)[TS]>(smem + NJ * KS * (kStagedA + kStagedB));

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kw = wave % KS, jw = wave / KS;
  const int i0 = by * TS, j0 = (bx * NJ + jw) * TS;
  const int rl = lane % TS, kg = lane / TS;
  const __amdgpu_buffer_rsrc_t a_rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void *)(g.a + rep * g.a_rs), 0, g.a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t b_rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void *)(g.b + rep * g.b_rs), 0, g.b_bytes, 0x00020000);

  // this wavefront's share of the contraction, in whole batches
  const int batches = (g.K + kFcBatch - 1) / kFcBatch, per = (batches + KS - 1) / KS;
  const int n_begin = kw * per, n_end = min(batches, n_begin + per);

  // batch n of an operand -> V vectors per lane, in memory order: rows of 32 k values (eight lanes on 128 bytes), or 32
  // rows k of TS columns.  What changes with the batch is the scalar offset of the load, so that a load costs no vector
  // instructions beside its own: with an address and a bounds check each, those took as long as the MFMAs.  Slow rows
  // beyond K lie beyond the buffer (zeros); contiguous vectors beyond K are cut off in the last batch.  Columns beyond
  // the operand only feed results that are not stored.
  uint32_t va[V], vb[V];
  auto base = [&](bool slow, int ld, int x0, int lim, uint32_t (&v)[V]) {
#pragma unroll
    for (int it = 0; it < V; ++it) {
      if (slow) {
        const int c = x0 + 4 * (lane % (TS / 4));
        v[it] = c < lim ? (uint32_t)((it * (256 / TS) + lane / (TS / 4)) * ld + c) * 4u : kOobOffset;
      } else {
        const int idx = x0 + 8 * it + (lane >> 3);
        v[it] = idx < lim ? (uint32_t)(idx * ld + 4 * (lane & 7)) * 4u : kOobOffset;
      }
    }
  };
  base(A_SLOW, g.lda, i0, g.I, va);
  base(B_SLOW, g.ldb, j0, g.J, vb);
  auto load = [&](bool slow, bool vec, __amdgpu_buffer_rsrc_t rsrc, int ld, int x0, int lim, const uint32_t (&v)[V], int n,
                  u4 (&r)[V]) {
    const int step = n * kFcBatch * 4 * (slow ? ld : 1);
    if (vec && (slow || (n + 1) * kFcBatch <= g.K)) {
#pragma unroll
      for (int it = 0; it < V; ++it) r[it] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, v[it], step, 0);
    } else {
      const int first = slow ? x0 + 4 * (lane % (TS / 4)) : n * kFcBatch + 4 * (lane & 7), end = slow ? lim : g.K;
#pragma unroll
      for (int it = 0; it < V; ++it)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          r[it][e] = __builtin_amdgcn_raw_buffer_load_b32(
              rsrc, v[it] != kOobOffset && first + e < end ? v[it] + 4u * e : kOobOffset, step, 0);
    }
  };
  // two chains of additions per wavefront, added at the end: half the rounding error of one, and no MFMA waits for the
  // one in front of it
  typename M::Acc acc, acc2;
#pragma unroll
  for (int v = 0; v < M::kVals; ++v) acc[v] = 0.f, acc2[v] = 0.f;
  float bsum = 0.f;
  const bool tally = A_SLOW && g.bias_out && bx == 0 && jw == 0;
  float *sa = lds[jw][kw], *sb = sa + kStagedA;  // this wavefront's own: its LDS accesses execute in order
  auto multiply = [&](const u4 (&ar)[V], const u4 (&br)[V]) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int it = 0; it < V; ++it) {
      const int oc = (8 * it + (lane >> 3)) * LDC + 4 * (lane & 7);
      const int os = (it * (256 / TS) + lane / (TS / 4)) * LDS + 4 * (lane % (TS / 4));
      *(u4 *)&sa[A_SLOW ? os : oc] = ar[it];
      *(u4 *)&sb[B_SLOW ? os : oc] = br[it];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // fragment of step u: the four values k = STEP*u + 4*kg + 0 .. 3 of this lane's row or column
    auto frag = [&](bool slow, const float *t, int u) -> f4 {
      if (!slow) return *(const f4 *)&t[rl * LDC + u * STEP + 4 * kg];
      const float *q = &t[(u * STEP + 4 * kg) * LDS + rl];
      return f4{q[0], q[LDS], q[2 * LDS], q[3 * LDS]};
    };
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const f4 af = frag(A_SLOW, sa, u), bf = frag(B_SLOW, sb, u);
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        acc = M::mma1(af[e], bf[e], acc);
        acc2 = M::mma1(af[e + 1], bf[e + 1], acc2);
      }
      if (tally) {  // rows beyond the range hold zeros
#pragma unroll
        for (int e = 0; e < 4; ++e) bsum += af[e];
      }
    }
  };
  // one batch in flight ahead of the one that is multiplied
  u4 ra[2][V], rb[2][V];
  auto fetch = [&](int n, int buf) {
    load(A_SLOW, g.vec_a, a_rsrc, g.lda, i0, g.I, va, n, ra[buf]);
    load(B_SLOW, g.vec_b, b_rsrc, g.ldb, j0, g.J, vb, n, rb[buf]);
  };
  if (n_begin < n_end) fetch(n_begin, 0);
  for (int n = n_begin; n < n_end; n += 2) {
    if (n + 1 < n_end) fetch(n + 1, 1);
    multiply(ra[0], rb[0]);
    if (n + 1 >= n_end) break;
    if (n + 2 < n_end) fetch(n + 2, 0);
    multiply(ra[1], rb[1]);
  }

  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int v = 0; v < M::kVals; ++v) sa[M::row(lane, v) * LD + rl] = acc[v] + acc2[v];  // the staged operands are dead
  if (tally) {
#pragma unroll
    for (int m = TS; m < 64; m <<= 1) bsum += __shfl_xor(bsum, m, 64);
    if (lane < TS) bpart[kw][lane] = bsum;
  }
  __syncthreads();
  float *out = g.out + rep * g.o_rs;
  const long long p0 = rep * g.o_rs + g.p_off;  // of the row that `out` belongs to
  const float gp = UPDATE ? (st->c.coupling ? st->c.coupling[0] : st->c.g) : 0.f;
  auto update1 = [&](long long at, float grad) {
    float y = st->y[at], v = st->vy[at], z = st->z[at];
    inner_update(st->c, gp, grad, st->x[at], y, v, z);
    st->y[at] = y, st->vy[at] = v, st->z[at] = z;
  };
  const float *bias = g.bias ? g.bias + rep * g.bias_rs : nullptr;
  const float *resid = g.resid ? g.resid + rep * g.resid_rs : nullptr;
  const float *mask = g.mask ? g.mask + rep * g.mask_rs : nullptr;
  for (int t = kw * 64 + lane; t < TS * TS / 4; t += KS * 64) {
    const int row = t / (TS / 4), col = (t - row * (TS / 4)) * 4;
    f4 v = *(const f4 *)&lds[jw][0][row * LD + col];
#pragma unroll
    for (int w = 1; w < KS; ++w) v += *(const f4 *)&lds[jw][w][row * LD + col];
    const int oi = i0 + row, oj = j0 + col;
    if (oi >= g.I || oj >= g.J) continue;
    const long long o = (long long)oi * g.ldo + oj;
    const int lim = min(4, g.J - oj);  // 4 whenever vec_out
    if (bias)
      for (int e = 0; e < lim; ++e) v[e] += bias[oj + e];
    if (g.vec_out) {
      if (resid) v += *(const f4 *)&resid[o];
      if (g.relu) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
      }
      if (mask) {
        const f4 mk = *(const f4 *)&mask[o];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = mk[e] > 0.f ? v[e] : 0.f;
      }
      if (g.accumulate) v += *(const f4 *)&out[o];
      *(f4 *)&out[o] = v;
      if constexpr (UPDATE) {
        f4 y = *(const f4 *)&st->y[p0 + o], vy = *(const f4 *)&st->vy[p0 + o], z = *(const f4 *)&st->z[p0 + o];
        inner_update(st->c, gp, v, *(const f4 *)&st->x[p0 + o], y, vy, z);
        *(f4 *)&st->y[p0 + o] = y, *(f4 *)&st->vy[p0 + o] = vy, *(f4 *)&st->z[p0 + o] = z;
      }
    } else {
      for (int e = 0; e < lim; ++e) {
        float t1 = v[e];
        if (resid) t1 += resid[o + e];
        if (g.relu) t1 = t1 > 0.f ? t1 : 0.f;
        if (mask) t1 = mask[o + e] > 0.f ? t1 : 0.f;
        if (g.accumulate) t1 += out[o + e];
        out[o + e] = t1;
        if constexpr (UPDATE) update1(p0 + o + e, t1);
      }
    }
  }
  if (A_SLOW && g.bias_out && bx == 0 && tid < TS && i0 + tid < g.I) {
    float t = bpart[0][tid];
#pragma unroll
    for (int w = 1; w < KS; ++w) t += bpart[w][tid];
    g.bias_out[rep * g.bias_out_rs + i0 + tid] = t;
    if constexpr (UPDATE) update1(p0 + (long long)g.I * g.J + i0 + tid, t);
  }
}

template <int TS, bool A_SLOW, bool B_SLOW, int KS, int NJ>
__global__ __launch_bounds__(KS *NJ * 64) void k_fc_f32(const FcArgs g) {
  __shared__ __attribute__((aligned(16))) float smem[kFcLds<TS, A_SLOW, B_SLOW, KS, NJ>];
  fc_tile<TS, A_SLOW, B_SLOW, KS, NJ>(g, smem, blockIdx.x, blockIdx.y, blockIdx.z);
}

// Weight gradients of several layers and the mean loss in one launch.  In a network of a few small layers each of these is a
// launch of 2 to 6 us that leaves most of the chip empty and waits for nothing but the classifier's gradient.  The MLP's two
// weight gradients and its loss were three launches of 3.5, 5.7 and 1.8 us: a step of it (three replicas) 30.1 -> 25.8 us; with the
// update, a fourth one of 4 us, 22.3.
constexpr int kFcGroup = 4;
struct FcGroup {
  FcArgs part[kFcGroup];
  int end[kFcGroup];  // workgroups of the parts up to this one; those behind the last part take a replica's loss each
  int count, B;
  const float *loss_img;
  float *loss_out;
  InnerState update;
};
// UPDATE: and the step's update, where the parts are all that a network has.
template <bool UPDATE>
__global__ __launch_bounds__(kThreads) void k_fc_group(const FcGroup a) {
  __shared__ __attribute__((aligned(16))) float smem[kFcLds<32, true, true, 4, 1>];
  int p = 0, first = 0;
  while (p < a.count && (int)blockIdx.x >= a.end[p]) first = a.end[p++];
  const int b = blockIdx.x - first;
  if (p == a.count) {
    mean_loss(a.B, a.loss_img, a.loss_out, b, smem);
    return;
  }
  const FcArgs &g = a.part[p];
  const int ts = g.small ? 16 : 32, nx = (g.J + ts - 1) / ts, ny = (g.I + ts - 1) / ts;
  const int rep = b / (nx * ny), t = b - rep * nx * ny, by = t / nx, bx = t - by * nx;
  if (g.small)
    fc_tile<16, true, true, 4, 1, UPDATE>(g, smem, bx, by, rep, &a.update);
  else
    fc_tile<32, true, true, 4, 1, UPDATE>(g, smem, bx, by, rep, &a.update);
}

template <int TS, bool A_SLOW, bool B_SLOW, int KS, int NJ>
hipError_t run_fc(hipStream_t st, int replicas, const FcArgs &g) {
  const dim3 grid((g.J + TS * NJ - 1) / (TS * NJ), (g.I + TS - 1) / TS, replicas);
  hipLaunchKernelGGL((k_fc_f32<TS, A_SLOW, B_SLOW, KS, NJ>), grid, dim3(KS * NJ * 64), 0, st, g);
  return hipGetLastError();
}

constexpr int kCus = 256;

long long fc_tiles(int I, int J, int ts) { return (long long)((I + ts - 1) / ts) * ((J + ts - 1) / ts); }

bool fc_small_tiles(int replicas, int I, int J, int K) { return fc_tiles(I, J, 32) * replicas < (K > 256 ? 144 : kCus); }

template <bool A_SLOW, bool B_SLOW>
hipError_t choose_fc(hipStream_t st, int replicas, FcArgs &g) {
  // Measured (us; forward / input gradient / weight gradient), six replicas of 128 x 800 x 500 (384 / 600 / 2400 tiles of
  // 32 x 32): <32, 4, 1> 13.5 / 18.4 / 14.7, <32, 2, 2> 17.4 / 17.3 / 13.9, <16, 4, 1> 14.1 / 17.7 / 18.8; three of
  // 128 x 784 x 128 (48 / 300 / 300 tiles): <32, 4, 1> 9.5 / 4.5 / 4.6, <16, 8, 1> 4.6 / 6.4 / 6.6.  So: small tiles while
  // large ones leave compute units empty, more wavefronts per tile the longer the contraction, and from two large tiles
  // per compute unit on fewer wavefronts per tile, each with more of the contraction.  Eight wavefronts to a small tile fill
  // the chip earlier than four: <16, 8, 1> / <32, 4, 1> at 160 large tiles (4 x 128 x 500 x 320 forward, 5 x 64 x 800 x 500
  // input gradient) 8.9 / 8.2 and 14.7 / 8.4, at 192 (3 x 128 x 500 x 500) 9.5 / 8.4, at 128 (8 x 32 x 1024 x 512) 7.8 / 7.9;
  // <16, 4, 1> / <32, 4, 1> at 192 (3 x 128 x 256 x 500) 4.9 / 5.5.
  const long long t32 = fc_tiles(g.I, g.J, 32) * replicas;
  if (fc_small_tiles(replicas, g.I, g.J, g.K)) {
    if (g.K > 256) return run_fc<16, A_SLOW, B_SLOW, 8, 1>(st, replicas, g);
    return run_fc<16, A_SLOW, B_SLOW, 4, 1>(st, replicas, g);
  }
  if (t32 <= 2 * kCus) return run_fc<32, A_SLOW, B_SLOW, 4, 1>(st, replicas, g);
  return run_fc<32, A_SLOW, B_SLOW, 2, 2>(st, replicas, g);
}

// 1 x 1 window, stride 1, no padding: row m of the product reads row m of the input
bool plain_product(const ConvGeom &g) {
  return g.R == 1 && g.S == 1 && g.sp == 1 && g.off == 0 && g.dshift == 0 && g.Hin == g.P && g.Win == g.Q;
}

}  // namespace

bool fc_f32_applicable(int dtype, int replicas, const ConvGeom &g) {
  if (dtype != 0 || !plain_product(g)) return false;
  const long long lim = 1LL << 31;
  if ((long long)g.M * g.K * 4 >= lim || (long long)g.N * g.K * 4 >= lim || (long long)g.M * g.N * 4 >= lim) return false;
  return fc_tiles(g.M, g.N, 64) * replicas <= kCus && (g.M + 31) / 32 <= 65535 && (g.N + 31) / 32 <= 65535;
}

hipError_t launch_fc_f32(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io) {
  FcArgs f{};
  f.a = (const float *)io.in, f.a_rs = io.in_rs, f.lda = g.K, f.a_bytes = g.M * g.K * 4;
  f.b = (const float *)io.w, f.b_rs = io.w_rs, f.ldb = io.w_kn ? g.N : g.K, f.b_bytes = g.N * g.K * 4;
  f.out = (float *)io.out, f.o_rs = io.out_rs, f.ldo = io.ldc;
  f.bias = io.bias, f.bias_rs = io.bias_rs;
  f.resid = (const float *)io.resid, f.resid_rs = io.resid_rs;
  f.mask = (const float *)io.mask, f.mask_rs = io.mask_rs;
  f.I = g.M, f.J = g.N, f.K = g.K;
  f.relu = io.relu, f.accumulate = io.accumulate;
  f.vec_a = f.lda % 4 == 0, f.vec_b = f.ldb % 4 == 0;
  f.vec_out = g.N % 4 == 0 && io.ldc % 4 == 0 && aligned_to(io.out, 16) && io.out_rs % 4 == 0 &&
              aligned_to(io.resid, 16) && (!io.resid || io.resid_rs % 4 == 0) && aligned_to(io.mask, 16) &&
              (!io.mask || io.mask_rs % 4 == 0);
  return io.w_kn ? choose_fc<false, true>(st, replicas, f) : choose_fc<false, false>(st, replicas, f);
}

// Weight gradient of such a layer (g: forward geometry).  A tile costs this kernel about 2.5 us of a workgroup beside its
// contraction (staging, partial tiles, the strided result), the generic kernel less, but that takes 1.8 us per 32 rows of
// the batch.  us, generic / this, at 256, 1024, 2400, 4096 and 16384 tiles of 32 x 32: 16 rows 3.6 / 4.2, 4.1 / 5.1,
// 6.4 / 11.9, 7.9 / 16.5, 16 / 53; 64 rows 6.4 / 4.3, 7.0 / 5.7, 11.5 / 12.5, 14.0 / 17.7, 39 / 59; 128 rows 10.1 / 4.4,
// 10.8 / 7.5, 18.2 / 17.3, 22.3 / 23.6, 68 / 83; 256 rows 13.4 / 5.4, 19.7 / 10.8, 30.8 / 28.6, 39.3 / 37.4, 127 / 132; at
// 512 rows this one leads at every size (245 / 233).  So the number of tiles it takes grows with the rows.
// Rows of no whole vectors are loaded and stored value by value here, which the generic kernel does with either, so it is
// ahead earlier: 304 tiles (5 x 175 x 307) at 32 rows 4.7 / 5.7, 65 7.3 / 6.6, 128 10.1 / 7.7, 300 15.4 / 12.8, 500 17.9 /
// 19.1; 560 (8 x 241 x 263) 4.8 / 6.6, 7.6 / 9.7, 10.4 / 11.7, 19.4 / 22.2, 22.7 / 32.6; 3700 (8 x 900 x 502) at 200 rows 32 / 47.
bool wgrad_fc_f32_applicable(int dtype, int replicas, const ConvGeom &g) {
  if (dtype != 0 || !plain_product(g) || g.M > 1024 || (g.N + 15) / 16 > 65535) return false;
  const long long lim = 1LL << 31;
  if ((long long)g.M * g.K * 4 >= lim || (long long)g.M * g.N * 4 >= lim || (long long)g.N * g.K * 4 >= lim) return false;
  const long long tiles = fc_tiles(g.N, g.K, 32) * replicas;
  if (g.N % 4 != 0 || g.K % 4 != 0) return tiles <= (g.M > 400 ? 200 : std::min(400, std::max(150, 4 * g.M + 70)));
  return g.M >= 512 || tiles <= std::max(192, 24 * (g.M - 8));
}

namespace {
FcArgs wgrad_fc_args(const ConvGeom &g, const WgradIO &io) {
  FcArgs f{};
  f.a = (const float *)io.dy, f.a_rs = io.dy_rs, f.lda = g.N, f.a_bytes = g.M * g.N * 4;
  f.b = (const float *)io.x, f.b_rs = io.x_rs, f.ldb = g.K, f.b_bytes = g.M * g.K * 4;
  f.out = io.out, f.o_rs = io.out_rs, f.ldo = g.K;
  f.I = g.N, f.J = g.K, f.K = g.M;
  f.vec_a = f.lda % 4 == 0, f.vec_b = f.ldb % 4 == 0;
  f.vec_out = g.K % 4 == 0 && aligned_to(io.out, 16) && io.out_rs % 4 == 0;
  if (io.with_bias) f.bias_out = io.out + (long long)g.N * g.K, f.bias_out_rs = io.out_rs;
  return f;
}
}  // namespace

hipError_t launch_wgrad_fc_f32(hipStream_t st, int replicas, const ConvGeom &g, const WgradIO &io) {
  if (io.splits != 1) return hipErrorInvalidValue;
  FcArgs f = wgrad_fc_args(g, io);
  return choose_fc<true, true>(st, replicas, f);
}

// Layers that choose_fc would give four wavefronts per tile; a launch of more tiles fills the chip by itself.
bool fc_group_takes(int dtype, int replicas, const ConvGeom &g) {
  if (wgrad_small_f32_applicable(dtype, g) || !wgrad_fc_f32_applicable(dtype, replicas, g)) return false;
  return fc_small_tiles(replicas, g.N, g.K, g.M) ? g.M <= 256 : fc_tiles(g.N, g.K, 32) * replicas <= 2 * kCus;
}

hipError_t launch_fc_group(hipStream_t st, int replicas, int count, const ConvGeom *g, const WgradIO *io, int B,
                           const float *loss_img, float *loss_out, const float *grad, const InnerState *update) {
  static_assert(kFcGroup == kFcGroupMax, "the callers' limit");
  if (count < 0 || count > kFcGroup) return hipErrorInvalidValue;
  FcGroup a{};
  a.count = count, a.B = B, a.loss_img = loss_img, a.loss_out = loss_out;
  int blocks = 0;
  for (int i = 0; i < count; ++i) {
    if (io[i].splits != 1) return hipErrorInvalidValue;
    FcArgs &f = a.part[i];
    f = wgrad_fc_args(g[i], io[i]);
    f.small = fc_small_tiles(replicas, f.I, f.J, f.K);
    f.p_off = f.out - grad;
    blocks += (int)fc_tiles(f.I, f.J, f.small ? 16 : 32) * replicas;
    a.end[i] = blocks;
  }
  if (loss_out) blocks += replicas;
  if (blocks == 0) return hipSuccess;
  if (update) {
    a.update = *update;
    hipLaunchKernelGGL(k_fc_group<true>, dim3(blocks), dim3(kThreads), 0, st, a);
  } else {
    hipLaunchKernelGGL(k_fc_group<false>, dim3(blocks), dim3(kThreads), 0, st, a);
  }
  return hipGetLastError();
}
