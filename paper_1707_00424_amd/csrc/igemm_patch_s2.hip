// Forward pass of a stride-2 3x3 convolution with padding 1 (bf16, channel counts in multiples of 8): operands loaded straight
// into LDS and the epilogue in registers, as in igemm_patch.hip.  Two kernels, for the two orders of sums that such layers have with
// a residual or column sums: by chunks of channels (k_patch_s2, several tiles per workgroup) and by taps (k_taps_s2, further down).
//
// The input of such a layer is four images, its pixels by the parity of row and column.  A patch is a tile's pixels of one
// parity class and 32 channels, a step one tap; the taps of a chunk of channels are taken row by row, which is the order of
// sums of k_conv_halo_s2, so that a layer's result does not depend on which of the two runs it (column sums, residuals and
// odd channel counts stay there).  Window rows 0 and 2 read odd rows, row 1 even rows; of each, columns 0 and 2 read odd columns:
//   step     0   1   2   3   4   5   6   7   8
//   class    OO  OE  OO  EO  EE  EO  OO  OE  OO     (row, column: odd or even)
//   buffer   X   Y   X   Z   Y   Z   X   Y   X      X and Z change places with every chunk
//   loads    Z       Y           Y   Z   Z   Y
// Three patches fit where four would leave one workgroup per compute unit less; OE is loaded twice for it, from L2.
//
// The kernel that runs the other layers of 128 channels and more stages whole patches through registers and waits for each of
// them, the gather kernels fetch each pixel 9/4 times.  us per pass, before -> now, 3 x 128 images unless said: 192 -> 192 on
// 16 x 16 36 -> 27, 128 -> 256 29 -> 25, 320 -> 640 123 -> 110, 160 -> 320 on 32 x 32 143 -> 113, 32 -> 64 15.5 -> 12.8, 3 x 64
// images of 128 -> 64 24 -> 19.  A step of 8 products asks for 2 to 3 KB per
// wavefront, and every barrier waits for the last of four.  (Class after class, four taps of odd-odd pixels first, needs no second
// load of OE and was 0 to 15 % faster, but is another order of sums.)
#include "igemm_halo.h"
#include <type_traits>

namespace {

using namespace igemm_dev;

constexpr uint32_t kOob = 0x80000000u;
constexpr int kPix = 64;  // bytes of a patch pixel or weight row in LDS: 32 channels, vectors exchanged as in igemm_patch.hip

// A tile is a number of whole output rows, counted through all images of a replica.  Its patches have one row and one column
// more than its outputs (an image that ends inside a tile: a row each), whichever class they are of: slot (u + 1, v + 1) holds
// input pixel (2u + a, 2v + c) of class (a, c), and window row 0 of output row p lies at u = p - 1, rows 1 and 2 at u = p.
struct S2Geom {
  int TH, HC, PRI, slots, rows;
  FastDiv dP, dQ, dHC, dPRI;
};
struct S2Args {
  ConvGeom g;
  GemmIO io;
  S2Geom sg;
  int items, groups, tiles;
  FastDiv dRep, dGroup;
};
typedef __attribute__((address_space(4))) const S2Args CArgs;

// The arguments, read again behind every call: what only a change of tile needs stays out of the scalar registers.
__device__ __forceinline__ CArgs *fresh(CArgs *a) {
  asm volatile("" : "+s"(a));
  return a;
}
__device__ __forceinline__ uint32_t fdivc(uint32_t n, __attribute__((address_space(4))) const FastDiv &f) {
  return (uint32_t)(((uint64_t)n * f.magic) >> f.shift);
}

constexpr int tap_class(int t) { return (t / 3 != 1 ? 2 : 0) + (t % 3 != 1 ? 1 : 0); }  // 2 * (odd row) + (odd column)

// Wavefront loads of a patch (H_IT of them) that step t issues: odd-odd pixels of the next chunk in two halves, else all at once.
template <int H_IT>
constexpr int step_pieces(int t) {
  return t == 0 || t == 2 || t == 5 || t == 8 ? H_IT : t == 6 ? (H_IT + 1) / 2 : t == 7 ? H_IT / 2 : 0;
}

// Outputs m0 .. mend - 1 of a tile as in igemm_patch.hip: lane l holds channels 16 * (l / 16 % 2) + 8 * (l / 32) .. + 7 of pixel
// l % 16 (+ 16) of a tile of 32 pixels x 32 channels.  bias, norm: LDS, the column block's bias; means, 1/sigma, gamma, beta.
template <int TM, int TN, bool NORM, typename Args>
__device__ __forceinline__ void store_outputs(Args *a, const f16v (&acc)[TM][TN], const char *bias, const char *norm, int rep, int m0, int mend, int n0,
                                              int wave, int lane) {
  typedef bf16_t T;
  constexpr int BN = TN * 32;
  const int h = lane >> 5, chan = 16 * ((lane >> 4) & 1) + 8 * h;
  auto out_like = [&](const void *p) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p + rep * a->io.out_rs), 0,
                                             p ? (int)((uint32_t)a->g.M * (uint32_t)a->io.ldc * 2u) : 0, 0x00020000);
  };
  const bool relu = a->io.relu;
  const int ldc = a->io.ldc, N = a->g.N;
  const __amdgpu_buffer_rsrc_t o_rsrc = out_like(a->io.out), n_rsrc = out_like(NORM ? a->io.bn_out : nullptr);
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      uint32_t d[4][2];
#pragma unroll
      for (int vg = 0; vg < 4; ++vg) {
        f4 v = f4{acc[tm][tn][4 * vg], acc[tm][tn][4 * vg + 1], acc[tm][tn][4 * vg + 2], acc[tm][tn][4 * vg + 3]} +
               *(const f4 *)(bias + (tn * 32 + vg * 8 + h * 4) * 4);
        if (relu) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_fmed3f(v[e], 0.f, __builtin_inff());  // NaN: 0
        }
        d[vg][0] = f32x2_to_bf16x2(v.x, v.y), d[vg][1] = f32x2_to_bf16x2(v.z, v.w);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) swap32(d[0][k], d[1][k]), swap32(d[2][k], d[3][k]);
#pragma unroll
      for (int k = 0; k < 2; ++k) swap16(d[0][k], d[2][k]), swap16(d[1][k], d[3][k]);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const u4 o = {d[2 * j][0], d[2 * j][1], d[2 * j + 1][0], d[2 * j + 1][1]};
        const int m = m0 + wave * (TM * 32) + tm * 32 + j * 16 + (lane & 15), n = n0 + tn * 32 + chan;
        const uint32_t at = m < mend && n < N ? ((uint32_t)m * (uint32_t)ldc + (uint32_t)n) * 2u : kOob;
        if (!NORM || !a->io.bn_only) __builtin_amdgcn_raw_buffer_store_b128(o, o_rsrc, at, 0, 0);
        if constexpr (NORM) {
          const char *p = norm + (tn * 32 + chan) * 4;  // means, 1/sigma, gamma, beta of the column block
          u4 r;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const f4 mu = *(const f4 *)(p + q * 16), rs = *(const f4 *)(p + BN * 4 + q * 16), gm = *(const f4 *)(p + BN * 8 + q * 16),
                     bt = *(const f4 *)(p + BN * 12 + q * 16);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float x = __uint_as_float(e & 1 ? o[2 * q + (e >> 1)] & 0xffff0000u : o[2 * q + (e >> 1)] << 16);
              const float t = (x - mu[e]) * rs[e] * gm[e] + bt[e];
              v[e] = t > 0.f ? t : 0.f;
            }
            r[2 * q] = f32x2_to_bf16x2(v[0], v[1]), r[2 * q + 1] = f32x2_to_bf16x2(v[2], v[3]);
          }
          __builtin_amdgcn_raw_buffer_store_b128(r, n_rsrc, at, 0, 0);
        }
      }
    }
}

// TM: 32-pixel tiles per wavefront (four wavefronts: 128 or 256 outputs); TN: 32-channel tiles; H_IT: wavefront loads of a patch
// per wavefront; NORM: io.bn_out.
template <int TM, int TN, int H_IT, bool NORM>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(TM == 1 && TN == 2 ? 3 : 2))) void k_patch_s2(const S2Args) {
  typedef bf16_t T;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  CArgs *args = (CArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int D = 2;                   // weight tiles in flight
  constexpr int BN = TN * 32, NB = D + 1;
  constexpr int WG = TN * 2;             // wavefront loads of a weight tile, 16 rows each
  constexpr int WI = (WG + 3) / 4;       // per wavefront, at most
  constexpr int STORES = TM * TN * 2;    // stores of a tile per wavefront, at least
  constexpr int TB = BN * kPix;          // bytes of a weight tile
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5;
  const int cv = (lane & 3) ^ ((lane >> 4) & 3);  // channel vector this lane loads
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  const int pbytes = (args->sg.slots + 15) / 16 * 16 * kPix;
  const int wring = 3 * pbytes, lbias = wring + NB * TB, ldump = lbias + 1024, lnorm = ldump + 1024;
  const int Cc = args->g.Cc, chunks = (Cc + 31) >> 5;
  const int b_l = (lane & 31) * kPix + ((h ^ ((lane >> 2) & 3)) << 4);
  int n0;

  // Items: eight tiles (counted through all replicas), column block, tile; a workgroup's are `groups` apart, a multiple of 8 x
  // column blocks: all of them have the same columns, and the column blocks of a tile share an XCD.
  auto item_at = [&](CArgs *a, int idx, int &rep, int &tile) {
    if (idx >= a->items) return false;
    const int group = (int)fdivc((uint32_t)idx, a->dGroup), w = idx - group * (int)a->dGroup.d, t = group * 8 + (w & 7);
    n0 = (w >> 3) * BN;
    rep = (int)fdivc((uint32_t)t, a->dRep), tile = t - rep * (int)a->dRep.d;
    return t < a->tiles;  // the last item of its workgroup where it is not
  };

  uint32_t h_off[H_IT], b_off[WI];  // of the even-even pixel of a slot
  uint32_t odd_ok = 0;              // bit `it`: the slot has a pixel in the odd row, bit 16 + it: in the odd column
  u4 a_rsrc, b_rsrc;
  uint64_t bn_base = 0;  // the next item's weights
  auto weights_at = [&](CArgs *a, int rep) { return (uint64_t)((const T *)a->io.w + rep * a->io.w_rs); };
  auto patch_of = [&](CArgs *a, int rep, int tile) {
    const int P = a->g.P, Hin = a->g.Hin, Win = a->g.Win, HC = a->sg.HC, PRI = a->sg.PRI, slots = a->sg.slots, rows = a->sg.rows;
    const int row0 = tile * a->sg.TH, b0 = (int)fdivc((uint32_t)row0, a->sg.dP), p0 = row0 - b0 * P;
    const int first_rows = P + 1 - p0;
    a_rsrc = buffer_desc((const T *)a->io.in + rep * a->io.in_rs, (uint32_t)a->io.in_bytes);
    odd_ok = 0;
#pragma unroll
    for (int it = 0; it < H_IT; ++it) {
      const int slot = (it * 4 + wave) * 16 + (lane >> 2);
      const int pr = (int)fdivc((uint32_t)slot, a->sg.dHC), v = slot - pr * HC - 1;
      int b = b0, u = p0 + pr - 1;
      if (pr >= first_rows) {
        const int rest = pr - first_rows, img = (int)fdivc((uint32_t)rest, a->sg.dPRI);
        b = b0 + 1 + img, u = rest - img * PRI - 1;
      }
      const bool ok = slot < slots && b * P < rows && u >= 0 && 2 * u < Hin && v >= 0 && 2 * v < Win;
      h_off[it] = ok ? (uint32_t)((((b * Hin + 2 * u) * Win + 2 * v) * Cc + cv * 8) * 2) : kOob;
      odd_ok |= (uint32_t)(2 * u + 1 < Hin) << it | (uint32_t)(2 * v + 1 < Win) << (16 + it);
      __builtin_amdgcn_sched_barrier(0);  // one after the other: side by side they need registers that the sums have taken
    }
  };
  // pieces `from` .. `to` - 1 of the patch of class 2 a + c and the chunk at byte `soff` of a pixel
  const uint32_t col_b = (uint32_t)Cc * 2u, row_b = (uint32_t)args->g.Win * col_b;
  auto load_pieces = [&](auto cls, int from, int to, int buf, uint32_t soff, bool live) {
    constexpr int CL = decltype(cls)::value;
    const uint32_t need = (CL & 2 ? 1u : 0u) | (CL & 1 ? 0x10000u : 0u);
#pragma unroll
    for (int it = from; it < to; ++it) {
      const int o = (it * 4 + wave) * 1024;
      const bool ok = live && (odd_ok & (need << it)) == need << it;
      dma16(lds0 + (uint32_t)(o < pbytes ? buf + o : ldump), a_rsrc, ok ? h_off[it] : kOob,
            soff + (CL & 2 ? row_b : 0u) + (CL & 1 ? col_b : 0u));
    }
  };
  auto load_w = [&](int ring, uint32_t soff, bool live) {
#pragma unroll
    for (int i = 0; i < WI; ++i)
      if (WG % 4 == 0 || wave + 4 * i < WG)
        dma16(lds0 + (uint32_t)(wring + ring + (wave + 4 * i) * 1024), b_rsrc, live ? b_off[i] : kOob, soff);
  };
  auto load_bias = [&](CArgs *a, int rep, int buf) {
    if (wave * 64 < BN) {
      const int n = n0 + wave * 64 + lane;
      const u4 rsrc = buffer_desc(a->io.bias + rep * a->io.bias_rs, a->io.bias ? (uint32_t)a->g.N * 4u : 0u);
      dma4(lds0 + (uint32_t)(lbias + buf * 512 + wave * 256), rsrc, n < a->g.N ? (uint32_t)n * 4u : kOob);
    }
  };
  // What the step before this one requested has arrived, the weight tile of the next step last; behind it came a tile, PIECES of
  // a patch and, with `stores`, those of the tile before.
  auto wait_step = [&](auto pieces, bool stores) {
    constexpr int P = decltype(pieces)::value, FULL = WI * (D - 1) + P, SHORT = (WI - 1) * (D - 1) + P;
    if (WG % 4 != 0 && wave >= WG % 4) {
      if (stores)
        wait_loads<SHORT + STORES>();
      else
        wait_loads<SHORT>();
    } else {
      if (stores)
        wait_loads<FULL + STORES>();
      else
        wait_loads<FULL>();
    }
  };
  auto meet = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  f16v acc[TM][TN];
  int a_b[TM];
  auto begin = [&](CArgs *a, int tile) {
    const int P = a->g.P, Q = a->g.Q, TH = a->sg.TH, HC = a->sg.HC, PRI = a->sg.PRI;
    const int row0 = tile * TH, b0 = (int)fdivc((uint32_t)row0, a->sg.dP), p0 = row0 - b0 * P;
    const int first_rows = P + 1 - p0;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      const int ml = wave * (TM * 32) + tm * 32 + (lane & 31);
      int i = (int)fdivc((uint32_t)ml, a->sg.dQ);
      const int q = ml - i * Q;
      i = i < TH ? i : 0;
      const int row = row0 + i, b = (int)fdivc((uint32_t)row, a->sg.dP), p = row - b * P;
      const int pr = b == b0 ? p - p0 : first_rows + (b - b0 - 1) * PRI + p;
      a_b[tm] = (pr * HC + q) * kPix + h * 16;
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.f;
  };

  int a_ad[TM];
  u4 fa_a[TM], fa_b[TN], fb_a[TM], fb_b[TN];
  const int row_step = args->sg.HC * kPix;
  auto read0 = [&](int t, int buf, int ring) {
    const int shift = buf + (t / 3 ? row_step : 0) + (t % 3 ? kPix : 0);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      const int a = a_b[tm] + shift;
      a_ad[tm] = a ^ ((a >> 4) & 0x30);
      fa_a[tm] = *(const u4 *)(smem + a_ad[tm]);
    }
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) fa_b[tn] = *(const u4 *)(smem + (wring + ring + b_l) + tn * 32 * kPix);
  };
  auto read1 = [&](int ring) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) fb_a[tm] = *(const u4 *)(smem + (a_ad[tm] ^ 32));
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) fb_b[tn] = *(const u4 *)(smem + (wring + ring + (b_l ^ 32)) + tn * 32 * kPix);
  };
  auto mma_sub = [&](const u4 (&af)[TM], const u4 (&bf)[TN]) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) mma<T>(bf[tn], af[tm], acc[tm][tn]);
  };
  auto interleave = [&]() {
#pragma unroll
    for (int i = 0; i < TM * TN; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, TM * TN < TM + TN ? 2 : 1, 0);
    }
  };

  constexpr int HALF = (H_IT + 1) / 2;
  int idx = blockIdx.x, rep, tile;
  if (!item_at(args, idx, rep, tile)) return;
  patch_of(args, rep, tile);
  b_rsrc = buffer_desc((const void *)weights_at(args, rep), (uint32_t)((long long)args->g.N * args->g.K * sizeof(T)));
#pragma unroll
  for (int i = 0; i < WI; ++i) {
    const int nrow = n0 + (wave + 4 * i) * 16 + (lane >> 2);
    b_off[i] = nrow < args->g.N ? (uint32_t)((nrow * args->g.K + cv * 8) * 2) : kOob;
  }
  {
    const bool live = cv * 8 < Cc;
    load_bias(args, rep, 0);
    load_pieces(std::integral_constant<int, tap_class(0)>{}, 0, H_IT, 0, 0, live);
    load_pieces(std::integral_constant<int, tap_class(1)>{}, 0, H_IT, pbytes, 0, live);
#pragma unroll
    for (int i = 0; i < D; ++i) load_w(i * TB, (uint32_t)i * col_b, live);
  }
  if (NORM && tid < BN) {
    const int n = min(n0 + tid, args->g.N - 1);
    float *p = (float *)(smem + lnorm) + tid;
    p[0] = args->io.bn_running[n], p[BN] = 1.0f / sqrtf(args->io.bn_running[args->g.N + n] + kBnEps);
    p[2 * BN] = args->io.bn_gamma[n], p[3 * BN] = args->io.bn_beta[n];
  }
  wait_step(std::integral_constant<int, 0>{}, false);
  meet();
  int ring = 0, base = 0, bbuf = 0;  // base: buffer X of the chunk
  bool later = false;                // not the first item: the stores of the one before it are in flight
  for (;;) {
    begin(fresh(args), tile);
    read0(0, base, ring);
    int rep1 = rep, tile1 = tile;
    bool more = true;
    for (int c = 0; c < chunks; ++c) {
      const bool last = c + 1 == chunks;
      const bool live = c * 32 + cv * 8 < Cc;
      const int c1 = last ? 0 : c + 1;
      bool live1 = c1 * 32 + cv * 8 < Cc;
      const int other = 2 * pbytes - base;  // buffer Z
      auto step = [&](auto tc) {
        constexpr int t = decltype(tc)::value;
        const int prev = ring == 0 ? (NB - 1) * TB : ring - TB, next = ring == (NB - 1) * TB ? 0 : ring + TB;
        read1(ring);
        // a buffer is loaded again one step or more behind the last tap that reads it, and two or more before its next tap
        if (t == 0) load_pieces(std::integral_constant<int, tap_class(3)>{}, 0, H_IT, other, (uint32_t)(c * 64), live);
        if (t == 2) load_pieces(std::integral_constant<int, tap_class(4)>{}, 0, H_IT, pbytes, (uint32_t)(c * 64), live);
        if (t == 5) load_pieces(std::integral_constant<int, tap_class(7)>{}, 0, H_IT, pbytes, (uint32_t)(c * 64), live);
        if (t == 6) {
          if (last) {
            CArgs *a = fresh(args);
            idx += a->groups;
            more = item_at(a, idx, rep1, tile1);
            if (more) {
              patch_of(a, rep1, tile1);
              bn_base = weights_at(a, rep1);
              load_bias(a, rep1, bbuf ^ 1);
            }
            live1 = live1 && more;
          }
          load_pieces(std::integral_constant<int, tap_class(0)>{}, 0, HALF, other, (uint32_t)(c1 * 64), live1);
        }
        if (t == 7) load_pieces(std::integral_constant<int, tap_class(0)>{}, HALF, H_IT, other, (uint32_t)(c1 * 64), live1);
        if (t == 8) load_pieces(std::integral_constant<int, tap_class(1)>{}, 0, H_IT, pbytes, (uint32_t)(c1 * 64), live1);
        constexpr int tw = (t + D) % 9;
        if (t + D == 9 && last && more) {
          b_rsrc.x = __builtin_amdgcn_readfirstlane((uint32_t)bn_base);
          b_rsrc.y = __builtin_amdgcn_readfirstlane((uint32_t)(bn_base >> 32) & 0xffffu);
        }
        load_w(prev, (uint32_t)tw * col_b + (uint32_t)((t + D >= 9 ? c1 : c) * 64), t + D >= 9 ? live1 : live);
        mma_sub(fa_a, fa_b);
        interleave();
        wait_step(std::integral_constant<int, step_pieces<H_IT>(t)>{}, t == 0 && c == 0 && later);
        meet();
        constexpr int t1 = (t + 1) % 9;
        if (t < 8)
          read0(t1, t1 == 3 || t1 == 5 ? other : t1 % 3 == 1 ? pbytes : base, next);
        else if (!last)
          read0(0, other, next);
        mma_sub(fb_a, fb_b);
        if (t < 8) interleave();
        ring = next;
      };
      step(std::integral_constant<int, 0>{}), step(std::integral_constant<int, 1>{}), step(std::integral_constant<int, 2>{});
      step(std::integral_constant<int, 3>{}), step(std::integral_constant<int, 4>{}), step(std::integral_constant<int, 5>{});
      step(std::integral_constant<int, 6>{}), step(std::integral_constant<int, 7>{}), step(std::integral_constant<int, 8>{});
      base = other;
    }
    {
      CArgs *a = fresh(args);
      const int m0 = tile * a->sg.TH * a->g.Q;
      store_outputs<TM, TN, NORM>(a, acc, smem + lbias + bbuf * 512, smem + lnorm, rep, m0, min(a->g.M, m0 + a->sg.TH * a->g.Q), n0, wave, lane);
    }
    if (!more) break;
    rep = rep1, tile = tile1, later = true, bbuf ^= 1;
  }
  wait_loads<0>();  // nothing may land in LDS after the workgroup has ended
}

// Layers of several chunks of channels that gather kernels run where there is a residual or column sums (33 to 127 input channels, more
// on sizes that k_conv_halo leaves to them): their order of sums takes all channels of a tap before the next tap, and so does this, to
// the same bits.  Nothing of a patch would be used twice in that order, so a step's 32 contraction values of every output come straight
// from the tensor into LDS, two steps ahead, whichever taps they lie in; those of a window row are consecutive in memory.  Small launches
// are bound by the latency of a step, large ones by what comes through L2, each output's window once per column block.  us per pass,
// gather kernels / this: 64 -> 128 on 32 x 32, 3 x 128 images 30.8 / 27.1, 96 -> 96 35.9 / 31.8, 2 x 128 of 120 -> 256 78 / 54; 16 images of
// 96 -> 256 on 12 x 12 22 / 9.6, 8 x 12 of 40 -> 320 36 / 7.5 (channels in no multiple of 32: 16-byte gathers with a mask each).
struct TapArgs {
  ConvGeom g;
  GemmIO io;
  int tiles, steps;
  FastDiv dRep, dGroup;
};
typedef __attribute__((address_space(4))) const TapArgs CTapArgs;

template <int TM, int TN, bool NORM>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(TM == 1 ? 3 : 2))) void k_taps_s2(const TapArgs) {
  typedef bf16_t T;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  CTapArgs *args = (CTapArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int BM = TM * 128, BN = TN * 32, NB = 3;
  constexpr int AI = TM * 2;        // wavefront loads of a step's outputs per wavefront, 16 outputs each
  constexpr int WG = TN * 2;        // ... of its weights, 16 rows each
  constexpr int WI = (WG + 3) / 4;  // per wavefront, at most
  constexpr int TA = BM * kPix, SLOT = TA + BN * kPix, lbias = NB * SLOT, lnorm = lbias + 512;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5;
  const int cv = (lane & 3) ^ ((lane >> 4) & 3);  // vector of a step's four that this lane loads
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  // items as in k_patch_s2, one per workgroup
  const int group = (int)fdivc((uint32_t)blockIdx.x, args->dGroup), w = (int)blockIdx.x - group * (int)args->dGroup.d, t = group * 8 + (w & 7);
  if (t >= args->tiles) return;
  const int rep = (int)fdivc((uint32_t)t, args->dRep), m0 = (t - rep * (int)args->dRep.d) * BM, n0 = (w >> 3) * BN;
  const int Cc = args->g.Cc, Win = args->g.Win;
  if (tid < BN) {
    const int n = n0 + tid, nc = min(n, args->g.N - 1);
    *(float *)(smem + lbias + tid * 4) = args->io.bias && n < args->g.N ? args->io.bias[rep * args->io.bias_rs + n] : 0.f;
    if (NORM) {
      float *p = (float *)(smem + lnorm) + tid;
      p[0] = args->io.bn_running[nc], p[BN] = 1.0f / sqrtf(args->io.bn_running[args->g.N + nc] + kBnEps);
      p[2 * BN] = args->io.bn_gamma[nc], p[3 * BN] = args->io.bn_beta[nc];
    }
  }
  const u4 a_rsrc = buffer_desc((const T *)args->io.in + rep * args->io.in_rs, (uint32_t)args->io.in_bytes);
  const u4 b_rsrc = buffer_desc((const T *)args->io.w + rep * args->io.w_rs, (uint32_t)((long long)args->g.N * args->g.K * sizeof(T)));
  uint32_t a_off[AI], a_taps[AI], b_off[WI];  // of the window's first pixel (which may lie outside) and this lane's vector; taps inside the image
#pragma unroll
  for (int it = 0; it < AI; ++it) {
    const int m = m0 + (it * 4 + wave) * 16 + (lane >> 2);
    const bool ok = m < args->g.M;
    const uint32_t mm = ok ? (uint32_t)m : 0u;
    const int b = (int)fdivc(mm, args->g.dPQ), rem = (int)mm - b * args->g.P * args->g.Q, p = (int)fdivc((uint32_t)rem, args->g.dQ), q = rem - p * args->g.Q;
    const uint32_t cols = (q > 0 ? 1u : 0u) | 2u | (2 * q + 1 < Win ? 4u : 0u);
    a_taps[it] = ok ? (p > 0 ? cols : 0u) | cols << 3 | (2 * p + 1 < args->g.Hin ? cols << 6 : 0u) : 0u;
    a_off[it] = (uint32_t)((((b * args->g.Hin + 2 * p - 1) * Win + 2 * q - 1) * Cc + cv * 8) * 2);
  }
#pragma unroll
  for (int i = 0; i < WI; ++i) {
    const int nrow = n0 + (wave + 4 * i) * 16 + (lane >> 2);
    b_off[i] = nrow < args->g.N ? (uint32_t)((nrow * args->g.K + cv * 8) * 2) : kOob;
  }
  // the step that is requested next: this lane's tap and channel, bytes from a window's first value, bytes from a weight row's first
  int tap = 0, chan = cv * 8;
  uint32_t a_add = 0, b_add = 0;
  const uint32_t next_row = (uint32_t)(Win - 3) * (uint32_t)Cc * 2u;
  auto load_step = [&](int ring) {
#pragma unroll
    for (int it = 0; it < AI; ++it)
      dma16(lds0 + (uint32_t)(ring + (it * 4 + wave) * 1024), a_rsrc, (a_taps[it] >> tap) & 1u ? a_off[it] + a_add : kOob, 0);
#pragma unroll
    for (int i = 0; i < WI; ++i)
      if (WG % 4 == 0 || wave + 4 * i < WG)
        dma16(lds0 + (uint32_t)(ring + TA + (wave + 4 * i) * 1024), b_rsrc, tap < 9 ? b_off[i] : kOob, b_add);
    chan += 32, a_add += 64, b_add += 64;
    if (chan >= Cc) {  // more than 32 channels: once per step at most
      chan -= Cc, ++tap;
      if (tap == 3 || tap == 6) a_add += next_row;
    }
  };
  auto wait_step = [&]() {
    if (WG % 4 != 0 && wave >= WG % 4)
      wait_loads<AI + WI - 1>();
    else
      wait_loads<AI + WI>();
  };
  auto meet = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  f16v acc[TM][TN];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.f;
  // the first 16 values of row r of a tile lie at r * kPix, their vectors exchanged as they were loaded; the others 32 bytes apart
  const int frag = (lane & 31) * kPix + ((h ^ ((lane >> 2) & 3)) << 4), a_at = wave * (TM * 32) * kPix + frag;
  u4 fa_a[TM], fa_b[TN], fb_a[TM], fb_b[TN];
  auto read = [&](int ring, int half, u4 (&fa)[TM], u4 (&fb)[TN]) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) fa[tm] = *(const u4 *)(smem + ring + tm * 32 * kPix + (a_at ^ half));
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) fb[tn] = *(const u4 *)(smem + ring + TA + tn * 32 * kPix + (frag ^ half));
  };
  auto mma_sub = [&](const u4 (&af)[TM], const u4 (&bf)[TN]) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) mma<T>(bf[tn], af[tm], acc[tm][tn]);
  };
  load_step(0);
  load_step(SLOT);
  wait_step();
  meet();
  int ring = 0;
  read(ring, 0, fa_a, fa_b);
  const int steps = args->steps;
  for (int s = 0; s < steps; ++s) {
    const int prev = ring == 0 ? (NB - 1) * SLOT : ring - SLOT, next = ring == (NB - 1) * SLOT ? 0 : ring + SLOT;
    read(ring, 32, fb_a, fb_b);
    load_step(prev);  // steps past the last one load zeros
    mma_sub(fa_a, fa_b);
    wait_step();
    meet();
    read(next, 0, fa_a, fa_b);
    mma_sub(fb_a, fb_b);
    ring = next;
  }
  store_outputs<TM, TN, NORM>(args, acc, smem + lbias, smem + lnorm, rep, m0, min(args->g.M, m0 + BM), n0, wave, lane);
  wait_loads<0>();  // nothing may land in LDS after the workgroup has ended
}

// The tiles of a layer; false where they would be less than three quarters full.
bool make_s2_geom(const ConvGeom &g, int outputs, int max_slots, S2Geom &sg) {
  sg.HC = g.Q + 1, sg.PRI = g.P + 1;
  for (sg.TH = outputs / g.Q; sg.TH > 0; --sg.TH) {
    // images a tile can touch: tiles start at multiples of TH rows
    const int images = g.P % sg.TH == 0 ? 1 : sg.TH % g.P == 0 ? sg.TH / g.P : (sg.TH + g.P - 2) / g.P + 1;
    sg.slots = (sg.TH + images) * sg.HC;
    if (sg.slots <= max_slots) break;
  }
  if (sg.TH * g.Q * 4 < outputs * 3) return false;
  sg.rows = g.M / g.Q;
  sg.dP = make_fastdiv(g.P), sg.dQ = make_fastdiv(g.Q), sg.dHC = make_fastdiv(sg.HC), sg.dPRI = make_fastdiv(sg.PRI);
  return true;
}

template <int TM, int TN, int H_IT, bool NORM>
hipError_t run_as(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io, const S2Geom &sg) {
  constexpr int kCus = 256, kLdsOfCu = 160 * 1024, kWaves = TM == 1 && TN == 2 ? 3 : 2;
  const int lds = 3 * ((sg.slots + 15) / 16 * 16 * kPix) + 3 * TN * 32 * kPix + 2048 + (NORM ? TN * 32 * 16 : 0);
  const int resident = kCus * (kLdsOfCu / lds < kWaves ? kLdsOfCu / lds : kWaves);
  const int nb = (g.N + TN * 32 - 1) / (TN * 32), rep_tiles = (sg.rows + sg.TH - 1) / sg.TH, tiles = rep_tiles * replicas;
  const long long items = (long long)((tiles + 7) / 8 * 8) * nb;
  if (items >= 1LL << 31 || lds > kLdsOfCu) return hipErrorInvalidValue;
  S2Args a{g, io, sg, (int)items, (int)items, tiles, make_fastdiv(rep_tiles), make_fastdiv(8 * nb)};
  const int step = 8 * nb;
  if (items > resident && step <= resident) a.groups = resident / step * step;
  static const hipError_t lds_ok =
      hipFuncSetAttribute((const void *)k_patch_s2<TM, TN, H_IT, NORM>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsOfCu);
  if (lds_ok != hipSuccess) return lds_ok;
  hipLaunchKernelGGL((k_patch_s2<TM, TN, H_IT, NORM>), dim3(a.groups), dim3(kThreads), lds, st, a);
  return hipGetLastError();
}
template <int TM, int TN, int H_IT>
hipError_t run(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io, const S2Geom &sg) {
  return io.bn_out ? run_as<TM, TN, H_IT, true>(st, replicas, g, io, sg) : run_as<TM, TN, H_IT, false>(st, replicas, g, io, sg);
}

template <int TM, int TN, bool NORM>
hipError_t run_taps_as(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io) {
  constexpr int BM = TM * 128, BN = TN * 32, kLds = 3 * (BM + BN) * kPix + 512 + (NORM ? BN * 16 : 0);
  const int nb = (g.N + BN - 1) / BN, rep_tiles = (g.M + BM - 1) / BM;
  const long long tiles = (long long)rep_tiles * replicas, items = (tiles + 7) / 8 * 8 * nb;
  if (items >= 1LL << 31) return hipErrorInvalidValue;
  const TapArgs a{g, io, (int)tiles, (g.K + 31) / 32, make_fastdiv(rep_tiles), make_fastdiv(8 * nb)};
  static const hipError_t lds_ok = hipFuncSetAttribute((const void *)k_taps_s2<TM, TN, NORM>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (lds_ok != hipSuccess) return lds_ok;
  hipLaunchKernelGGL((k_taps_s2<TM, TN, NORM>), dim3((int)items), dim3(kThreads), kLds, st, a);
  return hipGetLastError();
}
template <int TM, int TN>
hipError_t run_taps(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io) {
  return io.bn_out ? run_taps_as<TM, TN, true>(st, replicas, g, io) : run_taps_as<TM, TN, false>(st, replicas, g, io);
}

// 128 x 64 tiles up to 400 of them.  In larger launches the outputs that every column block fetches again weigh more: the blocks of 64,
// 96 or 128 channels by (channels / 32 + 1) each, and 256 outputs from 1000 tiles of 128.  us, 128 x 64 / 128 x 96 / 128 x 128 / 256 x 64 /
// 256 x 96 / 256 x 128: 344 tiles (5 x 123 images of 96 -> 128 on 12 x 12) 12.9 / 16.4 / 14.0 / 15.1 / 19.3 / 20.3, 460 (5 x 23 of 104 -> 128 on
// 32 x 32) 21 / 24 / 18 / 20 / 22 / 24, 576 (3 x 128 of 96 -> 192 on 16 x 16) 20 / 17 / 19 / 20 / 20 / 21, 1536 (64 -> 128 on 32 x 32) 33 / 36 / 27 /
// 30 / 36 / 28, 2184 (7 x 104 of 104 -> 320 on 16 x 32) 135 / 124 / 109 / 120 / 111 / 100, (7 x 78 of 104 -> 136 on 32 x 32) 107 / 98 / 106 / 101 / 88 / 93.
hipError_t launch_taps(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io) {
  const long long tiles = (long long)((g.M + 127) / 128) * replicas;
  auto blocks = [&](int tn) { return (g.N + tn * 32 - 1) / (tn * 32); };
  if (tiles * blocks(2) <= 400) return run_taps<1, 2>(st, replicas, g, io);
  int tn = 2;
  for (int t = 3; t <= 4; ++t)
    if (blocks(t) * (t + 1) <= blocks(tn) * (tn + 1)) tn = t;
  const bool tall = tiles * blocks(tn) > 1000;  // 256 x 128 with a batch-norm's constants does not fit in registers
  if (tn == 2) return tall ? run_taps<2, 2>(st, replicas, g, io) : run_taps<1, 2>(st, replicas, g, io);
  if (tn == 3) return tall ? run_taps<2, 3>(st, replicas, g, io) : run_taps<1, 3>(st, replicas, g, io);
  return tall && !io.bn_out ? run_taps_as<2, 4, false>(st, replicas, g, io) : run_taps<1, 4>(st, replicas, g, io);
}

// A single chunk of channels is the same order of sums for both.
bool tap_by_tap(int replicas, const ConvGeom &g, const GemmIO &io) { return g.Cc > 32 && !conv_halo_applicable(1, replicas, g, io, false); }

}  // namespace

bool patch_s2_applicable(int dtype, int replicas, const ConvGeom &g, const GemmIO &io, bool out_f32) {
  S2Geom sg;
  if (dtype != 1 || out_f32 || g.R != 3 || g.S != 3 || g.sp != 2 || g.off != -1 || g.sr != 1 || g.dshift != 0 || g.P != (g.Hin + 1) / 2 || g.Q != (g.Win + 1) / 2)
    return false;
  if (g.Cc % 8 != 0 || g.N % 8 != 0 || io.ldc % 8 != 0 || !io.vecA || !io.vecB || io.stat || io.resid || io.mask || io.accumulate || io.in_f32) return false;
  if (!aligned_to(io.out, 16) || io.out_rs % 8 != 0 || !aligned_to(io.bn_out, 16) || io.in_bytes <= 0 || io.in_bytes >= (1LL << 31)) return false;
  if ((long long)g.M * io.ldc * 4 >= (1LL << 31) || (long long)g.N * g.K * 2 >= (1LL << 31)) return false;
  return tap_by_tap(replicas, g, io) || make_s2_geom(g, 128, 192, sg);
}

hipError_t launch_patch_s2(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io) {
  if (tap_by_tap(replicas, g, io)) return launch_taps(st, replicas, g, io);
  // 96- or 64-wide column blocks, whichever pad the output channels least.  256 outputs with two workgroups per compute unit, as
  // far as three patches, the weight tiles and a batch-norm's constants fit in half of its LDS; 128 with three where the wide
  // ones would leave compute units empty.
  const bool tn3 = (g.N + 95) / 96 * 96 <= (g.N + 63) / 64 * 64;
  S2Geom sg;
  if (make_s2_geom(g, 256, tn3 ? (io.bn_out ? 304 : 320) : 336, sg) &&
      (long long)((sg.rows + sg.TH - 1) / sg.TH) * replicas * ((g.N + (tn3 ? 95 : 63)) / (tn3 ? 96 : 64)) > 256)
    return tn3 ? run<2, 3, 5>(st, replicas, g, io, sg) : run<2, 2, 6>(st, replicas, g, io, sg);
  if (!make_s2_geom(g, 128, 192, sg)) return hipErrorInvalidValue;
  return tn3 ? run<1, 3, 3>(st, replicas, g, io, sg) : run<1, 2, 3>(st, replicas, g, io, sg);
}
