// Stride-1 3x3 and 5x5 convolutions in bf16 (forward, and backward-data of such a layer), channel counts in multiples of 8: the
// input patch of a tile staged in LDS as in igemm_halo.hip, with nothing on its way through registers.
//
// What bounds them, from stamps in the kernel before this one (96 -> 96 channels, 32 x 32, batch 3 x 128: 512 of 1536
// workgroups at a time): of the 34 900 cycles of a workgroup the contraction loop took 22 600, for 20 700 cycles of matrix
// work that the two workgroups of a compute unit share; 7 400 went by until the first patch had come from memory and 4 000
// in the epilogue.  So
//   * operands go from memory to LDS directly (buffer loads with the LDS bit; lanes outside the image or the layer write
//     zeros): no staging registers, no LDS stores;
//   * a workgroup walks several tiles, and the patch, the first weight tiles and the bias of the next one are on their way
//     while the last channels of the current one are multiplied: only the first tile waits for memory;
//   * the epilogue exchanges lanes in registers (permlane swaps) until each lane holds eight channels of a pixel and a
//     store writes 64 bytes of sixteen pixels; LDS has no part in it, the next tile's loads run on beneath it.
// What is left is the matrix work at the clock that the power limit allows (1.4 to 1.6 GHz in these loops) and, in launches
// of one round, the first patch.  us per pass, before -> now: 96 -> 96 32 x 32, 3 x 128 images 93 -> 79; 320 -> 320
// 16 x 16 195 -> 161; 64 -> 64 32 x 32 47 -> 43; 96 -> 96 28 x 28, 100 images 31 -> 23; 256 -> 256 8 x 8 45 -> 35.
// 5 x 5: 128 -> 128 on 16 x 16, 64 images 41 -> 31; 32 -> 96 28 x 28, 100 images 42 -> 30; 64 -> 64 32 x 32, 128 images 52 -> 52.
// Backward-data reads the layer's weights as they lie, [Cout][k][k][Cin] (KN): a direct load puts rows of 32 input channels into
// LDS and the transposing read turns them round, in place of a pass over the weights in front of the kernel.  us, with that pass
// -> without: 96 -> 96 32 x 32, 3 x 128 images 78 -> 74; 320 -> 320 16 x 16 156 -> 146; 256 -> 256 8 x 8 41 -> 33; 96 -> 96
// 28 x 28, 100 images 25.5 -> 22.4; 3 x 16 images of 128 -> 128 on 16 x 16 16.4 -> 11.2.
// (Non-temporal stores took 2 to 5 % off the layer, and put as much on the batch-norm that reads its output next.)
//
// LDS: patch pixels and weight rows are 64 bytes (32 channels) without padding, as the direct loads write them; the four
// 16-byte vectors of pixel or row i lie at vector ^ (i / 4 % 4), which puts any sixteen consecutive pixels on different
// banks (the vector a lane loads is chosen accordingly).  Lanes that go on in the next row of an image skip its halo pixels and
// meet others: SQ_LDS_BANK_CONFLICT is 16 to 20 % of SQ_LDS_IDX_ACTIVE over layers of 32 x 32 and 16 x 16, 39 % on 8 x 8.  Two
// patches, a ring of D + 1 weight tiles.
//
// Step t = (channel chunk, tap): 2 x TM x TN products of 16 channels per wavefront.  While its first half is multiplied the
// weight tile of step t + D and a piece of the next chunk's patch are requested and the second half is read from LDS; then
// every wavefront waits until its own loads for step t + 1 have arrived (they return in order, so a count of younger ones
// is enough), the barrier makes all of them visible, and the first half of step t + 1 is read under the products of the
// second.  The barrier also says that tile t - 1 has been read by everyone: its place in the ring is filled in step t.
#include "igemm_halo.h"
#include <math.h>

namespace {

using namespace igemm_dev;
typedef short s4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4v lds_s4v;

constexpr uint32_t kOob = 0x80000000u;
constexpr int kPix = 64;  // bytes of a patch pixel or weight row in LDS: 32 channels

// The tiles of the column blocks of one width.  Items are numbered eight pixel tiles (counted through all replicas), column
// block, tile: ids that differ by 8 share an XCD (see halo_block), and a workgroup's items are `groups` apart, a multiple of
// 8 * nb, so that all of them have the same columns and the column blocks of a pixel tile run on one XCD.
struct PatchPlan {
  int nb;            // column blocks of this kind
  int col0;          // the first of them
  int items;         // pixel tiles of all replicas (padded to eights once, behind the last) x column blocks
  int groups;        // workgroups that share them
  int tiles;         // pixel tiles of all replicas
  FastDiv dRep, dGroup;  // tiles of a replica; items of eight tiles
};

struct PatchArgs {
  ConvGeom g;
  GemmIO io;
  HaloGeom hg;
  PatchPlan wide, last;
};
typedef __attribute__((address_space(4))) const PatchArgs CArgs;

// The kernel's arguments, read again behind every call: what only the change from one tile to the next needs would
// otherwise sit in scalar registers throughout, and spill.
__device__ __forceinline__ CArgs *fresh(CArgs *a) {
  asm volatile("" : "+s"(a));
  return a;
}
__device__ __forceinline__ uint32_t fdivc(uint32_t n, __attribute__((address_space(4))) const FastDiv &f) {
  return (uint32_t)(((uint64_t)n * f.magic) >> f.shift);
}

// S: window side; TM: 32-pixel tiles per wavefront (four wavefronts: 128 or 256 pixels); TN: 32-channel tiles; D: weight tiles in flight;
// LAST: this workgroup's column blocks are args->last; NORM: io.bn_out; KN: io.w_kn.
template <int S, int TM, int TN, int D, bool LAST, bool NORM, bool KN>
__device__ __forceinline__ void conv_patch_body(CArgs *args, char *smem, int first) {
  typedef bf16_t T;
  constexpr int BN = TN * 32, NB = D + 1, RS = S * S;
  constexpr int H_IT = TM == 1 ? 5 : TN == 4 && D == 3 ? 6 : 7;  // wavefront loads of a patch per wavefront, 64 pixels of the workgroup each time
  constexpr int WG = TN * 2;             // wavefront loads of a weight tile, 16 rows each
  constexpr int WI = (WG + 3) / 4;       // per wavefront, at most
  static_assert(H_IT <= RS + 2 - D, "a patch has to be older than the weight tiles that a wait leaves in flight");
  constexpr int STORES = TM * TN * 2;    // stores of a tile per wavefront
  constexpr int TB = BN * kPix;          // bytes of a weight tile
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5;
  const int cv = (lane & 3) ^ ((lane >> 4) & 3);  // channel vector this lane loads
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  const int pbytes = (args->hg.slots + 15) / 16 * 16 * kPix;
  const int wring = 2 * pbytes, lbias = wring + NB * TB, ldump = lbias + 1024, lnorm = ldump + 1024;
  const int Cc = args->g.Cc, chunks = (Cc + 31) >> 5;
  // KN: a weight row of LDS is an output channel of the layer (contraction) with 32 of its input channels (columns), no vectors
  // exchanged; a transposing read has lane l of sixteen address row l / 4, columns 4 (l % 4) .. + 3 of a 4 x 16 block and gives
  // it column l.  Four rows are all banks.
  const int b_l = KN ? (8 * h + ((lane & 15) >> 2)) * kPix + ((lane >> 4) & 1) * 32 + (lane & 3) * 8
                     : (lane & 31) * kPix + ((h ^ ((lane >> 2) & 3)) << 4);
  // bytes from one tap, and from one chunk of channels, to the next
  const uint32_t w_tap = (uint32_t)(KN ? args->g.N : Cc) * 2u, w_chunk = KN ? 32u * RS * w_tap : 64u;
  const int w_live = KN ? (wave & 1) * 16 + (lane >> 2) : cv * 8;  // this lane loads weights of channel w_live of a chunk
  int n0;  // all items of a workgroup have the same columns

  // the item `idx`, if there is one
  auto item_at = [&](CArgs *a, int idx, int &rep, int &tile) {
    const auto *pp = LAST ? &a->last : &a->wide;
    if (idx >= pp->items) return false;
    const int group = (int)fdivc((uint32_t)idx, pp->dGroup), w = idx - group * (int)pp->dGroup.d, t = group * 8 + (w & 7);
    n0 = (pp->col0 + (w >> 3)) * a->hg.bn;
    rep = (int)fdivc((uint32_t)t, pp->dRep), tile = t - rep * (int)pp->dRep.d;
    return t < pp->tiles;  // the last item of its workgroup where it is not: those behind it are further on
  };

  uint32_t h_off[H_IT], b_off[WI];
  u4 a_rsrc, b_rsrc;
  uint64_t bn_base = 0;  // the next item's weights
  auto weights_at = [&](CArgs *a, int rep) { return (uint64_t)((const T *)a->io.w + rep * a->io.w_rs); };
  auto set_weights = [&](uint64_t p) {
    b_rsrc.x = __builtin_amdgcn_readfirstlane((uint32_t)p);
    b_rsrc.y = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32) & 0xffffu);
  };
  auto patch_of = [&](CArgs *a, int rep, int tile) {
    const int P = a->g.P, Hin = a->g.Hin, Win = a->g.Win, HC = a->hg.HC, PRI = a->hg.PRI, slots = a->hg.slots, rows = a->hg.rows;
    const int omin_h = a->hg.omin_h, omin_w = a->hg.omin_w;
    const int row0 = tile * a->hg.TH, b0 = (int)fdivc((uint32_t)row0, a->hg.dP), p0 = row0 - b0 * P;
    const int first_rows = P - 1 - p0 + a->g.R;
    a_rsrc = buffer_desc((const T *)a->io.in + rep * a->io.in_rs, (uint32_t)a->io.in_bytes);
#pragma unroll
    for (int it = 0; it < H_IT; ++it) {
      const int slot = (it * 4 + wave) * 16 + (lane >> 2);
      const int pr = (int)fdivc((uint32_t)slot, a->hg.dHC), pc = slot - pr * HC;
      int b = b0, ih = p0 + pr + omin_h;
      if (pr >= first_rows) {
        const int rest = pr - first_rows, img = (int)fdivc((uint32_t)rest, a->hg.dPRI);
        b = b0 + 1 + img, ih = rest - img * PRI + omin_h;
      }
      const int iw = pc + omin_w;
      const bool ok = slot < slots && b * P < rows && (unsigned)ih < (unsigned)Hin && (unsigned)iw < (unsigned)Win;
      h_off[it] = ok ? (uint32_t)((((b * Hin + ih) * Win + iw) * Cc + cv * 8) * 2) : kOob;
    }
  };
  auto load_piece = [&](int it, int buf, uint32_t soff, bool live) {
    // a tile fills three quarters of its pixels at least; pieces beyond the patch go where nothing is read
    const int o = (it * 4 + wave) * 1024;
    dma16(lds0 + (uint32_t)(it * 64 + 64 <= TM * 96 || o < pbytes ? buf * pbytes + o : ldump), a_rsrc, live ? h_off[it] : kOob, soff);
  };
  auto load_w = [&](int ring, uint32_t soff, bool live) {
#pragma unroll
    for (int i = 0; i < WI; ++i)
      if (WG % 4 == 0 || wave + 4 * i < WG)
        dma16(lds0 + (uint32_t)(wring + ring + (wave + 4 * i) * 1024), b_rsrc, live ? b_off[i] : kOob, soff);
  };
  // the bias of a column block, zeros without one
  auto load_bias = [&](CArgs *a, int rep, int buf) {
    if (wave * 64 < BN) {
      const int n = n0 + wave * 64 + lane;
      const u4 rsrc = buffer_desc(a->io.bias + rep * a->io.bias_rs, a->io.bias ? (uint32_t)a->g.N * 4u : 0u);
      dma4(lds0 + (uint32_t)(lbias + buf * 512 + wave * 256), rsrc, n < a->g.N ? (uint32_t)n * 4u : kOob);
    }
  };
  // All but the D - 1 newest weight tiles of this wavefront have arrived, and what was requested before them; `extra`: the
  // stores of the tile before, or the loads for the epilogue, as many, are younger than the weight tile that is waited for.
  auto wait_tiles = [&](bool extra) {
    if (WG % 4 != 0 && wave >= WG % 4) {
      if (extra)
        wait_loads<(WI - 1) * (D - 1) + STORES>();
      else
        wait_loads<(WI - 1) * (D - 1)>();
    } else {
      if (extra)
        wait_loads<WI * (D - 1) + STORES>();
      else
        wait_loads<WI * (D - 1)>();
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
    const int P = a->g.P, Q = a->g.Q, TH = a->hg.TH, HC = a->hg.HC, PRI = a->hg.PRI;
    const int row0 = tile * TH, b0 = (int)fdivc((uint32_t)row0, a->hg.dP), p0 = row0 - b0 * P;
    const int first_rows = P - 1 - p0 + a->g.R;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      const int ml = wave * (TM * 32) + tm * 32 + (lane & 31);
      int i = (int)fdivc((uint32_t)ml, a->g.dQ);
      const int q = ml - i * Q;
      i = i < TH ? i : 0;
      const int row = row0 + i, b = (int)fdivc((uint32_t)row, a->hg.dP), p = row - b * P;
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

  // tap (r, c) of a forward pass lies r rows and c columns into the patch, of a backward-data pass S - 1 - r and S - 1 - c
  const int pix_step = args->g.sr > 0 ? kPix : -kPix, row_step = args->hg.HC * pix_step;
  const int tap0 = args->g.sr > 0 ? 0 : (S - 1) * (args->hg.HC + 1) * kPix;
  auto read_kn = [&](const char *p) {
    const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v *)p);
    const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v *)(p + 4 * kPix));
    return __builtin_bit_cast(u4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  int a_ad[TM];
  u4 fa_a[TM], fa_b[TN], fb_a[TM], fb_b[TN];
  auto read0 = [&](int shift, int ring) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      const int a = a_b[tm] + shift;
      a_ad[tm] = a ^ ((a >> 4) & 0x30);
      fa_a[tm] = *(const u4 *)(smem + a_ad[tm]);
    }
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) fa_b[tn] = KN ? read_kn(smem + (wring + ring + b_l) + tn * 32 * kPix) : *(const u4 *)(smem + (wring + ring + b_l) + tn * 32 * kPix);
  };
  auto read1 = [&](int ring) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) fb_a[tm] = *(const u4 *)(smem + (a_ad[tm] ^ 32));
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
      fb_b[tn] = KN ? read_kn(smem + (wring + ring + b_l) + (tn * 32 + 16) * kPix) : *(const u4 *)(smem + (wring + ring + (b_l ^ 32)) + tn * 32 * kPix);
  };
  auto mma_sub = [&](const u4 (&af)[TM], const u4 (&bf)[TN]) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) mma<T>(bf[tn], af[tm], acc[tm][tn]);
  };
  auto interleave = [&]() {
    if constexpr (KN) {
#pragma unroll
      for (int i = 0; i < TM * TN; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
    } else {
#pragma unroll
      for (int i = 0; i < TM + TN; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - TM - TN, 0);
    }
  };

  // Outputs: after the exchanges lane l holds channels 16 * (l / 16 % 2) + 8 * (l / 32) .. + 7 of pixel l % 16 (+ 16) of a tile
  // of 32 pixels x 32 channels.
  uint32_t row_off[TM][2];  // of channel n0 + chan of this lane's pixels
  const int chan = 16 * ((lane >> 4) & 1) + 8 * h;
  auto rows_of = [&](CArgs *a, int tile) {
    const int m0 = tile * a->hg.TH * a->g.Q, mend = min(a->g.M, m0 + a->hg.TH * a->g.Q), ldc = a->io.ldc;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int m = m0 + wave * (TM * 32) + tm * 32 + j * 16 + (lane & 15);
        row_off[tm][j] = m < mend ? ((uint32_t)m * (uint32_t)ldc + (uint32_t)(n0 + chan)) * 2u : kOob;
      }
  };
  auto off = [&](int N, int tm, int j, int tn) { return n0 + tn * 32 + chan < N ? row_off[tm][j] + tn * 64u : kOob; };
  // a tensor of the output's shape
  auto out_like = [&](CArgs *a, const void *p, long long rs, int rep) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p + rep * rs), 0, p ? (int)((uint32_t)a->g.M * (uint32_t)a->io.ldc * 2u) : 0,
                                             0x00020000);
  };
  // The first of mask, residual and old output that there is (mask and old output: the second one takes its place).  All of it
  // is requested before the tile's first store: a load behind a store is waited for until the store is done (residual of 64
  // channels on 32 x 32: 56 us a layer instead of 42).  Lanes beyond the layer's channels read what follows: offsets of their
  // own would be computed in registers that loads of the tile before may still be on their way to, behind a wait for everything.
  constexpr bool kEarly = TN < 4;  // registers for it beside the last fragments
  u4 ex[TM][2][TN];
  auto load_like = [&](__amdgpu_buffer_rsrc_t r, int tm, int tn) {
#pragma unroll
    for (int j = 0; j < 2; ++j) ex[tm][j][tn] = __builtin_amdgcn_raw_buffer_load_b128(r, row_off[tm][j] + tn * 64u, 0, 0);
  };
  auto load_extra = [&](CArgs *a, int rep, int tm) {
    const void *p = a->io.mask;
    long long rs = a->io.mask_rs;
    if (!p) p = a->io.resid, rs = a->io.resid_rs;
    if (!p && a->io.accumulate) p = a->io.out, rs = a->io.out_rs;
    if (!p) return;
    const __amdgpu_buffer_rsrc_t r = out_like(a, p, rs, rep);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) load_like(r, tm, tn);
  };
  // stores eight channels of a pixel; NORM: and what the batch-norm + ReLU behind the layer makes of them
  auto put = [&](CArgs *a, int rep, const u4 &o, uint32_t at, int tn, __amdgpu_buffer_rsrc_t o_rsrc, __amdgpu_buffer_rsrc_t n_rsrc) {
    if (!NORM || !a->io.bn_only) __builtin_amdgcn_raw_buffer_store_b128(o, o_rsrc, at, 0, 0);
    if constexpr (NORM) {
      const char *p = smem + lnorm + (tn * 32 + chan) * 4;  // means, 1/sigma, gamma, beta of the column block
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
  };
  auto half_of = [](uint32_t w, int e) { return __uint_as_float(e ? w & 0xffff0000u : w << 16); };
  auto store_item = [&](CArgs *a, int rep, int tile, int bias_buf) {
    const bool relu = a->io.relu, mask = !NORM && a->io.mask, resid = a->io.resid, accumulate = !NORM && a->io.accumulate;
    const __amdgpu_buffer_rsrc_t o_rsrc = out_like(a, a->io.out, a->io.out_rs, rep);
    auto bias_of = [&](int tn, int vg) { return *(const f4 *)(smem + lbias + bias_buf * 512 + (tn * 32 + vg * 8 + h * 4) * 4); };
    const bool two = mask && accumulate;
    const int N = a->g.N;
    const __amdgpu_buffer_rsrc_t n_rsrc = out_like(a, NORM ? a->io.bn_out : nullptr, a->io.out_rs, rep);
#pragma unroll
    for (int tm = kEarly ? TM : 0; tm < TM; ++tm) load_extra(a, rep, tm);
    // a tile's sums with the bias, exchanged: [channels 0 .. 15 / 16 .. 31][first / second four of a vector][e]
    auto exchanged = [&](int tm, int tn, uint32_t (&d)[2][2][4]) {
#pragma unroll
      for (int vg = 0; vg < 4; ++vg) {
        const f4 b = bias_of(tn, vg);
#pragma unroll
        for (int e = 0; e < 4; ++e) d[vg >> 1][vg & 1][e] = __float_as_uint(acc[tm][tn][4 * vg + e] + b[e]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        swap32(d[0][0][e], d[0][1][e]), swap32(d[1][0][e], d[1][1][e]);
        swap16(d[0][0][e], d[1][0][e]), swap16(d[0][1][e], d[1][1][e]);
      }
    };
    if (kEarly && two) {  // the masked sums stay where the sums were, the old output comes where the mask was
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
          uint32_t d[2][2][4];
          exchanged(tm, tn, d);
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              float v = __uint_as_float(d[j][e >> 2][e & 3]);
              if (relu) v = v > 0.f ? v : 0.f;
              acc[tm][tn][j * 8 + e] = half_of(ex[tm][j][tn][e >> 1], e & 1) > 0.f ? v : 0.f;
            }
          load_like(o_rsrc, tm, tn);
        }
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            u4 o;
#pragma unroll
            for (int k = 0; k < 4; ++k)
              o[k] = f32x2_to_bf16x2(acc[tm][tn][j * 8 + 2 * k] + half_of(ex[tm][j][tn][k], 0), acc[tm][tn][j * 8 + 2 * k + 1] + half_of(ex[tm][j][tn][k], 1));
            put(a, rep, o, off(N, tm, j, tn), tn, o_rsrc, n_rsrc);
          }
      return;
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      if (!resid && !accumulate) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
          uint32_t d[4][2];
#pragma unroll
          for (int vg = 0; vg < 4; ++vg) {
            f4 v = f4{acc[tm][tn][4 * vg], acc[tm][tn][4 * vg + 1], acc[tm][tn][4 * vg + 2], acc[tm][tn][4 * vg + 3]} + bias_of(tn, vg);
            if (relu) {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_fmed3f(v[e], 0.f, __builtin_inff());  // NaN: 0
            }
            d[vg][0] = f32x2_to_bf16x2(v.x, v.y), d[vg][1] = f32x2_to_bf16x2(v.z, v.w);
          }
#pragma unroll
          for (int k = 0; k < 2; ++k) swap32(d[0][k], d[1][k]), swap32(d[2][k], d[3][k]);
          u4 o[2] = {{d[0][0], d[0][1], d[1][0], d[1][1]}, {d[2][0], d[2][1], d[3][0], d[3][1]}};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            uint32_t lo = o[0][k], hi = o[1][k];
            swap16(lo, hi);
            o[0][k] = lo, o[1][k] = hi;
          }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            if (mask) {
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                // keeps where the mask is 1 .. 0x7f80, the positive numbers and infinity
                typedef unsigned short us2 __attribute__((ext_vector_type(2)));
                us2 t = __builtin_bit_cast(us2, (uint32_t)ex[tm][j][tn][k]) - us2{1, 1};
                t = __builtin_elementwise_sub_sat(us2{0x7f80, 0x7f80}, t);
                t = __builtin_elementwise_min(t, us2{1, 1});
                t = us2{0, 0} - t;
                o[j][k] &= __builtin_bit_cast(uint32_t, t);
              }
            }
            put(a, rep, o[j], off(N, tm, j, tn), tn, o_rsrc, n_rsrc);
          }
        }
      } else {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
          u4 ov[2] = {ex[tm][0][tn], ex[tm][1][tn]};
          if (!kEarly && two) {
#pragma unroll
            for (int j = 0; j < 2; ++j) ov[j] = __builtin_amdgcn_raw_buffer_load_b128(o_rsrc, row_off[tm][j] + tn * 64u, 0, 0);
          }
          uint32_t d[2][2][4];
          exchanged(tm, tn, d);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            u4 o;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              float v[2];
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                v[e] = __uint_as_float(d[j][k >> 1][2 * (k & 1) + e]);
                if (resid) v[e] += half_of(ex[tm][j][tn][k], e);
                if (relu) v[e] = v[e] > 0.f ? v[e] : 0.f;
                if (!kEarly && mask) v[e] = half_of(ex[tm][j][tn][k], e) > 0.f ? v[e] : 0.f;
                if (accumulate) v[e] += half_of(ov[j][k], e);
              }
              o[k] = f32x2_to_bf16x2(v[0], v[1]);
            }
            put(a, rep, o, off(N, tm, j, tn), tn, o_rsrc, n_rsrc);
          }
        }
      }
    }
  };

  int idx = first, rep, tile;
  if (!item_at(args, idx, rep, tile)) return;
  patch_of(args, rep, tile);
  b_rsrc = buffer_desc((const void *)weights_at(args, rep), (uint32_t)((long long)args->g.N * args->g.K * sizeof(T)));
#pragma unroll
  for (int i = 0; i < WI; ++i) {
    if (KN) {
      const int n = n0 + ((wave + 4 * i) >> 1) * 32 + (lane & 3) * 8;
      b_off[i] = n < args->g.N ? (uint32_t)w_live * RS * w_tap + (uint32_t)n * 2u : kOob;
    } else {
      const int nrow = n0 + (wave + 4 * i) * 16 + (lane >> 2);
      b_off[i] = nrow < args->g.N ? (uint32_t)((nrow * args->g.K + cv * 8) * 2) : kOob;
    }
  }
  {
    const bool live = cv * 8 < Cc;
    load_bias(args, rep, 0);
#pragma unroll
    for (int it = 0; it < H_IT; ++it) load_piece(it, 0, 0, live);
#pragma unroll
    for (int i = 0; i < D; ++i) load_w(i * TB, (uint32_t)i * w_tap, w_live < Cc);
  }
  if (NORM && tid < BN) {
    const int n = min(n0 + tid, args->g.N - 1);
    float *p = (float *)(smem + lnorm) + tid;
    p[0] = args->io.bn_running[n], p[BN] = 1.0f / sqrtf(args->io.bn_running[args->g.N + n] + kBnEps);
    p[2 * BN] = args->io.bn_gamma[n], p[3 * BN] = args->io.bn_beta[n];
  }
  wait_tiles(false);
  meet();
  int ring = 0, pbuf = 0, bbuf = 0;
  const bool has_extra = args->io.mask || args->io.resid || args->io.accumulate;
  bool later = false;  // not the first item: the stores of the one before it are in flight
  for (;;) {
    begin(fresh(args), tile);
    read0(tap0 + pbuf * pbytes, ring);
    int rep1 = rep, tile1 = tile;
    bool more = false;
    for (int c = 0; c < chunks; ++c) {
      const bool last = c + 1 == chunks;
      const bool live = c * 32 + w_live < Cc;
      if (last) {
        CArgs *a = fresh(args);
        idx += LAST ? a->last.groups : a->wide.groups;
        more = item_at(a, idx, rep1, tile1);
        if (more) {
          patch_of(a, rep1, tile1);
          bn_base = weights_at(a, rep1);
        } else {
#pragma unroll
          for (int it = 0; it < H_IT; ++it) h_off[it] = kOob;
        }
      }
      const int c1 = last ? 0 : c + 1;
      const bool live1 = c1 * 32 + cv * 8 < Cc, w_live1 = c1 * 32 + w_live < Cc;
      int shift = tap0 + pbuf * pbytes;                 // of the tap after this one
      uint32_t soff = D * w_tap + (uint32_t)c * w_chunk;  // of the weight tile that is requested
#pragma unroll
      for (int tap = 0; tap < RS; ++tap) {
        const int prev = ring == 0 ? (NB - 1) * TB : ring - TB, next = ring == (NB - 1) * TB ? 0 : ring + TB;
        read1(ring);
        // The buffer is the one that the item before this one took its bias from, behind its last barrier: with a single chunk
        // the barrier of tap 0 is the first that all wavefronts reach after it, and replicas differ.
        if (tap == 1 && last && more) load_bias(fresh(args), rep1, bbuf ^ 1);
        if (tap < H_IT) load_piece(tap, pbuf ^ 1, (uint32_t)(c1 * 64), live1);
        if (tap + D == RS) {
          soff = (uint32_t)c1 * w_chunk;
          if (last && more) set_weights(bn_base);
        }
        load_w(prev, soff, tap + D >= RS ? w_live1 : live);
        soff += w_tap;
        if (tap + D == RS && last) {
          // behind the weight tile that the last wait is for
          CArgs *a = fresh(args);
          rows_of(a, tile);
          if (kEarly) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) load_extra(a, rep, tm);
          }
        }
        mma_sub(fa_a, fa_b);
        interleave();
        wait_tiles((tap < D - 1 && c == 0 && later) || (kEarly && tap + D >= RS && last && has_extra));
        meet();
        shift += tap % S == S - 1 ? row_step - (S - 1) * pix_step : pix_step;
        if (tap + 1 < RS)
          read0(shift, next);
        else if (!last)
          read0(tap0 + (pbuf ^ 1) * pbytes, next);
        mma_sub(fb_a, fb_b);
        if (tap + 1 < RS) interleave();
        ring = next;
      }
      pbuf ^= 1;
    }
    store_item(fresh(args), rep, tile, bbuf);
    if (!more) break;
    rep = rep1, tile = tile1, later = true, bbuf ^= 1;
  }
  wait_loads<0>();  // nothing may land in LDS after the workgroup has ended
}

template <int S, int TM, int TN, int TL, int D, bool NORM, bool KN>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(TM == 1 ? 3 : 2))) void k_conv_patch(const PatchArgs) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  CArgs *args = (CArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  const int groups = args->wide.groups;
  if ((int)blockIdx.x < groups)
    conv_patch_body<S, TM, TN, D, false, NORM, KN>(args, smem, blockIdx.x);
  else if (TL != TN)
    conv_patch_body<S, TM, TL, D, true, NORM, KN>(args, smem, blockIdx.x - groups);
}

template <int S, int TM, int TN, int TL, int D, bool NORM, bool KN>
hipError_t run_patch_as(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io, HaloGeom hg) {
  constexpr int kCus = 256, kLdsOfCu = 160 * 1024;
  const int lds = 2 * ((hg.slots + 15) / 16 * 16) * kPix + (D + 1) * TN * 32 * kPix + 2048 + (NORM ? TN * 32 * 16 : 0);
  // workgroups that the chip holds at once: by registers, by LDS
  const int resident = kCus * (kLdsOfCu / lds < (TM == 1 ? 3 : 2) ? kLdsOfCu / lds : (TM == 1 ? 3 : 2));
  hg.tiles = (hg.rows + hg.TH - 1) / hg.TH;
  hg.bn = TN * 32;
  hg.nb = (g.N + hg.bn - 1) / hg.bn;
  const int tiles = hg.tiles * replicas;
  auto plan = [&](int nb, int col0) {
    PatchPlan p{};
    p.nb = nb, p.col0 = col0, p.tiles = tiles, p.items = (tiles + 7) / 8 * 8 * nb;
    p.dRep = make_fastdiv(hg.tiles), p.dGroup = make_fastdiv(8 * (nb > 0 ? nb : 1));
    return p;
  };
  PatchArgs pa{g, io, hg, plan(TL == TN ? hg.nb : hg.nb - 1, 0), plan(TL == TN ? 0 : 1, hg.nb - 1)};
  PatchPlan &wide = pa.wide, &last = pa.last;
  if ((long long)tiles * hg.nb <= resident) {  // workgroups of the padding end at once
    wide.groups = wide.items, last.groups = last.items;
  } else if (last.items == 0) {
    const int step = 8 * wide.nb;
    wide.groups = resident / step * step;
    if (wide.groups == 0 || wide.groups > wide.items) wide.groups = wide.items;
  } else {
    // shares of the two widths that end at about the same time
    long long best = -1;
    wide.groups = wide.items, last.groups = last.items;  // very wide layers: no share is a multiple
    for (int a = 8 * wide.nb; a < resident; a += 8 * wide.nb) {
      const long long ra = (wide.items + a - 1) / a * TN, rb = (last.items + resident - a - 1) / (resident - a) * TL;
      const long long worst = ra > rb ? ra : rb;
      if (best < 0 || worst < best) best = worst, wide.groups = a, last.groups = resident - a;
    }
  }
  static const hipError_t lds_ok =
      hipFuncSetAttribute((const void *)k_conv_patch<S, TM, TN, TL, D, NORM, KN>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsOfCu);
  if (lds_ok != hipSuccess) return lds_ok;
  hipLaunchKernelGGL((k_conv_patch<S, TM, TN, TL, D, NORM, KN>), dim3(wide.groups + last.groups), dim3(kThreads), lds, st, pa);
  return hipGetLastError();
}

template <int TM, int TN, int TL, int D>
hipError_t run_patch(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io, const HaloGeom &hg) {
  if (io.w_kn)
    return g.S == 5 ? run_patch_as<5, TM, TN, TL, D, false, true>(st, replicas, g, io, hg)
                    : run_patch_as<3, TM, TN, TL, D, false, true>(st, replicas, g, io, hg);
  if (g.S == 5) return run_patch_as<5, TM, TN, TL, D, false, false>(st, replicas, g, io, hg);
  return io.bn_out ? run_patch_as<3, TM, TN, TL, D, true, false>(st, replicas, g, io, hg)
                   : run_patch_as<3, TM, TN, TL, D, false, false>(st, replicas, g, io, hg);
}

// us per step of a workgroup that has its compute unit to itself, and what every further workgroup of it adds (measured over
// 23 layers of 64 to 320 channels, 7 x 7 to 32 x 32, 16 to 384 images, in each of the five shapes).  `extra`: us that a mask,
// residual or old output to read adds to an epilogue, twice that with two of them (fitted to 792 layers of 16 to 640 channels;
// 96 columns run short of registers for them, and 128 hold them in part only).  In a short contraction, of at most 18 steps
// (64 channels under 3 x 3), it comes with every workgroup, in a long one with the last: others of the compute unit hide it.
struct PatchShape {
  int tm, tn;
  float first, more, extra;
};
constexpr PatchShape kShapes[] = {
    {1, 2, .16f, .12f, 0.f}, {1, 3, .28f, .17f, 0.f}, {2, 2, .28f, .23f, 0.f}, {2, 3, .33f, .31f, 4.f}, {2, 4, .46f, .40f, 8.f}};

// The shape with the shortest estimate.  Within 3 % of the best one on 20 of the 23 layers, 4 to 11 % on the others.  The
// small ones keep launches of few tiles spread over the chip (16 images of 32 x 32 x 96: 10.1 us at 128 x 64, 15.0 at
// 256 x 96), the large ones need less of LDS and of the barriers per product (3 x 128 images: 90.7 and 68.8).  Short
// contractions with something to read in the epilogue run narrow: 32 -> 128 on 15 x 15, 240 images, residual, 22.4 us at 128
// columns, 13.8 at 64.
// False where the kernel through registers is the faster one: a residual, or an old output without a mask, is added in fp32
// behind twice the exchanges, which the 9 steps of a single chunk do not hide once workgroups have more than one tile (16 -> 256
// channels on 35 x 30, 8 x 66 images 216 us, the other 164; 32 -> 32 on 40 x 40 47 / 42).  Longer ones are 0.8 to 1.13 of it.
bool choose_shape(int replicas, const ConvGeom &g, const GemmIO &io, PatchShape &best, HaloGeom &hg_best) {
  HaloGeom geom[2];
  const bool ok[2] = {make_halo_geom(g, geom[0], true), make_halo_geom(g, geom[1], false)};
  const int steps = (g.Cc + 31) / 32 * g.R * g.S, extras = (io.mask ? 1 : 0) + (io.resid || io.accumulate ? 1 : 0);
  float least = 0.f;
  double least_groups = 0.;
  for (const PatchShape &s : kShapes) {
    if (!ok[s.tm - 1] || (s.tn > 2 && g.N <= 64)) continue;
    const HaloGeom &hg = geom[s.tm - 1];
    const int nb = (g.N + s.tn * 32 - 1) / (s.tn * 32), last = g.N - (nb - 1) * s.tn * 32;
    const double tiles = (double)((hg.rows + hg.TH - 1) / hg.TH) * replicas;
    double groups = tiles * nb;
    if (groups > 512. && s.tn > 2 && last <= 64) groups = tiles * (nb - 1 + 2. / s.tn);  // a narrow last block takes less
    const float ranks = (float)ceil(groups / 256.);
    const float t = (s.first + (ranks - 1.f) * s.more) * steps + extras * s.extra * (steps <= 18 ? ranks : 1.f);
    if (least == 0.f || t < least) least = t, least_groups = groups, best = s, hg_best = hg;
  }
  if (!io.bn_out && !io.mask && extras && steps <= 9 && least_groups > 512.) return false;
  return least > 0.f;
}

}  // namespace

bool conv_patch_applicable(int replicas, const ConvGeom &g, const GemmIO &io) {
  PatchShape s;
  HaloGeom hg;
  return g.R == g.S && (g.S == 3 || (g.S == 5 && !io.bn_out)) && g.sp == 1 && g.dshift == 0 && g.Cc % 8 == 0 && io.vecA && io.vecB && g.N % 8 == 0 && io.ldc % 8 == 0 &&
         !io.stat && aligned_to(io.out, 16) && io.out_rs % 8 == 0 && aligned_to(io.resid, 16) && io.resid_rs % 8 == 0 &&
         aligned_to(io.mask, 16) && io.mask_rs % 8 == 0 && !((io.resid || io.bn_out) && (io.mask || io.accumulate)) && aligned_to(io.bn_out, 16) && choose_shape(replicas, g, io, s, hg);
}

// In column blocks of 64 every product needs one transposing read or more beside its other operand.  us of the kernel, as they lie /
// turned round, 3 x 128 images: 64 -> 64 on 32 x 32 (256 x 64 tiles) 43.2 / 41.4, 128 -> 128 on 16 x 16 (128 x 64) 36.7 / 37.5, with
// the reads of a weight gradient beside it; in blocks of 96 192 -> 192 on 16 x 16 59 / 63.  A step with blocks of 64 either way:
// WRN-16-4 (three replicas of 128) 2.232 / 2.207 ms, one replica 1.202 / 1.187, All-CNN of 64 and 128 channels 0.657 / 0.650;
// with those of 96 turned round as well, All-CNN of 96 and 192 1.008 / 1.030.
bool dgrad_turned_is_faster(int dtype, int replicas, const ConvGeom &g, const GemmIO &io) {
  PatchShape s;
  HaloGeom hg;
  return dtype == 1 && g.dshift == 0 && conv_patch_applicable(replicas, g, io) && choose_shape(replicas, g, io, s, hg) && s.tn == 2;
}

hipError_t launch_conv_patch(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io) {
  PatchShape s;
  HaloGeom hg;
  if (!choose_shape(replicas, g, io, s, hg)) return hipErrorInvalidValue;
  const int width = s.tn * 32;
  const bool narrow = g.N - ((g.N + width - 1) / width - 1) * width <= 64;  // the last column block
  if (s.tm == 1) {
    if (s.tn == 2) return run_patch<1, 2, 2, 3>(st, replicas, g, io, hg);
    return narrow ? run_patch<1, 3, 2, 3>(st, replicas, g, io, hg) : run_patch<1, 3, 3, 3>(st, replicas, g, io, hg);
  }
  if (s.tn == 2) return run_patch<2, 2, 2, 3>(st, replicas, g, io, hg);
  if (s.tn == 3) return narrow ? run_patch<2, 3, 2, 3>(st, replicas, g, io, hg) : run_patch<2, 3, 3, 3>(st, replicas, g, io, hg);
  // two workgroups in the LDS of a compute unit: one weight tile less beside the larger patches
  if (hg.slots > 352) return narrow ? run_patch<2, 4, 2, 2>(st, replicas, g, io, hg) : run_patch<2, 4, 4, 2>(st, replicas, g, io, hg);
  return narrow ? run_patch<2, 4, 2, 3>(st, replicas, g, io, hg) : run_patch<2, 4, 4, 3>(st, replicas, g, io, hg);
}

bool conv_takes_bn(int dtype, int replicas, const ConvGeom &g, const GemmIO &io, bool out_f32) {
  if (replicas != 1 || conv_smallk_applicable(dtype, g, io)) return false;
  if (patch_s2_applicable(dtype, replicas, g, io, out_f32)) return true;
  return conv_halo_applicable(dtype, replicas, g, io, out_f32) && conv_patch_applicable(replicas, g, io);
}
