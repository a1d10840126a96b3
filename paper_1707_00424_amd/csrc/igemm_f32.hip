// fp32 convolutions (window larger than 1 x 1; forward with stride 1 or 2, backward-data of stride-1 layers) on the bf16
// matrix units, at fp32 accuracy.
//
// What bounds such a layer is the fp32 MFMA rate (157 TFLOP/s dense against 2.5 PFLOP/s in bf16).  An fp32 value is the
// sum of three bf16 values, x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 = x - x0 - x1 (8 + 8 + 8 bits of
// significand and two signs: nothing is lost while x2 is no denormal, from 2^-110 up), so a product is
//   x*y = x0*y0 + (x0*y1 + x1*y0 + x1*y1 + x0*y2 + x2*y0) + terms below 2^-24 |x*y|
// and six v_mfma_f32_32x32x16_bf16 (192 cycles) do what eight v_mfma_f32_32x32x2_f32 (512 cycles) did.  The products are
// exact in fp32; x0*y0 has an accumulator of its own, the five corrections share a second one, and the two are added once
// at the end.  Relative error against 64 bits on random operands, contraction 64 / 864 / 2880 / 32768: fp32 MFMA
// 1.0e-7 / 3.7e-7 / 6.7e-7 / 2.3e-6, this 0.41e-7 / 1.3e-7 / 2.6e-7 / 1.1e-6 (16 products are added per rounding instead
// of 2); with one accumulator for all six it would be 1.1e-7 / 4.2e-7 / 7.8e-7 / 2.8e-6.
// Where an operand is infinite or NaN the corrections are NaN (inf - inf), an operand beyond the largest bf16 value
// (3.39e38; the largest float is 3.40e38) has an infinite x0, and operands below 2^-110 lose bits.  A workgroup that finds
// a result that is not finite, or too small to be sure of (igemm_split.h), runs its contraction a second time with fp32
// MFMA on the values as they are, so such operands give what plain fp32 gives.
//
// The input patch of a workgroup's output pixels is staged once per 16 channels, split as it is stored to LDS (5.5 vector
// instructions per value), and serves all taps.  A tile is a number of whole output rows, counted through all images
// (row b*P + p), so any image size runs: an image that ends inside a tile only adds its own halo rows to the patch.
// 3 x 3, 96 -> 96 channels, 32 x 32, batch 3 x 128 (65 GFLOP): 720 us with fp32 MFMA, 345 us here (190 TFLOP/s of fp32
// work; the matrix units are busy 51 % of the time, the conversions and the epilogue take most of the rest).
#include "igemm_dev.h"
#include "igemm_split.h"

namespace {

using namespace igemm_dev;
typedef unsigned int u2 __attribute__((ext_vector_type(2)));

constexpr int kChunk = 16;             // channels per patch: one MFMA contraction step per tap
constexpr int kPlane = 32;             // bytes of one of the three parts of a pixel's 16 channels
constexpr int kSlotBytes = 3 * kPlane + 16;  // 112 = 28 banks: 16-byte reads of eight consecutive slots hit distinct banks
constexpr int kSlots1 = 368, kSlots2 = 432;  // patch capacity in pixels for 128 / 256 output pixels
constexpr int kSlotsS2 = 578;  // 128 output pixels of a stride-2 layer: 2 x 17 x 17, 17 x 33; two workgroups per compute unit

struct F32Geom {
  int TH;              // output rows per tile
  int HC, slots;       // patch columns; pixels of the largest patch
  int PRI;             // patch rows of a whole image
  int omin_h, omin_w;  // smallest tap offset (input row = sp * output row + offset)
  int rows, tiles, nb;  // output rows of all images, pixel tiles, column blocks
  FastDiv dP, dHC, dPRI;
};

template <int TN, int SLOTS>
constexpr int f32_lds_bytes() {
  constexpr int pipe = (SLOTS + 2 * TN * 32) * kSlotBytes;
  constexpr int stage = 4 * kStageFloats<TN> * (int)sizeof(float);
  return pipe > stage ? pipe : stage;
}

// VL: values per load instruction (4, 2 or 1: the largest that divides the channel count).  ROWS: epilogue through LDS in
// whole rows (output channels a multiple of 4), else straight from the accumulators.
template <int TM, int TN, int SLOTS, int VL, bool ROWS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_conv_f32x3(const ConvGeom g,
                                                                                                const GemmIO io,
                                                                                                const F32Geom fg) {
  constexpr int BN = TN * 32;
  constexpr int H_IT = (SLOTS * 4 + kThreads - 1) / kThreads, B_IT = (BN * 4 + kThreads - 1) / kThreads;
  __shared__ __attribute__((aligned(16))) char smem[f32_lds_bytes<TN, SLOTS>()];
  __shared__ int again;  // whether the tile takes the second pass
  char *const Hs = smem, *const Bs = smem + SLOTS * kSlotBytes;  // patch; two weight tiles

  // column blocks of one pixel tile differ by 8 in the workgroup id: the same XCD, whose L2 then holds the patch for all
  const int per_group = 8 * fg.nb;
  const int group = blockIdx.x / per_group, within = blockIdx.x - group * per_group;
  const int tile = group * 8 + (within & 7), col = within >> 3;
  if (tile >= fg.tiles) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rep = blockIdx.z;
  const int row0 = tile * fg.TH, m0 = row0 * g.Q, n0 = col * BN;
  const int RS = g.R * g.S;
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((const float *)io.in + rep * io.in_rs), 0, (int)io.in_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((const float *)io.w + rep * io.w_rs), 0, (int)((long long)g.N * g.K * 4), 0x00020000);

  const int b0 = (int)fdiv((uint32_t)row0, fg.dP), p0 = row0 - b0 * g.P;
  const int first_rows = g.sp * (g.P - 1 - p0) + g.R;  // patch rows of the first image, should the tile go beyond it
  // patch loader: piece it*256 + tid covers patch pixel piece/4, channels 4*(piece%4) .. +3 of the chunk
  uint32_t h_off[H_IT];
#pragma unroll
  for (int it = 0; it < H_IT; ++it) {
    const int piece = it * kThreads + tid, slot = piece >> 2;
    const int pr = (int)fdiv((uint32_t)slot, fg.dHC), pc = slot - pr * fg.HC;
    int b = b0, ih = g.sp * p0 + pr + fg.omin_h;
    if (pr >= first_rows) {
      const int rest = pr - first_rows, img = (int)fdiv((uint32_t)rest, fg.dPRI);
      b = b0 + 1 + img, ih = rest - img * fg.PRI + fg.omin_h;
    }
    const int iw = pc + fg.omin_w;
    const bool ok = slot < fg.slots && b * g.P < fg.rows && ih >= 0 && ih < g.Hin && iw >= 0 && iw < g.Win;
    h_off[it] = ok ? (uint32_t)(((b * g.Hin + ih) * g.Win + iw) * g.Cc + (piece & 3) * 4) * 4u : kOobOffset;
  }
  uint32_t b_off[B_IT];
#pragma unroll
  for (int i = 0; i < B_IT; ++i) {
    const int piece = i * kThreads + tid, row = piece >> 2, n = n0 + row;
    b_off[i] = row < BN && n < g.N ? (uint32_t)(n * g.K + (piece & 3) * 4) * 4u : kOobOffset;
  }
  // fragment rows of this lane: pixel -> patch slot of tap offset (0, 0)
  int a_lds[TM];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    const int ml = wave * (TM * 32) + tm * 32 + (lane & 31);
    int i = (int)fdiv((uint32_t)ml, g.dQ);
    const int q = ml - i * g.Q;
    i = i < fg.TH ? i : 0;  // rows beyond the tile are dropped by the epilogue
    const int b = (int)fdiv((uint32_t)(row0 + i), fg.dP), p = row0 + i - b * g.P;
    const int pr = b == b0 ? g.sp * (p - p0) : first_rows + (b - b0 - 1) * fg.PRI + g.sp * p;
    a_lds[tm] = (pr * fg.HC + g.sp * q) * kSlotBytes + (lane >> 5) * 16;
  }
  const int b_lds = (lane & 31) * kSlotBytes + (lane >> 5) * 16;

  // a piece of four channels starting at channel c of the chunk's row: beyond the layer's channels it is zero
  auto load_piece = [&](__amdgpu_buffer_rsrc_t rsrc, uint32_t off, uint32_t add, int c) -> u4 {
    if (VL == 4) return __builtin_amdgcn_raw_buffer_load_b128(rsrc, off != kOobOffset && c < g.Cc ? off + add : kOobOffset, 0, 0);
    u4 r;
    if (VL == 2) {
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        const u2 t = __builtin_bit_cast(u2, __builtin_amdgcn_raw_buffer_load_b64(
                                                rsrc, off != kOobOffset && c + e < g.Cc ? off + add + 4u * e : kOobOffset, 0, 0));
        r[e] = t.x, r[e + 1] = t.y;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        r[e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, off != kOobOffset && c + e < g.Cc ? off + add + 4u * e : kOobOffset, 0, 0);
    }
    return r;
  };
  u4 hreg[H_IT];
  auto load_halo = [&](int chunk) {
#pragma unroll
    for (int it = 0; it < H_IT; ++it) hreg[it] = load_piece(a_rsrc, h_off[it], (uint32_t)chunk * kChunk * 4u, chunk * kChunk + (tid & 3) * 4);
  };
  // PLAIN: the values as they are, 16 channels in 64 bytes, for the second pass
  auto store_piece = [&](auto plain, char *slot, int quarter, const u4 &v) {
    if constexpr (decltype(plain)::value) {
      *(u4 *)(slot + quarter * 16) = v;
    } else {
      const float f[4] = {__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
      uint32_t p[3][2];
      split_words<4>(f, p);
#pragma unroll
      for (int s = 0; s < 3; ++s) *(u2 *)(slot + quarter * 8 + s * kPlane) = u2{p[s][0], p[s][1]};
    }
  };
  auto store_halo = [&](auto plain) {
#pragma unroll
    for (int it = 0; it < H_IT; ++it) {
      const int piece = it * kThreads + tid;
      if (SLOTS * 4 % kThreads == 0 || piece < SLOTS * 4) store_piece(plain, Hs + (piece >> 2) * kSlotBytes, piece & 3, hreg[it]);
    }
  };
  // weight tile of step t: channels of chunk t / RS at tap t % RS
  const int chunks = (g.Cc + kChunk - 1) / kChunk, KT = chunks * RS;
  int ld_chunk = 0, ld_tap = 0;
  auto load_b = [&](u4 (&breg)[B_IT]) {
    const uint32_t kb = (uint32_t)(ld_tap * g.Cc + ld_chunk * kChunk) * 4u;
    const int c = ld_chunk * kChunk + (tid & 3) * 4;  // chunk == chunks: beyond the channels, nothing is loaded
#pragma unroll
    for (int i = 0; i < B_IT; ++i) breg[i] = load_piece(b_rsrc, b_off[i], kb, c);
    if (++ld_tap == RS) ld_tap = 0, ++ld_chunk;
  };
  auto store_b = [&](auto plain, int buf, const u4 (&breg)[B_IT]) {
#pragma unroll
    for (int i = 0; i < B_IT; ++i) {
      const int piece = i * kThreads + tid;
      if (BN * 4 % kThreads == 0 || piece < BN * 4)
        store_piece(plain, Bs + (buf * BN + (piece >> 2)) * kSlotBytes, piece & 3, breg[i]);
    }
  };
  auto shift_of = [&](int r, int c) {
    const int dh = g.sr > 0 ? r : g.R - 1 - r, dw = g.sr > 0 ? c : g.S - 1 - c;
    return (dh * fg.HC + dw) * kSlotBytes;
  };

  f16v hi[TM][TN], lo[TM][TN];
  // D = A x B with the pixel index in the registers (rows) for the direct epilogue, in the lanes for the one through LDS
  auto product = [&](auto type, const u4 (&a)[TM], const u4 (&b)[TN], f16v (&acc)[TM][TN]) {
    typedef decltype(type) T;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
        if (ROWS)
          mma<T>(b[tn], a[tm], acc[tm][tn]);
        else
          mma<T>(a[tm], b[tn], acc[tm][tn]);
      }
  };
  auto contract = [&](auto plain) {
    constexpr bool PLAIN = decltype(plain)::value;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int v = 0; v < 16; ++v) hi[tm][tn][v] = 0.f, lo[tm][tn][v] = 0.f;
    u4 rq[2][B_IT];  // weight tiles in flight: the tile stored in step t was requested in step t - 1
    ld_chunk = 0, ld_tap = 0;
    load_halo(0);
    load_b(rq[0]);
    load_b(rq[1]);
    store_halo(plain);
    load_halo(1);
    store_b(plain, 0, rq[0]);
    load_b(rq[0]);
    __syncthreads();
    int chunk = 0, tap_r = 0, tap_s = 0;
    auto step = [&](int t, u4 (&ra)[B_IT]) {  // `ra` holds tile t + 1 and then receives tile t + 3
      const int shift = shift_of(tap_r, tap_s);
      const char *bt = Bs + (t & 1) * BN * kSlotBytes + b_lds;
      constexpr int PARTS = PLAIN ? 2 : 3;  // three parts of 16 channels, or two times eight channels
      u4 a[PARTS][TM], b[PARTS][TN];
#pragma unroll
      for (int s = 0; s < PARTS; ++s) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) a[s][tm] = *(const u4 *)(Hs + a_lds[tm] + shift + s * kPlane);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) b[s][tn] = *(const u4 *)(bt + tn * 32 * kSlotBytes + s * kPlane);
      }
      if constexpr (PLAIN) {
        product(float{}, a[0], b[0], hi);
        product(float{}, a[1], b[1], hi);
      } else {
        product(bf16_t{}, a[0], b[0], hi);
        product(bf16_t{}, a[0], b[1], lo);
        product(bf16_t{}, a[1], b[0], lo);
        product(bf16_t{}, a[1], b[1], lo);
        product(bf16_t{}, a[0], b[2], lo);
        product(bf16_t{}, a[2], b[0], lo);
      }
      if (++tap_s == g.S) {
        tap_s = 0;
        if (++tap_r == g.R) tap_r = 0;
      }
      if (t + 1 < KT) {
        store_b(plain, (t + 1) & 1, ra);
        load_b(ra);
        if (tap_r == 0 && tap_s == 0) {
          __syncthreads();  // every wavefront has its fragments of the old patch
          ++chunk;
          store_halo(plain);
          load_halo(chunk + 1);
        }
        __syncthreads();
      }
    };
    int t = 0;
    for (; t + 1 < KT; t += 2) {
      step(t, rq[1]);
      step(t + 1, rq[0]);
    }
    if (t < KT) step(t, rq[1]);
  };
  if (tid == 0) again = 0;
  contract(std::false_type{});
  SplitRange range;
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) hi[tm][tn][v] += lo[tm][tn][v], range.add(hi[tm][tn][v]);
  if (range.in_doubt()) {
    bool left = false;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int v = 0; v < 16; ++v) left |= out_of_split_range(hi[tm][tn][v]);
    if (__any(left)) again = 1;
  }
  __syncthreads();  // patch and weight tiles are dead
  if (__builtin_expect(again, 0)) {
    // the pass works its addresses out anew: kept through the first pass, they would cost it registers
#pragma unroll
    for (int it = 0; it < H_IT; ++it) asm volatile("" : "+v"(h_off[it]));
#pragma unroll
    for (int i = 0; i < B_IT; ++i) asm volatile("" : "+v"(b_off[i]));
    contract(std::true_type{});
    __syncthreads();
  }
  ConvGeom gt = g;
  gt.M = min(g.M, m0 + fg.TH * g.Q);  // rows beyond the tile belong to the next one
  if (ROWS) {  // the LDS of patch and weight tiles becomes the staging strips
    store_tile_lds<float, TM, TN, false>(gt, io, rep, m0 + wave * TM * 32, n0, lane, hi,
                                         reinterpret_cast<float *>(smem) + wave * kStageFloats<TN>);
  } else {
    store_tile<float, TM, TN, false>(gt, io, rep, m0 + wave * TM * 32, n0, lane, hi);
  }
}

// Rows per tile of `bm` pixels and the patch that takes; false where no whole row, or no patch, fits.
bool tile_rows(const ConvGeom &g, int bm, int slots, F32Geom &fg) {
  fg.HC = g.sp * (g.Q - 1) + g.S;
  for (fg.TH = bm / g.Q; fg.TH > 0; --fg.TH) {
    // images a tile can touch: tiles start at multiples of TH rows
    const int images = g.P % fg.TH == 0 ? 1 : fg.TH % g.P == 0 ? fg.TH / g.P : (fg.TH + g.P - 2) / g.P + 1;
    const int rows = g.sp * (fg.TH - images) + g.R * images;
    if ((long long)rows * fg.HC <= slots) {
      fg.slots = rows * fg.HC;
      return true;
    }
  }
  return false;
}

struct F32Plan {
  int tile;  // index into kF32Tiles
  F32Geom fg;
};
struct F32Tile {
  int tm, tn, slots, sp;
};
constexpr F32Tile kF32Tiles[] = {{2, 2, kSlots2, 1}, {1, 4, kSlots1, 1}, {1, 3, kSlots1, 1}, {2, 1, kSlots2, 1},
                                 {1, 2, kSlots1, 1}, {1, 1, kSlots1, 1}, {1, 2, kSlotsS2, 2}};

bool plan_f32(const ConvGeom &g, int replicas, F32Plan &best) {
  if (g.dshift != 0 || g.R * g.S < 2 || (g.sp != 1 && g.sp != 2) || g.R < g.sp || g.S < g.sp) return false;
  long long best_cost = -1;
  for (int i = 0; i < (int)(sizeof(kF32Tiles) / sizeof(kF32Tiles[0])); ++i) {
    const F32Tile &v = kF32Tiles[i];
    F32Plan p;
    p.tile = i;
    if (v.sp != g.sp || !tile_rows(g, v.tm * 128, v.slots, p.fg)) continue;
    F32Geom &fg = p.fg;
    fg.rows = g.M / g.Q;
    fg.tiles = (fg.rows + fg.TH - 1) / fg.TH;
    fg.nb = (g.N + v.tn * 32 - 1) / (v.tn * 32);
    // cycles of a contraction step on the busiest compute unit: its workgroups' matrix work (192 per 32 x 32 tile), and
    // what a step costs in latency and barrier beside it (about 400), which two resident workgroups share
    const long long per_cu = ((long long)fg.tiles * fg.nb * replicas + 255) / 256;
    const long long cost = per_cu * v.tm * v.tn * 192 + (per_cu + 1) / 2 * 400;
    if (best_cost < 0 || cost < best_cost) best_cost = cost, best = p;
  }
  if (best_cost < 0) return false;
  F32Geom &fg = best.fg;
  // Stride 2 has the one tile of 128 x 64, and a workgroup alone on its compute unit is bound by its chain of steps, where
  // the gather kernel with twice as many workgroups is shorter.  us, gather kernel / here: 64 -> 128 channels on 32 x 32, 128
  // workgroups 20.1 / 23.4, 256 29.7 / 25.5; 128 -> 256 on 16 x 16, 128 34.1 / 42.4, 256 51.9 / 45.0; 96 -> 96 on 28 x 28, 100
  // 26.0 / 33.2, 200 38.7 / 34.4; 32 -> 32 on 32 x 32, 128 12.3 / 13.8, 256 17.9 / 15.1.
  // A long contraction (over 1000) into four or more column blocks, which fetch their weights each, takes a full tile to every
  // compute unit: 128 -> 320 on 28 x 28, 250 workgroups at 126 of 128 pixels 51.6 / 56.6; 256 -> 256 on 14 x 14, 264 at 119 pixels
  // 96 / 112; but 256 -> 50 on 28 x 28, 165 129 / 92.  Odd channel counts are gathered value by value, which a long
  // contraction makes slower than anything here: 65 -> 32 under 5 x 5, 27 workgroups 111 / 66.
  const long long groups = (long long)fg.tiles * fg.nb * replicas;
  if (g.sp == 2 && (g.Cc % 2 == 0 || g.K < 400) && groups * fg.TH * g.Q < (g.K > 1000 && fg.nb > 3 ? 250 : 156) * 128) return false;
  // Short contractions are mostly staging and epilogue, the latter value by value where the output channels are no multiple
  // of 4.  Time here over the gather kernel's, 3 x 3 windows, by (even) input channels: 10 to 50 outputs (no multiple of 4) in
  // large launches, 14 x 14 / 32 x 32 images, 8 1.7 / 1.5, 12 1.4 / 1.2, 16 1.2 / 1.0, 20 1.24 / 0.9 to 1.05, 24 1.15 / 0.95, 32
  // 0.95 / 0.8; 85 outputs 16 1.38; but 151 outputs from 12 up 1.0 / 0.96; 151 outputs in 256 to 512 workgroups 12 1.25, 20
  // 1.16, 24 1.04; small launches 8 1.15, 12 0.93 to 1.0; 16 and 20 outputs in large ones 8 1.15 / 0.98, 12 0.93 / 0.8.
  const int short_k = groups <= 128 || (groups > 512 && g.N > 128) ? 100 : g.Q >= 24 ? 150 : g.N > 32 ? 240 : 216;
  if (g.sp == 1 && g.N % 4 != 0 && g.Cc % 2 == 0 && g.K < short_k) return false;
  if (g.sp == 1 && g.K < 100 && g.N <= 32 && groups > 256) return false;
  fg.PRI = g.sp * (g.P - 1) + g.R;
  const int last_h = g.off + (g.R - 1) * g.sr, last_w = g.off + (g.S - 1) * g.sr;
  fg.omin_h = g.off < last_h ? g.off : last_h, fg.omin_w = g.off < last_w ? g.off : last_w;
  fg.dP = make_fastdiv(g.P), fg.dHC = make_fastdiv(fg.HC), fg.dPRI = make_fastdiv(fg.PRI);
  return true;
}

template <int I, int VL>
hipError_t run_f32(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io, const F32Geom &fg) {
  constexpr F32Tile v = kF32Tiles[I];
  const dim3 grid((fg.tiles + 7) / 8 * 8 * fg.nb, 1, replicas);
  if (g.N % 4 == 0 && io.ldc % 4 == 0)
    hipLaunchKernelGGL((k_conv_f32x3<v.tm, v.tn, v.slots, VL, true>), grid, dim3(kThreads), 0, st, g, io, fg);
  else
    hipLaunchKernelGGL((k_conv_f32x3<v.tm, v.tn, v.slots, VL, false>), grid, dim3(kThreads), 0, st, g, io, fg);
  return hipGetLastError();
}
template <int I>
hipError_t run_f32(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io, const F32Geom &fg) {
  if (g.Cc % 4 == 0) return run_f32<I, 4>(st, replicas, g, io, fg);
  if (g.Cc % 2 == 0) return run_f32<I, 2>(st, replicas, g, io, fg);
  return run_f32<I, 1>(st, replicas, g, io, fg);
}

}  // namespace

bool conv_f32x3_applicable(int dtype, int replicas, const ConvGeom &g, const GemmIO &io) {
  const long long lim = 1LL << 31;
  F32Plan p;
  return dtype == 0 && g.Cc >= 8 && io.in_bytes > 0 && io.in_bytes < lim && (long long)g.N * g.K * 4 < lim &&
         (long long)g.M * io.ldc * 4 < lim && plan_f32(g, replicas, p);
}

hipError_t launch_conv_f32x3(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io) {
  F32Plan p;
  if (!plan_f32(g, replicas, p)) return hipErrorInvalidValue;
  switch (p.tile) {
    case 0: return run_f32<0>(st, replicas, g, io, p.fg);
    case 1: return run_f32<1>(st, replicas, g, io, p.fg);
    case 2: return run_f32<2>(st, replicas, g, io, p.fg);
    case 3: return run_f32<3>(st, replicas, g, io, p.fg);
    case 4: return run_f32<4>(st, replicas, g, io, p.fg);
    case 5: return run_f32<5>(st, replicas, g, io, p.fg);
    default: return run_f32<6>(st, replicas, g, io, p.fg);
  }
}
