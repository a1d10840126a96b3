// Backward-data of a stride-2 3x3 convolution with padding 1 (bf16, channel counts in multiples of 8): output-gradient patch
// and weights loaded straight into LDS, all four parity classes of a position in one wavefront.
//
// Input pixel (2i + a, 2j + c) is reached by the taps of its parity class (a, c):
//   a = 0: window row 1 of dy row i;   a = 1: row 0 of dy row i + 1 and row 2 of dy row i   (columns alike)
// so position (i, j) of the output-gradient grid, which reads dy[i .. i + 1][j .. j + 1], owns four input pixels and nine taps.
//
// What bounded the kernel before this one (igemm_dgrad2.hip, which gives a class to each wavefront; 64 -> 128 channels,
// 32 x 32, 3 x 128 images, 35 us for 75 MB and 14.5 GFLOP): its wavefronts differ four to one in work, operands travelled
// through registers with two barriers per 32 channels, and a pass over the weights turned them round first (5 us).  Here
//   * a wavefront multiplies 32 positions x 4 classes x 32 input channels: the four shifted reads of dy serve nine taps, and
//     all wavefronts do the same work;
//   * patches and the weight tiles of a window row (three taps) come by direct loads, the rows three ahead in a ring;
//   * weights are read as the layer keeps them, [Cout][3][3][Cin]: the transposing LDS read turns a tile of 32 x 32 round;
//   * a workgroup walks several tiles, the first operands of the next one are on their way during the last products of the
//     current one, and mask or old output come with them.
// With all of it three workgroups share a compute unit.  What is left, by leaving parts out: 15 us of LDS reads (a wavefront
// reads 26 KB per 18 products of 32 cycles) and launch, 8 of waiting for operands, 5 of stores.  64 positions per wavefront
// read a third less, but two workgroups remain and the mask no longer fits in registers: 3 to 5 % ahead from 320 output
// channels, 5 to 20 % behind below.
// us per pass, the kernels before (with the turned weights) -> now, 3 x 128 images: 64 -> 128 on 32 x 32 40 -> 28, 96 -> 96 64 ->
// 42 (with mask), 192 -> 192 on 16 x 16 49 -> 32, 160 -> 320 on 32 x 32 190 -> 125, 16 -> 32 19 -> 8.4; images of no power of
// two, which a gather kernel ran: 96 -> 96 on 28 x 28 83 -> 35, 8 x 16 images of 256 -> 256 on 14 x 14 55 -> 19.
//
// LDS: patch pixels of 64 bytes (32 channels), their four vectors exchanged by the pixel's position as in igemm_patch.hip;
// weight rows (tap, output channel) of 32 input channels, 64 bytes: a transposing read takes 4 rows x 64 bytes, all banks.
// The order of an output's sums (channel chunk, window row, window column) is that of igemm_dgrad2.hip.  A gather kernel, which ran
// the other sizes, takes all channels of a tap before the next tap: there 3 to 11 in 100 000 bf16 results round the other way
// than with it; the error against 64 bits is the same to six digits.
#include "igemm_halo.h"
#include <type_traits>

namespace {

using namespace igemm_dev;
typedef short s4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4v lds_s4v;

constexpr uint32_t kOob = 0x80000000u;
constexpr int kPix = 64;                 // bytes of a patch pixel or weight row in LDS: 32 channels
constexpr int kRow = 3 * 32 * kPix;      // bytes of the weight tiles of a window row
constexpr int kRing = 4;                 // of these in LDS: one in use, three on their way
constexpr int kCols = 32;                // input channels of a workgroup

// A tile is a number of whole rows of positions, counted through all images of a replica.
struct PosGeom {
  int TH;     // rows per tile
  int HC;     // patch columns: one more than positions
  int PRI;    // patch rows of a whole image
  int slots;  // pixels of the largest patch
  int rows;   // rows of all images
  FastDiv dH, dW, dHC, dPRI;
};
struct DgradArgs {
  ConvGeom g;
  GemmIO io;
  PosGeom pg;
  int items, groups, tiles;  // see item_at
  FastDiv dRep, dGroup;
};
typedef __attribute__((address_space(4))) const DgradArgs CArgs;

// The arguments, read again behind every call: what only a change of tile needs stays out of the scalar registers.
__device__ __forceinline__ CArgs *fresh(CArgs *a) {
  asm volatile("" : "+s"(a));
  return a;
}
__device__ __forceinline__ uint32_t fdivc(uint32_t n, __attribute__((address_space(4))) const FastDiv &f) {
  return (uint32_t)(((uint64_t)n * f.magic) >> f.shift);
}

template <int N>
using Int = std::integral_constant<int, N>;

constexpr int TM = 1;             // 32-position tiles per wavefront
constexpr int kPositions = 128;   // of a workgroup's tile
constexpr int kMaxSlots = 192;    // pixels of a patch

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_dgrad_patch(const DgradArgs) {
  typedef bf16_t T;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  CArgs *args = (CArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int H_IT = (kMaxSlots / 16 + 3) / 4;  // wavefront loads of a patch per wavefront
  constexpr int EXTRA = TM * 8, STORES = TM * 8;      // loads for the epilogue, ahead of it, and its stores
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5;
  const int cv = (lane & 3) ^ ((lane >> 4) & 3);  // channel vector of a patch pixel this lane loads
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  const int pbytes = (args->pg.slots + 15) / 16 * 16 * kPix, wring = 2 * pbytes, ldump = wring + kRing * kRow;
  const int Cc = args->g.Cc, chunks = (Cc + 31) >> 5;
  int n0;

  // Items are numbered eight tiles (counted through all replicas), column block, tile: ids that differ by 8 share an XCD, so
  // the column blocks of a tile find its patch in that XCD's L2 and their partial lines of dx meet there.  A workgroup's items
  // are `groups` apart, a multiple of 8 x column blocks: all of them have the same columns.
  auto item_at = [&](CArgs *a, int idx, int &rep, int &tile) {
    if (idx >= a->items) return false;
    const int group = (int)fdivc((uint32_t)idx, a->dGroup), w = idx - group * (int)a->dGroup.d, t = group * 8 + (w & 7);
    n0 = (w >> 3) * kCols;
    rep = (int)fdivc((uint32_t)t, a->dRep), tile = t - rep * (int)a->dRep.d;
    return t < a->tiles;  // the last item of its workgroup where it is not
  };

  uint32_t h_off[H_IT];
  u4 a_rsrc, b_rsrc;
  auto operands_of = [&](CArgs *a, int rep, int tile) {
    const int Hin = a->g.Hin, Win = a->g.Win, HC = a->pg.HC, PRI = a->pg.PRI, slots = a->pg.slots, rows = a->pg.rows;
    const int row0 = tile * a->pg.TH, b0 = (int)fdivc((uint32_t)row0, a->pg.dH), p0 = row0 - b0 * Hin;
    const int first_rows = Hin + 1 - p0;
    a_rsrc = buffer_desc((const T *)a->io.in + rep * a->io.in_rs, (uint32_t)a->io.in_bytes);
    b_rsrc = buffer_desc((const T *)a->io.w + rep * a->io.w_rs, (uint32_t)((long long)a->g.N * a->g.K * sizeof(T)));
#pragma unroll
    for (int it = 0; it < H_IT; ++it) {
      const int slot = (it * 4 + wave) * 16 + (lane >> 2);
      const int pr = (int)fdivc((uint32_t)slot, a->pg.dHC), iw = slot - pr * HC;
      int b = b0, ih = p0 + pr;
      if (pr >= first_rows) {
        const int rest = pr - first_rows, img = (int)fdivc((uint32_t)rest, a->pg.dPRI);
        b = b0 + 1 + img, ih = rest - img * PRI;
      }
      const bool ok = slot < slots && b * Hin < rows && ih < Hin && iw < Win;
      h_off[it] = ok ? (uint32_t)((((b * Hin + ih) * Win + iw) * Cc + cv * 8) * 2) : kOob;
    }
  };
  auto load_patch = [&](int c, int buf, bool more) {
    const bool live = more && c * 32 + cv * 8 < Cc;
#pragma unroll
    for (int it = 0; it < H_IT; ++it) {
      const int o = (it * 4 + wave) * 1024;
      dma16(lds0 + (uint32_t)(o < pbytes ? buf + o : ldump), a_rsrc, live ? h_off[it] : kOob, (uint32_t)(c * 64));
    }
  };
  // Weight rows of this lane in the six loads of a window row, 16 rows each: output channel w_co of a chunk, window column
  // wave / 2, and for the first two wavefronts window column 2 as well.
  const int w_co = (wave & 1) * 16 + (lane >> 2);
  const uint32_t w_tap = (uint32_t)(args->g.N * 2), w_row = w_tap * 9u;  // bytes between taps and between output channels
  uint32_t w_off;
  auto load_w = [&](int c, int r, int slot, bool more) {
    const uint32_t off = more && c * 32 + w_co < Cc ? w_off : kOob, soff = (uint32_t)c * 32u * w_row + (uint32_t)(r * 3) * w_tap;
    dma16(lds0 + (uint32_t)(wring + slot + wave * 1024), b_rsrc, off, soff + (uint32_t)(wave >> 1) * w_tap);
    if (wave < 2) dma16(lds0 + (uint32_t)(wring + slot + (wave + 4) * 1024), b_rsrc, off, soff + 2u * w_tap);
  };

  f16v acc[4][TM];
  int a_b[TM];
  uint32_t row_off[TM][2];  // of channel n0 + chan of the even-even pixel of this lane's positions
  uint32_t odd_ok;          // bits 4 tm + 2 j: there is a pixel in the odd row, + 1: column
  const int chan = 16 * ((lane >> 4) & 1) + 8 * h;
  auto begin = [&](CArgs *a, int tile) {
    const int Hin = a->g.Hin, Win = a->g.Win, TH = a->pg.TH, HC = a->pg.HC, PRI = a->pg.PRI, P = a->g.P, Q = a->g.Q;
    const int row0 = tile * TH, b0 = (int)fdivc((uint32_t)row0, a->pg.dH), p0 = row0 - b0 * Hin;
    const int first_rows = Hin + 1 - p0;
    odd_ok = 0;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      {
        const int ml = wave * (TM * 32) + tm * 32 + (lane & 31);
        int i = (int)fdivc((uint32_t)ml, a->pg.dW);
        const int q = ml - i * Win;
        i = i < TH ? i : 0;
        const int row = row0 + i, b = (int)fdivc((uint32_t)row, a->pg.dH), p = row - b * Hin;
        const int pr = b == b0 ? p - p0 : first_rows + (b - b0 - 1) * PRI + p;
        a_b[tm] = (pr * HC + q) * kPix + h * 16;
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int ml = wave * (TM * 32) + tm * 32 + j * 16 + (lane & 15);
        const int i = (int)fdivc((uint32_t)ml, a->pg.dW), q = ml - i * Win;
        const int row = row0 + i, b = (int)fdivc((uint32_t)row, a->pg.dH), p = row - b * Hin;
        const bool ok = i < TH && row < a->pg.rows && n0 + chan < a->g.N;
        row_off[tm][j] = ok ? ((uint32_t)((b * P + 2 * p) * Q + 2 * q) * (uint32_t)a->io.ldc + (uint32_t)(n0 + chan)) * 2u : kOob;
        odd_ok |= (uint32_t)(2 * p + 1 < P) << (4 * tm + 2 * j) | (uint32_t)(2 * q + 1 < Q) << (4 * tm + 2 * j + 1);
      }
    }
#pragma unroll
    for (int cl = 0; cl < 4; ++cl)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[cl][tm][v] = 0.f;
  };
  auto pixel = [&](int cl, int tm, int j, uint32_t row_b, uint32_t col_b) {
    uint32_t o = row_off[tm][j] + (cl & 2 ? row_b : 0u) + (cl & 1 ? col_b : 0u);
    const uint32_t need = (uint32_t)(cl >> 1 | (cl & 1) << 1) << (4 * tm + 2 * j);
    return (odd_ok & need) == need && row_off[tm][j] != kOob ? o : kOob;
  };
  auto out_like = [&](CArgs *a, const void *p, long long rs, int rep) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p + rep * rs), 0, p ? (int)((uint32_t)a->g.M * (uint32_t)a->io.ldc * 2u) : 0,
                                             0x00020000);
  };
  u4 ex[4][TM][2];  // mask, or old output
  auto load_extra = [&](CArgs *a, int rep) {
    const void *p = a->io.mask ? a->io.mask : a->io.accumulate ? a->io.out : nullptr;
    if (!p) return;
    const __amdgpu_buffer_rsrc_t r = out_like(a, p, a->io.mask ? a->io.mask_rs : a->io.out_rs, rep);
    const uint32_t col_b = (uint32_t)a->io.ldc * 2u, row_b = (uint32_t)a->g.Q * col_b;
#pragma unroll
    for (int cl = 0; cl < 4; ++cl)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int j = 0; j < 2; ++j) ex[cl][tm][j] = __builtin_amdgcn_raw_buffer_load_b128(r, pixel(cl, tm, j, row_b, col_b), 0, 0);
  };
  auto half_of = [](uint32_t w, int e) { return __uint_as_float(e ? w & 0xffff0000u : w << 16); };
  auto store_item = [&](CArgs *a, int rep) {
    const bool mask = a->io.mask, accumulate = a->io.accumulate;
    const __amdgpu_buffer_rsrc_t o_rsrc = out_like(a, a->io.out, a->io.out_rs, rep);
    const uint32_t col_b = (uint32_t)a->io.ldc * 2u, row_b = (uint32_t)a->g.Q * col_b;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int cl = 0; cl < 4; ++cl) {
        if (!accumulate) {
          uint32_t d[4][2];
#pragma unroll
          for (int vg = 0; vg < 4; ++vg) {
            d[vg][0] = f32x2_to_bf16x2(acc[cl][tm][4 * vg], acc[cl][tm][4 * vg + 1]);
            d[vg][1] = f32x2_to_bf16x2(acc[cl][tm][4 * vg + 2], acc[cl][tm][4 * vg + 3]);
          }
#pragma unroll
          for (int k = 0; k < 2; ++k) swap32(d[0][k], d[1][k]), swap32(d[2][k], d[3][k]);
#pragma unroll
          for (int k = 0; k < 2; ++k) swap16(d[0][k], d[2][k]), swap16(d[1][k], d[3][k]);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            u4 o = {d[2 * j][0], d[2 * j][1], d[2 * j + 1][0], d[2 * j + 1][1]};
            if (mask) {
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                const uint32_t m = ex[cl][tm][j][k];
                o[k] = (half_of(m, 0) > 0.f ? o[k] & 0xffffu : 0u) | (half_of(m, 1) > 0.f ? o[k] & 0xffff0000u : 0u);
              }
            }
            __builtin_amdgcn_raw_buffer_store_b128(o, o_rsrc, pixel(cl, tm, j, row_b, col_b), 0, 0);
          }
        } else {
          uint32_t d[2][2][4];
#pragma unroll
          for (int vg = 0; vg < 4; ++vg)
#pragma unroll
            for (int e = 0; e < 4; ++e) d[vg >> 1][vg & 1][e] = __float_as_uint(acc[cl][tm][4 * vg + e]);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            swap32(d[0][0][e], d[0][1][e]), swap32(d[1][0][e], d[1][1][e]);
            swap16(d[0][0][e], d[1][0][e]), swap16(d[0][1][e], d[1][1][e]);
          }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const uint32_t at = pixel(cl, tm, j, row_b, col_b);
            u4 old = ex[cl][tm][j];
            if (mask) old = __builtin_amdgcn_raw_buffer_load_b128(o_rsrc, at, 0, 0);
            u4 o;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              float v[2];
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                v[e] = __uint_as_float(d[j][k >> 1][2 * (k & 1) + e]);
                if (mask) v[e] = half_of(ex[cl][tm][j][k], e) > 0.f ? v[e] : 0.f;
                v[e] += half_of(old[k], e);
              }
              o[k] = f32x2_to_bf16x2(v[0], v[1]);
            }
            __builtin_amdgcn_raw_buffer_store_b128(o, o_rsrc, at, 0, 0);
          }
        }
      }
  };

  // a transposing read: lane l of sixteen addresses row l / 4, channels 4 (l % 4) .. + 3 of a 4 x 16 block and receives
  // its column l; rows 8 h (+ 4) + 0 .. 3, columns 16 (lane / 16 % 2) + 0 .. 15
  const int t_l = ((8 * h + ((lane & 15) >> 2)) * kPix) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
  // window row r: dy row i + 1 for r = 0, else i
  auto multiply = [&](int r, int buf, int slot) {
    const int HC = args->pg.HC, di = r == 0;
#pragma unroll
    for (int dj = 1; dj >= 0; --dj)
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        u4 af[TM];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
          const int ad = a_b[tm] + buf + (di * HC + dj) * kPix;
          af[tm] = *(const u4 *)(smem + ((ad ^ ((ad >> 4) & 0x30)) ^ (sub * 32)));
        }
#pragma unroll
        for (int s = dj ? 0 : 2; s >= (dj ? 0 : 1); --s) {
          const int cl = (r != 1) * 2 + (s != 1);
          const char *p = smem + wring + slot + t_l + (s * 32 + sub * 16) * kPix;
          const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v *)p);
          const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v *)(p + 4 * kPix));
          const u4 bf = __builtin_bit_cast(u4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
          for (int tm = 0; tm < TM; ++tm) mma<T>(bf, af[tm], acc[cl][tm]);
        }
      }
  };
  // This wavefront's loads for the next window row have arrived: `YOUNGER` loads and stores, and two rows of weights, were
  // issued behind them.
  auto wait_row = [&](auto younger) {
    constexpr int YOUNGER = decltype(younger)::value;
    if (wave < 2)
      wait_loads<YOUNGER + 4>();
    else
      wait_loads<YOUNGER + 2>();
  };
  auto meet = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  int idx = blockIdx.x, rep, tile;
  if (!item_at(args, idx, rep, tile)) return;
  operands_of(args, rep, tile);
  w_off = n0 + (lane & 3) * 8 < args->g.N ? (uint32_t)w_co * w_row + (uint32_t)(n0 + (lane & 3) * 8) * 2u : kOob;
  load_patch(0, 0, true);
#pragma unroll
  for (int r = 0; r < 3; ++r) load_w(0, r, r * kRow, true);
  wait_row(Int<0>{});
  meet();
  int buf = 0, slot = 0;
  const bool has_extra = args->io.mask || args->io.accumulate;
  bool later = false;  // not the first item: the stores of the one before it are in flight
  for (;;) {
    begin(fresh(args), tile);
    int rep1 = rep, tile1 = tile;
    bool more = true;
    for (int c = 0; c < chunks; ++c) {
      const bool last = c + 1 == chunks;
      if (last) {
        CArgs *a = fresh(args);
        idx += a->groups;
        more = item_at(a, idx, rep1, tile1);
        if (more) operands_of(a, rep1, tile1);
      }
      const int c1 = last ? 0 : c + 1;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        // the row three ahead takes the place of the one before this, which everyone has read
        load_w(c1, r, slot == 0 ? (kRing - 1) * kRow : slot - kRow, more);
        if (r == 0) {
          load_patch(c1, pbytes - buf, more);
          if (last && has_extra) load_extra(fresh(args), rep);
        }
        multiply(r, buf, slot);
        if (r == 2) {
          wait_row(Int<0>{});  // the next patch too
        } else if (later && c == 0) {
          if (last && has_extra)
            wait_row(Int<H_IT + EXTRA + STORES>{});
          else
            wait_row(Int<H_IT + STORES>{});
        } else if (last && has_extra) {
          wait_row(Int<H_IT + EXTRA>{});
        } else {
          wait_row(Int<H_IT>{});
        }
        meet();
        slot = slot == (kRing - 1) * kRow ? 0 : slot + kRow;
      }
      buf = pbytes - buf;
    }
    store_item(fresh(args), rep);
    if (!more) break;
    rep = rep1, tile = tile1, later = true;
  }
  wait_loads<0>();  // nothing may land in LDS after the workgroup has ended
}

// The tiles of a layer; false where they would be less than three quarters full.
bool make_pos_geom(const ConvGeom &g, PosGeom &pg) {
  const int H = g.Hin, W = g.Win;
  pg.HC = W + 1, pg.PRI = H + 1;
  for (pg.TH = kPositions / W; pg.TH > 0; --pg.TH) {
    // images a tile can touch: tiles start at multiples of TH rows
    const int images = H % pg.TH == 0 ? 1 : pg.TH % H == 0 ? pg.TH / H : (pg.TH + H - 2) / H + 1;
    pg.slots = (pg.TH + images) * pg.HC;
    if (pg.slots <= kMaxSlots) break;
  }
  if (pg.TH * W * 4 < kPositions * 3) return false;
  pg.rows = g.M / (g.P * g.Q) * H;
  pg.dH = make_fastdiv(H), pg.dW = make_fastdiv(W), pg.dHC = make_fastdiv(pg.HC), pg.dPRI = make_fastdiv(pg.PRI);
  return true;
}

hipError_t run_dgrad_patch(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io, const PosGeom &pg) {
  constexpr int kCus = 256, kLdsOfCu = 160 * 1024;
  const int lds = 2 * ((pg.slots + 15) / 16 * 16 * kPix) + kRing * kRow + 1024;
  const int per_cu = 3 * lds <= kLdsOfCu ? 3 : 2;
  const int nb = (g.N + kCols - 1) / kCols, rep_tiles = (pg.rows + pg.TH - 1) / pg.TH, tiles = rep_tiles * replicas;
  const long long items = (long long)((tiles + 7) / 8 * 8) * nb;
  if (items >= 1LL << 31) return hipErrorInvalidValue;
  DgradArgs a{g, io, pg, (int)items, (int)items, tiles, make_fastdiv(rep_tiles), make_fastdiv(8 * nb)};
  const int resident = per_cu * kCus, step = 8 * nb;
  if (items > resident && step <= resident) a.groups = resident / step * step;
  static const hipError_t lds_ok =
      hipFuncSetAttribute((const void *)k_dgrad_patch, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsOfCu / 2);
  if (lds_ok != hipSuccess) return lds_ok;
  hipLaunchKernelGGL((k_dgrad_patch), dim3(a.groups), dim3(kThreads), lds, st, a);
  return hipGetLastError();
}

}  // namespace

// g: backward-data geometry of a stride-2 layer; io.w: its weights as they lie.
bool dgrad_patch_applicable(int dtype, const ConvGeom &g, const GemmIO &io) {
  PosGeom pg;
  return dtype == 1 && g.dshift == 1 && g.R == 3 && g.S == 3 && g.off == 1 && g.sr == -1 && g.sp == 1 &&
         g.Hin == (g.P + 1) / 2 && g.Win == (g.Q + 1) / 2 && g.Cc % 8 == 0 && g.N % 8 == 0 && io.vecA && io.vecB && aligned_to(io.w, 16) &&
         io.w_rs % 8 == 0 && aligned_to(io.out, 16) && io.out_rs % 8 == 0 && aligned_to(io.mask, 16) && io.mask_rs % 8 == 0 && io.ldc == g.N &&
         !io.resid && !io.bias && !io.relu && !io.stat && !io.bn_out &&
         (long long)g.M * g.N * 2 < (1LL << 31) && io.in_bytes > 0 && io.in_bytes < (1LL << 31) &&
         (long long)g.N * g.K * 2 < (1LL << 31) && make_pos_geom(g, pg);
}

hipError_t launch_dgrad_patch(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io) {
  PosGeom pg;
  if (!make_pos_geom(g, pg)) return hipErrorInvalidValue;
  return run_dgrad_patch(st, replicas, g, io, pg);
}
