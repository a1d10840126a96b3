// Backward-weight of "same" 3x3 convolutions (bf16) with the input patch staged ONCE in LDS
// and each output-gradient fragment reused by all nine window taps.
//
//   dW[n][r][s][c] = sum over pixels (b, p, q) of dy[b, p, q, n] * x[b, p + r - 1, q + s - 1, c]
//
// The contraction runs over pixels, which is the slow index of both operands in memory
// ([pixel][channel]); MFMA fragments need it contiguous, so they are fetched with the LDS transpose
// read (ds_read_b64_tr_b16), which delivers about half the bandwidth of a plain 16-byte read.  The
// kernel is built to need few of them:
//   * a wavefront owns one 32-channel tile of dy, one 32-channel tile of x and ALL nine taps
//     (nine 32x32 accumulators): one dy fragment serves nine MFMAs;
//   * a contraction sub-step is one row of 16 pixels; the x fragment of (row j, column shift s) is
//     the operand of tap (r, s) for dy row j + 1 - r, so the fragments of three consecutive x rows are
//     kept in registers and each dy row reads only the three fragments of the row that enters;
//   * per 9 MFMAs: 1 + 3 fragment reads (0.44 KiB of LDS traffic per MFMA instead of 1 KiB for a
//     plain 64x64 wavefront tile), and the patch is fetched from memory once, not once per tap.
// Images 8 pixels wide take sub-steps of two rows of 8 pixels: the fragment of the row pair that
// starts at x row t serves tap row r of the dy pair that starts at row t + 1 - r, pairs start at
// even dy rows, so one of three fragment sets is reused and two enter per sub-step.
// A workgroup is NTN x NTC wavefronts, dy tiles by x tiles.  It walks blocks of 128 pixels (8 rows x 16 columns, or two
// 8 x 8 images) of the images of its split.  Operands go from memory to LDS directly (buffer loads with the LDS bit; halo
// pixels outside the image write zeros), one block ahead in a second buffer, with one barrier per block: the form before
// took them through registers into a single buffer, two barriers and the LDS stores between a wavefront's last product of a
// block and its first of the next, with one wavefront per SIMD and nothing else to run (0.66 in the mean, matrix units 27 %
// busy).  Sixteen pixels of a tile are 64 bytes each, one behind the other, as the loads write them; a transpose read takes
// four consecutive pixels of 32 channels = 256 bytes per half wavefront, every bank once, without padding.
// us, weight gradient with its reduction, before -> now, 3 x 128 images: 96 channels 32 x 32 102 -> 87, 320 on 16 x 16
// 191 -> 162, 64 on 32 x 32 50 -> 41, 128 on 16 x 16 52 -> 41, 256 on 8 x 8 50 -> 41, 192 on 16 x 16 94 -> 69, 160 on 32 x 32
// 219 -> 193.  Three or five dy tiles (96, 160 channels) load the SIMDs unevenly: 75 and 63 % of the matrix units at best.
// Partial sums of the splits go to per-split buffers that a second kernel adds in a fixed order (no float atomics).
// BIAS: the wavefronts of the first x tile multiply their dy fragments by ones as well, a tenth product beside the nine, and
// write the layer's bias gradient, the column sums of dy, behind the weights.
#include <stdlib.h>

#include "igemm_dev.h"

namespace {

using namespace igemm_dev;
typedef short s4v __attribute__((ext_vector_type(4)));

constexpr int kBlockPixels = 128;                // 8 rows x 16 columns, or two images of 8 x 8
constexpr int kSub = 8;                          // contraction sub-steps (16 pixels) per block
// Patch of a block: one halo pixel around each image part.  Rows of whole 8 x 8 images have zeros on both sides: the one on the
// right of a row is the one on the left of the next, and one more lies behind the last row.  That keeps 2 x 2 tiles at 80 KB,
// two workgroups per compute unit (640 channels, 3 x 128 images, 300 workgroups: 196 us; 244 with columns of their own).
template <int KC>
struct Patch {
  static constexpr int PC = KC == 16 ? KC + 2 : KC + 1;  // columns
  static constexpr int IMG = KC == 16 ? 1 : 2;           // image parts per block
  static constexpr int PRI = kBlockPixels / KC / IMG + 2;  // rows per image part
  static constexpr int SLOTS = IMG * PRI * PC + (KC == 16 ? 0 : 1);  // 180 / 181
  static constexpr int LOADS = (SLOTS + 15) / 16;        // of 16 pixels
};

struct Wg9Geom {
  int H, W, Cin, N;          // image, channels in / out
  int B;                     // images per replica
  int bpi, cbn;              // blocks per image, column blocks per image row
  int total_blocks, bps;     // per replica; blocks per split
  int splits;
  FastDiv dBpi, dCbn;
};

__device__ __forceinline__ u4 tr_frag(const bf16_t *tile, int ld, int krow, int col) {
  // 8 contraction values (rows krow .. krow+7 as seen by this lane's 16-lane group) of column `col + l%16`
  const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4v *)(tile + krow * ld + col));
  const s4v hi =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4v *)(tile + (krow + 4) * ld + col));
  u4 r;
  r.x = (uint32_t)(unsigned short)lo.x | ((uint32_t)(unsigned short)lo.y << 16);
  r.y = (uint32_t)(unsigned short)lo.z | ((uint32_t)(unsigned short)lo.w << 16);
  r.z = (uint32_t)(unsigned short)hi.x | ((uint32_t)(unsigned short)hi.y << 16);
  r.w = (uint32_t)(unsigned short)hi.z | ((uint32_t)(unsigned short)hi.w << 16);
  return r;
}

// RAG: images that do not cut into blocks.  Loads beyond the image are zeros on both sides; x pixels that meet a dy pixel
// beyond its row are blanked as well, since they may be infinite, and rows beyond the image are left out.
template <int NTN, int NTC, int KC, bool BIAS, bool RAG>
__global__ __launch_bounds__(NTN * NTC * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad9(const Wg9Geom wg, const WgradIO io) {
  typedef Patch<KC> PT;
  constexpr int kPC = PT::PC, W = NTN * NTC;
  static_assert(!RAG || KC == 16, "8 x 8 images are whole");
  constexpr int XG = PT::LOADS;                           // loads of 16 pixels: one x tile, one dy tile (8)
  constexpr int PIECES = NTC * XG + NTN * 8;
  constexpr int IT = (PIECES + W - 1) / W;                // loads of a block per wavefront
  constexpr int BUF = PIECES * 1024;
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % NTN, wc = wave / NTN;             // this wavefront's dy tile and x tile
  const int cg = blockIdx.x, ng = blockIdx.y;
  const int rep = blockIdx.z / wg.splits, split = blockIdx.z - rep * wg.splits;
  const int blk_begin = split * wg.bps, blk_end = min(wg.total_blocks, blk_begin + wg.bps);
  const u4 x_rsrc = buffer_desc((const bf16_t *)io.x + rep * io.x_rs, (uint32_t)((long long)wg.B * wg.H * wg.W * wg.Cin * 2));
  const u4 d_rsrc = buffer_desc((const bf16_t *)io.dy + rep * io.dy_rs, (uint32_t)((long long)wg.B * wg.H * wg.W * wg.N * 2));
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;

  // Piece q = it * W + wave: sixteen pixels of an x tile (q < NTC * XG) or of a dy tile.  `rel`: offset of this lane's pixel
  // and channels from the block's first pixel; `pos`: patch row and column of an x pixel, to tell what lies inside the image.
  int rel[IT], pos[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int q = it * W + wave, px = lane >> 2, ch = (lane & 3) * 8;
    if (q < NTC * XG) {
      const int t = q / XG, slot = (q - t * XG) * 16 + px;
      const int img = slot / (PT::PRI * kPC), rem = slot - img * (PT::PRI * kPC);
      const int prow = rem / kPC, pcol = rem - prow * kPC;
      rel[it] = (((img * wg.H + prow - 1) * wg.W + (pcol - 1)) * wg.Cin + (cg * NTC + t) * 32 + ch) * 2;
      pos[it] = prow | pcol << 8 | img << 16;
      // a slot that belongs to no pixel: beyond the buffer from wherever a block begins
      if (slot >= PT::IMG * PT::PRI * kPC) rel[it] = (int)kOobOffset, pos[it] = 0;
    } else {
      const int d = q - NTC * XG, t = d >> 3, p = (d & 7) * 16 + px;  // pixel of the block
      const int img = p / (kBlockPixels / PT::IMG), r = p - img * (kBlockPixels / PT::IMG), row = r / KC, col = r - row * KC;
      rel[it] = (((img * wg.H + row) * wg.W + col) * wg.N + (ng * NTN + t) * 32 + ch) * 2;
      pos[it] = row | col << 8;
    }
  }
  auto load_block = [&](int blk, int buf) {
    int b, row0, col0;
    if (KC == 16) {
      b = (int)fdiv((uint32_t)blk, wg.dBpi);
      const int rem = blk - b * wg.bpi;
      const int rb = (int)fdiv((uint32_t)rem, wg.dCbn), cb = rem - rb * wg.cbn;
      row0 = rb * 8, col0 = cb * 16;
    } else {
      b = 2 * blk, row0 = 0, col0 = 0;
    }
    const int pix = (b * wg.H + row0) * wg.W + col0;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int q = it * W + wave;
      if (PIECES % W != 0 && it == IT - 1 && q >= PIECES) break;
      const uint32_t dst = lds0 + (uint32_t)(buf * BUF + q * 1024);
      if (q < NTC * XG) {
        const int row = row0 + (pos[it] & 0xff) - 1, col = col0 + (pos[it] >> 8 & 0xff) - 1;
        const bool ok = (unsigned)row < (unsigned)wg.H && (unsigned)col < (unsigned)wg.W && b + (pos[it] >> 16) < wg.B;
        dma16(dst, x_rsrc, ok ? (uint32_t)(pix * wg.Cin * 2 + rel[it]) : kOobOffset, 0);
      } else {
        // an image beyond the batch (odd batch, second 8 x 8 image of the last block) lies beyond the buffer: zeros
        const bool ok = !RAG || (row0 + (pos[it] & 0xff) < wg.H && col0 + (pos[it] >> 8) < wg.W);
        dma16(dst, d_rsrc, ok ? (uint32_t)(pix * wg.N * 2 + rel[it]) : kOobOffset, 0);
      }
    }
  };

  f16v acc[3][3], accb;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[r][c][v] = 0.f;
    accb[v] = 0.f;
  }
  const bool tally = BIAS && cg == 0 && wc == 0;
  const u4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};

  // fragment addressing of the transpose read: 16-lane group gq covers columns 16*(gq%2) .. +15 and
  // contraction half gq/2
  const int gq = lane >> 4, j = lane & 15;
  const int frag_k = 8 * (gq >> 1) + (j >> 2), frag_c = 16 * (gq & 1) + 4 * (j & 3);
  // contraction index e of the sub-step -> patch slot: one row of 16, or two rows of 8 (e / 8 is the
  // lane's contraction half gq / 2; the transpose read adds 4 slots for its second part)
  const int frag_x = KC == 16 ? frag_k : (gq >> 1) * kPC + (j >> 2);
  const char *xt, *dt;
  // x fragments of the sub-step whose first pixel is patch row `prow`, at the three column shifts;
  // dy fragment of sub-step p
  u4 inside;  // RAG: the contraction indexes of this lane that are pixels of the row
  auto read_x = [&](int prow, u4 (&f)[3]) {
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      f[s] = tr_frag((const bf16_t *)xt + (prow * kPC + s) * 32, 32, 0, 0);
      if (RAG) f[s] &= inside;
    }
  };
  // of contraction indexes k .. k + 7 those below `lim`
  auto below = [&](int k, int lim) {
    u4 m;
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = (k + 2 * e < lim ? 0xffffu : 0u) | (k + 2 * e + 1 < lim ? 0xffff0000u : 0u);
    return m;
  };
  auto read_d = [&](int p) { return tr_frag((const bf16_t *)dt + p * 16 * 32, 32, 0, 0); };

  load_block(blk_begin, 0);
  int buf = 0;
  for (int blk = blk_begin; blk < blk_end; ++blk) {
    wait_loads<0>();
    __syncthreads();  // the block has arrived, and every wavefront is done with the one before it
    asm volatile("" ::: "memory");
    if (blk + 1 < blk_end) load_block(blk + 1, buf ^ 1);
    xt = smem + buf * BUF + wc * XG * 1024 + (frag_x * 32 + frag_c) * 2;
    dt = smem + buf * BUF + (NTC * XG + wn * 8) * 1024 + (frag_k * 32 + frag_c) * 2;
    buf ^= 1;
    int rows = kSub;
    if (RAG) {
      const int rem = blk - (int)fdiv((uint32_t)blk, wg.dBpi) * wg.bpi, rb = (int)fdiv((uint32_t)rem, wg.dCbn);
      rows = min(kSub, wg.H - rb * kSub);
      inside = below(8 * (gq >> 1), wg.W - (rem - rb * wg.cbn) * 16);
    }
    u4 window[3][3], dfrag[2];
    if (KC == 16) {
      // x rows p-1, p, p+1 live in window[(p + 0, 1, 2) % 3]; patch row index = image row + 1
      read_x(0, window[0]);
      dfrag[0] = read_d(0);
      read_x(1, window[1]);
      read_x(2, window[2]);
#pragma unroll
      for (int p = 0; p < kSub; ++p) {
        if (RAG && p >= rows) break;
        const int w0 = p % 3, w1 = (p + 1) % 3, w2 = (p + 2) % 3;
        const u4 d = dfrag[p & 1];
        // taps of window row r = 0 use x row p-1; its registers then take x row p+2 for the next rows
#pragma unroll
        for (int s = 0; s < 3; ++s) mma<bf16_t>(d, window[w0][s], acc[0][s]);
        if (p + 1 < kSub) dfrag[(p + 1) & 1] = read_d(p + 1);
        u4 incoming[3];
        if (p + 2 < kSub + 1) read_x(p + 3, incoming);
        if (BIAS && tally) mma<bf16_t>(d, ones, accb);
#pragma unroll
        for (int s = 0; s < 3; ++s) mma<bf16_t>(d, window[w1][s], acc[1][s]);
#pragma unroll
        for (int s = 0; s < 3; ++s) mma<bf16_t>(d, window[w2][s], acc[2][s]);
        if (p + 2 < kSub + 1) {
#pragma unroll
          for (int s = 0; s < 3; ++s) window[w0][s] = incoming[s];
        }
      }
    } else {
      // the dy pair that starts at image row 2*mu meets the x pairs that start at patch rows 2*mu + r
      // (patch row = image row + 1); pair t lives in window[t % 3]
#pragma unroll
      for (int img = 0; img < 2; ++img) {
        const int pr0 = img * PT::PRI;
        read_x(pr0 + 0, window[0]);
        dfrag[0] = read_d(img * 4);
        read_x(pr0 + 1, window[1]);
        read_x(pr0 + 2, window[2]);
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
          const int w0 = (2 * mu) % 3, w1 = (2 * mu + 1) % 3, w2 = (2 * mu + 2) % 3;
          const u4 d = dfrag[mu & 1];
#pragma unroll
          for (int s = 0; s < 3; ++s) mma<bf16_t>(d, window[w0][s], acc[0][s]);
          if (mu + 1 < 4) dfrag[(mu + 1) & 1] = read_d(img * 4 + mu + 1);
          u4 in0[3], in1[3];
          if (mu + 1 < 4) read_x(pr0 + 2 * mu + 3, in0);
          if (BIAS && tally) mma<bf16_t>(d, ones, accb);
#pragma unroll
          for (int s = 0; s < 3; ++s) mma<bf16_t>(d, window[w1][s], acc[1][s]);
          if (mu + 1 < 4) read_x(pr0 + 2 * mu + 4, in1);
#pragma unroll
          for (int s = 0; s < 3; ++s) mma<bf16_t>(d, window[w2][s], acc[2][s]);
          if (mu + 1 < 4) {
#pragma unroll
            for (int s = 0; s < 3; ++s) window[w0][s] = in0[s], window[w1][s] = in1[s];
          }
        }
      }
    }
  }

  // acc[r][s]: lane holds column c = lane % 32 and rows n = 8*(v/4) + 4*(lane/32) + v%4
  float *out = io.out + rep * io.out_rs + split * io.split_stride;
  const int c = (cg * NTC + wc) * 32 + (lane & 31), h = lane >> 5;
  const int K = 9 * wg.Cin;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int n = (ng * NTN + wn) * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
        out[(long long)n * K + (r * 3 + s) * wg.Cin + c] = acc[r][s][v];
      }
  if (BIAS && tally && (lane & 31) == 0) {  // all columns hold the same sums
#pragma unroll
    for (int v = 0; v < 16; ++v) out[(long long)wg.N * K + (ng * NTN + wn) * 32 + 8 * (v >> 2) + 4 * h + (v & 3)] = accb[v];
  }
}

// Stride 2, padding 1, even input sizes (dy [H][W], x [2H][2W]):
//   dW[n][r][s][c] = sum over pixels (b, p, q) of dy[b, p, q, n] * x[b, 2p + r - 1, 2q + s - 1, c]
// The same walk in blocks of 64 pixels (4 rows x 16 columns, or one 8 x 8 image).  A patch row holds its odd input columns,
// -1, 1, 3, ..., and behind them the even ones: the pixels that a tap pairs with consecutive dy pixels are consecutive again.
// In blocks of 16 columns the x row of tap row 2 is that of tap row 0 for the next dy row and stays in registers: 1 + 6
// fragment reads per nine products, in pairs of 8-pixel rows 1 + 9.  Gathering each tap for itself (k_wgrad_tr) reads x nine
// times from L2 in pieces of 64 bytes two pixels apart.  us with the reduction, before -> now, 3 x 128 images: 64 -> 128
// channels 32 x 32 48 -> 36, 96 -> 96 50 -> 41, 160 -> 320 201 -> 127; 128 -> 256 on 16 x 16 44 -> 35, 192 -> 192 43 -> 42.
template <int KC>
struct Patch2 {
  static constexpr int QC = KC == 16 ? 16 : 8, ROWS = 64 / QC;  // dy columns and rows of a block
  static constexpr int PC = 2 * QC + 1;                         // QC + 1 odd columns, QC even ones
  static constexpr int PR = 2 * ROWS + 1;
  static constexpr int SLOTS = PR * PC;                         // 297 / 289
  static constexpr int LOADS = (SLOTS + 15) / 16;               // of 16 pixels
};

template <int NTN, int KC, bool BIAS>
__global__ __launch_bounds__(NTN * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad9_s2(const Wg9Geom wg, const WgradIO io) {
  typedef Patch2<KC> PT;
  constexpr int kPC = PT::PC, W = NTN, QC = PT::QC;
  constexpr int XG = PT::LOADS;                           // loads of 16 pixels: the x tile, one dy tile (4)
  constexpr int PIECES = XG + NTN * 4;
  constexpr int IT = (PIECES + W - 1) / W;
  constexpr int BUF = PIECES * 1024;
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ct = blockIdx.x, ng = blockIdx.y;
  const int rep = blockIdx.z / wg.splits, split = blockIdx.z - rep * wg.splits;
  const int blk_begin = split * wg.bps, blk_end = min(wg.total_blocks, blk_begin + wg.bps);
  const int Hx = 2 * wg.H, Wx = 2 * wg.W;
  const u4 x_rsrc = buffer_desc((const bf16_t *)io.x + rep * io.x_rs, (uint32_t)((long long)wg.B * Hx * Wx * wg.Cin * 2));
  const u4 d_rsrc = buffer_desc((const bf16_t *)io.dy + rep * io.dy_rs, (uint32_t)((long long)wg.B * wg.H * wg.W * wg.N * 2));
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;

  // rel: offset of this lane's pixel and channels from the block's first pixel; pos: what lies outside the image, bit 0 where
  // the block is in the first column, bit 1 in the first row, bit 2 always (beyond the patch)
  int rel[IT], pos[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int q = it * W + wave, px = lane >> 2, ch = (lane & 3) * 8;
    if (q < XG) {
      const int slot = q * 16 + px, prow = slot / kPC, i = slot - prow * kPC;
      const int col = i <= QC ? 2 * i - 1 : 2 * (i - QC - 1), row = prow - 1;
      rel[it] = ((row * Wx + col) * wg.Cin + ct * 32 + ch) * 2;
      pos[it] = (col < 0 ? 1 : 0) | (row < 0 ? 2 : 0) | (slot < PT::SLOTS ? 0 : 4);
    } else {
      const int d = q - XG, t = d >> 2, p = (d & 3) * 16 + px;
      const int row = p / QC, col = p - row * QC;
      rel[it] = ((row * wg.W + col) * wg.N + (ng * NTN + t) * 32 + ch) * 2;
      pos[it] = 0;
    }
  }
  auto load_block = [&](int blk, int buf) {
    const int b = (int)fdiv((uint32_t)blk, wg.dBpi);
    const int rem = blk - b * wg.bpi;
    const int rb = (int)fdiv((uint32_t)rem, wg.dCbn), cb = rem - rb * wg.cbn;
    const int row0 = rb * PT::ROWS, col0 = cb * QC;
    const int xbase = ((b * Hx + 2 * row0) * Wx + 2 * col0) * wg.Cin * 2, dbase = ((b * wg.H + row0) * wg.W + col0) * wg.N * 2;
    const int outside = 4 | (cb == 0 ? 1 : 0) | (rb == 0 ? 2 : 0);
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int q = it * W + wave;
      if (PIECES % W != 0 && it == IT - 1 && q >= PIECES) break;
      const uint32_t dst = lds0 + (uint32_t)(buf * BUF + q * 1024);
      if (q < XG)
        dma16(dst, x_rsrc, pos[it] & outside ? kOobOffset : (uint32_t)(xbase + rel[it]), 0);
      else
        dma16(dst, d_rsrc, (uint32_t)(dbase + rel[it]), 0);
    }
  };

  f16v acc[3][3], accb;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[r][c][v] = 0.f;
    accb[v] = 0.f;
  }
  const bool tally = BIAS && ct == 0;
  const u4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
  const int gq = lane >> 4, j = lane & 15;
  const int frag_k = 8 * (gq >> 1) + (j >> 2), frag_c = 16 * (gq & 1) + 4 * (j & 3);
  // a sub-step is a row of 16, or two rows of 8, two patch rows apart
  const int frag_x = KC == 16 ? frag_k : (gq >> 1) * 2 * kPC + (j >> 2);
  const char *xt, *dt;
  // x fragments of patch row `prow` at column shifts -1, 0, 1: odd columns from 0, even ones, odd ones from 1
  auto read_x = [&](int prow, u4 (&f)[3]) {
    const bf16_t *row = (const bf16_t *)xt + prow * kPC * 32;
    f[0] = tr_frag(row, 32, 0, 0);
    f[1] = tr_frag(row + (QC + 1) * 32, 32, 0, 0);
    f[2] = tr_frag(row + 32, 32, 0, 0);
  };
  auto read_d = [&](int p) { return tr_frag((const bf16_t *)dt + p * 16 * 32, 32, 0, 0); };

  load_block(blk_begin, 0);
  int buf = 0;
  for (int blk = blk_begin; blk < blk_end; ++blk) {
    wait_loads<0>();
    __syncthreads();  // the block has arrived, and every wavefront is done with the one before it
    asm volatile("" ::: "memory");
    if (blk + 1 < blk_end) load_block(blk + 1, buf ^ 1);
    xt = smem + buf * BUF + (frag_x * 32 + frag_c) * 2;
    dt = smem + buf * BUF + (XG + wave * 4) * 1024 + (frag_k * 32 + frag_c) * 2;
    buf ^= 1;
    constexpr int STEP = KC == 16 ? 2 : 4;  // patch rows from one sub-step to the next
    u4 top[3], mid[3], bot[3], d = read_d(0);
    read_x(0, top);
    read_x(1, mid);
    read_x(2, bot);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const u4 dn = p < 3 ? read_d(p + 1) : d;
#pragma unroll
      for (int s = 0; s < 3; ++s) mma<bf16_t>(d, top[s], acc[0][s]);
      if (p < 3 && KC == 8) read_x((p + 1) * STEP, top);
#pragma unroll
      for (int s = 0; s < 3; ++s) mma<bf16_t>(d, mid[s], acc[1][s]);
      if (p < 3) read_x((p + 1) * STEP + 1, mid);
      if (BIAS && tally) mma<bf16_t>(d, ones, accb);
#pragma unroll
      for (int s = 0; s < 3; ++s) mma<bf16_t>(d, bot[s], acc[2][s]);
      if (p < 3) {
        if (KC == 16) {
#pragma unroll
          for (int s = 0; s < 3; ++s) top[s] = bot[s];
        }
        read_x((p + 1) * STEP + 2, bot);
      }
      d = dn;
    }
  }

  float *out = io.out + rep * io.out_rs + split * io.split_stride;
  const int c = ct * 32 + (lane & 31), h = lane >> 5;
  const int K = 9 * wg.Cin;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int n = (ng * NTN + wave) * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
        out[(long long)n * K + (r * 3 + s) * wg.Cin + c] = acc[r][s][v];
      }
  if (BIAS && tally && (lane & 31) == 0) {
#pragma unroll
    for (int v = 0; v < 16; ++v) out[(long long)wg.N * K + (ng * NTN + wave) * 32 + 8 * (v >> 2) + 4 * h + (v & 3)] = accb[v];
  }
}

// Tiles per workgroup, dy x x.
struct Wg9Tiles {
  int n, c;
};
Wg9Tiles wg9_tiles(const ConvGeom &g) {
  const int nt32 = g.N / 32, ct32 = g.Cc / 32;
  if (g.sp == 2) {  // four, three or five dy tiles over one x tile: the patch is the larger load
    static const int order2[4] = {4, 3, 5, 2};
    for (int nt : order2)
      if (nt32 % nt == 0) return {nt, 1};
    return {0, 1};
  }
  // 2 x 2: an x tile and a dy tile each serve two wavefronts, and two workgroups put two wavefronts on every SIMD; three or
  // five dy tiles leave SIMDs with one beside others with two.  2 x 1 loads half as much again per product (192 channels on
  // 16 x 16, 3 x 128 images: 2 x 2 69.6 us, 3 x 1 69.9, 4 x 1 70.1, 2 x 1 92).
  if (nt32 % 2 == 0 && ct32 % 2 == 0) return {2, 2};
  static const int order[4] = {3, 4, 5, 2};
  for (int nt : order)
    if (nt32 % nt == 0) return {nt, 1};
  return {nt32 == 1 ? 1 : 0, 1};
}

bool small_images(const ConvGeom &g) { return g.Q <= 8 && g.P <= 8; }
bool whole_blocks(const ConvGeom &g) { return g.Q % 16 == 0 ? g.P % (g.sp == 2 ? 4 : 8) == 0 : g.Q == 8 && g.P == 8; }
int block_pixels(const ConvGeom &g) { return g.sp == 2 ? 64 : kBlockPixels; }

int wg9_lds(const ConvGeom &g, const Wg9Tiles &t) {
  if (g.sp == 2) return 2 * ((small_images(g) ? Patch2<8>::LOADS : Patch2<16>::LOADS) + t.n * 4) * 1024;
  return 2 * (t.c * (small_images(g) ? Patch<8>::LOADS : Patch<16>::LOADS) + t.n * 8) * 1024;
}

void make_wg9_geom(const ConvGeom &g, Wg9Geom &wg) {
  wg.H = g.P, wg.W = g.Q, wg.Cin = g.Cc, wg.N = g.N;
  wg.B = g.M / (g.P * g.Q);
  if (small_images(g)) {  // two whole images per block, one at stride 2
    wg.cbn = 1, wg.bpi = 1;
    wg.total_blocks = g.sp == 2 ? wg.B : (wg.B + 1) / 2;
  } else {
    const int rows = block_pixels(g) / 16;
    wg.cbn = (wg.W + 15) / 16;
    wg.bpi = (wg.H + rows - 1) / rows * wg.cbn;
    wg.total_blocks = wg.B * wg.bpi;
  }
  wg.dBpi = make_fastdiv(wg.bpi), wg.dCbn = make_fastdiv(wg.cbn);
}

template <int NTN, int NTC, int KC, bool BIAS, bool RAG>
hipError_t run_wgrad9(hipStream_t st, int replicas, const ConvGeom &g, const Wg9Geom &wg, const WgradIO &io) {
  const int lds = wg9_lds(g, {NTN, NTC});
  static const hipError_t lds_ok =
      hipFuncSetAttribute((const void *)k_wgrad9<NTN, NTC, KC, BIAS, RAG>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (lds_ok != hipSuccess) return lds_ok;
  dim3 grid(g.Cc / 32 / NTC, g.N / 32 / NTN, replicas * io.splits);
  hipLaunchKernelGGL((k_wgrad9<NTN, NTC, KC, BIAS, RAG>), grid, dim3(NTN * NTC * 64), lds, st, wg, io);
  return hipGetLastError();
}

template <int NTN, int KC, bool BIAS>
hipError_t run_wgrad9_s2(hipStream_t st, int replicas, const ConvGeom &g, const Wg9Geom &wg, const WgradIO &io) {
  const int lds = wg9_lds(g, {NTN, 1});
  static const hipError_t lds_ok =
      hipFuncSetAttribute((const void *)k_wgrad9_s2<NTN, KC, BIAS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (lds_ok != hipSuccess) return lds_ok;
  dim3 grid(g.Cc / 32, g.N / 32 / NTN, replicas * io.splits);
  hipLaunchKernelGGL((k_wgrad9_s2<NTN, KC, BIAS>), grid, dim3(NTN * 64), lds, st, wg, io);
  return hipGetLastError();
}

}  // namespace

bool wgrad9_applicable(int dtype, const ConvGeom &g) {
  if (dtype != 1 || g.R != 3 || g.S != 3 || (g.sp != 1 && g.sp != 2) || g.dshift != 0 || g.sr != 1 || g.off != -1) return false;
  if (g.sp * g.P != g.Hin || g.sp * g.Q != g.Win) return false;
  if (!whole_blocks(g)) {
    // Share of the products that are no padding.  us, this kernel / the transpose-read kernel: 28 x 28 (0.88) 96 channels, 100
    // images 35 / 46; 14 x 14 (0.88) 256 channels 48 / 61; 15 x 15 (0.94) 320 channels 44 / 69; 24 x 24 (0.75) 37 / 54;
    // 12 x 12 (0.75) 320 channels 44 / 61; 10 x 10 and 20 x 20 (0.63) 32.9 / 32.2 and 29.4 / 29.4; 9 x 9 32 / 29.  Images of
    // less than 8 x 8 would come two to a block whatever their size: 7 x 7, 65 images and more, 0.80 to 1.27 of the other's
    // time, 1.00 in the mean of 26 layers.  2 x 1 tiles load half as much again per product: 0.8 to 1.24, 1.00 of 33 layers.
    if (g.sp == 2 || small_images(g) || g.Q * 10 < 16 * ((g.Q + 15) / 16) * 7 || wg9_tiles(g).n * wg9_tiles(g).c == 2) return false;
  }
  if (g.Cc % 32 != 0 || g.N % 32 != 0 || wg9_tiles(g).n < 2) return false;
  const long long in_bytes = (long long)g.M * g.sp * g.sp * g.Cc * 2, dy_bytes = (long long)g.M * g.N * 2;
  return in_bytes < (1LL << 31) && dy_bytes < (1LL << 31) && g.M % (g.P * g.Q) == 0;
}

// Blocks of 128 pixels (64 at stride 2) per split so that the launch fills the chip; returns the split count and the
// pixels per split in *chunk_out.
int wgrad9_plan(int replicas, const ConvGeom &g, int *chunk_out) {
  Wg9Geom wg;
  make_wg9_geom(g, wg);
  const Wg9Tiles t = wg9_tiles(g);
  const long long tiles = (long long)(g.Cc / 32 / t.c) * (g.N / 32 / t.n) * replicas;
  // One or two workgroups per compute unit, never a few stragglers in another round, whichever ends sooner: the second
  // fills gaps of the first (8 %), and doubles the partial sums, which are written and read once more.  us with 256 / 512
  // workgroups at 3 x 128 images: 64 channels on 32 x 32 39.6 / 44.2, 128 on 16 x 16 39.5 / 43.9, 320 on 16 x 16 173 /
  // 160.  A network that has its leaves run beside a longer chain asks for fewer.
  // PARLE_WG9_WAVES: wavefronts in flight instead.
  static const int waves = [] {
    const char *e = getenv("PARLE_WG9_WAVES");
    return e ? atoi(e) : 0;
  }();
  constexpr int kCus = 256;
  const int target = g.leaf_waves > 0 ? g.leaf_waves : waves;
  long long want;
  if (target > 0) {
    want = (target / (t.n * t.c) + tiles - 1) / tiles;
  } else {
    const double product = 2.0 * wg.total_blocks * block_pixels(g) * g.N * (double)g.K * replicas / 1.45e9;  // us at what the chip sustains
    const double partial = 8.0 * g.N * (double)g.K * replicas / 8e6;                    // us per split
    // by LDS, and by two wavefronts of up to 256 registers per SIMD
    const int waves_of = t.n * t.c, lds = wg9_lds(g, t), per_cu = 160 * 1024 / lds < 8 / waves_of ? 160 * 1024 / lds : 8 / waves_of;
    double least = 0.;
    want = 1;
    for (int k = 1; k <= per_cu; ++k) {
      const long long splits = k * kCus / tiles;
      if (splits < 1) continue;
      const double busy = waves_of == 2 && g.sp == 1 ? k / (double)per_cu : k == 1 ? .92 : 1.;  // two wavefronts: half of the SIMDs
      const double us = product / ((double)splits * tiles / (k * kCus) * busy) + splits * partial;
      if (least == 0. || us < least) least = us, want = splits;
    }
  }
  // Four blocks per split at least, two where that leaves most of the chip idle (16 images of 8 x 8 x 128: 14.1 -> 11.8 us).
  const int blocks = wg.total_blocks / 4 * tiles < 96 ? 2 : 4;
  if (want > wg.total_blocks / blocks) want = wg.total_blocks / blocks;
  // Below eight blocks one split writes the gradient as it is; more pay a reduction of 2.6 us and 5 TB/s.  us, one split / more:
  // 32 -> 256 channels, 3 x 10 images of 8 x 8, 13.2 / 11.8; 224 -> 288, 4 x 9 images, 14.4 / 21.0.
  if (want > 1 && wg.total_blocks < 8) {
    const double left = wg.total_blocks - (wg.total_blocks + want - 1) / want;  // blocks a workgroup no longer walks
    const double mb = 4e-6 * g.N * (double)g.K * replicas;
    if (left * block_pixels(g) / kBlockPixels * (t.n == 5 ? 3. : 2.) < 2.6 + mb * (2. * want + 1.) / 5.) want = 1;
  }
  if (want < 1) want = 1;
  const long long cap = 65535 / replicas;
  if (want > cap) want = cap;
  const int bps = (int)((wg.total_blocks + want - 1) / want);
  const int splits = (wg.total_blocks + bps - 1) / bps;
  if (chunk_out) *chunk_out = bps * block_pixels(g);
  return splits;
}

hipError_t launch_wgrad9(hipStream_t st, int replicas, const ConvGeom &g, const WgradIO &io) {
  Wg9Geom wg;
  make_wg9_geom(g, wg);
  wg.bps = io.chunk / block_pixels(g);
  wg.splits = io.splits;
  if (wg.bps < 1 || (long long)wg.bps * io.splits < wg.total_blocks) return hipErrorInvalidValue;
  const Wg9Tiles t = wg9_tiles(g);
  const bool narrow = small_images(g);
#define WG9_S2(NV)                                                                                                            \
  if (t.n == NV)                                                                                                              \
    return io.with_bias ? narrow ? run_wgrad9_s2<NV, 8, true>(st, replicas, g, wg, io)                                        \
                                 : run_wgrad9_s2<NV, 16, true>(st, replicas, g, wg, io)                                       \
                        : narrow ? run_wgrad9_s2<NV, 8, false>(st, replicas, g, wg, io)                                       \
                                 : run_wgrad9_s2<NV, 16, false>(st, replicas, g, wg, io)
  if (g.sp == 2) {
    WG9_S2(2);
    WG9_S2(3);
    WG9_S2(4);
    WG9_S2(5);
    return hipErrorInvalidValue;
  }
#undef WG9_S2
  const bool rag = !whole_blocks(g);
#define WG9_RUN(NV, CV, KCV, RAGV)                                                \
  return io.with_bias ? run_wgrad9<NV, CV, KCV, true, RAGV>(st, replicas, g, wg, io) \
                      : run_wgrad9<NV, CV, KCV, false, RAGV>(st, replicas, g, wg, io)
#define WG9_CASE(NV, CV)                            \
  if (t.n == NV && t.c == CV) {                     \
    if (narrow) WG9_RUN(NV, CV, 8, false);          \
    if (rag) WG9_RUN(NV, CV, 16, (NV * CV != 2));   \
    WG9_RUN(NV, CV, 16, false);                     \
  }
  WG9_CASE(2, 2);
  WG9_CASE(2, 1);
  WG9_CASE(3, 1);
  WG9_CASE(4, 1);
  WG9_CASE(5, 1);
#undef WG9_CASE
#undef WG9_RUN
  return hipErrorInvalidValue;
}
