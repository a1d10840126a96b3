// Tiles of the kernels that stage the input patch of a convolution in LDS.
#pragma once
#include "igemm_dev.h"

// A tile is a number of whole output rows, counted through all images (row b*P + p), as many as BM pixels hold: 8 rows of
// 32, four images of 8 x 8, 9 rows of 28.  An image that ends inside a tile adds its own halo rows to the patch.
struct HaloGeom {
  int TH;              // output rows per tile
  int HC;              // patch columns = sp*(Q - 1) + S
  int PRI;             // patch rows of a whole image = sp*(P - 1) + R
  int slots;           // pixels of the largest patch
  int rows;            // output rows of all images
  int omin_h, omin_w;  // smallest tap offset (input row = sp * output row + offset)
  FastDiv dP, dHC, dPRI;  // no integer division on the device
  int tiles, nb, bn;   // pixel tiles, column blocks and their width in channels (set with the grid)
};

using igemm_dev::fdiv;

// Workgroups are handed to the eight XCDs in turn, so ids that differ by 8 share an L2: the column blocks
// of one pixel tile get such ids.  They run at the same time on the same XCD, the patch is fetched into
// that L2 once, and their partial output rows meet there before they are written back.
__device__ __forceinline__ bool halo_block(const HaloGeom &hg, int &tile, int &col) {
  const int per_group = 8 * hg.nb;
  const int group = blockIdx.x / per_group, within = blockIdx.x - group * per_group;
  tile = group * 8 + (within & 7), col = within >> 3;
  return tile < hg.tiles;  // the grid is padded to whole groups
}

// The tiles of a layer, 256 pixels or (half, stride 2) 128; false where they would fill less than three quarters (igemm_halo.hip).
bool make_halo_geom(const ConvGeom &g, HaloGeom &hg, bool half);
// Stride-1 3x3 and 5x5 layers with operands loaded straight into LDS (igemm_patch.hip).
bool conv_patch_applicable(int replicas, const ConvGeom &g, const GemmIO &io);
hipError_t launch_conv_patch(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io);
// Stride-2 3x3 layers likewise (igemm_patch_s2.hip): same results, bit for bit, as the kernels that run them with a residual or column sums.
bool patch_s2_applicable(int dtype, int replicas, const ConvGeom &g, const GemmIO &io, bool out_f32);
hipError_t launch_patch_s2(hipStream_t st, int replicas, const ConvGeom &g, const GemmIO &io);
