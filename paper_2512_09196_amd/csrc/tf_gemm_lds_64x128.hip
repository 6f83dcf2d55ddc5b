// Instances of the LDS-staged kernels (tf_gemm_lds.h) with tiles of 64 x 128.
#include "tf_gemm_lds.h"

namespace tf {

// For products whose 128 x 128 tiles leave CUs idle and whose 64 x 64 tiles come out at more than one per CU. What bounds
// them is what a CU fetches (about 95 GB/s of K tiles whatever the tile): 24 KB a K step here, 32 KB in a tile of 128 x 128
// or in two of 64 x 64. Eight waves of 32 x 32, 72 KB of LDS, so two work-groups may share a CU. Measured, us, 128 x 128 /
// 64 x 64 / here: 1418 x 1152 x 1856 16.2 / 13.5 / 12.4; 1172 x 928 x 2112, [N][K], 17.1 / 14.4 / 12.9; 1514 x 696 x 1208
// 15.5 / 13.1 / 11.4; 551 x 2880 x 1128 12.9 / 11.1 / 10.2; 2197 x 576 x 1088 11.2 / 9.3 / 8.9; 1694 x 1024 x 1920 15.9 / 15.2 /
// 13.2; 395 x 960 x 10176 in K slices 20.5 / - / 19.2. (Four waves of 32 x 64, five buffers: within 3 %, either way; tiles
// of 128 x 64: level to 11 % slower.)
//                            BM   BN   BK  WM WN ST  direct
using K64x128 = LdsCfg< 64, 128, 64, 2, 4, 3, true>;
using N64x128 = LdsCfg< 64, 128, 64, 2, 4, 3, true, false, 1, false, true>;

static const LdsKernelInfo g_64x128[] = {
    make_info<K64x128>(), make_info<N64x128>(), make_ragged_info<K64x128>(), make_ragged_info<N64x128>(),
};

const LdsKernelInfo* lds_64x128_table(int* n) {
  *n = (int)(sizeof(g_64x128) / sizeof(g_64x128[0]));
  return g_64x128;
}

}  // namespace tf
