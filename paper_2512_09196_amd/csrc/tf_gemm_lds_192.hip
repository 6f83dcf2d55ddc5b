// Instances of the LDS-staged kernels (tf_gemm_lds.h) with tiles of 192 x 256.
#include "tf_gemm_lds.h"

namespace tf {

// Eight waves of 96 x 64: a K step moves 56 KB into LDS and 160 KB out of it for 192 MFMAs, 1.13 KB per MFMA, an
// eighth more than the 256 x 256 tile and a fifth less than 256 x 128, so the matrix pipes stay the limit, and its row
// count falls between those of the others where a problem's rows or its number of tiles per CU do not suit 256.
// Measured against the best of the others (us): 1536 x 6144 x 2048 51.7 -> 49.4 and, B as [N][K], 51.1 -> 42.7;
// 3072 x 3072 x 3072 71.3 -> 66.7; 2048 x 5120 x 3072 73.5 -> 70.7; 6144 x 6144 x 1536 138.7 -> 123.3;
// 3000 x 3072 x 3072 66.2 -> 59.1; 805 x 9408 x 320, [N][K], 17.8 -> 15.0; 2105 x 4096 x 1984 44.9 -> 40.0;
// 1193 x 9024 x 5248, [N][K], 115.3 -> 110.8. Where the cost model takes it on rows that are a multiple of 128, 30
// drawn problems gained 10 % (geometric mean; the least 0.997).
// (192 x 128 was tried for 1500 x 4096 x 4096, whose 192 tiles of 256 x 128 leave 64 CUs idle: 52.2 against 51.9 us.
// With every CU busy the board's power limit lowers the clock by as much.)
//                            BM   BN   BK  WM WN ST  direct
using K192x256 = LdsCfg<192, 256, 64, 2, 4, 2, true>;
using N192x256 = LdsCfg<192, 256, 64, 2, 4, 2, true, false, 1, false, true>;

static const LdsKernelInfo g_192[] = {
    make_info<K192x256>(), make_info<N192x256>(), make_ragged_info<K192x256>(), make_ragged_info<N192x256>(),
};

const LdsKernelInfo* lds_192_table(int* n) {
  *n = (int)(sizeof(g_192) / sizeof(g_192[0]));
  return g_192;
}

}  // namespace tf
