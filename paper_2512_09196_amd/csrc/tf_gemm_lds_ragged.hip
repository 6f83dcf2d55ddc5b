// Instances of the LDS-staged kernels (tf_gemm_lds.h) for sizes that are no multiples of the tiles.
#include "tf_gemm_lds.h"

namespace tf {

// One or two per tile size, the ones that lead in their size range: every variant here has a rival of another size
// rather than of another wave shape.
//                               BM   BN   BK  WM WN ST  direct
using K256x256 = LdsCfg<256, 256, 64, 2, 4, 2, true>;
using K256x128 = LdsCfg<256, 128, 64, 4, 2, 3, true>;
using K128x256 = LdsCfg<128, 256, 64, 2, 4, 3, true>;
using K128x128 = LdsCfg<128, 128, 64, 2, 4, 3, true>;
using K64x64   = LdsCfg< 64,  64, 64, 2, 2, 3, true>;
using K32x128  = LdsCfg< 32, 128, 64, 1, 4, 3, true>;
using K32x64   = LdsCfg< 32,  64, 64, 1, 2, 4, true>;
using K32x32   = LdsCfg< 32,  32, 64, 1, 1, 4, true>;
// second operand as [N][K]
using N256x256 = LdsCfg<256, 256, 64, 2, 4, 2, true, false, 1, false, true>;
using N256x128 = LdsCfg<256, 128, 64, 4, 2, 3, true, false, 1, false, true>;
using N128x256 = LdsCfg<128, 256, 64, 2, 4, 3, true, false, 1, false, true>;
using N128x128 = LdsCfg<128, 128, 64, 2, 4, 3, true, false, 1, false, true>;
using N64x64   = LdsCfg< 64,  64, 64, 2, 2, 3, true, false, 1, false, true>;
using N32x128  = LdsCfg< 32, 128, 64, 1, 4, 3, true, false, 1, false, true>;
using N32x64   = LdsCfg< 32,  64, 64, 1, 2, 4, true, false, 1, false, true>;
using N32x32   = LdsCfg< 32,  32, 64, 1, 1, 4, true, false, 1, false, true>;

// rows in whole lines (RaggedKCfg::LINES): beside the instances with three buffers, where lines_offered says so
using KL128x128 = LdsCfg<128, 128, 64, 2, 4, 4, true>;
using KL64x128  = LdsCfg< 64, 128, 64, 2, 4, 4, true>;
using NL128x128 = LdsCfg<128, 128, 64, 2, 4, 4, true, false, 1, false, true>;
using NL64x128  = LdsCfg< 64, 128, 64, 2, 4, 4, true, false, 1, false, true>;

// first operand transposed: the persistent kernel for ragged tiles
using T128x128 = LdsCfg<128, 128, 64, 2, 4, 3, true, false, 1, true>;

static const LdsKernelInfo g_ragged[] = {
    make_ragged_info<K256x256>(), make_ragged_info<K256x128>(), make_ragged_info<K128x256>(), make_ragged_info<K128x128>(),
    make_ragged_info<K64x64>(),   make_ragged_info<K32x128>(),  make_ragged_info<K32x64>(),   make_ragged_info<K32x32>(),
    make_ragged_info<N256x256>(), make_ragged_info<N256x128>(), make_ragged_info<N128x256>(), make_ragged_info<N128x128>(),
    make_ragged_info<N64x64>(),   make_ragged_info<N32x128>(),  make_ragged_info<N32x64>(),   make_ragged_info<N32x32>(),
    make_persist_ragged_info<T128x128>(),
    make_ragged_info<KL128x128>(), make_ragged_info<KL64x128>(), make_ragged_info<NL128x128>(), make_ragged_info<NL64x128>(),
};

const LdsKernelInfo* lds_ragged_table(int* n) {
  *n = (int)(sizeof(g_ragged) / sizeof(g_ragged[0]));
  return g_ragged;
}

}  // namespace tf
