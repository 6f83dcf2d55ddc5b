// Instances of the LDS-staged kernels (tf_gemm_lds.h) for whole K tiles and for register staging, and the table of
// all instances.
#include <iterator>
#include <vector>

#include "tf_gemm_lds.h"

namespace tf {

//                         BM   BN   BK  WM WN ST  direct
using K256x128_d2 = LdsCfg<256, 128, 64, 2, 2, 2, true>;
using K128x256_d2 = LdsCfg<128, 256, 64, 2, 2, 2, true>;
using K128x128_d2 = LdsCfg<128, 128, 64, 2, 2, 2, true>;
using K128x128_d3 = LdsCfg<128, 128, 64, 2, 2, 3, true>;
using K128x128_r2 = LdsCfg<128, 128, 64, 2, 2, 2, false>;
using K64x64_r2   = LdsCfg< 64,  64, 64, 2, 2, 2, false>;
using K64x64_d3   = LdsCfg< 64,  64, 64, 2, 2, 3, true>;
using K32x128_d3  = LdsCfg< 32, 128, 64, 1, 4, 3, true>;
using K32x64_d4   = LdsCfg< 32,  64, 64, 1, 2, 4, true>;
using K32x128_r2  = LdsCfg< 32, 128, 64, 1, 4, 2, false>;
using K32x128_d6  = LdsCfg< 32, 128, 64, 1, 4, 6, true>;
using K32x64_d8   = LdsCfg< 32,  64, 64, 1, 2, 8, true>;
using K32x256_d4  = LdsCfg< 32, 256, 64, 1, 4, 4, true>;
using K32x32_d4   = LdsCfg< 32,  32, 64, 1, 1, 4, true>;
using K32x32_d8   = LdsCfg< 32,  32, 64, 1, 1, 8, true>;
using K128x128_w8a = LdsCfg<128, 128, 64, 2, 4, 3, true>;   // eight waves: two per SIMD cover each other's overheads
using K128x128_w8b = LdsCfg<128, 128, 64, 4, 2, 3, true>;
using K128x128_w8c = LdsCfg<128, 128, 64, 2, 4, 4, true>;
using K128x256_ab = LdsCfg<128, 256, 64, 4, 1, 2, true, true>;
using K128x128_k2a = LdsCfg<128, 128, 64, 2, 2, 3, true, false, 2>;   // two k groups of 2x2 waves
using K128x128_k2b = LdsCfg<128, 128, 64, 2, 2, 4, true, false, 2>;
// first operand transposed in memory ([K][M])
using T128x128_w8  = LdsCfg<128, 128, 64, 2, 4, 3, true, false, 1, true>;
using T128x128_d3  = LdsCfg<128, 128, 64, 2, 2, 3, true, false, 1, true>;
using T128x128_d2  = LdsCfg<128, 128, 64, 2, 2, 2, true, false, 1, true>;
using T256x256_w8  = LdsCfg<256, 256, 64, 4, 2, 2, true, false, 1, true>;
using T256x128_d2  = LdsCfg<256, 128, 64, 2, 2, 2, true, false, 1, true>;
using T64x64_d3    = LdsCfg< 64,  64, 64, 2, 2, 3, true, false, 1, true>;
// two buffers only: short K (a chunk) means few K steps per tile, and several work-groups per CU
// cover each other's start-up better than a deeper ring in one
using T128x128_w8s2 = LdsCfg<128, 128, 64, 2, 4, 2, true, false, 1, true>;
using T128x64_d2   = LdsCfg<128,  64, 64, 2, 2, 2, true, false, 1, true>;
using T64x128_d2   = LdsCfg< 64, 128, 64, 2, 2, 2, true, false, 1, true>;
using T64x64_d2    = LdsCfg< 64,  64, 64, 2, 2, 2, true, false, 1, true>;
using K256x256_w8a = LdsCfg<256, 256, 64, 2, 4, 2, true>;   // eight waves on the big tile: 128x64 or 64x128 per wave
using K256x256_w8b = LdsCfg<256, 256, 64, 4, 2, 2, true>;
// other K tiles. 128 wide: half as many hand-over barriers per K and 256-byte row pieces from memory, two buffers of
// 64 KB; 32 wide: four buffers of 32 KB behind the big tile, three K tiles in flight instead of one
using K128x128x128_w8a = LdsCfg<128, 128, 128, 2, 4, 2, true>;
using K128x128x128_w8b = LdsCfg<128, 128, 128, 4, 2, 2, true>;
using K128x128x128_k2  = LdsCfg<128, 128, 128, 2, 2, 2, true, false, 2>;
using K256x256x32_w8a  = LdsCfg<256, 256,  32, 2, 4, 4, true>;
using K256x256x32_w8b  = LdsCfg<256, 256,  32, 4, 2, 4, true>;
using K64x64x128_d3    = LdsCfg< 64,  64, 128, 2, 2, 3, true>;
using K32x64x128_d4    = LdsCfg< 32,  64, 128, 1, 2, 4, true>;
// eight waves of 64 x 64 on the rectangular tiles, three buffers of 48 KB
using K256x128_w8 = LdsCfg<256, 128, 64, 4, 2, 3, true>;
using K128x256_w8 = LdsCfg<128, 256, 64, 2, 4, 3, true>;
// second operand given as [N][K], k contiguous: staged and read like the A tile
using N256x256_w8a = LdsCfg<256, 256, 64, 2, 4, 2, true, false, 1, false, true>;
using N256x256_w8b = LdsCfg<256, 256, 64, 4, 2, 2, true, false, 1, false, true>;
using N128x128_w8a = LdsCfg<128, 128, 64, 2, 4, 3, true, false, 1, false, true>;
using N128x128_w8b = LdsCfg<128, 128, 64, 4, 2, 3, true, false, 1, false, true>;
using N128x128_d2  = LdsCfg<128, 128, 64, 2, 2, 2, true, false, 1, false, true>;
using N128x128x128 = LdsCfg<128, 128, 128, 2, 4, 2, true, false, 1, false, true>;
using N64x64_d3    = LdsCfg< 64,  64, 64, 2, 2, 3, true, false, 1, false, true>;
using N32x64_d4    = LdsCfg< 32,  64, 64, 1, 2, 4, true, false, 1, false, true>;
using N32x128_d3   = LdsCfg< 32, 128, 64, 1, 4, 3, true, false, 1, false, true>;
using N32x32_d4    = LdsCfg< 32,  32, 64, 1, 1, 4, true, false, 1, false, true>;
using N256x128_w8 = LdsCfg<256, 128, 64, 4, 2, 3, true, false, 1, false, true>;
// staged through registers: a ragged K tail is filled with zeros (K no multiple of the K tile)
using N128x128_r2 = LdsCfg<128, 128, 64, 2, 2, 2, false, false, 1, false, true>;
using N64x64_r2   = LdsCfg< 64,  64, 64, 2, 2, 2, false, false, 1, false, true>;
using N32x128_r2  = LdsCfg< 32, 128, 64, 1, 4, 2, false, false, 1, false, true>;
using N128x256_w8 = LdsCfg<128, 256, 64, 2, 4, 3, true, false, 1, false, true>;
// the big tile with only 192 of its 256 columns multiplied (4 x 2 waves of 64 x 96): the lighter last round
using K256x192_w8b = LdsCfg<256, 256, 64, 4, 2, 2, true, false, 1, false, false, 192>;
using N256x192_w8b = LdsCfg<256, 256, 64, 4, 2, 2, true, false, 1, false, true, 192>;     // the same with B staged as [n][k]

static LdsKernelInfo g_table[] = {
    make_info<K256x128_d2>(), make_info<K128x256_d2>(),
    make_info<K128x128_d2>(), make_info<K128x128_d3>(), make_info<K128x128_r2>(),
    make_info<K64x64_r2>(),   make_info<K64x64_d3>(),   make_info<K32x128_d3>(),
    make_info<K32x64_d4>(),   make_info<K32x128_r2>(),  make_info<K128x256_ab>(),
     make_info<K32x128_d6>(),  make_info<K32x64_d8>(),
    make_info<K32x256_d4>(),  make_info<K32x32_d4>(),   make_info<K32x32_d8>(),
    make_info<K128x128_w8a>(), make_info<K128x128_w8b>(), make_info<K128x128_w8c>(),
    make_info<K128x128_k2a>(), make_info<K128x128_k2b>(),
    make_info<T128x128_w8>(), make_info<T128x128_d3>(), make_info<T128x128_d2>(), make_info<T256x256_w8>(),
    make_info<T256x128_d2>(), make_info<T64x64_d3>(),
    make_info<T128x128_w8s2>(), make_info<T128x64_d2>(), make_info<T64x128_d2>(), make_info<T64x64_d2>(),
    make_info<K256x256_w8a>(), make_info<K256x256_w8b>(),
    make_persist_info<T128x128_w8>(), make_persist_info<T128x128_d3>(),
    make_info<StreamKCfg<K128x128_w8a>>(), make_info<StreamKCfg<K128x128_w8b>>(), make_info<StreamKCfg<K128x128_k2a>>(),
    make_info<K128x128x128_w8a>(), make_info<K128x128x128_w8b>(), make_info<K128x128x128_k2>(),
    make_info<K256x256x32_w8a>(), make_info<K256x256x32_w8b>(), make_info<K64x64x128_d3>(), make_info<K32x64x128_d4>(),
    make_info<K256x128_w8>(), make_info<K128x256_w8>(),
    make_info<N256x256_w8a>(), make_info<N256x256_w8b>(), make_info<N128x128_w8a>(), make_info<N128x128_w8b>(),
    make_info<N128x128_d2>(), make_info<N128x128x128>(), make_info<N64x64_d3>(), make_info<N32x64_d4>(),
    make_info<N32x128_d3>(), make_info<N32x32_d4>(), make_info<N256x128_w8>(), make_info<N128x256_w8>(),
    make_mixed_info<K256x256_w8a, K256x192_w8b>(), make_mixed_info<K256x256_w8b, K256x192_w8b>(),
    make_mixed_info<N256x256_w8a, N256x192_w8b>(), make_mixed_info<N256x256_w8b, N256x192_w8b>(),
    make_info<N128x128_r2>(), make_info<N64x64_r2>(), make_info<N32x128_r2>(),
};

// these first: the ids of a family's variants follow the order of the table
static const std::vector<LdsKernelInfo>& all_kernels() {
  static const std::vector<LdsKernelInfo> all = [] {
    std::vector<LdsKernelInfo> v(std::begin(g_table), std::end(g_table));
    int n = 0;
    const LdsKernelInfo* more = lds_ragged_table(&n);
    v.insert(v.end(), more, more + n);
    more = lds_192_table(&n);
    v.insert(v.end(), more, more + n);
    more = lds_64x128_table(&n);
    v.insert(v.end(), more, more + n);
    for (size_t i = v.size() - n; i < v.size(); ++i) v[i].appended = 1;
    for (LdsKernelInfo& k : v)
      if (k.lines) k.appended = 2;
    return v;
  }();
  return all;
}
int lds_kernel_count() { return (int)all_kernels().size(); }
const LdsKernelInfo* lds_kernel_table() { return all_kernels().data(); }

}  // namespace tf
