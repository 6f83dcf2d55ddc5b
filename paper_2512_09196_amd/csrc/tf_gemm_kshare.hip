// bf16 MFMA GEMM with the fused epilogues for problems with few output tiles, on gfx950: the waves of a work-group share K.
//
// A small or skinny problem, or one with a long sum, has too few tiles of 128 or 256 for 256 CUs, and the small tiles of
// the other LDS kernels (tf_gemm_lds.h) walk through K one barrier at a time with little in flight. Here
//  * the NW waves of a work-group share K, not the tile: wave w takes the K tiles (of 64) w, w + NW, ... of the work-group's
//    range, staged direct to LDS in a ring of its own (layouts and swizzles of tf_gemm_lds.h), and keeps accumulators of
//    the whole tile. No barrier in the main loop: a wave waits for its own transfers only, and hands a buffer to the next
//    transfer as soon as it has read it into registers (with one buffer the registers are the second one). 64 to 128 KB are
//    in flight per CU. The sums meet in LDS once, at the end, and are added in wave order.
//  * where tiles alone leave CUs idle, work-groups share K too. Slice s runs on the XCDs that 8 / S of them make up (or
//    an XCD takes S / 8 slices): every byte of A and B then enters one L2, or 8 / S of them, instead of all eight (with
//    the slices of a tile on one XCD and partial tiles exchanged through its L2, 283 x 448 x 8512 took 12.3 us, this way
//    10.9; 89 x 256 x 13952 9.1 and 7.9; 248 x 1024 x 11456 18.1 and 16.7). Partial tiles go past the
//    L2; the slice that arrives last adds them in slice order.
//  * CUT: tiles of fewer rows and columns than the kernel's largest, for problems whose whole tiles are fewer than the CUs or
//    mostly padding (8 rows of A in a tile of 32 are three quarters of its transfers). A kernel of its own: what it decides for
//    every transfer costs whole tiles 0.4 to 0.8 us. See tf::kshare_shape for the choice and what it gives.
// What bounds it: a CU fetches 76 to 97 GB/s this way (the tiles' row and column panels, mostly from L2), the L2s together
// fetch 7.4 TB/s, a launch takes 2.9 us and an exchange 1.5 to 3 (tf_predict_us has the fit). Hence no larger tiles:
// of 64 x 128, 128 x 64 and 128 x 128 (four waves) none led where the other LDS kernels do not, and four waves with two or
// four buffers in place of the table's choices were level or up to 15 % behind.
// Measured, pick of the other kernels / here (us, operands of three calls in turn): 25 x 6288 x 4584, B [N][K], fp32 21.6 /
// 12.9; 16 x 5392 x 6336 25.9 / 15.7; 13 x 9344 x 3776 20.0 / 13.1; 64 x 256 x 16384 35.4 / 8.2 (with slices);
// 613 x 256 x 1600 8.9 / 4.8; 248 x 1800 x 1752 11.8 / 8.7; 512 x 512 x 8192 23.8 / 13.4.
#include <algorithm>

#include "tf_gemm_lds.h"
#include "tf_loop.h"

namespace tf {

// One wave's part of the work: the whole tile over every NW-th K tile of 64, staged in a ring of its own. BM x BN is the
// largest tile; a launch of cut tiles takes 8 p.groups_a <= BM rows and (B as [N][K]) 8 p.groups_b <= BN columns for a tile,
// the same for every one, and p.ring_stages K tiles for a ring.
template <int BM_, int BN_, int NW_, int S_, bool TB_>
struct KshareCfg : LdsCfg<(BM_ < 32 ? 32 : BM_), BN_, 64, 1, 1, S_, true, false, 1, false, TB_> {
  static constexpr int BM = BM_, A_PER_WAVE = BM_ / 8;
  static constexpr int NW = NW_, WG_THREADS = 64 * NW_;
  static constexpr bool B_NT = false;
  // blocks of 16 x 16 over 32 of K: a wave has a K tile's fragments in half as many dependent MFMAs, of half the latency
  static constexpr int MB = 16, KMF = 32, TM = BM_ / 16, TN = BN_ / 16;
  static constexpr bool HAS_WHOLE = BM_ >= 32, HAS_CUT = !(BM_ == 32 && BN_ == 32);      // which kernels there are, see tf::kshare_shape
  // transfers of a K tile, at most, where a cut's ring holds two
  static constexpr int MAX_FLYING = BM_ > 32 || !HAS_CUT ? 0 : KSHARE_TWO_TILES_KB / NW_ < BM_ / 8 + BN_ / 8 ? KSHARE_TWO_TILES_KB / NW_ : BM_ / 8 + BN_ / 8;
  // what a launch may ask for: whole tiles, or a cut that the kernel has a main loop for
  static bool takes(int groups_a, int groups_b, int stages) {
    if (HAS_WHOLE && groups_a == BM_ / 8 && groups_b == BN_ / 8) return stages == S_;
    const bool cut = groups_a >= 1 && groups_a <= BM_ / 8 && groups_b <= BN_ / 8 && (TB_ ? groups_b >= 1 : groups_b == BN_ / 8);
    return HAS_CUT && cut && (stages == 1 || (stages == 2 && groups_a + groups_b <= MAX_FLYING));
  }
  static constexpr int SUMS = BM_ * BN_ * 4;                  // bytes of a wave's partial sums, where its ring was
  static constexpr int CPR = BN_ / 4, CHUNKS = BM_ * CPR;     // 16-byte pieces of fp32 sums: per row, per tile
  static constexpr int PER_THREAD = CHUNKS < WG_THREADS ? 1 : CHUNKS / WG_THREADS;
  static_assert(MAX_FLYING < 6, "a main loop for each count of transfers");
  static_assert(CHUNKS % WG_THREADS == 0 || CHUNKS < WG_THREADS, "the pieces divide over the threads");
};

// 16 bytes past this XCD's L2, written by work-groups of other XCDs
__device__ __forceinline__ f32x4 load_device(const float* src) {
  typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
  const u64x2 w = {__hip_atomic_load((unsigned long long*)src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                   __hip_atomic_load((unsigned long long*)src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
  return __builtin_bit_cast(f32x4, w);
}

template <class C, bool CUT>
__global__ void __launch_bounds__(C::WG_THREADS) tf_gemm_kshare_kernel(const GemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles = p.tiles_m * p.tiles_n;
  int tile, ks = 0;
  if (!CUT && p.split_k > 1) {
    const int x = blockIdx.x & 7;
    int j = (int)(blockIdx.x >> 3), g = 1, sub = 0;
    if (p.split_k <= 8) { g = 8 / p.split_k; ks = x / g; sub = x - ks * g; }
    else { const int per = p.split_k / 8; ks = x * per + j % per; j /= per; }
    const int base = tiles / g, rem = tiles - base * g;
    if (j >= base + (sub < rem ? 1 : 0)) return;
    tile = sub * base + (sub < rem ? sub : rem) + j;
  } else {
    tile = xcd_run(blockIdx.x, tiles);
  }
  const TileCoord tc = tile_at(p, tile);
  const int groups_a = CUT ? p.groups_a : C::BM / 8, groups_b = CUT && C::TRANSB ? p.groups_b : C::BN / 8;
  const int rows = 8 * groups_a, cols = 8 * groups_b;
  const int m0 = tc.tm * rows, n0 = tc.tn * cols;
  const int m_end = m0 + rows < p.M ? m0 + rows : p.M, n_end = n0 + cols < p.N ? n0 + cols : p.N;
  const int a_bytes = groups_a * 1024, stage_bytes = a_bytes + groups_b * 1024;
  const int per_tile = stage_bytes >> 10;                   // transfers of a K tile
  const int stages = CUT ? p.ring_stages : C::STAGES;
  const int ring_bytes = stages * stage_bytes > C::SUMS ? stages * stage_bytes : C::SUMS;
  char* const ring = smem + wave * ring_bytes;
  const unsigned ring_lds = (unsigned)(size_t)smem + wave * ring_bytes;

  TileLoader<C> ld;
  ld.init(p, m0, n0, 0, lane);
  const int nkt = (p.K + 63) >> 6, skip = 64 * nkt - p.K;
  const int kt0 = ks * p.ktiles_per_split + wave;
  const int kt1 = (ks + 1) * p.ktiles_per_split < nkt ? (ks + 1) * p.ktiles_per_split : nkt;
  const int n_own = kt1 > kt0 ? (kt1 - kt0 + C::NW - 1) / C::NW : 0;
  int issued = 0;
  unsigned to = ring_lds;                                   // where the next K tile goes
  auto issue = [&]() {
    const int t = kt0 + issued * C::NW;
    const long k0 = t == nkt - 1 ? (long)p.K - 64 : 64L * t;
    const uint16_t* const Ak = p.A + k0;
    const uint16_t* const Bk = p.B + (C::TRANSB ? k0 : k0 * p.ldb);
#pragma unroll
    for (int q = 0; q < C::A_PER_WAVE; ++q)
      if (q < groups_a) TileLoader<C>::gload_lds16(to + q * 1024, ld.a_src[q], Ak);
    const unsigned to_b = to + a_bytes;
#pragma unroll
    for (int q = 0; q < C::B_PER_WAVE; ++q)
      if (q < groups_b) TileLoader<C>::gload_lds16(to_b + q * 1024, ld.b_src[q], Bk);
    ++issued;
    to += stage_bytes;
    if (to == ring_lds + stages * stage_bytes) to = ring_lds;
  };
#pragma unroll
  for (int s = 0; s < 2; ++s)
    if (s < stages && s < n_own) issue();

  // this thread's four bias values: its pieces of the tile all lie in the same columns
  static_assert(C::WG_THREADS % C::CPR == 0, "one column group per thread");
  const int n = n0 + 4 * (tid % C::CPR);
  const bool n_ok = n < n_end;

  f32x4 acc[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int t = 0; t < C::TN; ++t) acc[i][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  const int fr = lane & 15, fg = lane >> 4;
  // rows of an operand that were not fetched are read as its last one: what comes of them is not stored
  int a_row[C::TM], b_row[C::TN];
#pragma unroll
  for (int x = 0; x < C::TM; ++x) a_row[x] = 16 * x + fr < rows ? 16 * x + fr : rows - 1;
#pragma unroll
  for (int x = 0; x < C::TN; ++x) b_row[x] = 16 * x + fr < cols ? 16 * x + fr : cols - 1;
  auto read_kc = [&](const char* base, int row, int kk) { return *(const bf16x8*)(base + row * 128 + (((4 * kk + fg) ^ C::row_swz(row)) << 4)); };
  // [K][N]: lane group g reads four rows of 16 columns from row 8 g on, then the next four
  const int tk = 8 * fg + (fr >> 2);
  int b_off[C::TN];
#pragma unroll
  for (int x = 0; x < C::TN; ++x) {
    const int c = 16 * x + 4 * (fr & 3);
    b_off[x] = tk * C::B_ROW_BYTES + (((c >> 3) ^ b_chunk_swz<C>(tk)) << 4) + (c & 7) * 2;
  }

  // FLYING: transfers of a second K tile in the ring, which may still fly when a tile is about to be read; one fewer than there
  // are where their number is odd. (A loop for each count: picking the wait inside the loop cost 32 x 32 tiles 15 to 20 %.)
  auto main_loop = [&](auto flying) {
  constexpr int FLYING = decltype(flying)::value;
  char* st = ring;
  for (int i = 0; i < n_own; ++i) {
    if (FLYING && i + 1 < n_own) wait_vmcnt<FLYING>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    if (skip && kt0 + i * C::NW == nkt - 1) {
      // the last K tile was fetched from K - 64 on: the k that the tile before holds are zeroed, in both operands
      const u32x4 zero = {0u, 0u, 0u, 0u};
      auto k_contiguous = [&](char* tile_lds, int rows) {
        for (int c = 0; c < skip / 8; ++c)
          for (int r = lane; r < rows; r += 64) *(u32x4*)(tile_lds + r * 128 + ((c ^ C::row_swz(r)) << 4)) = zero;
      };
      k_contiguous(st, rows);
      if constexpr (C::TRANSB) k_contiguous(st + a_bytes, cols);
      else
        for (int x = lane * 16; x < skip * C::B_ROW_BYTES; x += 1024) *(u32x4*)(st + a_bytes + x) = zero;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    bf16x8 af[2][C::TM], bfr[2][C::TN];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int x = 0; x < C::TM; ++x) af[kk][x] = read_kc(st, a_row[x], kk);
#pragma unroll
      for (int x = 0; x < C::TN; ++x) {
        if constexpr (C::TRANSB) {
          bfr[kk][x] = read_kc(st + a_bytes, b_row[x], kk);
        } else {
          const char* bp = st + a_bytes + b_off[x] + 32 * kk * C::B_ROW_BYTES;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp + 4 * C::B_ROW_BYTES));
          const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          bfr[kk][x] = __builtin_bit_cast(bf16x8, v);
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the buffer has been read: its next tile may come
    if (issued < n_own) issue();
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int x = 0; x < C::TM; ++x)
#pragma unroll
        for (int y = 0; y < C::TN; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[kk][y], af[kk][x], acc[x][y], 0, 0, 0);
    st += stage_bytes;
    if (st == ring + stages * stage_bytes) st = ring;
  }
  };
  if constexpr (!CUT) {
    main_loop(EpiTag<C::STAGES == 1 ? 0 : C::BM / 8 + C::BN / 8>{});
  } else {
    switch (stages == 1 ? 0 : per_tile / 2) {      // (one jump over the loops not taken: a chain of tests between them cost 0.8 us)
      case 0: main_loop(EpiTag<0>{}); break;
      case 1: if constexpr (C::MAX_FLYING >= 2) main_loop(EpiTag<2>{}); break;
      case 2: if constexpr (C::MAX_FLYING >= 4) main_loop(EpiTag<4>{}); break;
      default: break;                              // (the host launches none: KshareCfg::takes)
    }
  }

  const u32x2 braw = n_ok ? *(const u32x2*)(p.bias + n) : u32x2{0u, 0u};
  // ---- partial sums to this wave's LDS: [row][4-column piece ^ swizzle], 16 bytes each. Lane l, register e of a
  // 16 x 16 block: m = l & 15, n = 4 (l / 16) + e
  auto swz = [](int m) { return C::CPR >= 16 ? m & 15 : (m >> 1) & 7; };
#pragma unroll
  for (int i = 0; i < C::TM; ++i) {
    const int m = 16 * i + fr;
#pragma unroll
    for (int j = 0; j < C::TN; ++j) *(f32x4*)(ring + (m * C::CPR + ((4 * j + fg) ^ swz(m))) * 16) = acc[i][j];
  }
  __syncthreads();
  f32x4 z[C::PER_THREAD];
#pragma unroll
  for (int y = 0; y < C::PER_THREAD; ++y) {
    const int x = tid + y * C::WG_THREADS, r = C::CHUNKS < C::WG_THREADS && x >= C::CHUNKS ? C::BM - 1 : x / C::CPR, c = x % C::CPR;
    z[y] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < C::NW; ++w) z[y] += *(const f32x4*)(smem + w * ring_bytes + (r * C::CPR + (c ^ swz(r))) * 16);
  }

  if (!CUT && p.split_k > 1) {
    // the sums of a slice to the workspace, [slice][M][N]; the slice of a tile that arrives last adds them up in slice order
    const size_t slice = (size_t)p.M * p.N;
    float* const corner = p.ws + (size_t)m0 * p.N + n;
    bool ok[C::PER_THREAD];
#pragma unroll
    for (int y = 0; y < C::PER_THREAD; ++y) {
      const int x = tid + y * C::WG_THREADS, r = x / C::CPR;
      ok[y] = m0 + r < m_end && n_ok;
      if (ok[y]) store_through_f32x4(corner + ks * slice + (size_t)r * p.N, z[y]);
    }
    // every store of this wave has been acknowledged before the wave reaches the barrier, so the ticket taken behind
    // it is ordered behind the whole work-group's sums
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    __shared__ unsigned ticket;
    unsigned* const ctr = p.counters + 2 * tile;          // (one 8-byte counter per tile in the workspace)
    if (tid == 0) ticket = atomicAdd(ctr, 1u) + 1u;
    __syncthreads();
    if (ticket != (unsigned)p.split_k) return;
    if (tid == 0) *ctr = 0u;                              // ready for the next launch
#pragma unroll
    for (int y = 0; y < C::PER_THREAD; ++y) z[y] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int G = 8 / C::PER_THREAD;                  // slices per trip to memory
    static_assert(G >= 1, "register budget of the exchange");
    for (int s0 = 0; s0 < p.split_k; s0 += G) {
      f32x4 v[G][C::PER_THREAD];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int s = s0 + g < p.split_k ? s0 + g : p.split_k - 1;
#pragma unroll
        for (int y = 0; y < C::PER_THREAD; ++y)      // (a piece outside Y reads the workspace's first 16 bytes and is not stored)
          v[g][y] = load_device(ok[y] ? corner + s * slice + (size_t)((tid + y * C::WG_THREADS) / C::CPR) * p.N : p.ws);
      }
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int y = 0; y < C::PER_THREAD; ++y)
          if (s0 + g < p.split_k) z[y] += v[g][y];
    }
  }

  const float b0 = __builtin_bit_cast(float, braw[0] << 16), b1 = __builtin_bit_cast(float, braw[0] & 0xffff0000u);
  const float b2 = __builtin_bit_cast(float, braw[1] << 16), b3 = __builtin_bit_cast(float, braw[1] & 0xffff0000u);
#pragma unroll
  for (int y = 0; y < C::PER_THREAD; ++y) {
    const int x = tid + y * C::WG_THREADS, m = m0 + x / C::CPR;
    if (m >= m_end || !n_ok) continue;
    const float z0 = z[y][0] + b0, z1 = z[y][1] + b1, z2 = z[y][2] + b2, z3 = z[y][3] + b3;
    if (p.epi == TF_EPI_NONE_F32) {
      const f32x4 v = {z0, z1, z2, z3};
      *(f32x4*)((float*)p.Y + (size_t)m * p.ldy + n) = v;
    } else {
      u32x2 o;
      const f32x4 a = activate(f32x4{z0, z1, z2, z3}, p.epi);
      o[0] = pack_bf16x2(a[0], a[1]);
      o[1] = pack_bf16x2(a[2], a[3]);
      *(u32x2*)((uint16_t*)p.Y + (size_t)m * p.ldy + n) = o;
    }
  }
}

template <class C>
static void launch_kshare(const GemmParams& p, dim3 grid, hipStream_t stream) {
  const bool whole = p.groups_a == C::BM / 8 && p.groups_b == C::BN / 8;
  const int lds = C::NW * std::max(p.ring_stages * (p.groups_a + p.groups_b) * 1024, C::SUMS);
  if constexpr (C::HAS_CUT)
    if (!C::HAS_WHOLE || !whole) hipLaunchKernelGGL((tf_gemm_kshare_kernel<C, true>), grid, dim3(C::WG_THREADS), lds + KSHARE_CUT_MARK, stream, p);
  if constexpr (C::HAS_WHOLE)
    if (!C::HAS_CUT || whole) hipLaunchKernelGGL((tf_gemm_kshare_kernel<C, false>), grid, dim3(C::WG_THREADS), lds, stream, p);
}
template <class C>
static KshareKernelInfo make_kshare_info() {
  KshareKernelInfo k;
  k.bm = C::BM; k.bn = C::BN; k.waves = C::NW; k.stages = C::STAGES; k.trans_b = C::TRANSB ? 1 : 0;
  k.threads = C::WG_THREADS;
  k.func = k.func_cut = nullptr;
  if constexpr (C::HAS_WHOLE) k.func = (const void*)tf_gemm_kshare_kernel<C, false>;
  if constexpr (C::HAS_CUT) k.func_cut = (const void*)tf_gemm_kshare_kernel<C, true>;
  k.takes = C::takes;
  k.launch = launch_kshare<C>;
  return k;
}

static const KshareKernelInfo g_kshare_table[] = {
    make_kshare_info<KshareCfg<32, 32, 4, 2, false>>(), make_kshare_info<KshareCfg<32, 64, 8, 1, false>>(), make_kshare_info<KshareCfg<64, 64, 8, 1, false>>(),
    make_kshare_info<KshareCfg<32, 32, 4, 2, true>>(),  make_kshare_info<KshareCfg<32, 64, 8, 1, true>>(),  make_kshare_info<KshareCfg<64, 64, 8, 1, true>>(),
    make_kshare_info<KshareCfg<16, 32, 8, 1, false>>(), make_kshare_info<KshareCfg<16, 32, 16, 1, false>>(),
    make_kshare_info<KshareCfg<16, 32, 8, 1, true>>(),  make_kshare_info<KshareCfg<16, 32, 16, 1, true>>(),
};
int kshare_kernel_count() { return (int)(sizeof(g_kshare_table) / sizeof(g_kshare_table[0])); }
const KshareKernelInfo* kshare_kernel_table() { return g_kshare_table; }
bool kshare_takes(int kernel, int groups_a, int groups_b, int stages) { return g_kshare_table[kernel].takes(groups_a, groups_b, stages); }

}  // namespace tf
