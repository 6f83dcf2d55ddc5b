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
// What bounds it: a CU fetches 76 to 97 GB/s this way (the tiles' row and column panels, mostly from L2), the L2s together
// fetch 7.4 TB/s, a launch takes 2.9 us and an exchange 1.5 to 3 (tf_predict_us has the fit). Hence no larger tiles:
// of 64 x 128, 128 x 64 and 128 x 128 (four waves) none led where the other LDS kernels do not, and four waves with two or
// four buffers in place of the table's choices were level or up to 15 % behind.
// Measured, pick of the other kernels / here (us, operands of three calls in turn): 25 x 6288 x 4584, B [N][K], fp32 21.6 /
// 12.9; 16 x 5392 x 6336 25.9 / 15.7; 13 x 9344 x 3776 20.0 / 13.1; 64 x 256 x 16384 35.4 / 8.2 (with slices);
// 613 x 256 x 1600 8.9 / 4.8; 248 x 1800 x 1752 11.8 / 8.7; 512 x 512 x 8192 23.8 / 13.4.
#include "tf_gemm_lds.h"

namespace tf {

// One wave's part of the work: the whole BM x BN tile over every NW-th K tile of 64, staged in a ring of its own.
template <int BM_, int BN_, int NW_, int S_, bool TB_>
struct KshareCfg : LdsCfg<BM_, BN_, 64, 1, 1, S_, true, false, 1, false, TB_> {
  using Base = LdsCfg<BM_, BN_, 64, 1, 1, S_, true, false, 1, false, TB_>;
  static constexpr int NW = NW_, WG_THREADS = 64 * NW_;
  static constexpr bool B_NT = false;
  static constexpr int PER_TILE = Base::A_PER_WAVE + Base::B_PER_WAVE;
  static constexpr int RING = S_ * Base::STAGE_BYTES;
  static constexpr int WG_LDS = NW_ * RING;
  static constexpr int CPR = BN_ / 4, CHUNKS = BM_ * CPR;     // 16-byte pieces of fp32 sums: per row, per tile
  static constexpr int PER_THREAD = CHUNKS / WG_THREADS;
  static_assert(BM_ * BN_ * 4 <= RING, "the partial sums fit where the tiles were");
  static_assert(S_ <= 2 && PER_TILE < 64, "the main loop waits for at most one younger K tile; vmcnt range");
  static_assert(CHUNKS % WG_THREADS == 0, "the pieces divide over the threads");
  static_assert(WG_LDS <= 160 * 1024, "LDS budget of one CU");
};

// 16 bytes past this XCD's L2, for work-groups of other XCDs to read or written by them
__device__ __forceinline__ void store_device(float* dst, const f32x4 v) {
  typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
  const u64x2 w = __builtin_bit_cast(u64x2, v);
  __hip_atomic_store((unsigned long long*)dst, w[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store((unsigned long long*)dst + 1, w[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x4 load_device(const float* src) {
  typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
  const u64x2 w = {__hip_atomic_load((unsigned long long*)src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                   __hip_atomic_load((unsigned long long*)src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
  return __builtin_bit_cast(f32x4, w);
}

template <class C>
__global__ void __launch_bounds__(C::WG_THREADS) tf_gemm_kshare_kernel(const GemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles = p.tiles_m * p.tiles_n;
  int tile, ks = 0;
  if (p.split_k > 1) {
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
  const int m0 = tc.tm * C::BM, n0 = tc.tn * C::BN;
  char* const ring = smem + wave * C::RING;
  const unsigned ring_lds = (unsigned)(size_t)smem + wave * C::RING;

  TileLoader<C> ld;
  ld.init(p, m0, n0, 0, lane);
  const int nkt = (p.K + 63) >> 6, skip = 64 * nkt - p.K;
  const int kt0 = ks * p.ktiles_per_split + wave;
  const int kt1 = (ks + 1) * p.ktiles_per_split < nkt ? (ks + 1) * p.ktiles_per_split : nkt;
  const int n_own = kt1 > kt0 ? (kt1 - kt0 + C::NW - 1) / C::NW : 0;
  auto issue = [&](int i) {
    const int t = kt0 + i * C::NW;
    const long k0 = t == nkt - 1 ? (long)p.K - 64 : 64L * t;
    ld.issue_direct(p.A + k0, p.B + (C::TRANSB ? k0 : k0 * p.ldb), ring_lds + (i % C::STAGES) * C::STAGE_BYTES, 0);
  };
#pragma unroll
  for (int s = 0; s < C::STAGES; ++s)
    if (s < n_own) issue(s);

  // this thread's four bias values: its pieces of the tile all lie in the same columns
  static_assert(C::WG_THREADS % C::CPR == 0, "one column group per thread");
  const int n = n0 + 4 * (tid % C::CPR);
  const bool n_ok = n < p.N;

  f32x16 acc[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int t = 0; t < C::TN; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][t][r] = 0.0f;

  const int fr = lane & 31, fg = lane >> 5, fsw = C::row_swz(fr);
  const int tb = lane >> 4, ts = lane & 15;
  const int tk = 8 * (tb >> 1) + (ts >> 2), twithin = (16 * (tb & 1) + 4 * (ts & 3)) * 2;
  auto read_kc = [&](const char* base, int kk) { return *(const bf16x8*)(base + fr * 128 + (((2 * kk + fg) ^ fsw) << 4)); };

  int stage = 0;
  for (int i = 0; i < n_own; ++i) {
    // this tile has landed; with two buffers the next one may still fly
    if (C::STAGES > 1 && i + 1 < n_own) wait_vmcnt<(C::STAGES - 1) * C::PER_TILE>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    char* const st = ring + stage * C::STAGE_BYTES;
    if (skip && kt0 + i * C::NW == nkt - 1) {
      // the last K tile was fetched from K - 64 on: the k that the tile before holds are zeroed, in both operands
      const u32x4 zero = {0u, 0u, 0u, 0u};
      auto k_contiguous = [&](char* tile_lds, int rows) {
        for (int c = 0; c < skip / 8; ++c)
          for (int r = lane; r < rows; r += 64) *(u32x4*)(tile_lds + r * 128 + ((c ^ C::row_swz(r)) << 4)) = zero;
      };
      k_contiguous(st, C::BM);
      if constexpr (C::TRANSB) k_contiguous(st + C::A_BYTES, C::BN);
      else
        for (int x = lane * 16; x < skip * C::B_ROW_BYTES; x += 1024) *(u32x4*)(st + C::A_BYTES + x) = zero;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    bf16x8 af[4][C::TM], bfr[4][C::TN];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
      for (int x = 0; x < C::TM; ++x) af[kk][x] = read_kc(st + x * 4096, kk);
#pragma unroll
      for (int x = 0; x < C::TN; ++x) {
        if constexpr (C::TRANSB) {
          bfr[kk][x] = read_kc(st + C::A_BYTES + x * 4096, kk);
        } else {
          const int piece = x ^ b_swz<C::B_PIECES>(tk);
          const char* bp = st + C::A_BYTES + (16 * kk + tk) * C::B_ROW_BYTES + piece * 64 + twithin;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp + 4 * C::B_ROW_BYTES));
          const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          bfr[kk][x] = __builtin_bit_cast(bf16x8, v);
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the buffer has been read: its next tile may come
    if (i + C::STAGES < n_own) issue(i + C::STAGES);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int x = 0; x < C::TM; ++x)
#pragma unroll
        for (int y = 0; y < C::TN; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[kk][y], af[kk][x], acc[x][y], 0, 0, 0);
    if (++stage == C::STAGES) stage = 0;
  }

  const u32x2 braw = n_ok ? *(const u32x2*)(p.bias + n) : u32x2{0u, 0u};
  // ---- partial sums to this wave's LDS: [row][4-column piece ^ swizzle], 16 bytes each. Lane l, register e of a
  // 32 x 32 block: m = l & 31, n = 8 (e / 4) + 4 (l / 32) + e % 4
  auto swz = [](int m) { return C::CPR >= 16 ? m & 15 : (m >> 1) & 7; };
#pragma unroll
  for (int i = 0; i < C::TM; ++i) {
    const int m = 32 * i + fr;
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        *(f32x4*)(ring + (m * C::CPR + ((8 * j + 2 * q + fg) ^ swz(m))) * 16) = v;
      }
  }
  __syncthreads();
  f32x4 z[C::PER_THREAD];
#pragma unroll
  for (int y = 0; y < C::PER_THREAD; ++y) {
    const int x = tid + y * C::WG_THREADS, r = x / C::CPR, c = x % C::CPR;
    z[y] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < C::NW; ++w) z[y] += *(const f32x4*)(smem + w * C::RING + (r * C::CPR + (c ^ swz(r))) * 16);
  }

  if (p.split_k > 1) {
    // the sums of a slice to the workspace, [slice][M][N]; the slice of a tile that arrives last adds them up in slice order
    const size_t slice = (size_t)p.M * p.N;
    float* const corner = p.ws + (size_t)m0 * p.N + n;
    bool ok[C::PER_THREAD];
#pragma unroll
    for (int y = 0; y < C::PER_THREAD; ++y) {
      const int x = tid + y * C::WG_THREADS, r = x / C::CPR;
      ok[y] = m0 + r < p.M && n_ok;
      if (ok[y]) store_device(corner + ks * slice + (size_t)r * p.N, z[y]);
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
    if (m >= p.M || !n_ok) continue;
    const float z0 = z[y][0] + b0, z1 = z[y][1] + b1, z2 = z[y][2] + b2, z3 = z[y][3] + b3;
    if (p.epi == TF_EPI_NONE_F32) {
      const f32x4 v = {z0, z1, z2, z3};
      *(f32x4*)((float*)p.Y + (size_t)m * p.ldy + n) = v;
    } else {
      u32x2 o;
      o[0] = pack_bf16x2(activate(z0, p.epi), activate(z1, p.epi));
      o[1] = pack_bf16x2(activate(z2, p.epi), activate(z3, p.epi));
      *(u32x2*)((uint16_t*)p.Y + (size_t)m * p.ldy + n) = o;
    }
  }
}

template <class C>
static void launch_kshare(const GemmParams& p, dim3 grid, hipStream_t stream) {
  hipLaunchKernelGGL(tf_gemm_kshare_kernel<C>, grid, dim3(C::WG_THREADS), C::WG_LDS, stream, p);
}
template <class C>
static KshareKernelInfo make_kshare_info() {
  KshareKernelInfo k;
  k.bm = C::BM; k.bn = C::BN; k.waves = C::NW; k.stages = C::STAGES; k.trans_b = C::TRANSB ? 1 : 0;
  k.threads = C::WG_THREADS; k.lds_bytes = C::WG_LDS;
  k.func = (const void*)tf_gemm_kshare_kernel<C>;
  k.launch = launch_kshare<C>;
  return k;
}

static const KshareKernelInfo g_kshare_table[] = {
    make_kshare_info<KshareCfg<32, 32, 4, 2, false>>(), make_kshare_info<KshareCfg<32, 64, 8, 1, false>>(), make_kshare_info<KshareCfg<64, 64, 8, 1, false>>(),
    make_kshare_info<KshareCfg<32, 32, 4, 2, true>>(),  make_kshare_info<KshareCfg<32, 64, 8, 1, true>>(),  make_kshare_info<KshareCfg<64, 64, 8, 1, true>>(),
};
int kshare_kernel_count() { return (int)(sizeof(g_kshare_table) / sizeof(g_kshare_table[0])); }
const KshareKernelInfo* kshare_kernel_table() { return g_kshare_table; }

}  // namespace tf
