// bf16 MFMA GEMM with the fused epilogues for operands whose rows start at any two-byte address (odd dimensions,
// leading dimensions or pointers), on gfx950; also what the static pick of a small problem takes.
//
// The tile kernels copy 16-byte pieces that must not straddle a row end; here nothing is known about alignment. What
// is left is a problem of latency (the sizes are small: a few hundred to a few thousand per dimension), so the
// design keeps many loads in flight and no barrier in the main loop:
//  * a work-group computes a 32 T x 32 T tile of Y; its NW waves share K, not the tile: wave w takes the K tiles (of
//    64) w, w + NW, ... and keeps accumulators of the whole tile. The partial sums meet in LDS once, at the end,
//    and are added in wave order.
//  * a wave loads its A and B tiles by 16-byte loads of two-byte alignment, eight (T = 1) or sixteen (T = 2) of them
//    per K tile, 128 bytes of a row per eight lanes, into one of two register sets: two K tiles are in flight.
//    It passes them through its own piece of LDS (the layouts of the other tile kernels: k-contiguous rows
//    with XOR-swizzled 16-byte chunks, read by ds_read_b128; [k][n] rows read by the transposing
//    ds_read_b64_tr_b16) - fragments straight from memory would touch 32 rows per load instead of eight.
//  * every load stays inside its operand without a check per element: rows past M (or N, B as [N][K]) repeat the last
//    one; the last K tile starts at K - 64 and the k that the tile before holds are zeroed in registers, in
//    both operands; the last column tile of a [K][N] B starts at N - 32 T and stores only its own columns.
//    Hence K >= 64, and N >= 32 T where B is [K][N].
// 509 x 1021 x 763 (fp32 result): 53.8 us a call on the one-wave-per-tile kernel that gathers element by element, 6.8 us
// here; the kernel alone takes 42.7 and 8.4 us there with cold operands. Matrix pipes 2 %
// busy, 92 % of the reads hit in L2: what is left is the trip to memory and back. Where K is long and the tiles are
// fewer than the CUs, a CU's own rate bounds it (64 x 256 x 16384 35 us, 60 GB/s per CU).
#include "tf_device.h"

namespace tf {

template <int T_, int NW_, bool TB_>
struct AnyCfg {
  static constexpr int T = T_, NW = NW_, TILE = 32 * T_, THREADS = 64 * NW_;
  static constexpr bool TB = TB_;                       // B is [N][ldb], k contiguous
  static constexpr int NL = 4 * T;                      // 16-byte loads per lane, operand and K tile
  static constexpr int OP_BYTES = TILE * 128;           // one operand's K tile
  static constexpr int WAVE_BYTES = 2 * OP_BYTES;       // a wave's LDS: its A and B tile, later its partial sums
  static_assert(TILE * TILE * 4 <= WAVE_BYTES, "the partial sums fit where the tiles were");
  static constexpr int LDS_BYTES = NW * WAVE_BYTES;
  static constexpr int CPR = TILE / 4;                  // 16-byte chunks per row of the partial sums
  static constexpr int B_ROW_BYTES = TILE * 2, B_PIECES = B_ROW_BYTES / 64, B_CHUNKS = B_ROW_BYTES / 16;   // [k][n] tile
};

typedef u32x4 u32x4_any __attribute__((aligned(2)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));

template <class C>
__global__ void __launch_bounds__(C::THREADS, C::T == 1 ? 2 : 1) tf_gemm_any_kernel(const GemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const TileCoord tc = map_tile(p, blockIdx.x);
  const int m0 = tc.tm * C::TILE, n_own = tc.tn * C::TILE;       // first row; first column this tile stores
  const int n0 = !C::TB && n_own > p.N - C::TILE ? p.N - C::TILE : n_own;
  char* const a_lds = smem + wave * C::WAVE_BYTES;
  char* const b_lds = a_lds + C::OP_BYTES;

  // ---- byte offsets of this lane's pieces from the tile's corner (32 bits: the host bounds the leading dimensions)
  unsigned a_src[C::NL], b_src[C::NL];
  int b_dst[C::NL];
  const int row8 = lane >> 3, c8 = lane & 7;            // k-contiguous tiles: eight lanes per row of 64 k
  const int a_dst = row8 * 128 + ((c8 ^ (lane >> 4)) << 4);      // + 1024 q: slot = chunk ^ (row / 2 mod 8)
#pragma unroll
  for (int q = 0; q < C::NL; ++q) {
    int r = 8 * q + row8;
    if (m0 + r >= p.M) r = p.M - 1 - m0;
    a_src[q] = ((unsigned)r * (unsigned)p.lda + 8u * c8) * 2u;
    if constexpr (C::TB) {
      int n = 8 * q + row8;
      if (n0 + n >= p.N) n = p.N - 1 - n0;
      b_src[q] = ((unsigned)n * (unsigned)p.ldb + 8u * c8) * 2u;
      b_dst[q] = 0;
    } else {
      const int x = 64 * q + lane, k = x / C::B_CHUNKS, c = x % C::B_CHUNKS;
      const int sw = C::B_PIECES == 2 ? (k >> 1) & 1 : 0;
      b_src[q] = ((unsigned)k * (unsigned)p.ldb + 8u * c) * 2u;
      b_dst[q] = k * C::B_ROW_BYTES + ((c ^ (sw << 2)) << 4);
    }
  }
  // slot = chunk ^ (row / 2 mod 8) with row = 8 q + lane / 8: (4 q + lane / 16) mod 8
  auto kc_dst = [&](int q) { return 1024 * q + (q & 1 ? a_dst ^ (4 << 4) : a_dst); };

  const char* const Abase = (const char*)(p.A + (size_t)m0 * p.lda);
  const char* const Bbase = (const char*)(C::TB ? p.B + (size_t)n0 * p.ldb : p.B + n0);
  const int nkt = (p.K + 63) >> 6, skip = 64 * nkt - p.K;
  struct Regs { u32x4 a[C::NL], b[C::NL]; };
  auto load = [&](Regs& r, int t) {
    const int k0 = t == nkt - 1 ? p.K - 64 : 64 * t;
    const char* Ak = Abase + (size_t)k0 * 2;
    const char* Bk = Bbase + (C::TB ? (size_t)k0 * 2 : (size_t)k0 * p.ldb * 2);
#pragma unroll
    for (int q = 0; q < C::NL; ++q) r.a[q] = *(const u32x4_any*)(Ak + a_src[q]);
#pragma unroll
    for (int q = 0; q < C::NL; ++q) r.b[q] = *(const u32x4_any*)(Bk + b_src[q]);
  };
  // zeroes the first `skip` k of a tile in its registers
  auto zero_skipped = [&](Regs& r) {
    u32x4 keep;                                          // k-contiguous pieces: the lane's chunk is the same for every q
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int left = skip - 8 * c8 - 2 * e;            // of this dword's two values, how many go
      keep[e] = left >= 2 ? 0u : left == 1 ? 0xffff0000u : 0xffffffffu;
    }
#pragma unroll
    for (int q = 0; q < C::NL; ++q) {
      r.a[q] &= keep;
      if constexpr (C::TB) r.b[q] &= keep;
      else if ((64 * q + lane) / C::B_CHUNKS < skip) r.b[q] = u32x4{0u, 0u, 0u, 0u};
    }
  };

  f32x16 acc[C::T][C::T];
#pragma unroll
  for (int i = 0; i < C::T; ++i)
#pragma unroll
    for (int t = 0; t < C::T; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][t][e] = 0.0f;

  const int fr = lane & 31, fg = lane >> 5, fsw = (fr >> 1) & 7;
  const int tb = lane >> 4, ts = lane & 15;
  const int tk = 8 * (tb >> 1) + (ts >> 2), twithin = (16 * (tb & 1) + 4 * (ts & 3)) * 2;   // (k / 2 mod 2 of tk + 4 and tk + 16 is tk's)
  const int tsw = C::B_PIECES == 2 ? (tk >> 1) & 1 : 0;
  auto multiply = [&](Regs& r, int t) {
    if (t == nkt - 1 && skip) zero_skipped(r);
    // (a wave's LDS instructions run in order; the fences keep the compiler from reordering them across lanes)
#pragma unroll
    for (int q = 0; q < C::NL; ++q) *(u32x4*)(a_lds + kc_dst(q)) = r.a[q];
#pragma unroll
    for (int q = 0; q < C::NL; ++q) *(u32x4*)(b_lds + (C::TB ? kc_dst(q) : b_dst[q])) = r.b[q];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (t + 2 * C::NW < nkt) load(r, t + 2 * C::NW);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8 af[C::T], bf[C::T];
#pragma unroll
      for (int i = 0; i < C::T; ++i) af[i] = *(const bf16x8*)(a_lds + (32 * i + fr) * 128 + (((2 * kk + fg) ^ fsw) << 4));
#pragma unroll
      for (int i = 0; i < C::T; ++i) {
        if constexpr (C::TB) {
          bf[i] = *(const bf16x8*)(b_lds + (32 * i + fr) * 128 + (((2 * kk + fg) ^ fsw) << 4));
        } else {
          const char* bp = b_lds + (16 * kk + tk) * C::B_ROW_BYTES + ((i ^ tsw) << 6) + twithin;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp + 4 * C::B_ROW_BYTES));
          const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          bf[i] = __builtin_bit_cast(bf16x8, v);
        }
      }
#pragma unroll
      for (int i = 0; i < C::T; ++i)
#pragma unroll
        for (int j = 0; j < C::T; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[j], af[i], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };

  // This thread's bias values: all its chunks of the tile lie in the same four columns. Asked for with the first K tiles, so that the
  // epilogue waits for no memory; with B as [N][K] behind the main loop, where registers are free (before it they cost a fourth
  // wave per SIMD: 719 x 865 x 81 3.8 / 4.0 us). Asked for chunk by chunk behind the barrier / so (us): 509 x 1021 x 763 with fp32 result
  // 7.04 / 6.95, 170 x 455 x 493 4.65 / 4.37, 789 x 145 x 431 4.53 / 4.20; [N][K] 45 x 1879 x 355 4.33 / 4.12. (A third K tile in
  // flight: 4 to 11 % slower where K has four to a wave.)
  static_assert(C::THREADS % C::CPR == 0, "one column group per thread");
  uint16_t b16[4];
  auto load_bias = [&]() {
    const int n = n0 + 4 * (tid % C::CPR);
#pragma unroll
    for (int e = 0; e < 4; ++e) b16[e] = p.bias[n + e < p.N ? n + e : p.N - 1];
  };
  if constexpr (!C::TB) load_bias();
  {
    Regs r0, r1;
    if (wave < nkt) load(r0, wave);
    if (wave + C::NW < nkt) load(r1, wave + C::NW);
    for (int t = wave; t < nkt; t += 2 * C::NW) {
      multiply(r0, t);
      if (t + C::NW < nkt) multiply(r1, t + C::NW);
    }
  }

  if constexpr (C::TB) load_bias();

  // ---- partial sums to this wave's LDS: [row][4-column chunk ^ swizzle], 16 bytes each. Lane l, register e of a
  // 32 x 32 block: m = l & 31, n = 8 (e / 4) + 4 (l / 32) + e % 4
  constexpr int CPR = C::CPR;
#pragma unroll
  for (int i = 0; i < C::T; ++i) {
    const int m = 32 * i + fr;
    const int sw = C::T == 2 ? m & 15 : (m >> 1) & 7;
#pragma unroll
    for (int j = 0; j < C::T; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        *(f32x4*)(a_lds + (m * CPR + ((8 * j + 2 * q + fg) ^ sw)) * 16) = v;
      }
  }
  __syncthreads();
  const int n_end = n_own + C::TILE < p.N ? n_own + C::TILE : p.N;
  float b[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) b[e] = bf16_bits_to_f32(b16[e]);
#pragma unroll
  for (int x = tid; x < C::TILE * CPR; x += C::THREADS) {
    const int r = x / CPR, c = x % CPR;
    const int sw = C::T == 2 ? r & 15 : (r >> 1) & 7;
    f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < C::NW; ++w) z += *(const f32x4*)(smem + w * C::WAVE_BYTES + (r * CPR + (c ^ sw)) * 16);
    const int m = m0 + r, n = n0 + 4 * c;
    if (m >= p.M) continue;
    const size_t at = (size_t)m * p.ldy + n;
    const bool whole = n >= n_own && n + 4 <= n_end;
    if (p.epi == TF_EPI_NONE_F32) {
      float* y = (float*)p.Y + at;
      if (whole) {
        const f32x4 v = {z[0] + b[0], z[1] + b[1], z[2] + b[2], z[3] + b[3]};
        *(f32x4_any*)y = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e >= n_own && n + e < n_end) y[e] = z[e] + b[e];
      }
    } else {
      uint16_t* y = (uint16_t*)p.Y + at;
      u32x2 o;
      const f32x4 v = activate(f32x4{z[0] + b[0], z[1] + b[1], z[2] + b[2], z[3] + b[3]}, p.epi);
      o[0] = pack_bf16x2(v[0], v[1]);
      o[1] = pack_bf16x2(v[2], v[3]);
      if (whole) {
        *(u32x2_any*)y = o;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e >= n_own && n + e < n_end) y[e] = (uint16_t)(o[e >> 1] >> (16 * (e & 1)));
      }
    }
  }
}

template <class C>
static void launch_any(const GemmParams& p, dim3 grid, hipStream_t stream) {
  hipLaunchKernelGGL(tf_gemm_any_kernel<C>, grid, dim3(C::THREADS), C::LDS_BYTES, stream, p);
}
template <class C>
static AnyKernelInfo make_any_info() {
  AnyKernelInfo k;
  k.tile = C::TILE; k.waves = C::NW; k.trans_b = C::TB ? 1 : 0; k.threads = C::THREADS; k.lds_bytes = C::LDS_BYTES;
  k.func = (const void*)tf_gemm_any_kernel<C>;
  k.launch = launch_any<C>;
  return k;
}

// (eight waves instead of four: slower or the same except here for the larger tile with B as [N][K], 1024 x 2047 x 1023
// 18.7 against 21.1 us)
static const AnyKernelInfo g_any_table[] = {
    make_any_info<AnyCfg<1, 4, false>>(), make_any_info<AnyCfg<2, 4, false>>(),
    make_any_info<AnyCfg<1, 4, true>>(),  make_any_info<AnyCfg<2, 8, true>>(),
};
int any_kernel_count() { return (int)(sizeof(g_any_table) / sizeof(g_any_table[0])); }
const AnyKernelInfo* any_kernel_table() { return g_any_table; }

}  // namespace tf
