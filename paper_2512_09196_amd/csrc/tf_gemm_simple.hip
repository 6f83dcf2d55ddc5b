// The two unstaged members of the family.
//
//  * naive: the baseline kernel K of the variant loop. One thread per output element, a
//    scalar fp32 FMA loop over K, no MFMA, no LDS; accepts any shape, stride and alignment.
//  * mfma_direct: one wave per 32x32 output tile; MFMA operands are gathered straight from
//    memory, element by element, so it also accepts any shape. It pins the MFMA operand and accumulator
//    lane layouts with nothing else in the way, and is the quickest where K is below 64 and rows are odd.
#include <type_traits>

#include "tf_device.h"

namespace tf {

__global__ void __launch_bounds__(256) tf_gemm_naive_kernel(const GemmParams p) {
  const int n = blockIdx.x * 64 + (threadIdx.x & 63);
  const int m = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (m >= p.M || n >= p.N) return;
  const uint16_t* a = p.A + (size_t)m * p.lda;
  // B as [K][ldb] (consecutive k are ldb apart) or, trans_b, as [N][ldb] (k contiguous)
  const uint16_t* b = p.trans_b ? p.B + (size_t)n * p.ldb : p.B + n;
  const size_t bstep = p.trans_b ? 1 : (size_t)p.ldb;
  float acc = 0.0f;
  for (int k = 0; k < p.K; ++k)
    acc = __builtin_fmaf(bf16_bits_to_f32(a[k]), bf16_bits_to_f32(b[(size_t)k * bstep]), acc);
  const float z = acc + bf16_bits_to_f32(p.bias[n]);
  if (p.epi == TF_EPI_NONE_F32) ((float*)p.Y)[(size_t)m * p.ldy + n] = z;
  else ((uint16_t*)p.Y)[(size_t)m * p.ldy + n] = f32_to_bf16_bits(activate(z, p.epi));
}

__global__ void __launch_bounds__(64) tf_gemm_mfma_direct_kernel(const GemmParams p) {
  const int lane = threadIdx.x;
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  const int r = lane & 31, g = lane >> 5;
  // v_mfma_f32_32x32x16_bf16 operand layout: lane l supplies row (A) / column (B) l % 32
  // and the eight k values 8 (l / 32) .. 8 (l / 32) + 7 of the 16-wide k step.
  // Bound by trips to memory: the operands of 64 of K are all asked for before the first is used (element by element behind a
  // guard each, a step of 16 was a trip of its own, and the activations a chain of sixteen; us, so / now: 365 x 87 x 53 with fp32 result 6.2 / 4.2,
  // 36 x 253 x 59 6.9 / 4.4, 491 x 379 x 33 with GELU 6.1 / 4.6, 202 x 43 x 51 with B as [N][K] and GELU 6.5 / 5.0).
  // Rows and k outside the operands repeat their last ones; what such rows give is not stored, such k are zeroed in both operands.
  const int am = m0 + r < p.M ? m0 + r : p.M - 1, bn = n0 + r < p.N ? n0 + r : p.N - 1;
  const uint16_t* const a_row = p.A + (size_t)am * p.lda;
  const uint16_t* const b_col = p.B + (p.trans_b ? (size_t)bn * p.ldb : (size_t)bn);
  const size_t b_step = p.trans_b ? 1 : (size_t)p.ldb;
  const float bias = bf16_bits_to_f32(p.bias[bn]);
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
  for (int k0 = 0; k0 < p.K; k0 += 64) {
    uint16_t a[4][8], b[4][8];
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (k0 + 16 * s < p.K) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int ke = k0 + 16 * s + 8 * g + e, k = ke < p.K ? ke : p.K - 1;
          a[s][e] = a_row[k];
          b[s][e] = b_col[(size_t)k * b_step];
        }
      }
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (k0 + 16 * s < p.K) {
        s16x8 av, bv;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool kin = k0 + 16 * s + 8 * g + e < p.K;
          av[e] = kin ? (short)a[s][e] : (short)0;
          bv[e] = kin ? (short)b[s][e] : (short)0;
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv), acc, 0, 0, 0);
      }
  }
  // accumulator layout: register i of lane l is row 8 (i / 4) + 4 (l / 32) + i % 4, column l % 32
  const int n = n0 + r;
  if (n >= p.N) return;
  auto finish = [&](auto epi) {            // (one branch on the epilogue, so that the sixteen activations overlap)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = activate<decltype(epi)::value>(acc[i] + bias);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int m = m0 + 8 * (i >> 2) + 4 * g + (i & 3);
      if (m < p.M) {
        if (decltype(epi)::value == TF_EPI_NONE_F32) ((float*)p.Y)[(size_t)m * p.ldy + n] = acc[i];
        else ((uint16_t*)p.Y)[(size_t)m * p.ldy + n] = f32_to_bf16_bits(acc[i]);
      }
    }
  };
  switch (p.epi) {
    case TF_EPI_NONE_F32: finish(std::integral_constant<int, TF_EPI_NONE_F32>{}); break;
    case TF_EPI_BIAS_GELU_ERF: finish(std::integral_constant<int, TF_EPI_BIAS_GELU_ERF>{}); break;
    case TF_EPI_BIAS_GELU_TANH: finish(std::integral_constant<int, TF_EPI_BIAS_GELU_TANH>{}); break;
    default: finish(std::integral_constant<int, TF_EPI_BIAS>{}); break;
  }
}

// What the chip sustains, measured rather than quoted: an MFMA loop on registers only, with
// operands that look like data (bf16 values about normal, sigma 0.014: the clock the chip holds under MFMA load
// depends on what the multipliers toggle), and a streaming read of a large buffer.
// BLOCK: outputs per side of the matrix instruction, 32 (over 16 of k) or 16 (over 32), the two the tile kernels use; 4 x 4
// blocks in serpentine order (every instruction shares an operand with the one before) or, at 32, 2 x 2. TFLOP/s on two
// boards: 1845 and 1860 at 32, 2060 and 2080 at 16.
template <int BLOCK>
__global__ void __launch_bounds__(256) tf_calib_mfma_kernel(float* sink, int iters, unsigned seed) {
  constexpr int T = BLOCK == 16 ? 4 : 2;
  typedef float Acc __attribute__((ext_vector_type(BLOCK * BLOCK / 64)));
  unsigned h = (threadIdx.x + blockIdx.x * 256u + 1u) * 2654435761u ^ seed;
  auto next = [&]() { h ^= h << 13; h ^= h >> 17; h ^= h << 5; return h; };
  auto value = [&]() {             // (the sum of six uniform numbers; its upper half is the bf16)
    float v = 0.0f;
    for (int i = 0; i < 6; ++i) v += (float)(next() >> 8) * (1.0f / 16777216.0f) - 0.5f;
    return __builtin_bit_cast(unsigned, 0.02f * v);
  };
  auto operand = [&]() {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned lo = value(), hi = value();
      r[i] = (lo >> 16) | (hi & 0xffff0000u);
    }
    return __builtin_bit_cast(bf16x8, r);
  };
  bf16x8 a[T], b[T];
#pragma unroll
  for (int x = 0; x < T; ++x) {
    a[x] = operand();
    b[x] = operand();
  }
  Acc c[T][T];
#pragma unroll
  for (int x = 0; x < T; ++x)
#pragma unroll
    for (int y = 0; y < T; ++y)
#pragma unroll
      for (int i = 0; i < BLOCK * BLOCK / 64; ++i) c[x][y][i] = 0.0f;
  // (the small blocks in asm: of the builtin the compiler makes a loop with up to four register moves an instruction, 1260 to 1490
  // TFLOP/s. What it cannot see then it cannot space either: an accumulator comes round every 16 instructions, far beyond
  // what a chain of them needs, and the waits on either side of the loop cover the operands and the sums.)
  asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll 1
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int x = 0; x < T; ++x)
#pragma unroll
      for (int u = 0; u < T; ++u) {
        const int y = x & 1 ? T - 1 - u : u;
        if constexpr (BLOCK == 16) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c[x][y]) : "v"(b[y]), "v"(a[x]));
        else c[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[y], a[x], c[x][y], 0, 0, 0);
      }
  }
  asm volatile("s_nop 15\n\ts_nop 15");
  float s = 0.0f;
#pragma unroll
  for (int x = 0; x < T; ++x)
#pragma unroll
    for (int y = 0; y < T; ++y)
#pragma unroll
      for (int i = 0; i < BLOCK * BLOCK / 64; ++i) s += c[x][y][i];
  if (s == 1.2345e-30f) sink[0] = s;      // keeps the loop alive; never true
}

__global__ void __launch_bounds__(256) tf_calib_read_kernel(const u32x4* src, size_t n16, unsigned* sink) {
  // every wave reads 8 KB of its own, contiguous, as eight 16-byte non-temporal loads per lane that are all in flight
  // together, and ends: the pattern that read fastest of those tried (134 MB: 19.9 us; the same bytes as column
  // strips of 128 to 2048 bytes per row 20.4 to 33 us; a grid-stride walk with ordinary loads 25.7 us)
  const size_t wave = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const size_t base = wave * 512 + (threadIdx.x & 63);            // in 16-byte units: 8 KB per wave
  u32x4 acc = {0u, 0u, 0u, 0u};
  if (base + 7 * 64 < n16) {
    u32x4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = __builtin_nontemporal_load(src + base + j * 64);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc ^= v[j];
  } else {
    for (int j = 0; j < 8; ++j)
      if (base + j * 64 < n16) acc ^= src[base + j * 64];
  }
  if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x12345678u) sink[0] = 1u;   // never true for the buffer the host fills
}

double launch_calib_mfma(float* sink, int block, int wgs, int iters, hipStream_t s) {
  if (block == 16) hipLaunchKernelGGL(tf_calib_mfma_kernel<16>, dim3((unsigned)wgs), dim3(256), 0, s, sink, iters, 0x9e3779b9u);
  else hipLaunchKernelGGL(tf_calib_mfma_kernel<32>, dim3((unsigned)wgs), dim3(256), 0, s, sink, iters, 0x9e3779b9u);
  return (double)wgs * 4.0 * iters * (block == 16 ? 16.0 * 16384.0 : 4.0 * 32768.0);
}
void launch_calib_read(const void* src, size_t bytes, unsigned* sink, int /*wgs*/, hipStream_t s) {
  const size_t n16 = bytes / 16, waves = (n16 + 511) / 512;
  hipLaunchKernelGGL(tf_calib_read_kernel, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, (const u32x4*)src, n16, sink);
}

// Batched product with the first operand transposed in memory (C[b] = A[b]^T B[b], A[b] = [K][lda]):
// the baseline kernel, one thread per output element, scalar loop over k.
__global__ void __launch_bounds__(256) tf_bgemm_tn_naive_kernel(const GemmParams p) {
  const int n = blockIdx.x * 64 + (threadIdx.x & 63);
  const int m = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (m >= p.M || n >= p.N) return;
  const uint16_t* a = p.A + (size_t)blockIdx.z * p.stride_a + m;
  const uint16_t* b = p.B + (size_t)blockIdx.z * p.stride_b + n;
  float acc = 0.0f;
  for (int k = 0; k < p.K; ++k)
    acc = __builtin_fmaf(bf16_bits_to_f32(a[(size_t)k * p.lda]), bf16_bits_to_f32(b[(size_t)k * p.ldb]), acc);
  ((float*)p.Y)[(size_t)blockIdx.z * p.stride_y + (size_t)m * p.ldy + n] = acc;
}

// The separate-pass alternative to staging A transposed: At[b][m][k] = A[b][k][m], 64 x 64 tiles
// through LDS (padded rows), reads and writes both coalesced.
__global__ void __launch_bounds__(256) tf_transpose_kernel(const uint16_t* A, uint16_t* At, int K, int M, long lda,
                                                           long stride_a, long ldt, long stride_t) {
  __shared__ uint16_t tile[64][66];
  const uint16_t* a = A + (size_t)blockIdx.z * stride_a;
  uint16_t* t = At + (size_t)blockIdx.z * stride_t;
  const int m0 = blockIdx.x * 64, k0 = blockIdx.y * 64;
  const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
  for (int r = r0; r < 64; r += 4)
    if (k0 + r < K && m0 + c < M) tile[r][c] = a[(size_t)(k0 + r) * lda + m0 + c];
  __syncthreads();
  for (int r = r0; r < 64; r += 4)
    if (m0 + r < M && k0 + c < K) t[(size_t)(m0 + r) * ldt + k0 + c] = tile[c][r];
}

void launch_bgemm_tn_naive(const GemmParams& p, int batch, hipStream_t s) {
  dim3 grid((p.N + 63) / 64, (p.M + 3) / 4, batch);
  hipLaunchKernelGGL(tf_bgemm_tn_naive_kernel, grid, dim3(256), 0, s, p);
}
const void* bgemm_tn_naive_func() { return (const void*)tf_bgemm_tn_naive_kernel; }
void launch_transpose(const uint16_t* A, uint16_t* At, int K, int M, long lda, long stride_a, long ldt, long stride_t,
                      int batch, hipStream_t s) {
  dim3 grid((M + 63) / 64, (K + 63) / 64, batch);
  hipLaunchKernelGGL(tf_transpose_kernel, grid, dim3(256), 0, s, A, At, K, M, lda, stride_a, ldt, stride_t);
}

__global__ void tf_fill_u32_kernel(unsigned* p, size_t n, unsigned v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Second kernel of the two-kernel split-K: Y = epilogue(sum_s ws[s] + bias), slices summed in
// slice order. One thread per four consecutive n (N is a multiple of 8 for every tile kernel; the slices are tiles of one or two
// rounds of the CUs, so the quads fit 32 bits). Bound by memory: all slices of a thread's quad are asked for at once, with
// non-temporal loads, or the lines would stay in this XCD's L2 and slow down the next call's stores to them. (us a call, one 64-bit
// division per thread, a loop over the slices and ordinary loads / this, the partial tiles written with ordinary stores: 478 x 768 x 7872
// in eight slices 19.9 / 17.2 on one workspace, 17.2 / 15.7 on two in turn; 1024 x 1024 x 16384 42.9 / 41.0; 2048^3 in two 36.0 /
// 34.2. Non-temporal stores there: 15.2, 15.2, 40.0, 34.6.) The loads at once apart from their kind: one slice after another, non-temporal
// too, takes 1.11 of the time of the whole call over 58 launches in 2 to 32 slices (1.58 at the most, 100 x 512 x 16384 in sixteen 10.5 / 16.6), four
// at a time 1.01 (11.7).
template <int S, bool PAST_L2>
__global__ void __launch_bounds__(256) tf_splitk_reduce_kernel(const GemmParams p) {
  const unsigned quads_per_row = (unsigned)p.N / 4;
  const unsigned i = blockIdx.x * 256u + threadIdx.x;
  if (i >= (unsigned)p.M * quads_per_row) return;
  const unsigned m = i / quads_per_row;
  const int n = (int)(i - m * quads_per_row) * 4;
  const size_t slice = (size_t)p.M * p.N;
  const float* src = p.ws + (size_t)i * 4;
  f32x4 v[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    if constexpr (PAST_L2) v[s] = __builtin_nontemporal_load((const f32x4*)(src + (size_t)s * slice));
    else v[s] = *(const f32x4*)(src + (size_t)s * slice);
  }
  const u32x2 braw = *(const u32x2*)(p.bias + n);
  f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < S; ++s) sum += v[s];
  const float z0 = sum[0] + __builtin_bit_cast(float, braw[0] << 16);
  const float z1 = sum[1] + __builtin_bit_cast(float, braw[0] & 0xffff0000u);
  const float z2 = sum[2] + __builtin_bit_cast(float, braw[1] << 16);
  const float z3 = sum[3] + __builtin_bit_cast(float, braw[1] & 0xffff0000u);
  if (p.epi == TF_EPI_NONE_F32) {
    const f32x4 o = {z0, z1, z2, z3};
    __builtin_nontemporal_store(o, (f32x4*)((float*)p.Y + (size_t)m * p.ldy + n));
  } else {
    u32x2 o;
    const f32x4 a = activate(f32x4{z0, z1, z2, z3}, p.epi);
    o[0] = pack_bf16x2(a[0], a[1]);
    o[1] = pack_bf16x2(a[2], a[3]);
    __builtin_nontemporal_store(o, (u32x2*)((uint16_t*)p.Y + (size_t)m * p.ldy + n));
  }
}

// (an instance for each number of slices: one of another number would read past the workspace, or leave slices out)
static auto splitk_reduce_kernel(int slices, bool past_l2) -> void (*)(const GemmParams) {
  switch (slices) {
    case 2: return past_l2 ? tf_splitk_reduce_kernel<2, true> : tf_splitk_reduce_kernel<2, false>;
    case 4: return past_l2 ? tf_splitk_reduce_kernel<4, true> : tf_splitk_reduce_kernel<4, false>;
    case 8: return past_l2 ? tf_splitk_reduce_kernel<8, true> : tf_splitk_reduce_kernel<8, false>;
    case 16: return past_l2 ? tf_splitk_reduce_kernel<16, true> : tf_splitk_reduce_kernel<16, false>;
    case 32: return past_l2 ? tf_splitk_reduce_kernel<32, true> : tf_splitk_reduce_kernel<32, false>;
    default: return nullptr;
  }
}
bool splitk_reduce_takes(int slices) { return splitk_reduce_kernel(slices, true) != nullptr; }
// Partial tiles pass the L2s by (epilogue_staged has what that gives) but where much of them lies in rows off 128-byte lines: a
// line that two tiles share goes out in halves, and the memory-side cache no longer makes up for it. Time against ordinary stores
// and loads: rows of whole lines 0.89 over 29 launches up to 16 MB of slices, 0.98 over 91 above 25 (worst 1.035); others 0.90 over 119
// up to 20 MB (none loses 2 %), 1.00 over 44 above (928 x 2072 x 11776 with B as [N][K] in eight slices, 62 MB, 72.6 / 80.3 us; 838 x
// 2040 x 6320 [N][K] in four, 27 MB, 33.7 / 36.2; 804 x 2184 x 8416 [N][K] in four, 28 MB, 41.6 / 42.8), and with this line 0.99.
bool splitk_past_l2(int M, int N, int slices) { return N % 32 == 0 || 4.0 * slices * M * N <= 20e6; }
void launch_splitk_reduce(const GemmParams& p, hipStream_t s) {
  const dim3 grid((unsigned)(((size_t)p.M * (p.N / 4) + 255) / 256));
  hipLaunchKernelGGL(splitk_reduce_kernel(p.split_k, p.ws_past_l2), grid, dim3(256), 0, s, p);
}

void launch_naive(const GemmParams& p, hipStream_t s) {
  dim3 grid((p.N + 63) / 64, (p.M + 3) / 4);
  hipLaunchKernelGGL(tf_gemm_naive_kernel, grid, dim3(256), 0, s, p);
}
void launch_mfma_direct(const GemmParams& p, hipStream_t s) {
  dim3 grid((p.N + 31) / 32, (p.M + 31) / 32);
  hipLaunchKernelGGL(tf_gemm_mfma_direct_kernel, grid, dim3(64), 0, s, p);
}
const void* naive_func() { return (const void*)tf_gemm_naive_kernel; }
const void* mfma_direct_func() { return (const void*)tf_gemm_mfma_direct_kernel; }
void launch_fill_u32(unsigned* p, size_t n, unsigned v, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(tf_fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
}

// Fills the first row_bytes of every row (ld_bytes apart) with a 16-bit pattern, two bytes per thread and
// step: the rows of an output matrix without touching the padding between them, whatever its alignment.
__global__ void __launch_bounds__(256) tf_fill_rows_kernel(uint16_t* y, size_t rows, size_t row_halves, size_t ld_halves,
                                                           unsigned lo, unsigned hi) {
  const size_t total = rows * row_halves;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const size_t r = i / row_halves, c = i % row_halves;
    y[r * ld_halves + c] = (uint16_t)((c & 1) ? hi : lo);
  }
}
void launch_fill_rows(void* y, size_t rows, size_t row_bytes, size_t ld_bytes, unsigned pattern, hipStream_t s) {
  const size_t total = rows * (row_bytes / 2);
  if (total == 0) return;
  size_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  // 2-byte elements: both halves are the low half of the pattern; 4-byte elements: low then high half
  const bool four = (pattern >> 16) != (pattern & 0xffffu);
  hipLaunchKernelGGL(tf_fill_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint16_t*)y, rows, row_bytes / 2, ld_bytes / 2,
                     pattern & 0xffffu, four ? (pattern >> 16) : (pattern & 0xffffu));
}

// Placement probe: work-group i records the XCD it runs on.
__global__ void __launch_bounds__(64) tf_xcc_probe_kernel(unsigned* out) {
  if (threadIdx.x == 0) out[blockIdx.x] = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15u;   // HW_REG_XCC_ID, bits 0..3
}
void launch_xcc_probe(unsigned* out, int wgs, hipStream_t s) {
  if (wgs <= 0) return;
  hipLaunchKernelGGL(tf_xcc_probe_kernel, dim3((unsigned)wgs), dim3(64), 0, s, out);
}

// Euclidean norms of bf16 vectors (one wave per vector, lanes stride through it, lane-exchange sum).
__global__ void __launch_bounds__(256) tf_norms_kernel(const uint16_t* X, long n_outer, long outer_stride, long n_inner,
                                                       long inner_stride, long len, long elem_stride, float* out) {
  const long v = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (v >= n_outer * n_inner) return;
  const int lane = threadIdx.x & 63;
  const long o = v / n_inner, i = v % n_inner;
  const uint16_t* x = X + o * outer_stride + i * inner_stride;
  float acc = 0.0f;
  for (long e = lane; e < len; e += 64) {
    const float f = bf16_bits_to_f32(x[e * elem_stride]);
    acc = __builtin_fmaf(f, f, acc);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  // rounded up a little: the gate uses the product of two norms as an upper bound of sum |a b|
  if (lane == 0) out[v] = __builtin_sqrtf(acc) * 1.0001f;
}
void launch_norms(const uint16_t* X, long n_outer, long outer_stride, long n_inner, long inner_stride, long len,
                  long elem_stride, float* out, hipStream_t s) {
  const long n = n_outer * n_inner;
  if (n <= 0) return;
  hipLaunchKernelGGL(tf_norms_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, X, n_outer, outer_stride, n_inner,
                     inner_stride, len, elem_stride, out);
}

}  // namespace tf
