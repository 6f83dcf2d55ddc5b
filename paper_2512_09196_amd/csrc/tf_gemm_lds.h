// LDS-staged bf16 MFMA GEMM with fused bias + GELU(erf) epilogue for gfx950.
//
// One work-group computes one BM x BN tile of Y (or one K slice of it). Per K step of
// BK (32, 64 or 128) it stages an A tile [BM][BK] and a B tile [BK][BN] in LDS, multi-buffered,
// and each of the WM x WN waves accumulates a (BM/WM) x (BN/WN) sub-tile in fp32 with
// v_mfma_f32_16x16x32_bf16 or v_mfma_f32_32x32x16_bf16 (see LdsCfg::MB).
//
// LDS layouts (chosen from measured bank behaviour: 64 banks x 4 B, b128 reads are
// conflict free when 16 consecutive lanes cover 16 distinct 16-byte slots of a 256-byte line):
//   A tile: row-major, 2 BK bytes per row, BK / 8 16-byte chunks per row; chunk c of row r is
//           stored in slot c ^ f(r), f(r) = (r / rows per 256-byte line) mod chunks per row
//           (BK = 64: c ^ ((r >> 1) & 7)). MFMA A operands are ds_read_b128.
//   B tile: row-major as in memory ([k][n], n contiguous), BN*2 bytes per row, split in
//           64-byte pieces; piece j of row k is stored in slot j ^ f(k) so that four
//           consecutive k rows fall in four different bank groups (blocks of 16 x 16 also swap the halves of a
//           piece by bit 3 of k, see b_chunk_swz). MFMA B operands, which
//           need 8 consecutive k per lane, are read with the transposing
//           ds_read_b64_tr_b16 (two per operand), so B is never transposed by ALU code.
// Both tiles are written either by global_load_lds_dwordx4 (memory -> LDS without passing
// through registers; the lane -> slot map is fixed by hardware, the swizzle is applied to
// the global address instead) or by 16-byte global loads into registers followed by
// ds_write_b128, which allows zero fill of a ragged K tail.
#pragma once
#include "tf_device.h"

namespace tf {

template <int BM_, int BN_, int BK_, int WM_, int WN_, int STAGES_, bool DIRECT_, bool ABYPASS_ = false, int WK_ = 1, bool TRANSA_ = false,
          bool TRANSB_ = false, int BN_ACT_ = BN_>
struct LdsCfg {
  // BN_ACT < BN: a narrower tile that shares everything else with the BN-wide one. The B tile is staged BN wide as
  // always (same ring, same transfers), but only the first BN_ACT columns are multiplied and written out: the
  // tiles of a last, deliberately lighter round of a launch (see tf_gemm_mixed_kernel).
  static constexpr int BN_ACT = BN_ACT_;
  static_assert(BN_ACT_ <= BN_ && BN_ACT_ % (32 * WN_) == 0, "active width: whole 32-column blocks per wave column");
  // TRANSA: A is given transposed, [K][lda] with m contiguous (the dO^T A product of the paper's
  // Case Study 3). Its tile is then staged exactly like the B tile, [64][BM] row-major with the
  // same 64-byte piece swizzle, and its MFMA operands come from the transposing LDS read too:
  // the loads from memory stay fully coalesced and nothing is transposed by ALU code or by a
  // separate pass.
  static constexpr bool TRANSA = TRANSA_;
  static constexpr int A_ROW_BYTES = BM_ * 2, A_PIECES = A_ROW_BYTES / 64, A_ROWS_PER_INSTR = 1024 / A_ROW_BYTES;
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, STAGES = STAGES_;
  static_assert(BK == 32 || BK == 64 || BK == 128, "K tile of 32, 64 or 128");
  // TRANSB: B is given as [N][ldb] with k contiguous (weights stored output-major). Its tile is then staged
  // exactly like the A tile, [BN][BK] with the same chunk swizzle, and its MFMA operands are ds_read_b128.
  static constexpr bool TRANSB = TRANSB_;
  // A tile rows (and B tile rows under TRANSB): BK / 8 chunks of 16 bytes; slot = chunk ^ row_swz(row)
  static constexpr int K_ROW_BYTES = BK * 2, K_CHUNKS = BK / 8, K_ROWS_PER_LINE = 16 / K_CHUNKS, K_ROWS_PER_INSTR = 64 / K_CHUNKS;
  // The matrix instruction: blocks of MB x MB outputs over KMF of k, 32 x 32 over 16 or 16 x 16 over 32. Both take the
  // same cycles per flop and the same fragment bytes per wave, but the second reads and writes half as many accumulators
  // per flop, and under load this board's clock is what its power limit leaves: register-only loops on operands
  // about normal sustain 1810 to 1860 TFLOP/s with the first and 2020 to 2040 with the second, 2050 to 2080 in the serpentine order
  // below (on zeros both 2400 to 2490). It is used where the matrix pipes set the pace, in the eight-wave tiles with wave tiles of 64
  // rows and more; smaller ones wait for operands and keep the first, which needs half as many instructions, and so do
  // tiles of four waves, one to a SIMD, where nothing fills the pipe while its wave issues or waits (with the second, over 28 to 92
  // problems, 128 x 256 tiles took 12 % longer, 256 x 128 7 %, 128 x 128 13 % with three buffers and 2 % with two).
  static constexpr int MB = DIRECT_ && !ABYPASS_ && !TRANSA_ && WK_ == 1 && BK_ >= 64 && WM_ * WN_ >= 8 && BM_ / WM_ >= 64 ? 16 : 32;
  static constexpr int KMF = MB == 16 ? 32 : 16;
  static constexpr int QN = MB / 16 * (MB / 16);           // runs of four accumulators a lane holds of a block
  static constexpr int KSTEPS = BK / KMF;                  // MFMA steps per K tile
  // WK: wave groups along k. With WK = 2 a second set of WM x WN waves works on the same
  // BM x BN tile but takes the other half of every 64-wide K step; the two sets add their
  // accumulators through LDS after the main loop. Eight waves then keep the LDS busier than
  // four can (a wave issues one LDS instruction every twenty-odd cycles) without the extra
  // fragment reads that a finer split of the tile along m or n costs.
  static constexpr int WK = WK_, KS = KSTEPS / WK_;        // MFMA steps per wave per K step
  static_assert(KS >= 2 && KS % 2 == 0, "the pipeline alternates two fragment sets per MFMA step");
  // ORDERED: a step's blocks in serpentine order, its MFMAs pinned to it (see the main loops). Not where a wave has two MFMA
  // steps of 32 x 32 blocks in a K tile: there the compiler's own order is the faster (128 x 128 tiles with two k groups 2.3 %
  // over 95 problems, 256 x 256 tiles with a K tile of 32 1.6 % over 16).
  static constexpr bool ORDERED = MB == 16 || KS > 2;
  static constexpr bool DIRECT = DIRECT_;
  // ABYPASS: the A operand never enters LDS. Each wave loads its own A fragments from memory
  // straight into registers (WN must be 1, so no two waves need the same A rows) and only B is
  // staged. This halves the LDS write traffic, which is what bounds the two-operand scheme.
  static constexpr bool ABYPASS = ABYPASS_;
  static constexpr int NWAVES = WM * WN * WK, THREADS = NWAVES * 64;
  static constexpr int WTM = BM / WM, WTN = BN_ACT / WN;   // wave tile
  static constexpr int TM = WTM / MB, TN = WTN / MB;       // MFMA blocks per wave
  static constexpr int ACC = TM * TN * MB * MB / 64;       // accumulator registers per lane
  typedef float Acc __attribute__((ext_vector_type(MB * MB / 64)));
  // QUAD: the two-buffer eight-wave tiles of 256 columns are staged and multiplied in quadrants. A tile is made of four
  // units, the first 128 rows of A, its other rows, and the two halves of B's columns, and every wave owns a piece of all
  // four quadrants (see the main loop: a unit's buffer is free for the tile after next as soon as it has been read).
  static constexpr bool QUAD = MB == 16 && BK == 64 && STAGES == 2 && WM * WN == 8 && BN == 256 && BM >= 192;
  static constexpr int TM0 = QUAD ? 128 / (16 * WM) : TM, TN0 = QUAD ? TN / 2 : TN;     // blocks per wave in the first A and B unit
  static constexpr int B_UNITS = QUAD ? 2 : 1, B_UNIT_COLS = BN / B_UNITS;
  // first row and column (inside the tile) of a wave's block i, t
  __device__ __forceinline__ static constexpr int row_off(int i, int wave_m) {
    return i < TM0 ? wave_m * TM0 * MB + MB * i : WM * TM0 * MB + wave_m * (TM - TM0) * MB + MB * (i - TM0);
  }
  __device__ __forceinline__ static constexpr int col_off(int t, int wave_n) {
    return t < TN0 ? wave_n * TN0 * MB + MB * t : WN * TN0 * MB + wave_n * (TN - TN0) * MB + MB * (t - TN0);
  }
  static constexpr int A_BYTES = ABYPASS ? 0 : BM * BK * 2, B_BYTES = BK * BN * 2;
  static_assert(!ABYPASS || (WN == 1 && DIRECT && STAGES == 2 && WK_ == 1 && BK == 64 && !TRANSB_), "A bypass: one wave column, direct B staging, two buffers, K tile of 64");
  static_assert(DIRECT || BK == 64, "register staging: K tile of 64");
  static_assert(!TRANSB_ || !TRANSA_, "one transposed operand at a time");
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int RING_BYTES = STAGES * STAGE_BYTES;
  // behind the ring: this tile's BN bias values, fetched at kernel start so that the epilogue
  // does not begin with a trip to memory
  static constexpr int BIAS_OFF = RING_BYTES, BIAS_BYTES = 512;
  static constexpr int LDS_BYTES = RING_BYTES + BIAS_BYTES;
  static constexpr int A_INSTR = A_BYTES / 1024;           // wave-wide 1 KB transfers per tile
  static constexpr int B_INSTR = B_BYTES / 1024;
  static constexpr int A_PER_WAVE = A_INSTR / NWAVES, B_PER_WAVE = B_INSTR / NWAVES;
  static constexpr int B_ROW_BYTES = TRANSB ? K_ROW_BYTES : B_UNIT_COLS * 2;
  static constexpr int B_ROWS_PER_INSTR = 1024 / B_ROW_BYTES;
  static constexpr int B_SLOTS_PER_ROW = B_ROW_BYTES / 16;  // 16-byte slots per B row
  static constexpr int B_PIECES = B_ROW_BYTES / 64;         // 64-byte pieces per B row
  static constexpr int B_UNIT_BYTES = B_BYTES / B_UNITS;
  // Ring layout: K tile by K tile, A before B; quadrant tiles all A tiles before all B tiles, so that the 16-bit offset of
  // an LDS read reaches every buffer from one address register.
  static constexpr int A_STRIDE = QUAD ? A_BYTES : STAGE_BYTES, B_STRIDE = QUAD ? B_BYTES : STAGE_BYTES;
  static constexpr int B_BASE = QUAD ? STAGES * A_BYTES : A_BYTES;
  static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be made of 32x32 blocks");
  static_assert(A_INSTR % NWAVES == 0 && B_INSTR % NWAVES == 0, "tile loads must divide over the waves");
  static_assert(BN == 32 || BN == 64 || BN == 128 || BN == 256, "B row must be 64, 128, 256 or 512 bytes");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget of one CU");
  static_assert(WK == 1 || (WK == 2 && TM % 2 == 0 && DIRECT && !ABYPASS), "k groups: two, each keeps half of the row blocks");
  static_assert(WK == 1 || WM * WN > 1, "one wave per k group and several groups: how a descriptor names the kernels of tf_gemm_kshare.hip");
  static_assert(!TRANSA || (DIRECT && !ABYPASS && (BM == 32 || BM == 64 || BM == 128 || BM == 256)), "transposed A: direct staging, A row of 64 to 512 bytes");
  static_assert(WK == 1 || RING_BYTES >= NWAVES * ACC * 128, "the accumulator exchange reuses the tile buffers");
  static constexpr int TM_OUT = TM / WK;                   // row blocks a wave writes out
  // The in-kernel split-K reduction is only compiled for wave tiles of at most 64 accumulator
  // registers: behind bigger ones its code makes the compiler spill, and the scratch memory
  // that reserves per wave slows every launch of the kernel, split or not.
  static constexpr bool FUSED_OK = ACC <= 64;
  static constexpr bool SEGMENTS = false;                  // see StreamKCfg
  static constexpr bool KTAIL = false;                     // see RaggedKCfg
  static constexpr bool LINES = false;                     // see RaggedKCfg
  // Output staging (see epilogue_staged): each pass moves 32 rows per wave row (and k group) through the tile
  // ring, rows padded by 16 bytes; used for an output type when one pass fits into the ring.
  static constexpr int ST_ROWS = 32 * WM * WK_;
  // (not behind wave tiles of 256 accumulator registers: the extra code makes the compiler spill there)
  // the persistent kernel's fp32 staging area lies behind the ring
  static constexpr int PERSIST_LDS_BYTES = RING_BYTES + ST_ROWS * (BN * 4 + 16);
  static constexpr bool stage_ok(int esz) { return ACC <= 128 && ST_ROWS * (BN_ACT * esz + 16) <= RING_BYTES; }
  // 32-row tiles serve problems of few rows, where every B element is read by one work-group only: its
  // loads are marked non-temporal
  static constexpr bool B_NT = BM <= 32;
  // slot permutation of the 16-byte chunks of a k-contiguous tile row (see the file header)
  __device__ __forceinline__ static constexpr int row_swz(int r) { return (r / K_ROWS_PER_LINE) & (K_CHUNKS - 1); }
};

// Slot permutation of the 64-byte pieces of B row k (see header).
template <int PIECES>
__device__ __forceinline__ int b_swz(int k) {
  if (PIECES >= 4) return k & 3;
  if (PIECES == 2) return (k >> 1) & 1;
  return 0;
}
// The same in 16-byte chunks, as TileLoader and the transposing reads of 32-column (MB 32) or 16-column (MB 16) blocks
// use it. A transposing read of 16 columns takes 32 bytes of the rows 8 g .. 8 g + 3 in lane group g: the half of the
// 64-byte piece is permuted by bit 3 of k too, so that groups g and g + 1 fall in different banks.
template <class C>
__device__ __forceinline__ int b_chunk_swz(int k) {
  return (b_swz<C::B_PIECES>(k) << 2) | (C::MB == 16 ? ((k >> 3) & 1) << 1 : 0);
}

// An operand whose rows are contiguous along k, staged in whole 128-byte lines. Rows of a length that is no multiple of 128
// bytes start anywhere in a line, and the 128 bytes a K tile takes of each of them are two requests to the L2, not one. Here
// buffer w takes line w of every row, counted from the one its first k lies in: chunk j of 16 bytes of K tile t lies in buffer
// t + (j + shift) / 8, in the slot it would have in a tile's own buffer (with slots in the order of the line the reads conflict:
// 1160 x 3080 x 1864 24.7 us instead of 23.0; the staging of tiles took 24.3). Rows a multiple of eight apart have the same
// shift (a row is whole chunks), so a lane has one for all its blocks, and one for all its transfers. Where the ragged last K
// tile comes first, chunks in front of the range are its (a line shared by the two holds both).
struct LineRows {
  int shift;                     // of this lane's rows as it reads them
  int cs;                        // slot minus shift in its transfers
  int k0, begin, chunks;         // chunk that slot 0 of buffer 0 stands for where the shift is 0; first chunk of the range; chunks in a row
  bool wrap;                     // the ragged K tile comes first
  __device__ __forceinline__ static int shift_of(const uint16_t* base, long ld, int row) {
    return (int)(((unsigned long long)base >> 4) + (unsigned long long)row * (unsigned long long)(ld >> 3)) & 7;
  }
  // chunk to fetch for buffer w, inside the row whatever w is (what no K tile holds is not read)
  __device__ __forceinline__ int chunk(int w) const {
    int c = k0 + 8 * w + cs;
    if (wrap && c < begin) c += chunks - begin;
    return c < 0 ? 0 : c >= chunks ? chunks - 1 : c;
  }
};

template <class C>
struct TileLoader {
  // Per-lane, per-transfer source offsets (in elements, relative to the tile's first k) and
  // validity. Computed once; the K step only moves the base pointers.
  // (byte offsets from the tile's first k; 32 bits: the host rejects tensors of 4 GiB or more)
  static constexpr int NA = C::A_PER_WAVE > 0 ? C::A_PER_WAVE : 1;   // (no zero-length arrays)
  unsigned a_src[NA];
  unsigned b_src[C::B_PER_WAVE];
  int a_k[NA];                   // k offset (elements) of the lane's chunk inside the tile
  int b_k[C::B_PER_WAVE];        // k row of the lane inside the tile
  bool b_ok[C::B_PER_WAVE];      // column chunk inside N
  bool a_ok[NA];                 // row inside M
  // Quadrant tiles have no registers to spare for an offset per transfer. The transfers of a wave are 64 rows (of a
  // k-contiguous operand) or 32 k (of a [K][N] one) apart, and a lane's chunk is the same in all of them and in both
  // operands: the offsets of its first rows and of the chunk are enough, the rest is scalar.
  unsigned a_first, b_first, chunk;
  unsigned a_row, b_row, a_last, b_last;     // bytes from one row to the next, to the last row (scalar)

  __device__ __forceinline__ void init(const GemmParams& p, int m0, int n0, int wave, int lane) {
    if constexpr (C::QUAD) {
      a_row = (unsigned)p.lda * 2u;
      b_row = (unsigned)p.ldb * 2u;
      a_last = (unsigned)(p.M - 1) * a_row;
      b_last = (unsigned)(p.N - 1) * b_row;
      const int row = C::K_ROWS_PER_INSTR * wave + lane / C::K_CHUNKS;
      chunk = 16u * ((lane % C::K_CHUNKS) ^ C::row_swz(row));
      a_first = (unsigned)(m0 + row < p.M ? m0 + row : p.M - 1) * a_row;
      b_first = (unsigned)(n0 + row < p.N ? n0 + row : p.N - 1) * b_row;
    }
#pragma unroll
    for (int q = 0; q < C::A_PER_WAVE; ++q) {
      const int ia = wave + C::NWAVES * q;
      if constexpr (C::TRANSA) {
        // rows of the tile are k, columns m: the scheme of the B tile with m in place of n
        constexpr int LPR = 64 / C::A_ROWS_PER_INSTR;
        const int krow = C::A_ROWS_PER_INSTR * ia + lane / LPR;
        const int s16 = lane % LPR;
        const int piece = (s16 >> 2) ^ b_swz<C::A_PIECES>(krow);
        int m = m0 + 32 * piece + 8 * (s16 & 3);
        a_ok[q] = m < p.M;
        if (m >= p.M) m = 0;
        a_src[q] = ((unsigned)krow * (unsigned)p.lda + (unsigned)m) * 2u;
        a_k[q] = krow;
      } else {
        const int row = C::K_ROWS_PER_INSTR * ia + lane / C::K_CHUNKS;
        const int slot = lane % C::K_CHUNKS;
        const int c = slot ^ C::row_swz(row);
        int m = m0 + row;
        a_ok[q] = m < p.M;
        if (m >= p.M) m = p.M - 1;
        a_src[q] = ((unsigned)m * (unsigned)p.lda + 8u * c) * 2u;
        a_k[q] = 8 * c;
      }
    }
#pragma unroll
    for (int q = 0; q < C::B_PER_WAVE; ++q) {
      const int ib = wave + C::NWAVES * q;
      if constexpr (C::TRANSB) {
        // rows of the tile are n, columns k: the scheme of the A tile with n in place of m
        const int row = C::K_ROWS_PER_INSTR * ib + lane / C::K_CHUNKS;
        const int slot = lane % C::K_CHUNKS;
        const int c = slot ^ C::row_swz(row);
        int n = n0 + row / C::B_UNIT_COLS * (C::BN_ACT / C::B_UNITS) + row % C::B_UNIT_COLS;
        b_ok[q] = n < p.N;
        if (n >= p.N) n = p.N - 1;
        b_src[q] = ((unsigned)n * (unsigned)p.ldb + 8u * c) * 2u;
        b_k[q] = 8 * c;
      } else {
        constexpr int LPR = 64 / C::B_ROWS_PER_INSTR;          // lanes per row
        const int unit = C::B_ROWS_PER_INSTR * ib / C::BK;
        const int krow = C::B_ROWS_PER_INSTR * ib % C::BK + lane / LPR;
        int n = n0 + unit * (C::BN_ACT / C::B_UNITS) + 8 * ((lane % LPR) ^ b_chunk_swz<C>(krow));
        b_ok[q] = n < p.N;
        if (n >= p.N) n = 0;
        b_src[q] = ((unsigned)krow * (unsigned)p.ldb + (unsigned)n) * 2u;
        b_k[q] = krow;
      }
    }
  }

  // memory -> LDS without registers. Requires every k of the tile to be < K.
  // Written as inline assembly: M0 carries the wave-uniform LDS destination, each lane lands
  // at M0 + 16 * lane, the source is an SGPR base plus this lane's 32-bit byte offset. The
  // transfers are counted by vmcnt; the kernel waits for them explicitly before the barrier
  // that publishes a tile, so the compiler needs no knowledge of them (given the builtin, it
  // would make every later LDS read wait for all transfers in flight, including the tiles
  // prefetched for later steps). Nothing else in these kernels uses M0.
  template <bool NT = false>
  __device__ __forceinline__ static void gload_lds16(unsigned lds_addr, unsigned voff, const void* base) {
    // the base is the same for every lane; say so, or it may be handed over in vector registers
    const unsigned long long b = (unsigned long long)base;
    // (the builtin returns a signed int: go through unsigned, or the low half sign-extends)
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    const unsigned long long sb = (unsigned long long)lo | ((unsigned long long)hi << 32);
    const void* sbase = (const void*)sb;
    if constexpr (NT)      // non-temporal: data that no other work-group reads again need not stay in the caches
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                   :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
    else
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
  }
  // same, four bytes per lane (lane l lands at M0 + 4 l; lanes switched off transfer nothing)
  __device__ __forceinline__ static void gload_lds4(unsigned lds_addr, unsigned voff, const void* base) {
    const unsigned long long b = (unsigned long long)base;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    const unsigned long long sb = (unsigned long long)lo | ((unsigned long long)hi << 32);
    const void* sbase = (const void*)sb;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
  }
  __device__ __forceinline__ void issue_direct(const uint16_t* Ak, const uint16_t* Bk, unsigned stage_lds, int wave) const {
#pragma unroll
    for (int q = 0; q < C::A_PER_WAVE; ++q) {
      const int ia = wave + C::NWAVES * q;
      gload_lds16(__builtin_amdgcn_readfirstlane(stage_lds + ia * 1024), a_src[q], Ak);
    }
#pragma unroll
    for (int q = 0; q < C::B_PER_WAVE; ++q) {
      const int ib = wave + C::NWAVES * q;
      gload_lds16<C::B_NT>(__builtin_amdgcn_readfirstlane(stage_lds + C::A_BYTES + ib * 1024), b_src[q], Bk);
    }
  }

  // LINES: buffer w of an operand. EDGE: any w; otherwise one whose lines lie inside the range of every row (offsets that
  // begin 7 chunks ahead, so that none is negative)
  template <bool EDGE, bool NT, int PER_WAVE>
  __device__ __forceinline__ static void issue_lines(const LineRows& r, const unsigned (&src)[PER_WAVE], const uint16_t* base, int w,
                                                     unsigned lds, int wave) {
    const int c = EDGE ? r.chunk(w) - (r.cs + 7) : 0;
    const char* from = (const char*)base + (EDGE ? 0l : 16l * (r.k0 + 8 * w - 7));
#pragma unroll
    for (int q = 0; q < PER_WAVE; ++q)
      gload_lds16<NT>(__builtin_amdgcn_readfirstlane(lds + (wave + C::NWAVES * q) * 1024), src[q] + 16u * (unsigned)c, from);
  }

  // min(first + further, last) + chunk, in three instructions where it is needed (the compiler would compute every offset
  // ahead of the main loop and keep them all)
  __device__ __forceinline__ unsigned row_chunk(unsigned first, unsigned further, unsigned last) const {
    unsigned off;
    asm volatile("v_add_u32 %0, %2, %1\n\tv_min_u32 %0, %3, %0\n\tv_add_u32 %0, %4, %0"
                 : "=&v"(off) : "v"(first), "s"(further), "s"(last), "v"(chunk));
    return off;
  }
  __device__ __forceinline__ void issue_a_one(int q, const uint16_t* Ak, unsigned stage_lds, int wave) const {
    const int ia = wave + C::NWAVES * q;
    unsigned off = a_src[q < NA ? q : 0];
    if constexpr (C::QUAD) {
      off = row_chunk(a_first, (unsigned)q * (64u * a_row), a_last);
    }
    gload_lds16(__builtin_amdgcn_readfirstlane(stage_lds + ia * 1024), off, Ak);
  }
  __device__ __forceinline__ void issue_b_one(int q, const uint16_t* Bk, unsigned stage_lds, int wave) const {
    const int ib = wave + C::NWAVES * q;
    unsigned off = b_src[q];
    if constexpr (C::QUAD) {
      constexpr int PER_UNIT = C::B_PER_WAVE / C::B_UNITS;
      const int unit = q / PER_UNIT, x = q % PER_UNIT;
      if constexpr (C::TRANSB) {
        off = row_chunk(b_first, (unsigned)(unit * (C::BN_ACT / C::B_UNITS) + 64 * x) * b_row, b_last);
      } else {
        off = b_src[unit * PER_UNIT];
        Bk = (const uint16_t*)((const char*)Bk + (size_t)(32 * x) * b_row);
      }
    }
    gload_lds16<C::B_NT>(__builtin_amdgcn_readfirstlane(stage_lds + C::A_BYTES + ib * 1024), off, Bk);
  }
  __device__ __forceinline__ void issue_a_all(const uint16_t* Ak, unsigned stage_lds, int wave) const {
#pragma unroll
    for (int q = 0; q < C::A_PER_WAVE; ++q) issue_a_one(q, Ak, stage_lds, wave);
  }
  __device__ __forceinline__ void issue_b_direct(const uint16_t* Bk, unsigned stage_lds, int wave) const {
#pragma unroll
    for (int q = 0; q < C::B_PER_WAVE; ++q) {
      const int ib = wave + C::NWAVES * q;
      gload_lds16<C::B_NT>(__builtin_amdgcn_readfirstlane(stage_lds + C::A_BYTES + ib * 1024), b_src[q], Bk);
    }
  }

  // memory -> registers, zero where k >= K (ragged tail) or outside M / N.
  __device__ __forceinline__ void load_regs(const uint16_t* Ak, const uint16_t* Bk, int k0, int K,
                                            u32x4 (&ra)[NA], u32x4 (&rb)[C::B_PER_WAVE]) const {
#pragma unroll
    for (int q = 0; q < C::A_PER_WAVE; ++q) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (a_ok[q] && k0 + a_k[q] < K) v = *(const u32x4*)((const char*)Ak + a_src[q]);
      ra[q] = v;
    }
#pragma unroll
    for (int q = 0; q < C::B_PER_WAVE; ++q) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (b_ok[q] && k0 + b_k[q] < K) v = *(const u32x4*)((const char*)Bk + b_src[q]);
      rb[q] = v;
    }
  }
  __device__ __forceinline__ void store_regs(char* stage, int wave, int lane,
                                             const u32x4 (&ra)[NA], const u32x4 (&rb)[C::B_PER_WAVE]) const {
#pragma unroll
    for (int q = 0; q < C::A_PER_WAVE; ++q) {
      const int ia = wave + C::NWAVES * q;
      *(u32x4*)(stage + ia * 1024 + lane * 16) = ra[q];
    }
#pragma unroll
    for (int q = 0; q < C::B_PER_WAVE; ++q) {
      const int ib = wave + C::NWAVES * q;
      *(u32x4*)(stage + C::A_BYTES + ib * 1024 + lane * 16) = rb[q];
    }
  }
};

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding:
// vmcnt = bits [3:0] and [15:14], expcnt [6:4] and lgkmcnt [11:8] left at "no wait").
// Work-group barrier for the direct-to-LDS pipeline: this wave's LDS reads have returned
// (lgkmcnt 0), then s_barrier. Unlike __syncthreads() it does not wait for vector-memory
// operations, so tiles prefetched for later steps stay in flight across it; the caller waits
// for the tile it is about to publish with wait_vmcnt<> first. The asm memory clobber keeps
// the compiler from moving LDS accesses across it.
__device__ __forceinline__ void barrier_lds() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Four fp32 stored with device ("agent") scope: written through the L2 of this XCD, so a
// work-group on another XCD (another L2) reads the new value from memory. Split-K uses it for
// the partial sums instead of a device-wide fence, which would write back and invalidate the
// whole L2 twice per work-group.
// (One 16-byte store with the device-scope bit, as the compiler emits for a relaxed device-scope atomic store
// of one dword; the atomic builtins themselves stop at 8 bytes. ptr is 16-byte aligned.)
__device__ __forceinline__ void store_through_f32x4(float* ptr, const f32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1" :: "v"(ptr), "v"(v) : "memory");
}
// The matching load: 16 bytes past this XCD's L2. Only issues it; the data is there after wait_through().
__device__ __forceinline__ void load_through_f32x4(f32x4& dst, const float* ptr) {
  asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=&v"(dst) : "v"(ptr) : "memory");
}
// Waits for every load above; the values pass through it, so that no use of them can be moved ahead of the wait.
__device__ __forceinline__ void wait_through(f32x4& a, f32x4& b, f32x4& c, f32x4& d) {
  asm volatile("s_waitcnt vmcnt(0)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) :: "memory");
}

// Split-K: one slice's partial tile -> workspace (fp32, [slice][M][N]).
template <class C, bool FULL, bool THROUGH>
__device__ __forceinline__ void store_partial(const typename C::Acc (&acc)[C::TM][C::TN], float* wsk, const GemmParams& p,
                                              int wm0, int wn0, int wave_m, int wave_n) {
#pragma unroll
  for (int i = 0; i < C::TM_OUT; ++i) {
    const int m = wm0 + C::row_off(i, wave_m);
#pragma unroll
    for (int t = 0; t < C::TN; ++t)
#pragma unroll
      for (int q = 0; q < C::QN; ++q) {
        const int n = wn0 + C::col_off(t, wave_n) + 8 * q;
        if (FULL || (m < p.M && n < p.N)) {
          const f32x4 v = {acc[i][t][4 * q], acc[i][t][4 * q + 1], acc[i][t][4 * q + 2], acc[i][t][4 * q + 3]};
          if (THROUGH) store_through_f32x4(wsk + (size_t)m * p.N + n, v);
          else *(f32x4*)(wsk + (size_t)m * p.N + n) = v;
        }
      }
  }
}

// Split-K: sum of all slices, always in slice order 0, 1, ... so the result does not depend on
// which slice arrived last.
// THROUGH: device-scope loads (the slices may have been written through other XCDs' L2s);
// otherwise plain 16-byte loads, for slices known to sit in this XCD's L2.
template <class C, bool FULL, bool THROUGH>
__device__ __forceinline__ void sum_partials(typename C::Acc (&acc)[C::TM][C::TN], const GemmParams& p, int wm0, int wn0, int wave_m,
                                             int wave_n) {
  const size_t slice = (size_t)p.M * p.N;
  // 16-byte loads (device scope, or plain ones for slices that sit in this XCD's L2), whole slices in flight at a
  // time: a loop over the slices per element is one long chain of dependent trips to memory, and everything behind
  // the K loop of a memory-bound problem is time in which nothing is streamed. The accumulator registers are free
  // by now: their contents have been published. Pieces outside M or N (ragged tiles) count as zero.
  constexpr int NV = C::TM_OUT * C::TN * C::QN;
  static_assert(NV % 4 == 0 && NV <= 16, "register budget of the exchange");
  f32x4 sum[NV];
  bool ok[NV];
#pragma unroll
  for (int x = 0; x < NV; ++x) {
    const int i = x / (C::TN * C::QN), t = (x / C::QN) % C::TN, q = x % C::QN;
    sum[x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    ok[x] = FULL || (wm0 + C::row_off(i, wave_m) < p.M && wn0 + C::col_off(t, wave_n) + 8 * q < p.N);
  }
  // G slices are loaded together (as many as sixteen 16-byte vectors per lane allow: small tiles with two or four
  // slices make one trip to memory in all), then added in slice order
  constexpr int G = NV <= 4 ? 4 : (NV <= 8 ? 2 : 1);
  for (int s0 = 0; s0 < p.split_k; s0 += G) {
    f32x4 v[G][NV];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      // (a slice past the last one reads the last one again and is not added)
      const int sidx = s0 + g < p.split_k ? s0 + g : p.split_k - 1;
      const float* base = p.ws + (size_t)sidx * slice;
#pragma unroll
      for (int x = 0; x < NV; ++x) {
        const int i = x / (C::TN * C::QN), t = (x / C::QN) % C::TN, q = x % C::QN;
        // (a piece outside the matrix reads the slice's first 16 bytes instead: no branch round the load, whose
        // result only counts after the wait below)
        const float* src = ok[x] ? base + (size_t)(wm0 + C::row_off(i, wave_m)) * p.N + (wn0 + C::col_off(t, wave_n) + 8 * q) : base;
        if constexpr (THROUGH) load_through_f32x4(v[g][x], src);
        else v[g][x] = *(const f32x4*)src;
      }
    }
    if constexpr (THROUGH) {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int x = 0; x < NV; x += 4) wait_through(v[g][x], v[g][x + 1], v[g][x + 2], v[g][x + 3]);
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int x = 0; x < NV; ++x)
        if (ok[x] && s0 + g < p.split_k) sum[x] += v[g][x];
  }
#pragma unroll
  for (int x = 0; x < NV; ++x) {
    const int i = x / (C::TN * C::QN), t = (x / C::QN) % C::TN, q = x % C::QN;
    acc[i][t][4 * q] = sum[x][0]; acc[i][t][4 * q + 1] = sum[x][1];
    acc[i][t][4 * q + 2] = sum[x][2]; acc[i][t][4 * q + 3] = sum[x][3];
  }
}

template <int E> struct EpiTag { static constexpr int value = E; };
// f(EpiTag<0>{}), ..., f(EpiTag<N - 1>{})
template <int N, class F>
__device__ __forceinline__ void static_for(const F& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(EpiTag<N - 1>{});
  }
}

// wm0, wn0: first row and column of this lane, without the wave's part; bias_lds: the tile's bias from column wn0 on
template <class C, bool FULL, int EPI>
__device__ __forceinline__ void epilogue(const typename C::Acc (&acc)[C::TM][C::TN], const GemmParams& p, int wm0, int wn0, int wave_m,
                                         int wave_n, const char* bias_lds, int n_end) {
#pragma unroll
  for (int t = 0; t < C::TN; ++t) {
#pragma unroll
    for (int q = 0; q < C::QN; ++q) {
      const int col = C::col_off(t, wave_n) + 8 * q, n = wn0 + col;
      const bool n_ok = FULL || n < n_end;
      const u32x2 braw = *(const u32x2*)(bias_lds + col * 2);   // (columns past N hold values nobody stores)
      const float b0 = __builtin_bit_cast(float, braw[0] << 16), b1 = __builtin_bit_cast(float, braw[0] & 0xffff0000u);
      const float b2 = __builtin_bit_cast(float, braw[1] << 16), b3 = __builtin_bit_cast(float, braw[1] & 0xffff0000u);
#pragma unroll
      for (int i = 0; i < C::TM_OUT; ++i) {
        const int m = wm0 + C::row_off(i, wave_m);
        if (FULL || (n_ok && m < p.M)) {
          const float z0 = acc[i][t][4 * q] + b0, z1 = acc[i][t][4 * q + 1] + b1;
          const float z2 = acc[i][t][4 * q + 2] + b2, z3 = acc[i][t][4 * q + 3] + b3;
          if (EPI == TF_EPI_NONE_F32) {
            const f32x4 v = {z0, z1, z2, z3};
            *(f32x4*)((float*)p.Y + (size_t)m * p.ldy + n) = v;
          } else {
            u32x2 o;
            o[0] = pack_bf16x2(activate<EPI>(z0), activate<EPI>(z1));
            o[1] = pack_bf16x2(activate<EPI>(z2), activate<EPI>(z3));
            *(u32x2*)((uint16_t*)p.Y + (size_t)m * p.ldy + n) = o;
          }
        }
      }
    }
  }
}

// The same epilogue for whole tiles with 16-byte aligned output rows, with the stores coalesced through LDS.
// Written straight from the accumulators, a store instruction touches 32 rows with 16 or 32 bytes each, and
// the memory side handles every such piece as a request of its own: that, not the byte count, bounds the
// write-back. Here the work-group lays 32 rows per wave row out in LDS (the tile ring is free by now),
// and reads them back so that consecutive lanes hold consecutive 16-byte pieces of a row: a store
// instruction then writes whole rows of the tile, 64 x 16 bytes contiguous per BN * esz bytes.
// The lines go out complete, so the stores are marked non-temporal: nothing is left in the L2 for the
// write-back at the end of the kernel. PARTIAL: the raw accumulators (no bias) go to `dst`, a split-K slice of
// the workspace with rows of `ld` floats, instead of Y.
// Every wave of the work-group must call it (barriers inside).
template <class C, int EPI, bool PARTIAL = false>
__device__ __forceinline__ void epilogue_staged(const typename C::Acc (&acc)[C::TM][C::TN], const GemmParams& p, char* smem, int m0,
                                                int n0, int tid, int wave_m, int wave_n, int wave_k, int lane_m, int lane_g,
                                                char* dst, size_t ld, int ncols = C::BN_ACT) {
  // ncols: columns of the tile that exist / belong to it (a multiple of 8); pieces past them are not stored
  static_assert(!PARTIAL || EPI == TF_EPI_NONE_F32, "partial sums are fp32");
  constexpr int ESZ = EPI == TF_EPI_NONE_F32 ? 4 : 2;
  constexpr int ROWB = C::BN_ACT * ESZ + 16;             // staged row, padded: the 32 rows a store hits spread over the banks
  constexpr int CPR = C::BN_ACT * ESZ / 16;              // 16-byte pieces per row
  constexpr int PER_THREAD = C::ST_ROWS * CPR / C::THREADS;
  static_assert(C::ST_ROWS * CPR % C::THREADS == 0, "pieces divide over the threads");
  const char* bias_lds = smem + C::BIAS_OFF + 8 * lane_g;
  char* wr = smem + ((wave_m * C::WK + wave_k) * 32 + lane_m) * ROWB + 4 * lane_g * ESZ;
  constexpr int RB = 32 / C::MB;                         // row blocks a pass takes
  static_assert(C::TM0 % RB == 0, "a pass takes consecutive rows of a wave");
  wait_vmcnt<0>();          // no transfer into LDS is in flight any more (the K loops leave none; the bias of a work-group without K tiles may be)
  barrier_lds();            // and nobody reads tile fragments any more
#pragma unroll
  for (int i = 0; i < C::TM_OUT / RB; ++i) {
    if (i) barrier_lds();   // the previous pass has been read back
#pragma unroll
    for (int t = 0; t < C::TN; ++t)
#pragma unroll
      for (int q = 0; q < C::QN * RB; ++q) {
        const int b = i * RB + q / C::QN, e = 4 * (q % C::QN), col = C::col_off(t, wave_n) + 2 * e;
        char* const at = wr + (q / C::QN) * C::MB * ROWB;
        float z0 = acc[b][t][e], z1 = acc[b][t][e + 1], z2 = acc[b][t][e + 2], z3 = acc[b][t][e + 3];
        if (!PARTIAL) {
          const u32x2 braw = *(const u32x2*)(bias_lds + col * 2);
          z0 += __builtin_bit_cast(float, braw[0] << 16);
          z1 += __builtin_bit_cast(float, braw[0] & 0xffff0000u);
          z2 += __builtin_bit_cast(float, braw[1] << 16);
          z3 += __builtin_bit_cast(float, braw[1] & 0xffff0000u);
        }
        if (EPI == TF_EPI_NONE_F32) {
          const f32x4 v = {z0, z1, z2, z3};
          *(f32x4*)(at + col * 4) = v;
        } else {
          u32x2 o;
          o[0] = pack_bf16x2(activate<EPI>(z0), activate<EPI>(z1));
          o[1] = pack_bf16x2(activate<EPI>(z2), activate<EPI>(z3));
          *(u32x2*)(at + col * 2) = o;
        }
      }
    barrier_lds();
#pragma unroll
    for (int j = 0; j < PER_THREAD; ++j) {
      const int c = tid + C::THREADS * j;
      const int rs = c / CPR, cc = c % CPR;
      const int g = rs >> 5;                               // wave row and k group the staged row came from
      const int m = m0 + C::row_off(RB * i, g / C::WK) + (g % C::WK) * (C::WTM / 2) + (rs & 31);
      const u32x4 v = *(const u32x4*)(smem + rs * ROWB + cc * 16);
      // not read again by this launch: non-temporal. A partial tile too: ordinary stores leave 4 MB of it in this XCD's L2 until the
      // launch ends, and the lines that the reducing kernel of the call before has left in other L2s make them slower still (one
      // workspace for call after call, us, with ordinary loads there too / both non-temporal: 512 x 768 x 8192 in eight slices
      // 19.7 / 15.2, 288 x 1152 x 7360 18.9 / 15.0, 1912 x 488 x 3976 in four 20.0 / 18.3, 1024 x 1024 x 16384 42.9 / 40.0).
      // Not where many rows start off 128-byte lines, whose ends would go out in halves: p.ws_past_l2.
      if (cc * 16 < ncols * ESZ) {
        u32x4* const to = (u32x4*)(dst + ((size_t)m * ld + n0) * ESZ + cc * 16);
        if (PARTIAL && !p.ws_past_l2) {
          // (two stores to one place, of which the compiler would make one, an ordinary one, if the branches began or ended alike)
          asm volatile("" ::: "memory");
          *to = v;
          asm volatile("" ::: "memory");
        } else {
          __builtin_nontemporal_store(v, to);
        }
      }
    }
  }
}

template <class C>
__device__ __forceinline__ void gemm_tile_body(const GemmParams& p_in) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  // batched problems: blockIdx.y is the batch item, whose operands are a stride away
  GemmParams p = p_in;
  int tile_id = blockIdx.x;
  if (gridDim.y > 1) {
    int item = blockIdx.y;
    if (p.batch_xcd) {
      // Work-groups go to the eight XCDs in turn, in launch order (x fastest). Renumber them so that all tiles
      // of a batch item run on one XCD, whose L2 then fetches the item's operands once, not once per XCD:
      // XCD x takes items x, x + 8, ... (the host sets the flag only for a batch that is a multiple of 8).
      const unsigned launch_id = blockIdx.y * gridDim.x + blockIdx.x;
      const unsigned local = launch_id >> 3;
      item = (int)((launch_id & 7u) + 8u * (local / gridDim.x));
      tile_id = (int)(local % gridDim.x);
    }
    p.A += (size_t)item * p.stride_a;
    p.B += (size_t)item * p.stride_b;
    p.Y = (char*)p.Y + (size_t)item * p.stride_y * (p.epi == TF_EPI_NONE_F32 ? 4 : 2);
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_k = wave / (C::WM * C::WN), wave_mn = wave % (C::WM * C::WN);
  const int wave_m = wave_mn / C::WN, wave_n = wave_mn % C::WN;

  // A work-group computes one segment = one tile over one range of K tiles - except the stream-K work-groups,
  // which take an equal share of the K steps of the last tiles each, a share that may span up to three tiles
  // (the end of one, a whole one, the beginning of the next). The host arranges that a tile has at most two
  // contributors: they exchange partial tiles like two split-K slices (slice 0 = the part that begins the
  // tile), and since a sum of two terms does not depend on their order the result is the same whoever
  // arrives last.
  const int ktiles_total = (p.K + C::BK - 1) / C::BK;
  // (Compiled only into the stream-K instances, StreamKCfg<>; in every other kernel the loop below is one pass
  // and costs nothing: wrapped around the ordinary kernels it cost them 1-2 % through register pressure.)
  constexpr bool SEGMENTS = C::SEGMENTS;
  static_assert(!SEGMENTS || C::FUSED_OK, "stream-K needs the in-kernel reduction");
  int sk_cur = 0, sk_end = 0;
  const bool stream_k = SEGMENTS && p.stream_k;
  const bool stream_wg = stream_k && tile_id >= p.sk_first_wg;
  if (stream_wg) {
    // (the shares of the work-groups of one XCD lie side by side: they work on neighbouring tiles)
    const long g = xcd_run(tile_id - p.sk_first_wg, p.sk_wgs), total_steps = (long)p.sk_tiles * ktiles_total;
    sk_cur = (int)(g * total_steps / p.sk_wgs);
    sk_end = (int)((g + 1) * total_steps / p.sk_wgs);
  }
  bool more = true;
  for (int seg = 0; more; ++seg) {
  if (seg) {                       // the ring, the bias copy and the staging area are about to be reused
    wait_vmcnt<0>();
    __syncthreads();
  }
  TileCoord tc;
  int kt_begin, kt_end;
  bool split = p.split_k > 1;      // this segment is one of several contributions to its tile
  int n0_mixed = -1, n_end = p.N;  // (mixed grid) origin of a tile of the narrow round; first column that is not the tile's
  if (p.mix_main_wgs > 0) {
    // A launch of whole rounds of BN-wide tiles over the first columns, then one round of narrower tiles that
    // share out the remaining columns of every row panel evenly (see tf_gemm_mixed_kernel). No K slices.
    if constexpr (C::BN_ACT == C::BN) {
      tc = tile_at(p, xcd_run(tile_id, p.mix_main_wgs));          // p.tiles_n = tile columns of the wide part
    } else {
      const int t = xcd_run(tile_id - p.mix_main_wgs, p.tiles_m * p.mix_tiles);
      tc.tm = t / p.mix_tiles; tc.tn = 0; tc.ks = 0;
      const int j = t - tc.tm * p.mix_tiles;
      // tile j of the row panel starts at block floor(j R / T) of the remaining R blocks of 32 columns and owns the
      // blocks up to the start of tile j + 1 (at most BN_ACT / 32 of them; the host checked)
      const int b0 = (int)((long)j * p.mix_blocks / p.mix_tiles), b1 = (int)((long)(j + 1) * p.mix_blocks / p.mix_tiles);
      n0_mixed = p.mix_n_origin + 32 * b0;
      const int lim = p.mix_n_origin + 32 * b1;
      n_end = lim < p.N ? lim : p.N;
    }
    kt_begin = 0; kt_end = ktiles_total; split = false; more = false;
  } else if (!stream_k) {
    tc = map_tile(p, tile_id);
    kt_begin = tc.ks * p.ktiles_per_split;
    kt_end = kt_begin + p.ktiles_per_split;
    if (kt_end > ktiles_total) kt_end = ktiles_total;
    more = false;
  } else if (!stream_wg) {
    tc = tile_at(p, p.xcd_swizzle ? xcd_run(tile_id, p.sk_first_wg) : tile_id);
    kt_begin = 0; kt_end = ktiles_total; split = false; more = false;
  } else {
    if (sk_cur >= sk_end) break;   // (an empty share: more work-groups than steps)
    const int t = sk_cur / ktiles_total;
    kt_begin = sk_cur - t * ktiles_total;
    kt_end = kt_begin + (sk_end - sk_cur);
    if (kt_end > ktiles_total) kt_end = ktiles_total;
    tc = tile_at(p, p.sk_first_wg + t);
    split = !(kt_begin == 0 && kt_end == ktiles_total);
    tc.ks = kt_begin == 0 ? 0 : 1;
    sk_cur += kt_end - kt_begin;
    more = sk_cur < sk_end;
  }
  const int m0 = tc.tm * C::BM, n0 = n0_mixed >= 0 ? n0_mixed : tc.tn * C::BN;
  // K tiles dealt to the slices in turn (slice s takes the tiles s, s + S, s + 2 S, ...) instead of a contiguous range
  // each: at any moment all work-groups then read inside one narrow band of rows of B, which a streaming read of
  // column strips rewards (134 MB: 21.2 us against 23.2 us with two halves of K; host: direct staging only)
  const bool k_deal = C::DIRECT && p.k_interleave && split && !stream_k;
  // (the same for every lane: said so, the K loop keeps its counters and addresses in scalar registers)
  const int nkt = __builtin_amdgcn_readfirstlane(k_deal ? (ktiles_total - tc.ks + p.split_k - 1) / p.split_k
                                                        : kt_end - kt_begin);   // may be <= 0 for a trailing empty slice: contributes zeros

  // ---- LDS read offsets of this lane (bytes inside a stage)
  int a_off[C::KS];
  {
    const int r = C::row_off(0, wave_m) + lane % C::MB;
    const int g = lane / C::MB;
    const int sw = C::row_swz(r);          // (the same for the rows MB, 2 MB, ... further down)
#pragma unroll
    for (int kk = 0; kk < C::KS; ++kk) a_off[kk] = r * C::K_ROW_BYTES + (((C::KMF / 8 * (wave_k * C::KS + kk) + g) ^ sw) << 4);
  }
  // from a wave's first block of A to block i: the same for every wave but in a tile of unequal units
  auto a_block = [&](int i) { return (C::row_off(i, wave_m) - C::row_off(0, wave_m)) * C::K_ROW_BYTES; };
  auto a_block_const = [](int i) { return (C::row_off(i, 0) - C::row_off(0, 0)) * C::K_ROW_BYTES; };
  constexpr bool EVEN_UNITS = C::TM == C::TM0 || C::TM == 2 * C::TM0;
  // B given as [N][K]: its tile is read like the A tile. Its offsets are derived per read from two values (the
  // chunk index KMF / 8 k + g only differs from g above g's bits, so the swizzled slot of step k is (g ^ sw) ^ (KMF / 8 k)):
  // a table per k16-step as for A costs registers the big tiles do not have.
  int bt_row = 0, bt_c0 = 0;
  int bt_off[C::QUAD ? C::KS : 1];
  if constexpr (C::TRANSB) {
    const int r = wave_n * C::TN0 * C::MB + lane % C::MB;
    bt_row = C::B_BASE + r * C::K_ROW_BYTES;
    bt_c0 = ((lane / C::MB) ^ C::row_swz(r)) << 4;
    if constexpr (C::QUAD)
#pragma unroll
      for (int kk = 0; kk < C::KS; ++kk) bt_off[kk] = bt_row + (bt_c0 ^ (kk * (C::KMF * 2)));
  }
  int a_toff[C::TRANSA ? C::TM : 1];     // transposed A: offsets for the transposing read, as for B
  if constexpr (C::TRANSA) {
    const int b = lane >> 4, s = lane & 15;
    const int krow = 8 * (b >> 1) + (s >> 2);
    const int within = (16 * (b & 1) + 4 * (s & 3)) * 2;
#pragma unroll
    for (int i = 0; i < C::TM; ++i) {
      const int j = (wave_m * C::WTM) / 32 + i;
      const int piece = j ^ b_swz<C::A_PIECES>(krow);
      a_toff[i] = (krow + wave_k * C::KS * 16) * C::A_ROW_BYTES + piece * 64 + within;
    }
  }
  // one A operand of MFMA step kk (relative to the wave's first step), row block i
  auto read_a = [&](const char* stage, int kk, int i) -> bf16x8 {
    if constexpr (C::TRANSA) {
      const char* ap = stage + a_toff[i] + (16 * kk) * C::A_ROW_BYTES;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(ap));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(ap + 4 * C::A_ROW_BYTES));
      const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      return __builtin_bit_cast(bf16x8, v);
    } else {
      return *(const bf16x8*)(stage + a_off[kk] + (EVEN_UNITS ? a_block_const(i) : a_block(i)));
    }
  };
  int b_off[C::TN0];                       // the second unit's are B_UNIT_BYTES further
  {
    const int b = lane >> 4, s = lane & 15;
    // a lane group reads four rows of 16 columns, its lanes 4 columns each; MB 32: two groups side by side, then 8 k on
    const int krow = 8 * (C::MB == 16 ? b : b >> 1) + (s >> 2);      // + KMF kk + 4 h
    const int col = wave_n * C::TN0 * C::MB + (C::MB == 16 ? 0 : 16 * (b & 1)) + 4 * (s & 3);
#pragma unroll
    for (int t = 0; t < C::TN0; ++t) {
      const int n = col + C::MB * t;
      b_off[t] = C::B_BASE + (krow + wave_k * C::KS * C::KMF) * C::B_ROW_BYTES + (((n >> 3) ^ b_chunk_swz<C>(krow)) << 4) + (n & 7) * 2;
    }
  }
  // one B operand of MFMA step kk (relative to the wave's first step), column block t
  auto read_b1 = [&](const char* stage, int kk, int t) -> bf16x8 {
    if constexpr (C::TRANSB && C::QUAD) {
      return *(const bf16x8*)(stage + bt_off[kk] + t / C::TN0 * C::B_UNIT_BYTES + t % C::TN0 * C::MB * C::K_ROW_BYTES);
    } else if constexpr (C::TRANSB) {
      return *(const bf16x8*)(stage + bt_row + (bt_c0 ^ ((wave_k * C::KS + kk) * (C::KMF * 2))) + t * C::MB * C::K_ROW_BYTES);
    } else {
      const char* bp = stage + b_off[t % C::TN0] + t / C::TN0 * C::B_UNIT_BYTES + (C::KMF * kk) * C::B_ROW_BYTES;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp + 4 * C::B_ROW_BYTES));
      const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      return __builtin_bit_cast(bf16x8, v);
    }
  };
  // LINES: where chunk KMF / 8 kk + g lies, for rows of this lane's shift
  LineRows la{}, lb{};
  int la_off[C::LINES ? C::KS : 1], lb_off[C::LINES ? C::KS : 1];
  bool la_next[C::LINES ? C::KS : 1], lb_next[C::LINES ? C::KS : 1];
  if constexpr (C::LINES) {
    const int ra = C::row_off(0, wave_m) + lane % C::MB, rb = wave_n * C::TN0 * C::MB + lane % C::MB;
    la.shift = LineRows::shift_of(p.A, p.lda, m0 + ra);
    lb.shift = LineRows::shift_of(p.B, p.ldb, n0 + rb);
#pragma unroll
    for (int kk = 0; kk < C::KS; ++kk) {
      const int ua = C::KMF / 8 * kk + lane / C::MB + la.shift, ub = C::KMF / 8 * kk + lane / C::MB + lb.shift;
      la_off[kk] = ra * C::K_ROW_BYTES + (((ua - la.shift) ^ C::row_swz(ra)) << 4);
      la_next[kk] = ua >= 8;
      lb_off[kk] = C::B_BASE + rb * C::K_ROW_BYTES + (((ub - lb.shift) ^ C::row_swz(rb)) << 4);
      lb_next[kk] = ub >= 8;
    }
  }
  auto line_a = [&](const char* stage, const char* next, int kk, int i) -> bf16x8 {
    return *(const bf16x8*)((la_next[kk] ? next : stage) + la_off[kk] + a_block_const(i));
  };
  auto line_b = [&](const char* stage, const char* next, int kk, int t) -> bf16x8 {
    return *(const bf16x8*)((lb_next[kk] ? next : stage) + lb_off[kk] + t * C::MB * C::K_ROW_BYTES);
  };
  auto mma = [](const bf16x8 b, const bf16x8 a, const typename C::Acc c) -> typename C::Acc {
    if constexpr (C::MB == 16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, c, 0, 0, 0);
  };

  typename C::Acc acc[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int t = 0; t < C::TN; ++t)
#pragma unroll
      for (int r = 0; r < 4 * C::QN; ++r) acc[i][t][r] = 0.0f;

  TileLoader<C> ld;
  ld.init(p, m0, n0, wave, lane);
  // bias of this tile -> LDS (two values per lane), ahead of the first tile: it is in place when
  // the first hand-over barrier has been passed
  if (wave == 0) {
#pragma unroll
    for (int r = 0; r < (C::BN + 127) / 128; ++r) {
      const int c = 128 * r + 2 * lane;                 // column inside the tile
      if (c < C::BN) {
        const int n = n0 + c;
        if (p.bias == nullptr) {
          *(unsigned*)(smem + C::BIAS_OFF + c * 2) = 0u;      // no bias: the epilogue adds zeros
        } else if constexpr (C::DIRECT) {
          TileLoader<C>::gload_lds4(__builtin_amdgcn_readfirstlane((unsigned)(size_t)smem + C::BIAS_OFF + 256 * r),
                                    n < p.N ? (unsigned)n * 2u : 0u, p.bias);
        } else {
          unsigned v = 0u;
          if (n < p.N) v = *(const unsigned*)(p.bias + n);
          *(unsigned*)(smem + C::BIAS_OFF + c * 2) = v;
        }
      }
    }
  }
  const long a_tile = C::TRANSA ? (long)C::BK * p.lda : (long)C::BK;     // one K tile further in A
  const long b_tile = C::TRANSB ? (long)C::BK : (long)C::BK * p.ldb;      // one K tile further in B
  const int first_kt = k_deal ? tc.ks : kt_begin;
  const long a_step = k_deal ? a_tile * p.split_k : a_tile;              // this work-group's next K tile
  const long b_step = k_deal ? b_tile * p.split_k : b_tile;
  const uint16_t* Ak = p.A + (long)first_kt * a_tile;
  const uint16_t* Bk = p.B + (long)first_kt * b_tile;

  // ---- main loop, software pipelined by hand (one wave per SIMD has nobody to hide behind):
  //  * fragments are double buffered in registers: the LDS reads of MFMA step kk+1 are issued
  //    before the MFMAs of step kk;
  //  * the loop is rotated: the barrier that hands over the next tile, the global loads of the
  //    tile after it and the first fragment reads of the next tile are all issued BEFORE the
  //    last step of the current tile, whose MFMAs cover their latency.
  bf16x8 af[2][C::TM], bfr[2][C::TN];
  auto read_frags = [&](const char* stage, int kk, int set) {
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
      af[set][i] = read_a(stage, kk, i);
#pragma unroll
    for (int t = 0; t < C::TN; ++t) bfr[set][t] = read_b1(stage, kk, t);
  };
  // (blocks in serpentine order: an MFMA shares one operand with the one before it, which costs less power)
  auto mfma_step = [&](int set) {
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int u = 0; u < C::TN; ++u) {
        const int t = C::ORDERED && (i & 1) ? C::TN - 1 - u : u;
        acc[i][t] = mma(bfr[set][t], af[set][i], acc[i][t]);
      }
  };
  // Scheduling hint for a step of MFMAs behind which LDS reads go out: one read per MFMA until they are all issued, so that
  // the matrix pipe never waits for the whole batch and the hand-over at the end of the step finds most of them done (two per
  // MFMA: 2048^3 20.0 -> 20.8 us). The MFMAs left over are named too: what is not, the compiler moves across steps.
  constexpr int DS_B = C::TRANSB ? 1 : 2;                  // LDS reads per B operand
  constexpr int N_DS = C::TM + DS_B * C::TN, N_MFMA = C::TM * C::TN;
  auto spread = [&](auto reads, auto mfmas) {
    constexpr int R = decltype(reads)::value, N = decltype(mfmas)::value;
    static_for<(R < N ? R : N)>([&](auto) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one DS read
    });
    if constexpr (C::ORDERED && R > N) __builtin_amdgcn_sched_group_barrier(0x100, R - N, 0);
    if constexpr (C::ORDERED && N > R) __builtin_amdgcn_sched_group_barrier(0x008, N - R, 0);
  };
  auto interleave_hint = [&]() { spread(EpiTag<N_DS>{}, EpiTag<N_MFMA>{}); };

  // The last tile is peeled off the loop, and so are the ones behind which nothing more is fetched: the
  // loop body has no branch inside and is scheduled as one block, with constant vmcnt waits. (The A-bypass kernel
  // re-fetches the last tile past the end, into a buffer nobody reads any more, and the register-staged kernels into
  // registers. With every kernel doing that, a work-group fetched STAGES - 1 K tiles more than it has, at the rate that
  // bounds the K loop, and waited for them before its epilogue.)
  const int last = nkt - 1;
  // Order of the K tiles (a sum: any order is right). Without split-K the work-groups of XCD x start an
  // eighth of the way further into K than those of XCD x - 1 and wrap round: at any moment the eight XCDs
  // then fetch eight different slabs of A and B, and seven times out of eight a line has already been
  // brought into the memory-side cache by another XCD instead of all eight waiting for it together.
  // (All work-groups of an XCD keep the same order, so they still share panels in its L2.)
  // RaggedKCfg (K no multiple of BK; a multiple of 8, at least BK): the last K tile of the problem is fetched from
  // K - BK on, so that every transfer stays inside the operands, and its first `skip` k, which the tile before it holds
  // too, are zeroed in LDS in BOTH operands (an infinity or NaN among them must not meet a zero) before its fragments are
  // read. The work-group that has this tile takes it first, ahead of the main loop and before there are accumulators
  // (at the end of the loop the zeroing made the 256 x 256 tiles spill). The host offers no rotated order here.
  const int k_over = ktiles_total * C::BK - p.K;
  const int skip = __builtin_amdgcn_readfirstlane(
      C::KTAIL && k_over > 0 && first_kt + last * (k_deal ? p.split_k : 1) == ktiles_total - 1 ? k_over : 0);
  const int k_rot = C::KTAIL ? (skip ? last : 0) : (p.k_rotate && nkt > 0) ? (int)(((blockIdx.x & 7u) * (unsigned)nkt) >> 3) : 0;
  auto k_order = [&](int t) { const int u = t + k_rot; return u >= nkt ? u - nkt : u; };
  const long a_back = C::TRANSA ? skip * p.lda : (long)skip, b_back = C::TRANSB ? (long)skip : skip * p.ldb;
  // Where the next K tile to fetch lies in A and B: moved on a tile at a time, with one wrap (a multiplication per
  // tile and operand cost the loop some thirty scalar or, where the compiler chose so, vector instructions a step).
  struct Fetch {
    unsigned long long a, b;
    int left;                              // tiles from here to the end of the range
  } nx;
  auto uniform = [](const void* x) {
    const unsigned long long v = (unsigned long long)x;
    return (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v) |
           ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32)) << 32);
  };
  const unsigned long long a_first = uniform(Ak), b_first = uniform(Bk);
  const long a_move = 2 * a_step, b_move = 2 * b_step;       // bytes
  nx.left = nkt - k_rot;
  nx.a = uniform((const void*)(a_first + (unsigned long long)(k_rot * a_move) - (C::KTAIL ? 2 * a_back : 0)));
  nx.b = uniform((const void*)(b_first + (unsigned long long)(k_rot * b_move) - (C::KTAIL ? 2 * b_back : 0)));
  auto next_tile = [&]() {
    --nx.left;
    nx.a = nx.left == 0 ? a_first : nx.a + a_move;
    nx.b = nx.left == 0 ? b_first : nx.b + b_move;
  };
  auto next_a = [&]() { return (const uint16_t*)nx.a; };
  auto next_b = [&]() { return (const uint16_t*)nx.b; };
  if constexpr (C::LINES) {
    const int row = C::K_ROWS_PER_INSTR * wave + lane / C::K_CHUNKS, c = (lane % C::K_CHUNKS) ^ C::row_swz(row);
    auto set = [&](LineRows& r, unsigned* src, int per_wave, const uint16_t* base, long ld_elems, int first, int count) {
      const int s = LineRows::shift_of(base, ld_elems, first + row);
      r.cs = ((c + s) & 7) - s;
      r.begin = first_kt * 8;
      r.k0 = r.begin - (skip ? 8 : 0);
      r.chunks = p.K / 8;
      r.wrap = skip != 0;
      for (int q = 0; q < per_wave; ++q) {
        int m = first + row + C::K_ROWS_PER_INSTR * C::NWAVES * q;
        if (m >= count) m = count - 1;
        src[q] = ((unsigned)m * (unsigned)ld_elems + 8u * (unsigned)(r.cs + 7)) * 2u;
      }
    };
    static_assert(!C::LINES || C::K_ROWS_PER_INSTR * C::NWAVES % 16 == 0, "one slot and one shift for all transfers of a lane");
    set(la, ld.a_src, C::A_PER_WAVE, p.A, p.lda, m0, p.M);
    if constexpr (C::TRANSB) set(lb, ld.b_src, C::B_PER_WAVE, p.B, p.ldb, n0, p.N);
  }
  auto zero_skipped = [&]() {                  // every wave calls it; the first tile has landed and has not been read
    if (!C::KTAIL || skip == 0) return;
    char* const a_tile = smem;
    char* const b_tile = smem + C::B_BASE;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    auto k_contiguous = [&](char* tile, int rows) {
      for (int c = 0; c < skip / 8; ++c)
        for (int r = tid; r < rows; r += C::THREADS) *(u32x4*)(tile + r * C::K_ROW_BYTES + ((c ^ C::row_swz(r)) << 4)) = zero;
    };
    auto k_rows = [&](char* tile, int row_bytes) {
      for (int x = tid * 16; x < skip * row_bytes; x += C::THREADS * 16) *(u32x4*)(tile + x) = zero;
    };
    auto k_lines = [&](char* tile, int rows, const uint16_t* base, long ld_elems, int first) {
      for (int r = tid; r < rows; r += C::THREADS) {
        const int s = LineRows::shift_of(base, ld_elems, first + r);
        for (int c = 0; c < skip / 8; ++c)
          *(u32x4*)(tile + ((c + s) >> 3) * C::STAGE_BYTES + r * C::K_ROW_BYTES + ((c ^ C::row_swz(r)) << 4)) = zero;
      }
    };
    if constexpr (C::TRANSA) k_rows(a_tile, C::A_ROW_BYTES);
    else if constexpr (C::LINES) k_lines(a_tile, C::BM, p.A, p.lda, m0);
    else k_contiguous(a_tile, C::BM);
    if constexpr (C::TRANSB && C::LINES) k_lines(b_tile, C::BN, p.B, p.ldb, n0);
    else if constexpr (C::TRANSB) k_contiguous(b_tile, C::BN);
    else
      for (int u = 0; u < C::B_UNITS; ++u) k_rows(b_tile + u * C::B_UNIT_BYTES, C::B_ROW_BYTES);
    barrier_lds();
  };
  if constexpr (C::ABYPASS) {
    // A straight from memory into MFMA operand registers: lane l of a wave needs, for row block
    // i and k16-step kk, the 16 bytes at row 32 i + (l & 31), k = 16 kk + 8 (l >> 5): one
    // global_load_dwordx4. Two register sets alternate per tile (the loop is unrolled by two so
    // both are addressed statically); the loads of tile kt+1 are issued at the top of tile kt.
    // These loads are ordinary loads the compiler tracks; the B transfers are not, so every
    // hand-over waits for vmcnt 0, which by then only covers loads issued a tile earlier.
    const unsigned lds0 = (unsigned)(size_t)smem;
    unsigned a_goff[C::TM];
#pragma unroll
    for (int i = 0; i < C::TM; ++i) {
      int m = m0 + wave_m * C::WTM + 32 * i + (lane & 31);
      if (m >= p.M) m = p.M - 1;
      a_goff[i] = ((unsigned)m * (unsigned)p.lda + 8u * (lane >> 5)) * 2u;
    }
    auto tile_a = [&](int t) { return Ak + (long)k_order(t < last ? t : last) * a_step; };
    auto tile_b = [&](int t) { return Bk + (long)k_order(t < last ? t : last) * b_step; };
    auto load_a = [&](u32x4 (&dst)[C::TM][4], const uint16_t* base) {
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) dst[i][kk] = *(const u32x4*)((const char*)base + a_goff[i] + kk * 32);
    };
    auto read_b = [&](const char* stage, int kk, int set) {
#pragma unroll
      for (int t = 0; t < C::TN; ++t) {
        const char* bp = stage + b_off[t] + (16 * kk) * C::B_ROW_BYTES;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(bp + 4 * C::B_ROW_BYTES));
        const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        bfr[set][t] = __builtin_bit_cast(bf16x8, v);
      }
    };
    auto mfma_a = [&](const u32x4 (&as)[C::TM][4], int kk, int set) {
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int t = 0; t < C::TN; ++t)
          acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][t], __builtin_bit_cast(bf16x8, as[i][kk]), acc[i][t], 0, 0, 0);
    };
    auto hint_b = [&]() {
#pragma unroll
      for (int x = 0; x < (2 * C::TN < C::TM * C::TN ? 2 * C::TN : C::TM * C::TN); ++x) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    };
    // one non-final tile t computed from register set `cur`, while `nxt` receives tile t+1
    auto half = [&](const u32x4 (&cur)[C::TM][4], u32x4 (&nxt)[C::TM][4], int t) {
      const char* sb = smem + (t & 1) * C::STAGE_BYTES;
      load_a(nxt, tile_a(t + 1));
      __builtin_amdgcn_sched_barrier(0);   // keep the loads up here: a whole tile of MFMAs covers their latency
#pragma unroll
      for (int kk = 0; kk < 3; ++kk) {
        read_b(sb, kk + 1, (kk + 1) & 1);
        mfma_a(cur, kk, kk & 1);
        hint_b();
      }
      wait_vmcnt<0>();      // B tile t+1 (issued one tile ago) and A tile t+1 have arrived
      barrier_lds();        // ... for every wave; every wave is done reading B tile t
      ld.issue_b_direct(tile_b(t + 2), lds0 + (t & 1) * C::STAGE_BYTES, wave);
      read_b(smem + ((t + 1) & 1) * C::STAGE_BYTES, 0, 0);
      mfma_a(cur, 3, 1);
      hint_b();
    };
    auto final_tile = [&](const u32x4 (&cur)[C::TM][4], int t) {
      const char* sb = smem + (t & 1) * C::STAGE_BYTES;
#pragma unroll
      for (int kk = 0; kk < 3; ++kk) {
        read_b(sb, kk + 1, (kk + 1) & 1);
        mfma_a(cur, kk, kk & 1);
        hint_b();
      }
      mfma_a(cur, 3, 1);
    };
    if (nkt > 0) {
      u32x4 A0[C::TM][4], A1[C::TM][4];
      ld.issue_b_direct(tile_b(0), lds0, wave);
      load_a(A0, tile_a(0));
      wait_vmcnt<0>();
      barrier_lds();
      ld.issue_b_direct(tile_b(1), lds0 + C::STAGE_BYTES, wave);
      read_b(smem, 0, 0);
      int kt = 0;
      for (; kt + 2 <= last; kt += 2) {
        half(A0, A1, kt);
        half(A1, A0, kt + 1);
      }
      if (kt < last) {
        half(A0, A1, kt);
        final_tile(A1, last);
      } else {
        final_tile(A0, last);
      }
      wait_vmcnt<0>();
    }
  } else if constexpr (C::DIRECT && C::ACC * C::KS * C::KMF <= 8 * 16 * 16) {
    // Small wave tiles (skinny problems): an MFMA step has only one or two MFMAs of 32 x 32, far too few to
    // cover an LDS read, so the step-by-step pipeline above would stall four times per tile.
    // Here all fragments of a tile are read at once, into one of two register sets, while the
    // MFMAs of the previous tile run; one wait + barrier per tile. Unrolled by two so that both
    // sets are addressed statically.
    constexpr int D = C::STAGES - 1;
    constexpr int PER_TILE = C::A_PER_WAVE + C::B_PER_WAVE;
    static_assert((D - 1) * PER_TILE < 64, "vmcnt range");
    const unsigned lds0 = (unsigned)(size_t)smem;
    bf16x8 fa[2][C::KS][C::TM], fb[2][C::KS][C::TN];
    // the K tile in buffer `buf` (LINES: and the next one)
    auto read_tile = [&](int buf, bf16x8 (&a)[C::KS][C::TM], bf16x8 (&b)[C::KS][C::TN]) {
      const char* const stage = smem + buf * C::STAGE_BYTES;
      const char* const next = smem + (buf + 1 == C::STAGES ? 0 : buf + 1) * C::STAGE_BYTES;
#pragma unroll
      for (int kk = 0; kk < C::KS; ++kk) {
#pragma unroll
        for (int i = 0; i < C::TM; ++i) {
          if constexpr (C::LINES) a[kk][i] = line_a(stage, next, kk, i);
          else a[kk][i] = read_a(stage, kk, i);
        }
#pragma unroll
        for (int t = 0; t < C::TN; ++t) {
          if constexpr (C::LINES && C::TRANSB) b[kk][t] = line_b(stage, next, kk, t);
          else b[kk][t] = read_b1(stage, kk, t);
        }
      }
    };
    // what buffer w takes: K tile w, or the lines of that number, of which there is one more. EDGE: see issue_lines
    auto fetch_buffer = [&](auto edge, int w, int slot) {
      constexpr bool EDGE = decltype(edge)::value != 0;
      const unsigned to = lds0 + slot * C::STAGE_BYTES;
      if constexpr (!C::LINES) {
        ld.issue_direct(next_a(), next_b(), to, wave);
        next_tile();
      } else {
        TileLoader<C>::template issue_lines<EDGE, false>(la, ld.a_src, p.A, w, to, wave);
        if constexpr (C::TRANSB) {
          TileLoader<C>::template issue_lines<EDGE, C::B_NT>(lb, ld.b_src, p.B, w, to + C::A_BYTES, wave);
        } else if (!EDGE || w < nkt) {
          ld.issue_b_direct(next_b(), to, wave);
          next_tile();
        }
      }
    };
    constexpr int MORE = C::LINES ? 1 : 0;            // buffers beyond the last K tile
    // transfers that may still fly when a K tile is about to be read: all behind it, but for the next lines
    constexpr int FLYING = (D - 1) * PER_TILE - (C::LINES ? (C::TRANSB ? PER_TILE : C::A_PER_WAVE) : 0);
    auto mfma_tile = [&](const bf16x8 (&a)[C::KS][C::TM], const bf16x8 (&b)[C::KS][C::TN]) {
#pragma unroll
      for (int kk = 0; kk < C::KS; ++kk)
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
          for (int u = 0; u < C::TN; ++u) {
            const int t = C::ORDERED && (i & 1) ? C::TN - 1 - u : u;
            acc[i][t] = mma(b[kk][t], a[kk][i], acc[i][t]);
          }
    };
    if (nkt > 0) {
#pragma unroll
      for (int s = 0; s < D; ++s)
        if (s < nkt + MORE) fetch_buffer(EpiTag<1>{}, s, s);
      if (nkt >= D) wait_vmcnt<FLYING>();
      else wait_vmcnt<0>();
      barrier_lds();
      if (D < nkt + MORE) fetch_buffer(EpiTag<1>{}, D, D);
      zero_skipped();
      read_tile(0, fa[0], fb[0]);
      int stage = 0;
      // one non-final tile t: its fragments are in (ca, cb); (na, nb) receive tile t+1. FETCH: tile t + 1 + D exists and
      // is fetched; otherwise what there is
      auto step = [&](auto fetch, int t, const bf16x8 (&ca)[C::KS][C::TM], const bf16x8 (&cb)[C::KS][C::TN],
                      bf16x8 (&na)[C::KS][C::TM], bf16x8 (&nb)[C::KS][C::TN]) {
        constexpr bool FETCH = decltype(fetch)::value != 0;
        int nstage = stage + 1;
        if (nstage == C::STAGES) nstage = 0;
        if (FETCH || t + D <= last) wait_vmcnt<FLYING>();    // tile t+1 has landed
        else wait_vmcnt<0>();
        barrier_lds();                       // ... for every wave; every wave holds tile t in registers
        if (FETCH || t + 1 + D < nkt + MORE) fetch_buffer(EpiTag<!FETCH>{}, t + 1 + D, stage);
        read_tile(nstage, na, nb);
        mfma_tile(ca, cb);
        if constexpr (C::MB == 16) spread(EpiTag<C::KS * N_DS>{}, EpiTag<C::KS * N_MFMA>{});
        if constexpr (C::ORDERED) __builtin_amdgcn_sched_barrier(0);
        stage = nstage;
      };
      int kt = 0;
      for (; kt + 1 < last - D; kt += 2) {
        step(EpiTag<1>{}, kt, fa[0], fb[0], fa[1], fb[1]);
        step(EpiTag<1>{}, kt + 1, fa[1], fb[1], fa[0], fb[0]);
      }
      kt = __builtin_amdgcn_readfirstlane(kt);   // (the same value: keeps the compiler from making one loop of the two)
      for (; kt + 2 <= last; kt += 2) {
        step(EpiTag<0>{}, kt, fa[0], fb[0], fa[1], fb[1]);
        step(EpiTag<0>{}, kt + 1, fa[1], fb[1], fa[0], fb[0]);
      }
      if (kt < last) {
        step(EpiTag<0>{}, kt, fa[0], fb[0], fa[1], fb[1]);
        mfma_tile(fa[1], fb[1]);
      } else {
        mfma_tile(fa[0], fb[0]);
      }
    }
  } else if constexpr (C::QUAD) {
    // Quadrants. A K tile takes four phases, one quadrant of every wave's tile over the whole 64 of K each: A0 B0, A0 B1,
    // A1 B1, A1 B0. Behind the MFMAs of a phase the one unit that the next phase needs is read into registers: B1, A1,
    // then A0 and B0 of the next tile. A unit is read once, so its buffer can take the tile after next as soon as the
    // two phases that read it and its neighbour are over: the transfers run 1.5 K tiles ahead with the two buffers that
    // give one tile otherwise, and a wait only ever meets transfers that went out five phases before. Without it the
    // compiler, or a burst of waves that arrive late, met transfers of half a tile ago. 256 x 256 tiles, us per 64 of K
    // (random operands / zeros, which leave the clock at 2.4 GHz; 0.85 us of MFMA there): one tile ahead in 32 x 32
    // blocks 1.49 / 1.44, here 1.35 / 1.07; 192 x 256 1.32 / 1.22 and 1.07 / 0.82. 4096 x 11008 x 4096 306 -> 285 us,
    // 3072^3 55.0 -> 52.4, 3000 x 5000 x 3000 83.2 -> 76.3 and with B as [N][K] 86.3 -> 77.6.
    // Two K tiles per pass: the buffers and the register sets (B0 in set t & 1) are then addressed statically.
    constexpr int PER_TILE = C::A_PER_WAVE + C::B_PER_WAVE;
    constexpr int TM1 = C::TM - C::TM0, TN1 = C::TN - C::TN0;
    constexpr int A0_PER_WAVE = 128 * 128 / 1024 / C::NWAVES, B0_PER_WAVE = C::B_PER_WAVE / 2;
    static_assert(TM1 > 0 && TM1 <= C::TM0 && TN1 == C::TN0 && C::KS == 2 && C::WK == 1, "units of a quadrant tile");
    const unsigned lds0 = (unsigned)(size_t)smem;
    bf16x8 qa[2][C::KS][C::TM0], qb[2][C::KS][C::TN0];
    auto read_au = [&](int buf, auto u) {                     // A unit u of the tile in buffer buf
#pragma unroll
      for (int kk = 0; kk < C::KS; ++kk)
#pragma unroll
        for (int i = 0; i < (decltype(u)::value ? TM1 : C::TM0); ++i)
          qa[decltype(u)::value][kk][i] = read_a(smem + buf * C::A_STRIDE, kk, decltype(u)::value * C::TM0 + i);
    };
    auto read_bu = [&](int buf, auto u, int set) {
#pragma unroll
      for (int kk = 0; kk < C::KS; ++kk)
#pragma unroll
        for (int t = 0; t < C::TN0; ++t) qb[set][kk][t] = read_b1(smem + buf * C::B_STRIDE, kk, decltype(u)::value * C::TN0 + t);
    };
    auto issue_au = [&](int buf, int u) {
#pragma unroll
      for (int q = u ? A0_PER_WAVE : 0; q < (u ? C::A_PER_WAVE : A0_PER_WAVE); ++q) ld.issue_a_one(q, next_a(), lds0 + buf * C::A_STRIDE, wave);
    };
    auto issue_bu = [&](int buf, int u) {
#pragma unroll
      for (int q = u ? B0_PER_WAVE : 0; q < (u ? C::B_PER_WAVE : B0_PER_WAVE); ++q) ld.issue_b_one(q, next_b(), lds0 + buf * C::B_STRIDE + (C::B_BASE - C::A_BYTES), wave);
    };
    // (u, v): the quadrant; B in register set `set`
    auto quadrant = [&](auto u, auto v, int set) {
      constexpr int U = decltype(u)::value, V = decltype(v)::value;
#pragma unroll
      for (int kk = 0; kk < C::KS; ++kk)
#pragma unroll
        for (int i = 0; i < (U ? TM1 : C::TM0); ++i)
#pragma unroll
          for (int x = 0; x < C::TN0; ++x) {
            const int t = (i + kk) & 1 ? C::TN0 - 1 - x : x;
            acc[U * C::TM0 + i][V * C::TN0 + t] = mma(qb[set][kk][t], qa[U][kk][i], acc[U * C::TM0 + i][V * C::TN0 + t]);
          }
    };
    constexpr int N_B = C::KS * C::TN0 * DS_B, N_A0 = C::KS * C::TM0, N_A1 = C::KS * TM1;
    // tile t in buffer P = t & 1. STEADY: tile t + 2 exists; otherwise what there is
    auto tile_quad = [&](auto parity, auto steady, int t) {
      constexpr int P = decltype(parity)::value, Q = 1 - P;
      constexpr bool STEADY = decltype(steady)::value != 0;
      const bool fetch = STEADY || t + 2 <= last;
      if (fetch) issue_au(P, 0);
      read_bu(P, EpiTag<1>{}, Q);
      quadrant(EpiTag<0>{}, EpiTag<0>{}, P);
      spread(EpiTag<N_B>{}, EpiTag<C::KS * C::TM0 * C::TN0>{});
      __builtin_amdgcn_sched_barrier(0);           // (a phase keeps its reads: their registers are the last one's)
      if (fetch) issue_bu(P, 0);
      read_au(P, EpiTag<1>{});
      quadrant(EpiTag<0>{}, EpiTag<1>{}, Q);
      spread(EpiTag<N_A1>{}, EpiTag<C::KS * C::TM0 * C::TN0>{});
      __builtin_amdgcn_sched_barrier(0);
      if (fetch) wait_vmcnt<PER_TILE>();           // A0, B0 of tile t + 1 have landed
      else if (t < last) wait_vmcnt<C::A_PER_WAVE - A0_PER_WAVE + B0_PER_WAVE>();
      barrier_lds();                               // ... for every wave, and every wave holds B1 and A1 of tile t
      if (fetch) issue_bu(P, 1);
      read_au(Q, EpiTag<0>{});                     // (behind the last tile: what the buffer holds, not used)
      quadrant(EpiTag<1>{}, EpiTag<1>{}, Q);
      spread(EpiTag<N_A0>{}, EpiTag<C::KS * TM1 * C::TN0>{});
      __builtin_amdgcn_sched_barrier(0);
      if (fetch) issue_au(P, 1);
      read_bu(Q, EpiTag<0>{}, Q);
      quadrant(EpiTag<1>{}, EpiTag<0>{}, P);
      spread(EpiTag<N_B>{}, EpiTag<C::KS * TM1 * C::TN0>{});
      __builtin_amdgcn_sched_barrier(0);
      if (fetch) { next_tile(); wait_vmcnt<PER_TILE>(); }    // B1, A1 of tile t + 1 have landed
      else wait_vmcnt<0>();
      barrier_lds();                               // ... for every wave, and every wave holds A0 and B0 of tile t + 1
    };
    if (nkt > 0) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (s < nkt) {
          issue_au(s, 0); issue_bu(s, 0); issue_bu(s, 1); issue_au(s, 1);
          next_tile();
        }
      if (nkt > 1) wait_vmcnt<PER_TILE>();
      else wait_vmcnt<0>();
      barrier_lds();
      zero_skipped();
      read_au(0, EpiTag<0>{});
      read_bu(0, EpiTag<0>{}, 0);
      barrier_lds();
      int kt = 0;
      for (; kt + 3 <= last; kt += 2) {
        tile_quad(EpiTag<0>{}, EpiTag<1>{}, kt);
        tile_quad(EpiTag<1>{}, EpiTag<1>{}, kt + 1);
      }
      kt = __builtin_amdgcn_readfirstlane(kt);   // (the same value: keeps the compiler from making one loop of the two)
      for (; kt <= last; kt += 2) {
        tile_quad(EpiTag<0>{}, EpiTag<0>{}, kt);
        if (kt + 1 <= last) tile_quad(EpiTag<1>{}, EpiTag<0>{}, kt + 1);
      }
    }
  } else if constexpr (C::DIRECT) {
    constexpr int D = C::STAGES - 1;                            // tiles in flight ahead of the one computed
    constexpr int PER_TILE = C::A_PER_WAVE + C::B_PER_WAVE;   // transfers per wave per tile
    static_assert((D - 1) * PER_TILE < 64, "vmcnt range");
    const unsigned lds0 = (unsigned)(size_t)smem;
    // A wave issues in order: a burst of transfers right after the barrier would hold back the
    // MFMAs behind it for as long as the load unit takes to accept the burst (the four waves of a
    // CU share one, at about 16 cycles per transfer). So the transfers of a tile are dealt out
    // one at a time between the fragment reads of two k16-steps: its A part during the last step
    // of the tile whose buffer it takes over, its B part during the first step of the next tile.
    // which: 1 = A part, 2 = B part; the fragment reads and the transfers keep this order, the
    // MFMAs are spread between them by the scheduling hint.
    auto read_frags_issue = [&](const char* stage, int kk, int set, int which, const uint16_t* src, unsigned dst_lds) {
      constexpr int NR = C::TM + C::TN;                   // fragment reads (A: one b128, B: a tr pair)
      const int nx = which == 1 ? C::A_PER_WAVE : which == 2 ? C::B_PER_WAVE : 0;
#pragma unroll
      for (int x = 0; x < (NR > 8 ? NR : 8); ++x) {
        if (x < C::TM) af[set][x] = read_a(stage, kk, x);
        else if (x < NR) bfr[set][x - C::TM] = read_b1(stage, kk, x - C::TM);
        if (x < nx) {
          if (which == 1) ld.issue_a_one(x, src, dst_lds, wave);
          else ld.issue_b_one(x, src, dst_lds, wave);
        }
      }
    };
    static_assert(C::A_PER_WAVE <= 8 && C::B_PER_WAVE <= 8, "transfers of one part fit between the reads of one step");
    if (nkt > 0) {
#pragma unroll
      for (int s = 0; s < D; ++s)
        if (s < nkt) {
          ld.issue_direct(next_a(), next_b(), lds0 + s * C::STAGE_BYTES, wave);
          next_tile();
        }
      if (nkt >= D) wait_vmcnt<(D - 1) * PER_TILE>();      // tile 0 has landed, D-1 younger tiles may still fly
      else wait_vmcnt<0>();
      barrier_lds();
      // tile D: A part now, B part during the first step of tile 0 (as in the steady state)
      if (D < nkt) ld.issue_a_all(next_a(), lds0 + D * C::STAGE_BYTES, wave);
      zero_skipped();
      read_frags(smem, 0, 0);
      int stage = 0, kt = 0;
      // one tile but the last. FETCH: the B part of tile kt + D and the A part of tile kt + 1 + D are on their way
      // behind it (there are such tiles); otherwise the B part of the last tile, if that is tile kt + D, and no more
      auto tile_step = [&](auto fetch) {
        constexpr bool FETCH = decltype(fetch)::value != 0;
        const char* cur = smem + stage * C::STAGE_BYTES;
        int nstage = stage + 1;
        if (nstage == C::STAGES) nstage = 0;
        int pstage = stage + D;               // buffer of tile kt + D (freed by the barrier before this tile)
        if (pstage >= C::STAGES) pstage -= C::STAGES;
        const bool last_b = kt + D == last;
        if (!FETCH && last_b) ld.issue_b_direct(next_b(), lds0 + pstage * C::STAGE_BYTES, wave);
        if constexpr (FETCH) {
          read_frags_issue(cur, 1, 1, 2, next_b(), lds0 + pstage * C::STAGE_BYTES);
          next_tile();
        }
        else read_frags(cur, 1, 1);
        mfma_step(0);
        interleave_hint();
#pragma unroll
        for (int kk = 1; kk < C::KS - 1; ++kk) {
          read_frags(cur, kk + 1, (kk + 1) & 1);
          mfma_step(kk & 1);
          interleave_hint();
        }
        if constexpr (C::ORDERED) __builtin_amdgcn_sched_barrier(0);   // (the MFMAs above stay above)
        if (FETCH || last_b) wait_vmcnt<(D - 1) * PER_TILE>();    // tile kt+1 has landed
        else wait_vmcnt<0>();
        barrier_lds();                       // ... for every wave, and every wave is done reading tile kt
        if constexpr (FETCH) read_frags_issue(smem + nstage * C::STAGE_BYTES, 0, 0, 1, next_a(), lds0 + stage * C::STAGE_BYTES);
        else read_frags(smem + nstage * C::STAGE_BYTES, 0, 0);
        mfma_step(1);                        // the last MFMA step of tile kt covers the latencies above
        interleave_hint();
        stage = nstage;
      };
      for (; kt < last - D; ++kt) tile_step(EpiTag<1>{});
      kt = __builtin_amdgcn_readfirstlane(kt);   // (the same value: keeps the compiler from making one loop of the two)
      for (; kt < last; ++kt) tile_step(EpiTag<0>{});
      {
        const char* cur = smem + stage * C::STAGE_BYTES;
        read_frags(cur, 1, 1);
        mfma_step(0);
        interleave_hint();
#pragma unroll
        for (int kk = 1; kk < C::KS - 1; ++kk) {
          read_frags(cur, kk + 1, (kk + 1) & 1);
          mfma_step(kk & 1);
          interleave_hint();
        }
        mfma_step(1);
      }
    }
  } else {
    // Register-staged double buffering: the global loads of tile kt+1 fly during tile kt and are
    // written to the other LDS buffer before the hand-over barrier.
    static_assert(C::DIRECT || C::STAGES == 2, "register staging uses two buffers");
    u32x4 ra[TileLoader<C>::NA], rb[C::B_PER_WAVE];
    const int kbase = kt_begin * C::BK;
    auto load_tile = [&](int t) {
      const int tt = t < last ? t : last;
      ld.load_regs(Ak + (long)tt * a_step, Bk + (long)tt * b_step, kbase + tt * C::BK, p.K, ra, rb);
    };
    if (nkt > 0) {
      load_tile(0);
      ld.store_regs(smem, wave, lane, ra, rb);
      __syncthreads();
      load_tile(1);
      read_frags(smem, 0, 0);
      for (int kt = 0; kt < last; ++kt) {
        const char* cur = smem + (kt & 1) * C::STAGE_BYTES;
        char* nxt = smem + ((kt + 1) & 1) * C::STAGE_BYTES;
#pragma unroll
        for (int kk = 0; kk < C::KS - 1; ++kk) {
          read_frags(cur, kk + 1, (kk + 1) & 1);
          mfma_step(kk & 1);
          interleave_hint();
        }
        ld.store_regs(nxt, wave, lane, ra, rb);   // buffer last read in iteration kt-1, released by its barrier
        __syncthreads();
        load_tile(kt + 2);
        read_frags(nxt, 0, 0);
        mfma_step(1);
      }
      {
        const char* cur = smem + (last & 1) * C::STAGE_BYTES;
#pragma unroll
        for (int kk = 0; kk < C::KS - 1; ++kk) {
          read_frags(cur, kk + 1, (kk + 1) & 1);
          mfma_step(kk & 1);
          interleave_hint();
        }
        mfma_step(1);
      }
    }
  }

  // ---- accumulator layout. The MFMA is issued with the B fragment as its first operand and
  // the A fragment as its second, so each block is held transposed: lane l, register r
  // holds  m = block_m + l % MB,  n = block_n + 8 (r / 4) + 4 (l / MB) + (r % 4).
  // A lane therefore owns runs of four consecutive n, which pack into one 8-byte (bf16) or
  // 16-byte (fp32) store without any cross-lane exchange.
  int lane_out = lane;
  if constexpr (C::QUAD) {       // found anew: no register for it (or for tid) has to live through the main loop
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane_out));
    lane_out &= 63;              // (its range: without it the staged epilogue works out rows, columns and whether to store anew for
  }                              // every store: 2560 x 4096 x 256 14.6 us against 14.0, 4096^2 x 128 with fp32 results 19.0 / 18.6)
  const int tid_out = C::QUAD ? (wave & (C::NWAVES - 1)) * 64 + lane_out : tid;
  const int lane_m = lane_out % C::MB, lane_g = lane_out / C::MB;
  if constexpr (C::WK == 2) {
    static_assert(C::WK == 1 || C::MB == 32, "the exchange of the k groups: blocks of 32 x 32");
    // The two k groups hold partial sums of the same wave tile. Group 0 keeps its first TM/2 row
    // blocks and hands the others to its partner wave of group 1, which does the reverse;
    // afterwards acc[0 .. TM/2) of every wave holds complete sums of the rows it writes out.
    constexpr int H = C::TM / 2;
    wait_vmcnt<0>();
    barrier_lds();                          // nobody reads tiles any more, no transfer is in flight
    char* mine = smem + wave * (H * C::TN * 4096);
    const char* theirs = smem + ((wave_mn + (1 - wave_k) * C::WM * C::WN)) * (H * C::TN * 4096);
#pragma unroll
    for (int i = 0; i < H; ++i)
#pragma unroll
      for (int t = 0; t < C::TN; ++t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = wave_k ? acc[i][t][4 * q + e] : acc[i + H][t][4 * q + e];
          *(f32x4*)(mine + (((i * C::TN + t) * 4 + q) * 64 + lane) * 16) = v;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][t][r] = wave_k ? acc[i + H][t][r] : acc[i][t][r];
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < H; ++i)
#pragma unroll
      for (int t = 0; t < C::TN; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = *(const f32x4*)(theirs + (((i * C::TN + t) * 4 + q) * 64 + lane) * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i][t][4 * q + e] += v[e];
        }
  }
  const int wm0 = m0 + lane_m + (C::WK == 2 ? wave_k * (C::WTM / 2) : 0);   // + row_off
  const int wn0 = n0 + 4 * lane_g;                                          // + col_off + 8 q
  const int ncols = n_end - n0 < C::BN_ACT ? n_end - n0 : C::BN_ACT;     // columns this tile writes (a multiple of 8)
  const bool rows_full = m0 + C::BM <= p.M;
  const bool full = rows_full && ncols == C::BN_ACT;

  if (split) {
    // publish the partial tile; the last slice to arrive sums all slices in slice order
    const size_t slice = (size_t)p.M * p.N;
    float* wsk = p.ws + (size_t)tc.ks * slice;
    if (!C::FUSED_OK || !p.fused_reduce) {
      // two-kernel split-K: a reduce kernel launched behind this one sums the slices in slice order and applies the
      // epilogue (the kernel boundary orders the two). Whole tiles go out staged, past the L2s where p.ws_past_l2 says so;
      // ragged ones, and those of kernels that cannot stage floats (stage_ok), in ordinary stores
      if (C::stage_ok(4) && full && p.ws_vec16) {
        if constexpr (C::stage_ok(4))
          epilogue_staged<C, TF_EPI_NONE_F32, true>(acc, p, smem, m0, n0, tid_out, wave_m, wave_n, wave_k, lane_m, lane_g, (char*)wsk, (size_t)p.N);
      } else if (full) store_partial<C, true, false>(acc, wsk, p, wm0, wn0, wave_m, wave_n);
      else store_partial<C, false, false>(acc, wsk, p, wm0, wn0, wave_m, wave_n);
      continue;
    }
    if constexpr (C::FUSED_OK) {
    // Two ways to hand the partial tiles to the last slice:
    //  fused_reduce 1: device-scope (write-through) stores and loads, valid wherever the slices run;
    //  fused_reduce 2: plain stores and loads. The host offers it only when the tile order puts
    //    all slices of a tile on one XCD (work-group i runs on XCD i mod 8), whose L2 then holds
    //    the partial tiles: a store acknowledged by the L2 (vmcnt) is what any CU of the same XCD
    //    reads afterwards, and no CU has read these addresses earlier in the launch. Every slice
    //    reports the XCD it really ran on with its ticket; if they differ, the tile is poisoned
    //    with NaN rather than summed from memory that may be stale, and the status word of the
    //    workspace is set (the host probes the placement once per device before it launches this mode).
    const bool local = p.fused_reduce == 2;
    if (local) {
      if (full) store_partial<C, true, false>(acc, wsk, p, wm0, wn0, wave_m, wave_n);
      else store_partial<C, false, false>(acc, wsk, p, wm0, wn0, wave_m, wave_n);
    } else {
      if (full) store_partial<C, true, true>(acc, wsk, p, wm0, wn0, wave_m, wave_n);
      else store_partial<C, false, true>(acc, wsk, p, wm0, wn0, wave_m, wave_n);
    }
    // every store of this wave has been acknowledged before the wave reaches the barrier, so
    // the ticket taken after it is ordered behind the whole work-group's partials
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // ticket word: arrivals in bits 0..7, arrivals per XCD in 7-bit fields above
    __shared__ unsigned long long ticket;
    unsigned long long* ctr = (unsigned long long*)p.counters + (tc.tm * p.tiles_n + tc.tn);
    const unsigned xcc = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 7u;      // HW_REG_XCC_ID, bits 0..3
    const unsigned long long mine = 1ull + (1ull << (8 + 7 * xcc));
    // (the L2-local mode takes its ticket in this XCD's L2 as well: an atomic of narrower scope is carried out there,
    // one of device scope past it, at several times the latency; all slices of the tile sit on this XCD)
    if (tid_out == 0)
      ticket = (local ? __hip_atomic_fetch_add(ctr, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : atomicAdd(ctr, mine)) + mine;
    __syncthreads();
    const unsigned long long tk = ticket;
    if ((unsigned)(tk & 255u) != (unsigned)p.split_k) continue;
    if (tid_out == 0) *ctr = 0ull;        // ready for the next launch
    if (local) {
      if (full) sum_partials<C, true, false>(acc, p, wm0, wn0, wave_m, wave_n);
      else sum_partials<C, false, false>(acc, p, wm0, wn0, wave_m, wave_n);
      if ((unsigned)((tk >> (8 + 7 * xcc)) & 127u) != (unsigned)p.split_k) {
        if (tid_out == 0) atomicOr(p.status, 1u);   // reported by the next synchronous call of the library
        const float nan = __builtin_nanf("");
#pragma unroll
        for (int i = 0; i < C::TM_OUT; ++i)
#pragma unroll
          for (int t = 0; t < C::TN; ++t)
#pragma unroll
            for (int r = 0; r < 4 * C::QN; ++r) acc[i][t][r] = nan;
      }
    } else {
      if (full) sum_partials<C, true, true>(acc, p, wm0, wn0, wave_m, wave_n);
      else sum_partials<C, false, true>(acc, p, wm0, wn0, wave_m, wave_n);
    }
    }
  }

  // ---- epilogue: + bias, GELU, round to bf16 (or raw fp32 pre-activation)
  if (nkt <= 0) {            // no K step, so no hand-over has published the bias copy yet
    wait_vmcnt<0>();
    __syncthreads();
  }
  const char* bias_lds = smem + C::BIAS_OFF + 8 * lane_g;
  // whole rows of the tile go out coalesced through LDS, also when the tile's last columns do not exist or belong
  // to its neighbour (their pieces are skipped)
  const bool staged = rows_full && ncols > 0 && p.y_vec16;      // the same for every wave of the work-group
  auto finish = [&](auto tag) {
    constexpr int EPI = decltype(tag)::value;
    constexpr int ESZ = EPI == TF_EPI_NONE_F32 ? 4 : 2;
    if (C::stage_ok(ESZ) && staged) {
      if constexpr (C::stage_ok(ESZ))
        epilogue_staged<C, EPI>(acc, p, smem, m0, n0, tid_out, wave_m, wave_n, wave_k, lane_m, lane_g, (char*)p.Y, (size_t)p.ldy, ncols);
    } else if (full) epilogue<C, true, EPI>(acc, p, wm0, wn0, wave_m, wave_n, bias_lds, n_end);
    else epilogue<C, false, EPI>(acc, p, wm0, wn0, wave_m, wave_n, bias_lds, n_end);
  };
  if (p.epi == TF_EPI_BIAS_GELU_ERF) finish(EpiTag<TF_EPI_BIAS_GELU_ERF>{});
  else if (p.epi == TF_EPI_NONE_F32) finish(EpiTag<TF_EPI_NONE_F32>{});
  else if (p.epi == TF_EPI_BIAS) finish(EpiTag<TF_EPI_BIAS>{});
  else finish(EpiTag<TF_EPI_BIAS_GELU_TANH>{});
  }   // segments
}

template <class C>
__global__ void __launch_bounds__(C::THREADS) tf_gemm_lds_kernel(const GemmParams p) {
  gemm_tile_body<C>(p);
}

// The same kernel for a K that is no multiple of its K tile (1160 x 3080 x 1864: 34.0 us on the register-staged
// kernels, 22.7 us on the direct ones). An instance of its own, since it takes no rotated order of K: what it does beside costs where K
// is whole tiles about 1 % or nothing (us, the ordinary kernel / this: 4096 x 11008 x 4096 in tiles of 256 x 256 290.7 / 291.8, 192 x 256
// 308.5 / 312.1, 256 x 128 331.8 / 331.1; 4096^3 101.6 / 101.7; 3000 x 3000 x 2048 with B as [N][K] in 192 x 256 39.4 / 39.5; 2048^3 20.0 /
// 20.4; 64 x 64 tiles 1418 x 1152 x 1856 13.8 / 13.5, 700 x 1024^2 [N][K] 7.4 / 7.1). It was 1 to 3 % while the ragged tile was zeroed last.
template <class Base>
struct RaggedKCfg : Base {
  static_assert(Base::DIRECT && !Base::ABYPASS, "both operands staged directly");
  static constexpr bool KTAIL = true;
  // LINES: operands whose rows are contiguous along k are staged in whole 128-byte lines (see LineRows). One buffer more than
  // the pipeline needs otherwise: a K tile lies in two of them.
  static constexpr bool LINES = Base::STAGES >= 4 && Base::BM >= 64 && Base::BK == 64 && !Base::TRANSA && Base::WK == 1 && !Base::QUAD &&
                                Base::ACC * Base::KS * Base::KMF <= 8 * 16 * 16;
};

template <class C>
__global__ void __launch_bounds__(C::THREADS) tf_gemm_lds_ktail_kernel(const GemmParams p) {
  gemm_tile_body<RaggedKCfg<C>>(p);
}

// A launch with a lighter last round. Equal tiles leave the chip badly filled whenever the tile count is a little
// above a multiple of the CU count (688 tiles on 256 CUs: the third round runs on 176 of them). Here the first
// work-groups (whole rounds) compute BN-wide tiles over the leading columns, and one more round of exactly one
// work-group per CU shares out the remaining columns of every row panel in narrower tiles (CN: the same staging,
// fewer columns multiplied): every CU gets the same number of tiles and nearly the same work. Work-groups are
// handed to the CUs in id order, so the narrow round comes last.
template <class CM, class CN>
__global__ void __launch_bounds__(CM::THREADS) tf_gemm_mixed_kernel(const GemmParams p) {
  static_assert(CM::THREADS == CN::THREADS && CM::LDS_BYTES == CN::LDS_BYTES && CM::BM == CN::BM && CM::BN == CN::BN &&
                CM::BK == CN::BK && CN::BN_ACT < CN::BN, "the two tile shapes share the work-group shape and the staging");
  if ((int)blockIdx.x < p.mix_main_wgs) gemm_tile_body<CM>(p);
  else gemm_tile_body<CN>(p);
}

// Persistent kernel for the batched transposed-operand product with few K steps per tile
// (C[b] = A[b]^T B[b]). With four K steps a work-group spends most of its life waiting for
// its first tiles and for the end of its stores; here one work-group per CU walks through many output tiles
// and the ring never drains: the transfers of the next tile's K steps are issued while the current tile still
// multiplies and writes out. The output goes through a staging area of its own behind the ring, so the ring
// stays free for those transfers.
//   * work-group w runs on XCD w mod 8; XCD x takes the batch items x, x + 8, ..., so an item's operands are
//     fetched into one L2; the work-groups of an XCD deal that XCD's tiles out among themselves in turn.
//   * RAGGED (M or N no multiple of the tile, but at least one tile; or the batch no multiple of eight): an XCD takes
//     an eighth of the tiles of all items, in item order, instead; the last tile of a row or column of tiles begins at
//     M - BM or N - BN, so every transfer stays inside the item, and stores only what its neighbour does not.
//     An instance of its own: in one kernel for both, 32 x 1024 x 1024 x 256 went from 35.2 to 38.3 us. Against the
//     one-tile work-groups that had such sizes to themselves, tile picked / best tile / here (us): 48 x 568 x 896 x
//     128 37.0 / 28.3 / 22.2, 57 x 880 x 288 x 64 26.3 / 21.0 / 14.4, 27 x 320 x 848 x 256 23.2 / 16.6 / 14.1,
//     64 x 264 x 392 x 512 30.5 / 22.6 / 22.1. Items of many tiles: 32 x 1000 x 1000 x 192 54.3 / 37.7 / 38.4,
//     K = 256 56.3 / 39.8 / 41.9, K = 512 93.1 / 54.7 / 71.2, K = 1024 155.0 / 82.8 / 114.9 - tiles of 256 x 256 are
//     faster there from K = 320 on, and of whole tiles from K = 384 on (tf_predict_us does not see that yet).
//   * one "flat step" = one K step of one tile. At flat step f the transfers of step f + D (D = STAGES - 1)
//     are issued into the buffer that step f - 1 has just left. Past the end the last step is fetched again
//     (into a buffer nobody reads), which keeps the number of transfers in flight, and so the vmcnt waits,
//     constant.
//   * vector-memory operations of a wave complete in issue order, stores included, so a transfer issued
//     behind a tile's stores would only count as landed once those stores (a trip to memory) are done. The
//     waves therefore split the memory work: the first half of the waves issue all transfers into the ring,
//     the second half all stores of the output; every wave multiplies.
//   * tried and dropped: setting the finished tile's accumulators aside and writing them out pass by pass
//     during the next tile's first K steps (T2: 48 us against 42 us, also with the waves split as above: the
//     second barrier in the middle of a step costs more than the overlap gains), and a fourth buffer with
//     half-size output passes (43 us against 39 us).
template <class C, bool RAGGED>
__device__ __forceinline__ void bgemm_persist_body(const GemmParams& p) {
  static_assert(C::TRANSA && !C::TRANSB && C::DIRECT && C::WK == 1 && !C::ABYPASS && C::STAGES >= 3, "transposed staging, direct, three buffers or more");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  constexpr int D = C::STAGES - 1;
  // the loading half of the waves moves the tiles exactly as a work-group of half as many wave columns would
  static_assert(C::WN % 2 == 0, "an even number of wave columns");
  using CL = LdsCfg<C::BM, C::BN, C::BK, C::WM, C::WN / 2, C::STAGES, true, false, 1, true>;
  constexpr int LW = CL::NWAVES, STORE_THREADS = C::THREADS - LW * 64;
  static_assert(CL::STAGE_BYTES == C::STAGE_BYTES && CL::A_BYTES == C::A_BYTES, "same ring layout");
  constexpr int PER_TILE = CL::A_PER_WAVE + CL::B_PER_WAVE;
  constexpr int ROWB = C::BN * 4 + 16, CPR = C::BN * 4 / 16;
  constexpr int PER_THREAD = C::ST_ROWS * CPR / STORE_THREADS;
  static_assert(C::ST_ROWS * CPR % STORE_THREADS == 0, "pieces divide over the storing threads");
  static_assert((D - 1) * PER_TILE < 64, "vmcnt range");
  static_assert(C::PERSIST_LDS_BYTES <= 160 * 1024, "LDS budget of one CU");
  char* const staging = smem + C::RING_BYTES;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_m = wave / C::WN, wave_n = wave % C::WN;
  const int lane_m = lane & 31, lane_g = lane >> 5;

  // ---- this work-group's tiles
  const int tiles = p.tiles_m * p.tiles_n;                       // per batch item
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, per_xcd = gridDim.x >> 3;
  const long all = (long)p.batch * tiles;
  const int items_x = (p.batch - xcd + 7) / 8;                   // items x, x + 8, ... < batch
  const int first = RAGGED ? (int)(xcd * all / 8) : 0;
  const int n_flat = RAGGED ? (int)((xcd + 1) * all / 8) - first : items_x * tiles;
  const int my_tiles = local < n_flat ? (n_flat - local + per_xcd - 1) / per_xcd : 0;
  const int nkt = p.K / C::BK;
  const int total = my_tiles * nkt;
  if (total <= 0) return;
  struct Where { const uint16_t* a; const uint16_t* b; char* y; int m0, n0, skip_m, skip_n; };    // skip_: leading rows and columns that are the neighbour's
  auto where = [&](int k) -> Where {                               // k-th tile of this work-group
    const int j = first + local + k * per_xcd;
    const int item = RAGGED ? j / tiles : xcd + 8 * (j / tiles), tile = j % tiles;
    const int m_own = (tile % p.tiles_m) * C::BM, n_own = (tile / p.tiles_m) * C::BN;
    Where w;
    w.m0 = !RAGGED || m_own + C::BM <= p.M ? m_own : p.M - C::BM;
    w.n0 = !RAGGED || n_own + C::BN <= p.N ? n_own : p.N - C::BN;
    w.skip_m = m_own - w.m0; w.skip_n = n_own - w.n0;
    w.a = p.A + (size_t)item * p.stride_a + w.m0;                  // A[b] is [K][lda], m contiguous
    w.b = p.B + (size_t)item * p.stride_b + w.n0;
    w.y = (char*)p.Y + (size_t)item * p.stride_y * 4;
    return w;
  };

  // ---- LDS read offsets of this lane (bytes inside a stage), as in tf_gemm_lds_kernel
  int a_toff[C::TM], b_off[C::TN];
  {
    const int b = lane >> 4, s = lane & 15;
    const int krow = 8 * (b >> 1) + (s >> 2);
    const int within = (16 * (b & 1) + 4 * (s & 3)) * 2;
#pragma unroll
    for (int i = 0; i < C::TM; ++i) {
      const int j = (wave_m * C::WTM) / 32 + i;
      a_toff[i] = krow * C::A_ROW_BYTES + (j ^ b_swz<C::A_PIECES>(krow)) * 64 + within;
    }
#pragma unroll
    for (int t = 0; t < C::TN; ++t) {
      const int j = (wave_n * C::WTN) / 32 + t;
      b_off[t] = C::A_BYTES + krow * C::B_ROW_BYTES + (j ^ b_swz<C::B_PIECES>(krow)) * 64 + within;
    }
  }
  auto read_tr = [&](const char* ptr, int row_bytes) -> bf16x8 {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(ptr));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(ptr + 4 * row_bytes));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };

  f32x16 acc[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int t = 0; t < C::TN; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][t][r] = 0.0f;

  const bool loader = wave < LW;                 // wave-uniform
  TileLoader<CL> ld;
  ld.init(p, 0, 0, loader ? wave : 0, lane);     // offsets relative to the tile's corner
  const unsigned lds0 = (unsigned)(size_t)smem;
  const size_t a_step = (size_t)C::BK * p.lda, b_step = (size_t)C::BK * p.ldb;

  // the loader runs D flat steps ahead of the multiplier
  int l_tile = 0, l_kt = 0, l_stage = 0;
  Where lw = where(0);
  auto issue_next = [&]() {
    if (loader) ld.issue_direct(lw.a + (size_t)l_kt * a_step, lw.b + (size_t)l_kt * b_step, lds0 + l_stage * C::STAGE_BYTES, wave);
    if (++l_stage == C::STAGES) l_stage = 0;
    if (l_tile * nkt + l_kt + 1 < total) {       // else: stay on the last step (fetched again, never read)
      if (++l_kt == nkt) { l_kt = 0; ++l_tile; lw = where(l_tile); }
    }
  };
#pragma unroll
  for (int s = 0; s < D; ++s) issue_next();

  int c_tile = 0, c_kt = 0, c_stage = 0;
  Where cw = where(0);
  for (int f = 0; f < total; ++f) {
    if (loader) wait_vmcnt<(D - 1) * PER_TILE>();   // this wave's transfers of step f have landed (it issues nothing else)
    barrier_lds();                 // step f has landed for every wave; every wave has left the buffer of step f - 1
    issue_next();                  // step f + D into that buffer
    const char* cur = smem + c_stage * C::STAGE_BYTES;
#pragma unroll
    for (int kk = 0; kk < C::KSTEPS; ++kk) {
      bf16x8 af[C::TM], bfr[C::TN];
#pragma unroll
      for (int i = 0; i < C::TM; ++i) af[i] = read_tr(cur + a_toff[i] + (16 * kk) * C::A_ROW_BYTES, C::A_ROW_BYTES);
#pragma unroll
      for (int t = 0; t < C::TN; ++t) bfr[t] = read_tr(cur + b_off[t] + (16 * kk) * C::B_ROW_BYTES, C::B_ROW_BYTES);
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int t = 0; t < C::TN; ++t)
          acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[t], af[i], acc[i][t], 0, 0, 0);
    }
    if (++c_stage == C::STAGES) c_stage = 0;
    if (++c_kt == nkt) {
      // ---- the tile is complete: out through the staging area, 32 rows per wave row at a time
      char* wr = staging + (wave_m * 32 + lane_m) * ROWB + (wave_n * C::WTN + 4 * lane_g) * 4;
#pragma unroll
      for (int i = 0; i < C::TM; ++i) {
        if (i) barrier_lds();      // the previous pass has been read back
#pragma unroll
        for (int t = 0; t < C::TN; ++t)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = {acc[i][t][4 * q], acc[i][t][4 * q + 1], acc[i][t][4 * q + 2], acc[i][t][4 * q + 3]};
            *(f32x4*)(wr + (32 * t + 8 * q) * 4) = v;
          }
        barrier_lds();
        auto put = [&](bool ragged) {
#pragma unroll
          for (int j = 0; j < PER_THREAD; ++j) {
            const int c = (tid - LW * 64) + STORE_THREADS * j;
            const int rs = c / CPR, cc = c % CPR;
            const int r = (rs >> 5) * C::WTM + 32 * i + (rs & 31), m = cw.m0 + r;
            const u32x4 v = *(const u32x4*)(staging + rs * ROWB + cc * 16);
            if (!ragged || (r >= cw.skip_m && 4 * cc >= cw.skip_n))
              __builtin_nontemporal_store(v, (u32x4*)(cw.y + ((size_t)m * p.ldy + cw.n0) * 4 + cc * 16));
          }
        };
        // (a branch of its own for whole tiles: with the test at every store the LDS reads no longer run ahead)
        if (!loader) {
          if (!RAGGED || (cw.skip_m == 0 && cw.skip_n == 0)) put(false);
          else put(true);
        }
      }
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int t = 0; t < C::TN; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][t][r] = 0.0f;
      c_kt = 0; ++c_tile;
      if (c_tile < my_tiles) cw = where(c_tile);
    }
  }
  wait_vmcnt<0>();                 // no transfer may still be on its way into this work-group's LDS when it ends
}

template <class C>
__global__ void __launch_bounds__(C::THREADS) tf_bgemm_persist_kernel(const GemmParams p) {
  bgemm_persist_body<C, false>(p);
}
template <class C>
__global__ void __launch_bounds__(C::THREADS) tf_bgemm_persist_ragged_kernel(const GemmParams p) {
  bgemm_persist_body<C, true>(p);
}

template <class C>
static void launch_persist(const GemmParams& p, dim3 grid, hipStream_t stream) {
  hipLaunchKernelGGL(tf_bgemm_persist_kernel<C>, grid, dim3(C::THREADS), C::PERSIST_LDS_BYTES, stream, p);
}
template <class C>
static void launch_persist_ragged(const GemmParams& p, dim3 grid, hipStream_t stream) {
  hipLaunchKernelGGL(tf_bgemm_persist_ragged_kernel<C>, grid, dim3(C::THREADS), C::PERSIST_LDS_BYTES, stream, p);
}

template <class C>
static LdsKernelInfo make_persist_info();

template <class C>
static void launch_lds(const GemmParams& p, dim3 grid, hipStream_t stream) {
  hipLaunchKernelGGL(tf_gemm_lds_kernel<C>, grid, dim3(C::THREADS), C::LDS_BYTES, stream, p);
}
template <class CM, class CN>
static void launch_mixed(const GemmParams& p, dim3 grid, hipStream_t stream) {
  hipLaunchKernelGGL((tf_gemm_mixed_kernel<CM, CN>), grid, dim3(CM::THREADS), CM::LDS_BYTES, stream, p);
}

// The same kernel with the loop over segments compiled in: work-groups may take several (tile, K range) pieces.
template <class Base>
struct StreamKCfg : Base { static constexpr bool SEGMENTS = true; };

template <class C>
static LdsKernelInfo describe() {
  LdsKernelInfo k{};
  k.bm = C::BM; k.bn = C::BN; k.bk = C::BK; k.waves_m = C::WM; k.waves_n = C::WN; k.waves_k = C::WK;
  k.stages = C::STAGES; k.direct_to_lds = C::DIRECT ? 1 : 0; k.a_bypass_lds = C::ABYPASS ? 1 : 0; k.trans_a = C::TRANSA ? 1 : 0;
  k.trans_b = C::TRANSB ? 1 : 0;
  k.threads = C::THREADS; k.lds_bytes = C::LDS_BYTES; k.fused_ok = C::FUSED_OK ? 1 : 0;
  k.persistent = 0; k.stream_k = C::SEGMENTS ? 1 : 0; k.bn_tail = 0; k.k_tail = 0; k.lines = 0;
  return k;
}
template <class C>
static LdsKernelInfo make_info() {
  LdsKernelInfo k = describe<C>();
  k.func = (const void*)tf_gemm_lds_kernel<C>;
  k.launch = launch_lds<C>;
  return k;
}

template <class C>
static void launch_lds_ragged(const GemmParams& p, dim3 grid, hipStream_t stream) {
  hipLaunchKernelGGL(tf_gemm_lds_ktail_kernel<C>, grid, dim3(C::THREADS), C::LDS_BYTES, stream, p);
}
template <class C>
static LdsKernelInfo make_ragged_info() {
  LdsKernelInfo k = describe<C>();
  k.k_tail = 1; k.lines = RaggedKCfg<C>::LINES ? 1 : 0;
  k.func = (const void*)tf_gemm_lds_ktail_kernel<C>;
  k.launch = launch_lds_ragged<C>;
  return k;
}

template <class CM, class CN>
static LdsKernelInfo make_mixed_info() {
  LdsKernelInfo k = make_info<CM>();
  k.bn_tail = CN::BN_ACT;
  k.func = (const void*)tf_gemm_mixed_kernel<CM, CN>;
  k.launch = launch_mixed<CM, CN>;
  return k;
}

template <class C>
static LdsKernelInfo make_persist_info() {
  LdsKernelInfo k = make_info<C>();
  k.persistent = 1;
  k.lds_bytes = C::PERSIST_LDS_BYTES;
  k.func = (const void*)tf_bgemm_persist_kernel<C>;
  k.launch = launch_persist<C>;
  return k;
}
template <class C>
static LdsKernelInfo make_persist_ragged_info() {
  LdsKernelInfo k = describe<C>();
  k.persistent = 1; k.ragged_mn = 1;
  k.lds_bytes = C::PERSIST_LDS_BYTES;
  k.func = (const void*)tf_bgemm_persist_ragged_kernel<C>;
  k.launch = launch_persist_ragged<C>;
  return k;
}

}  // namespace tf
