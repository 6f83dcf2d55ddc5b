// Host logic of the profiling-guided variant loop (paper Sec. 3.3, Algorithm 1).
// Pure functions of reports and descriptors: nothing here touches the GPU, so the loop can
// be tested on synthetic reports.
//
// The paper names the roles (Proposal, BuildRun, Profile, Arbiter, RefineHint), the
// Arbiter's criteria (speedup, robustness, resource limits, diminishing returns), two
// example hints (memory stalls -> tiling/staging, low occupancy -> register pressure), the
// 1.05x success bar (Sec. 4.2) and the cap of 8 rounds; it gives no threshold values and its
// Proposal / RefineHint are an LLM. Here both are rules over a finite kernel family.
#include <math.h>
#include <string.h>

#include "tf_loop.h"

extern "C" void tf_theta_default(tf_theta* t) {
  if (!t) return;
  t->first_accept_speedup = 1.05;  // the paper's success bar against the baseline kernel
  t->later_accept_gain = 1.02;     // a new best must beat the old best by more than timing noise
  t->robust_spread = 0.10;
  t->patience = 4;   // Case Study 3 runs four consecutive non-improving rounds before it stops
  t->max_rounds = 8;
  t->cold_bytes = 512ll << 20;
}

extern "C" void tf_hw_nominal(tf_hw* h) {
  if (!h) return;
  memset(h, 0, sizeof(*h));
  strncpy(h->name, "AMD Instinct MI355X (published figures)", sizeof(h->name) - 1);
  h->cus = 256; h->simds_per_cu = 4; h->wave_size = 64; h->xcds = 8;
  h->lds_bytes_per_cu = 160 * 1024; h->vgprs_per_simd_lane = 512; h->max_waves_per_simd = 8;
  h->l2_bytes = 4ll << 20; h->hbm_bytes = 288ll << 30;
  h->clock_mhz = 2400.0; h->hbm_gbs_peak = 8000.0;
  h->bf16_tflops_peak = 256 * 4096.0 * 2400.0e6 / 1e12;   // 2516.6
}

// ------------------------------------------------------------------ Arbiter
extern "C" int32_t tf_arbiter(const tf_report* cand, const tf_report* best, const tf_theta* th,
                              int32_t best_is_baseline, int32_t stall_rounds, int32_t round) {
  if (!cand || !best || !th) return TF_DEC_FINISH;
  const bool usable = cand->status == TF_OK && cand->parity_ok != 0 && cand->t_med_us > 0.0 &&
                      best->t_med_us > 0.0;
  if (usable) {
    const double spread = (cand->t_med_us - cand->t_min_us) / cand->t_med_us;
    const double need = best_is_baseline ? th->first_accept_speedup : th->later_accept_gain;
    if (spread <= th->robust_spread && best->t_med_us / cand->t_med_us >= need) return TF_DEC_ACCEPT;
  }
  if (stall_rounds + 1 >= th->patience) return TF_DEC_FINISH;   // diminishing returns
  if (round >= th->max_rounds) return TF_DEC_FINISH;
  return TF_DEC_CONTINUE;
}

// ------------------------------------------------------------------ RefineHint
static int classify(const tf_report* r, const tf_hw* hw) {
  const double ridge = hw->bf16_tflops_peak * 1e3 / hw->hbm_gbs_peak;   // flop per byte
  const double mfma = r->have_counters ? r->mfma_busy_pct : r->pct_mfma_peak;
  const double hbm = r->have_counters ? 100.0 * (r->hbm_read_gbs + r->hbm_write_gbs) / hw->hbm_gbs_peak
                                      : r->pct_hbm_peak;
  if (r->grid_fill < 0.75) return TF_BN_UNDERFILLED;
  if (r->arithmetic_intensity < ridge && hbm >= 60.0) return TF_BN_HBM;
  if (mfma >= 70.0) return TF_BN_MFMA;
  if (r->have_counters && r->lds_bank_conflict_pct > 5.0) return TF_BN_LDS_CONFLICT;
  if (r->occupancy_pct < 25.0 && mfma < 50.0 && hbm < 50.0) return TF_BN_OCCUPANCY;
  return TF_BN_LATENCY;
}

extern "C" int32_t tf_refine_hint(const tf_report* prev, const tf_report* cand, const tf_hw* hw) {
  if (!cand || !hw) return TF_BN_UNKNOWN;
  if (cand->status != TF_OK || cand->t_med_us <= 0.0) return TF_BN_UNKNOWN;
  int c = classify(cand, hw);
  // The delta against the previous report: the candidate was proposed under the hint the previous report
  // carries (its bottleneck field; a report without one is read by its own figures). When that step made
  // things slower and the candidate's figures call for the same remedy again, the remedy has just failed:
  // swap between the two "nothing is saturated" diagnoses so that the next proposal goes the other way.
  // This reproduces the hints behind the rounds of Case Study 3 (Sec. 5): coalescing / staging, then lower
  // register use, then deeper pipelining, then less shared memory per work-group, each after a slower round.
  if (prev && prev->status == TF_OK && prev->t_med_us > 0.0 && cand->t_med_us > 1.02 * prev->t_med_us) {
    const int followed = prev->bottleneck != TF_BN_UNKNOWN ? prev->bottleneck : classify(prev, hw);
    if (followed == c) {
      if (c == TF_BN_OCCUPANCY) c = TF_BN_LATENCY;
      else if (c == TF_BN_LATENCY) c = TF_BN_OCCUPANCY;
    }
  }
  return c;
}

// ------------------------------------------------------------------ static cost model
static inline long cdiv(long a, long b) { return (a + b - 1) / b; }
static inline int at_least(int least, int x) { return x < least ? least : x; }      // (a caller's descriptor may hold anything)
static inline bool is_tile_kernel(const tf_variant_desc* v) { return v->kind == TF_KIND_MFMA_LDS || (v->kind == TF_KIND_MFMA_LDS_ANY && !tf::is_kshare(v)); }

extern "C" int32_t tf_resident_wgs(const tf_hw* hw, const tf_variant_desc* v) {
  if (v->kind == TF_KIND_MFMA_STREAM) {
    // about 128 registers per lane: four waves per SIMD; LDS only holds the final exchange
    const int waves = v->waves_k > 0 ? v->waves_k : 1;
    int r = 4 * hw->simds_per_cu / waves;
    const int by_lds = v->lds_bytes > 0 ? hw->lds_bytes_per_cu / v->lds_bytes : 8;
    if (by_lds < r) r = by_lds;
    return r < 1 ? 1 : (r > 8 ? 8 : r);
  }
  if (tf::is_kshare(v)) {
    int r = v->lds_bytes > 0 ? hw->lds_bytes_per_cu / (v->lds_bytes + 64) : 8;
    const int by_waves = hw->simds_per_cu * hw->max_waves_per_simd / at_least(1, v->waves_k);
    if (by_waves < r) r = by_waves;
    return r < 1 ? 1 : (r > 8 ? 8 : r);
  }
  if (!is_tile_kernel(v)) return 8;
  const int acc_regs = (v->bm / v->waves_m) * (v->bn / v->waves_n) / 64;
  const int regs = acc_regs + 96;                      // fragments, staging, addresses
  int wps = hw->vgprs_per_simd_lane / regs;
  if (wps < 1) wps = 1;
  if (wps > hw->max_waves_per_simd) wps = hw->max_waves_per_simd;
  const int wg_waves = v->waves_m * v->waves_n * (v->waves_k > 1 ? v->waves_k : 1);
  int by_regs = wps * hw->simds_per_cu / wg_waves;
  if (by_regs < 1) by_regs = 1;
  int by_lds = v->lds_bytes > 0 ? hw->lds_bytes_per_cu / v->lds_bytes : 8;
  if (by_lds < 1) by_lds = 1;
  int r = by_regs < by_lds ? by_regs : by_lds;
  return r > 8 ? 8 : r;
}

extern "C" double tf_grid_fill(const tf_hw* hw, const tf_variant_desc* v) {
  const long slots = (long)hw->cus * tf_resident_wgs(hw, v);
  if (v->grid <= 0) return 0.0;
  return (double)v->grid / (double)(cdiv(v->grid, slots) * slots);
}

// The shape of a launch whose waves share K, and its predicted time. Without slices the tiles are cut to what suits the problem,
// whatever the kernel's largest is: as many tiles as there are CUs, no more rows of A than the problem has, the rest shared out
// evenly (us, the pick in whole tiles / the cut: 8 x 2048 x 7432 with B as [N][K] in 64 tiles of 32 x 32 15.2, in 256 of 8 x 8 8.7;
// 32 x 2576 x 2856 [N][K] 9.7 / 7.1; 12 x 1552 x 5352 [N][K] 10.4 / 6.8; 5 x 11008 x 4096 [N][K] 19.1 / 17.5; 30 x 2048 x 4920 in 64
// tiles of 32 x 32 15.9, in 256 of 8 x 32 11.4; 368 x 1408 x 2240 [N][K] 10.9 / 9.5). Not the tiles of 32 x 32, whose four waves have
// nothing to hide the cut kernel's tests behind (12 x 1552 x 5352 10.7 whole, 12.1 cut), and no slices, which fill the chip by
// themselves: over 147 problems, what is left out was 0.6 % faster where it was the best.
//   * A wave's ring takes a second K tile where the work-groups of a CU have no more than 40 KB in flight without (the second
//     gains 17 % at 16 KB, 8 % at 32, 4 % at 40, nothing from 48 KB on, and a third gains nothing).
//   * The time: fitted (log error, 9 % rms within 1.25 times the best) to 3400 timings of these kernels on 147 problems, operands
//     of several calls in turn. A CU fetches k-contiguous rows at 106 GB/s and rows of a [K][N] B at 94 in pieces of 128 bytes, 73
//     in pieces of 64, less by a half where rows start off 128-byte lines; a wave takes 0.09 us for a K tile and every 32 x 32
//     outputs, 0.11 more in cut tiles, which start 0.4 us later; the L2s together fetch 6.2 TB/s; the three overlap. The
//     variant and shape predicted to be the fastest is 2.4 % behind the fastest of all.
//   * Shapes that cannot be the fastest are left before the overlap is worked out, and what has no cut is priced once: 64 shapes of four
//     powers each, twice for every variant, took half of a small problem's proposal (79 x 256 x 11448 with B as [N][K] 24 us, now 13; 32 x 2576 x 2856
//     [N][K] 10 and 7; without any cuts 8 and 5).
struct KsharePricer {
  const tf_problem_desc* pr;
  const tf_hw* hw;
  const tf_variant_desc* v;
  int nw, max_a, max_b, sums;
  long nkt;
  double off_a, off_b, rate_b;
  KsharePricer(const tf_problem_desc* pr_, const tf_hw* hw_, const tf_variant_desc* v_) : pr(pr_), hw(hw_), v(v_) {
    nw = at_least(1, v->waves_k); max_a = at_least(1, v->bm / 8); max_b = at_least(1, v->bn / 8); sums = v->bm * v->bn * 4;
    nkt = cdiv(pr->K, 64);
    off_a = pr->lda % 64 ? 1.47 : 1.0; off_b = pr->ldb % 64 ? 1.47 : 1.0;
    rate_b = pr->trans_b ? 105.6e3 : v->bn > 32 ? 93.6e3 : 73.4e3;
  }
  // The launch in tiles of ga x gb eights, or groups_a = 0 if there is none or it takes `bound` or longer.
  tf::KshareShape price(int ga, int gb, bool whole, double bound) const {
    const long tm = cdiv(pr->M, 8 * ga), tn = cdiv(pr->N, 8 * gb), tiles = tm * tn;
    const double load = (double)tiles / hw->cus, on_cu = fmax(1.0, ceil(load - 1e-9));
    const int stages = whole ? v->stages : v->bm <= 32 && nw * (ga + gb) * on_cu <= tf::KSHARE_TWO_TILES_KB && nkt > nw ? 2 : 1;
    const int ring = stages * (ga + gb) * 1024 > sums ? stages * (ga + gb) * 1024 : sums;
    const int lds = nw * ring + (whole ? 0 : tf::KSHARE_CUT_MARK);
    if (!whole && lds > hw->lds_bytes_per_cu) return {};
    const int by_lds = hw->lds_bytes_per_cu / (lds + 64), by_waves = hw->simds_per_cu * hw->max_waves_per_simd / nw;
    const double res = fmax(1.0, by_lds < by_waves ? by_lds : by_waves), rounds = fmax(1.0, ceil(load / res - 1e-9));
    const double at_once = fmin(on_cu, res);
    const double fetch = nkt * on_cu * (ga * 1024.0 * off_a / 105.6e3 + gb * 1024.0 * off_b / rate_b);
    const double serial = rounds * cdiv(nkt, nw) * ((whole ? 0.0 : 0.108) + 0.088 * v->bm * v->bn / 1024.0 * at_once * nw / 8.0);
    // an XCD's run of neighbouring tiles, in columns of group_m
    const double run = tiles / 8.0, gm = tm < 8 ? (double)tm : 8.0;
    const double rows = fmin((double)tm, run < gm ? fmax(1.0, run) : gm * fmax(1.0, ceil(run / (gm * tn)))), cols = fmin((double)tn, fmax(1.0, run / gm));
    const double fabric = fmax(8.0 * (rows * ga + cols * gb) * 1024.0 * nkt, 2.0 * ((double)pr->M * pr->K + (double)pr->K * pr->N)) / 6.24e6;
    const double start = 3.03 + (whole ? 0.0 : 0.4) - (nw == 4 ? 0.15 : 0.0) + (v->bm == 64 ? 0.71 : 0.0) + 0.068 * nw * at_once / 16.0;
    // (the three overlap to no less than the longest)
    if (start + fmax(fmax(fetch, serial), fabric) + 2.55 * (rounds - 1.0) > bound * (1.0 + 1e-9)) return {};
    const double us = start + pow(pow(fetch, 2.29) + pow(serial, 2.29) + pow(fabric, 2.29), 1.0 / 2.29) + 2.55 * (rounds - 1.0);
    if (bound != INFINITY && !(us < bound)) return {};
    return tf::KshareShape{ga, gb, stages, tm, tn, lds, us, 0.0, false};
  }
  // Tiles of the kernel's own size, if it has them.
  tf::KshareShape whole() const {
    return 8 * max_a == v->bm && 8 * max_b == v->bn && v->bm >= 32 ? price(max_a, max_b, true, INFINITY) : tf::KshareShape{};
  }
};

tf::KshareShape tf::kshare_shape(const tf_problem_desc* pr, const tf_hw* hw, const tf_variant_desc* v) {
  const KsharePricer k(pr, hw, v);
  const KshareShape all = k.whole();
  KshareShape cut{};
  if (v->split_k == 1 && !(v->bm == 32 && v->bn == 32)) {
    double bound = INFINITY;
    for (int ga = 1; ga <= k.max_a; ++ga) {
      const long tm = cdiv(pr->M, 8 * ga);
      if (ga > 1 && ga < k.max_a && cdiv(pr->M, 8 * (ga - 1)) == tm) continue;                  // fewer rows make as many tiles
      for (int gb = pr->trans_b ? 1 : k.max_b; gb <= k.max_b; ++gb) {
        const long tn = cdiv(pr->N, 8 * gb);
        if (tm * tn > hw->cus || (gb > 1 && pr->trans_b && cdiv(pr->N, 8 * (gb - 1)) == tn)) continue;
        if (all.groups_a == ga && all.groups_b == gb) continue;
        const KshareShape one = k.price(ga, gb, false, bound);
        if (one.groups_a != 0) { cut = one; bound = one.us; }
      }
    }
  }
  const bool is_cut = cut.groups_a != 0 && (all.groups_a == 0 || cut.us < 0.97 * all.us);
  KshareShape best = is_cut ? cut : all;
  best.is_cut = is_cut;
  best.whole_us = all.us;
  return best;
}

// A launch of whole tiles.
static double kshare_whole_us(const tf_problem_desc* pr, const tf_hw* hw, const tf_variant_desc* v) {
  // Fitted (log error, 12 % rms) to 893 timings of these kernels on 176 problems from 1 x 4096 x 11008 to 2965 x 1104 x 2224
  // (13 % rms over three thousand timings on 700 others), when these kernels ran MFMAs of 32 x 32 x 16. (With those of 16 x 16 x 32 they take 0.98
  // of the time in the mean. On 130 problems of any size 292 launches in slices are within 11 % rms; 211 without are predicted 12 % low, 19 % rms.)
  // A CU fetches the panels of its tiles at 76 to 101 GB/s (rows of 32 columns of a [K][N] B are half a 128-byte line), the
  // L2s together what their tiles need at 7.4 TB/s (the two overlap in part), a launch takes 2.9 us and a further round of
  // work-groups costs 2.3 beside its bytes.
  const int s = at_least(1, v->split_k), lds_whole = v->waves_k * v->stages * (v->bm + v->bn) * 128;
  const int res = fmax(1.0, fmin(8.0, hw->lds_bytes_per_cu / at_least(1, lds_whole)));
  const long tm = cdiv(pr->M, at_least(1, v->bm)), tn = cdiv(pr->N, at_least(1, v->bn)), nkt = cdiv(pr->K, 64);
  const double load = (double)(tm * tn * s) / hw->cus;
  const double rate = v->bm > 32 ? 76.3e3 : v->bn > 32 ? 96.4e3 : pr->trans_b ? 101.2e3 : 89.7e3;
  const double fetch = (v->bm + v->bn) * 128.0 * cdiv(nkt, s) * fmax(1.0, ceil(load - 1e-9)) / rate;
  // an XCD's run of neighbouring tiles (8 / s XCDs share the tiles of a slice), in columns of group_m
  const double run = (double)(tm * tn) / (s >= 8 ? 1 : 8 / s), gm = v->group_m > 0 ? v->group_m : 1;
  const double rows = fmin((double)tm, run < gm ? fmax(1.0, run) : gm * fmax(1.0, ceil(run / (gm * tn)))), cols = fmin((double)tn, fmax(1.0, run / gm));
  const double fabric = fmax(8.0 * (rows * v->bm + cols * v->bn) * 128.0 * nkt / (s < 8 ? s : 8), 2.0 * ((double)pr->M * pr->K + (double)pr->K * pr->N)) / 7.35e6;
  double us = 2.9 + pow(pow(fetch, 1.55) + pow(fabric, 1.55), 1.0 / 1.55) + 2.3 * fmax(0.0, ceil(load / res - 1e-9) - 1.0);
  // slices: the acknowledgement of the partial tile, the ticket, the other slices' tiles
  const double tile_bytes = v->bm * (double)v->bn * 4.0;
  if (s > 1) us += 1.45 + 1.16e-5 * s * tile_bytes + 6.1e-7 * load * hw->cus * tile_bytes;
  return us;
}

double tf::base_predict_us(const tf_problem_desc* pr, const tf_hw* hw, const tf_variant_desc* v) {
  const double flops = 2.0 * pr->M * (double)pr->N * pr->K;
  const double bytes = 2.0 * ((double)pr->M * pr->K + (double)pr->K * pr->N + (double)pr->M * pr->N + pr->N);
  const double hbm_us = bytes / (hw->hbm_gbs_peak * 1e3);
  if (v->kind == TF_KIND_SIN) {
    // 8 bytes per element through HBM; a work-group costs about 0.45 us of one of the CU's slots to start and
    // retire whatever it does (few elements per work-group: that is all there is), and one- or two-element
    // accesses per lane reach about half the rate of 16-byte ones
    const double floor_us = 8.0 * (double)pr->N / (0.75 * hw->hbm_gbs_peak * 1e3);
    const double wg_us = (double)v->grid * 0.45 / ((double)hw->cus * 8.0);
    const double width = v->bk >= 4 ? 1.0 : (v->bk == 2 ? 0.9 : 0.55);
    // many passes per work-group hold many registers and leave few waves per SIMD; a grid-stride launch of
    // few work-groups loses the hardware's own balancing of the tail
    const double shape = 1.0 + 0.02 * (v->stages - 1) + (v->group_m ? 0.03 : 0.0) - (v->nontemporal ? 0.01 : 0.0);
    return fmax(floor_us / width * shape, wg_us) + 3.0;
  }
  if (pr->op == TF_OP_BATCHED_GEMM_TN) {
    // C[b] = A[b]^T B[b]: the tile model on one item with the whole grid, an HBM floor that counts the
    // fp32 output, and the transposing pass where the variant has one
    const double items = pr->batch > 0 ? (double)pr->batch : 1.0;
    const double tbytes = items * (2.0 * (double)pr->K * ((double)pr->M + pr->N) + 4.0 * (double)pr->M * pr->N);
    const double floor_us = tbytes / (0.75 * hw->hbm_gbs_peak * 1e3);
    if (v->kind == TF_KIND_BGEMM_TN_NAIVE) return items * 2.0 * pr->M * (double)pr->N * pr->K / (0.004 * hw->bf16_tflops_peak * 1e6) + 3.0;
    tf_problem_desc one = *pr;
    one.op = TF_OP_GEMM_EPILOGUE;
    tf_variant_desc v1 = *v;
    v1.trans_a = 0;
    if (v->persistent) {
      // one work-group per CU walks through the tiles and never lets its ring drain: the tile model over all
      // tiles, without the start-up that every work-group of the plain kernels pays. (Right up to four or five K
      // steps, 32 x 1024 x 1024 x 256 32 predicted, 35.2 us measured; with more of them it takes up to 1.5 times as
      // long, 16 x 2048 x 2048 x 2048 251 predicted, 380 us, where 256 x 256 tiles take 282. The 128 x 128 tiles that
      // would be the pick without it are slower still, 449 us, and so for ragged sizes: 16 x 2000 x 2000 x 2048 504
      // against 417 us.)
      v1.persistent = 0;
      v1.xcd_swizzle = 1;
      v1.grid = (int32_t)(((pr->M + v->bm - 1) / v->bm) * (long)((pr->N + v->bn - 1) / v->bn) * (long)items);
      // (dealt out as whole items, eight XCDs wait for the ones with the most)
      const double share = v->xcd_swizzle ? 8.0 * cdiv((long)items, 8) / items : 1.0;
      return fmax(0.8 * tf::base_predict_us(&one, hw, &v1), floor_us + 4.0) * share;
    }
    // (a work-group of the plain kernels reads, multiplies and then writes, and the chip's reads and writes overlap
    // less for it: 32 x 1024 x 1024 x 256, 168 MB, takes 44.7-52.2 us in their tiles, 34.9 us in the persistent kernel)
    double us = fmax(tf::base_predict_us(&one, hw, &v1), 1.4 * floor_us + 4.0);
    // with few K steps per tile a work-group is a short read - multiply - write sequence; alone on its CU
    // it leaves memory idle while it multiplies and the matrix pipes idle while it writes (measured 1.4-1.6x)
    const long slots_one = (long)hw->cus * tf_resident_wgs(hw, v);
    long co = cdiv(v->grid, hw->cus);
    if (co > slots_one / hw->cus) co = slots_one / hw->cus;
    if (co < 2) us *= 1.5;
    if (!v->trans_a) us += 3.0 + items * 4.0 * (double)pr->K * pr->M / (0.6 * hw->hbm_gbs_peak * 1e3);
    return us;
  }
  if (v->kind == TF_KIND_VECMAT_NAIVE || v->kind == TF_KIND_VECMAT_STREAM) {
    // C[m][n] = sum_k A[m][k] B[m][n][k]: B is read once; everything else is small
    const double vbytes = 2.0 * ((double)pr->M * pr->K + (double)pr->M * pr->N * pr->K) + 4.0 * (double)pr->M * pr->N;
    const double floor_us = vbytes / (hw->hbm_gbs_peak * 1e3);
    if (v->kind == TF_KIND_VECMAT_NAIVE) return floor_us / 0.12 + 3.0;     // 64 lines per load instruction
    // bytes a CU keeps in flight: resident waves (at most 16 by registers) x rows x chunks x 1 KB; about
    // 48 KB are needed for the rate the chip sustains (0.72 of the peak)
    double waves_per_cu = (double)v->grid * v->waves_k / hw->cus;
    if (waves_per_cu > 16.0) waves_per_cu = 16.0;
    double feed = waves_per_cu * v->bm * v->stages * 1024.0 / 49152.0;
    if (feed > 1.0) feed = 1.0;
    // a wave that takes many row groups in turn pays the memory latency once per group
    const double groups = (double)pr->M * (double)((pr->N + v->bm - 1) / v->bm);
    const double per_wave = groups / ((double)v->grid * v->waves_k);
    const double serial_us = per_wave * 2.0 / (waves_per_cu > 4.0 ? waves_per_cu / 4.0 : 1.0);
    return fmax(floor_us / (0.72 * feed), serial_us) + 3.0;
  }
  if (v->kind == TF_KIND_NAIVE) return fmax(flops / (0.004 * hw->bf16_tflops_peak * 1e6), hbm_us) + 2.0;
  // one wave per tile that gathers element by element: a chain of trips to memory, 1.2 to 2.3 us for 64 of K, however few tiles there are
  // (256^3 9.0 us, 6 x 3008 x 1856 43.6, 5 x 11008 x 4096 101 and with B as [N][K] 156, 19 x 2432 x 3392 78.9). The figure below, 3 us, is of the
  // time when 16 of K were a trip (16.7, 98.6, 170, 225). Nothing hangs on it: where another kernel but the naive one takes the problem and K is 64
  // or more, it is 1.5 to 8 times as fast as this one is now (18 drawn problems).
  if (v->kind == TF_KIND_MFMA_DIRECT) return fmax(fmax(flops / (0.02 * hw->bf16_tflops_peak * 1e6), hbm_us), 0.75 * (pr->K / 16.0)) + 2.0;
  if (v->kind == TF_KIND_MFMA_ANY) {
    // every tile fetches its row and column panel (mostly from L2): 13 TB/s in tiles of 32, 9.5 in tiles of 64 (two
    // loads in flight per byte of LDS against one); below that a wave takes its share of the K tiles one after the
    // other, 0.65 and 1.6 us each (measured on thirty shapes from 36 x 61 x 139 to 4096 x 4095 x 4097). Operands that
    // come from memory arrive at about 0.55 of the peak rate (2 x 8000 x 13120 40 us, 3 x 10912 x 7920 with B as
    // [N][K] 43 us, 1 x 7544 x 14256 49 us; 2.7 to 5.2 TB/s over ten such shapes)
    const bool t64 = v->bm > 32;
    const double traffic = (double)v->grid * 2.0 * v->bm * 2.0 * pr->K;
    const double serial = (double)cdiv(cdiv(pr->K, 64), v->waves_k) * (t64 ? 1.6 : 0.65);
    return 4.0 + fmax(fmax(traffic / (t64 ? 9.5e6 : 13.0e6), hbm_us / 0.55), serial);
  }
  if (tf::is_kshare(v)) {
    const int s = v->split_k;
    const long nkt = cdiv(pr->K, 64);
    // What is known of whole tiles, and how much less their cut takes (the tiles of 16 rows go by those of 32 x 32).
    tf_variant_desc whole = *v;
    if (v->bm < 32) { whole.bm = whole.bn = 32; whole.waves_k = 4; whole.stages = 2; }
    double us = kshare_whole_us(pr, hw, &whole);
    const KshareShape shape = s == 1 ? kshare_shape(pr, hw, v) : KshareShape{};        // (slices are of whole tiles)
    if (shape.is_cut) {
      const double cut = fmax(us * shape.us / (v->bm < 32 ? KsharePricer(pr, hw, &whole).whole().us : shape.whole_us), shape.us);
      // Where the two fits leave the tiles of 16 rows level with those of 32 x 32, which come first in a family, they are ahead by a hair if each of
      // eight waves has more than one K tile: a chain half as long (over 200 such problems, us, 32 x 32 / eight waves to 16 rows, 0.85 of the
      // time, 1.01 at the worst: 2 x 32 x 11120 14.6 / 8.8, 3 x 104 x 5824 8.9 / 6.0, 164 x 96 x 7312 18.2 / 12.3; with no more than one 0.99, 1.05).
      us = cut < us ? cut : v->bm < 32 && nkt > 8 ? 0.999 * us : us;
    }
    // On the scale of what it is compared with. Small problems, the any-address kernels, which are the faster where K is short or rows
    // start off 128-byte lines. (Over 136 drawn problems the faster of the two is picked but for 2.3 %, with a factor of 1.15 in
    // place of this 3.4 %: 105 x 648 x 360 with B as [N][K] 5.3 us where the any-address kernel takes 3.5, 93 x 6480 x 264 [N][K] 6.3 / 4.9.)
    if (v->kind == TF_KIND_MFMA_LDS_ANY) return 1.05 * us + (pr->lda % 64 ? 0.7 : 0.0) + 0.6 * exp(-(double)nkt / 8.0);
    // Otherwise the tile kernels. Operands that no cache holds (three such sets are more than the memory-side cache's 256 MB)
    // arrive at 3.6 TB/s in half lines of B, at 4.2 in slices (16 x 8192 x 8192 31.8 us, the tile kernels' 26.5), at 4.6 in
    // whole lines and whole sums (11008 x 5120 24.3).
    const double opnd_bytes = 2.0 * ((double)pr->M * pr->K + (double)pr->K * pr->N);
    if (!pr->trans_b && opnd_bytes > 95e6) us = fmax(us, 2.9 + opnd_bytes / (v->bn <= 32 ? 3.6e6 : s > 1 ? 4.25e6 : 4.6e6));
    // Where K is whole tiles their 64 x 64 tiles, with the K order rotated or a K tile of 128, are 5 to 15 % faster than these
    // without slices up to a K of about 2000; where it is ragged, 0 to 10 % slower. Cut ones a little more: 277 x 2368 x 1792 with B
    // as [N][K] 10.7 us, the tile kernel 10.1.
    if (v->bm > 32 && s == 1 && pr->K % 64 == 0) us *= 1.0 + (shape.is_cut ? 0.36 : 0.3) * exp(-(double)nkt / 40.0);
    // The tile kernels' figure below is high by what it counts for start-up: 1.4 us, up to 3.4 where K is short (917 x 640 x
    // 320 4.0 us measured, 6.7 predicted). With one factor, 1.15, in place of all this, 101 of 1350 picks were 2 to 23 % slower
    // than the other kernels' (917 x 640 x 320 4.8 / 4.0 us, 1103 x 640 x 448 5.5 / 4.9, 25 x 7808 x 6208 25.5 / 21.5) and the
    // picks 4.4 % behind the best; now 44 are, and 3.0 %.
    return (s > 1 ? 0.97 : 1.0) * us + 1.4 + (v->bm > 32 ? 2.0 : 1.2) * exp(-(double)nkt / 12.0);
  }
  if (v->kind == TF_KIND_MFMA_STREAM) {
    // B is read once at the rate the chip sustains from HBM, if enough waves keep loads in flight
    // (about 96 KB per CU; a wave keeps stages - 1 blocks of 8 KB outstanding)
    const double waves = (double)v->grid * (v->waves_k > 0 ? v->waves_k : 1);
    double feed = waves * (v->stages > 1 ? v->stages - 1 : 1) * 8192.0 / (98304.0 * hw->cus);
    if (feed > 1.0) feed = 1.0;
    const long kblocks = cdiv(cdiv(pr->K, 32), (long)v->split_k * (v->waves_k > 0 ? v->waves_k : 1));
    const double startup = 1.0 + 4.0 / (double)(kblocks > 0 ? kblocks : 1);      // short runs never reach the steady state
    // a CU draws at most about 37 GB/s from HBM (less in row pieces under 256 bytes): few work-groups cannot use the chip
    const double active = v->grid < hw->cus ? (double)v->grid : (double)hw->cus;
    const double cap_gbs = active * 37.0 * (v->bn >= 128 ? 1.0 : 0.65);
    double rate = 0.72 * feed * hw->hbm_gbs_peak;
    if (rate > cap_gbs) rate = cap_gbs;
    double us = bytes / (rate * 1e3) + startup + 2.5;
    // slices: the last work-group to arrive sums them after one more trip to memory, or a second launch does
    if (v->split_k > 1) us += (v->fused_reduce == 2 ? 2.0 : (v->fused_reduce ? 5.5 : 4.5)) + 2.0 * v->split_k * 4.0 * pr->M * (double)pr->N / (hw->hbm_gbs_peak * 1e3);
    return us;
  }
  const int resident = tf_resident_wgs(hw, v);
  const long slots = (long)hw->cus * resident;
  const int bk = v->bk > 0 ? v->bk : 64;
  const double kr = bk / 64.0;                      // the figures below are per 64 of K: a tile of bk is kr of them
  const long ktiles = cdiv(cdiv(pr->K, bk), v->split_k);
  const int mn_waves = v->waves_m * v->waves_n, wg_waves = mn_waves * (v->waves_k > 1 ? v->waves_k : 1);
  // Cycles one CU spends on one K tile (64 wide) of one work-group. The form of each term is what the kernels
  // do; the constants are a least-squares fit (of log predicted / measured, variants within 1.5x of the best) to
  // this family's measured times on MI355X on eight shapes (2048^3, 4096 x 11008 x 4096, 16 x 8192^2,
  // 1024^2 x 16384, 3072^3, 1024 x 8192 x 4096, 256 x 8192^2, 4096 x 2048^2) and were then checked on eight others:
  //  * the clock under MFMA load with every CU busy is about 1650 MHz, whatever the nominal figure says (the board
  //    is power limited); with fewer work-groups than CUs it is higher, by about 0.38 of the idle share; all
  //    cycle counts below are at that clock;
  //  * an MFMA 32x32x16 costs 36.5 cycles of its pipe, not 32 (every tile kernel ran it then; the eight-wave tiles with rows of 64
  //    and more per wave have since gone over to 16x16x32, on which the board holds about a tenth more clock: tf_predict_us);
  //  * tiles enter LDS at about 167 B/clk, fragments leave it at about 203 B/clk; reads and writes take turns;
  //  * a CU receives A tiles (short row pieces) at 82 B/clk and B tiles (long ones) at 52 B/clk when all CUs
  //    ask at once; 0.38 of that time is not hidden behind the matrix pipes;
  //  * per K step a chain of barrier, transfer issue, first fragment reads and first MFMA is
  //    exposed: about 490 cycles with two buffers, 237 with three or more, and a second wave per
  //    SIMD hides nearly all of it; register staging adds 300, the A-bypass loads 400.
  const double mfma = kr * v->bm * (double)v->bn / 32.0 * 1.14;
  const double stage_bytes = kr * (v->a_bypass_lds ? v->bn : v->bm + v->bn) * 128.0;
  const double lds_w = stage_bytes / 167.0;
  long co_resident = cdiv(v->grid, hw->cus);       // work-groups really sharing a CU, not how many would fit
  if (co_resident > resident) co_resident = resident;
  const double cu_waves = (double)wg_waves * co_resident;
  const double a_rows = v->a_bypass_lds ? 0.0 : (double)(v->bm / v->waves_m);
  const double lds_r = kr * mn_waves * (a_rows + (v->bn / v->waves_n)) * 128.0 / 203.0;
  const double ta = kr * (v->bm * 128.0 / 82.0 + v->bn * 128.0 / 52.0);         // global -> CU
  double chain = v->stages >= 3 ? 237.0 : 490.0;
  if (cu_waves >= 8) chain *= v->waves_k > 1 ? 0.455 : 0.05;    // k groups: half the MFMAs per wave and step to hide it behind
  // a K tile of 32 pays the chain twice per 64 of K
  if (bk < 64) chain *= 64.0 / bk;
  if (!v->direct_to_lds) chain += 300.0;
  if (v->a_bypass_lds) chain += 400.0;
  // the tile transfers are never fully hidden behind the matrix pipes: they share the LDS port with the fragment
  // reads and the L2 with the other CUs, and most of their time shows (measured: the 256 x 128 and 128 x 256
  // tiles, whose other figures match the 256 x 256 tile's, need 12-15 % more time per flop; they move 1.5 times
  // the bytes per flop)
  double ktile = fmax(fmax(mfma, lds_w + lds_r), ta) + chain + 0.376 * ta;
  // the in-kernel reductions keep the slices of a tile side by side, so the work-groups of an XCD work on
  // different K ranges and share fewer operand panels in its L2 than in the slice-by-slice order of the
  // two-kernel reduction (measured: about a quarter more time per K step)
  // (big tiles; the skinny tiles' operands are read once anyway)
  const double big = fmin(1.0, v->bm * (double)v->bn / 16384.0);
  if (v->split_k > 1 && v->fused_reduce) ktile *= 1.0 + 0.166 * big;
  // per tile: pipeline fill (first tiles from memory), then bias + GELU + pack at about 11 VALU
  // issue slots per element, or the fp32 partial tile at 32 B/clk when a second kernel reduces
  const double fill = 2900.0 / (double)co_resident;
  // (the raw fp32 output has no activation to evaluate: 16-byte stores at about 64 B/clk)
  // VALU issue slots per output element of the epilogue: erf-GELU 11, tanh-GELU 7, plain conversions 2
  const double epi_valu = pr->epi == TF_EPI_BIAS_GELU_ERF ? 11.0 : pr->epi == TF_EPI_BIAS_GELU_TANH ? 7.0 : 2.0;
  double tile_end = v->bm * (double)v->bn * epi_valu / 64.0;
  // accumulator exchange of the k groups (with less, or none behind a second kernel that reduces, the 2 x 2 x 2 waves were
  // predicted level with the 2 x 4 ones; measured they are 1.0 to 2.0 us slower in 128 x 128 tiles wherever both were
  // timed, e.g. 477 x 1616 x 4992 20.4 / 18.6, 217 x 4928 x 2368 18.1 / 16.1, 408 x 832 x 10944 21.6 / 20.0)
  const double exchange = v->waves_k > 1 ? v->bm * (double)v->bn * 0.12 : 0.0;
  double reduce_us = 0.0, fused_tail_us = 0.0;
  const double active = v->grid < hw->cus ? (double)v->grid / hw->cus : 1.0;
  const double mhz = (hw->clock_mhz < 1650.0 ? hw->clock_mhz : 1650.0) * (1.0 + 0.38 * (1.0 - active));
  if (v->split_k > 1) {
    if (v->fused_reduce == 2) {
      // partial tiles stay in the L2 the slices share: 16-byte stores and loads, one round of tickets
      // ... but the last slice of a tile still sums all slices and runs the epilogue alone, on one CU
      fused_tail_us = 2.0 + 3.0 * big + v->bm * (double)v->bn * 4.0 * (1.0 + 2.0 * v->split_k) / 64.0 / mhz;
    } else if (v->fused_reduce) {
      // partial tiles go out and come back through 16-byte device-scope accesses; the store acknowledgement,
      // the ticket and one load round trip per slice are dependent trips to memory on the last slice's path
      fused_tail_us = 4.0 + 2.5 * v->split_k + v->bm * (double)v->bn * 4.0 * (1.0 + v->split_k) / 32.0 / mhz;
    } else {
      tile_end = v->bm * (double)v->bn * 4.0 / 32.0;
      reduce_us = 4.5 + (v->split_k + 0.5) * 4.0 * pr->M * (double)pr->N / (0.686 * hw->hbm_gbs_peak * 1e3);
    }
  }
  // CUs take the next work-group as they finish one: whole rounds, then a last round that takes between half a
  // round's time (few work-groups left: they have the chip's memory system and power budget to themselves)
  // and all of it, plus a ragged end
  double rounds = (double)v->grid / (double)slots;
  if (rounds <= 1.0) {
    rounds = 1.0;
  } else {
    const double whole = floor(rounds + 1e-9), part = rounds - whole;
    rounds = whole + (part < 1e-9 ? 0.0 : 0.51 + 0.49 * part) + 0.09;
  }
  // a lighter last round: whole rounds of full tiles, then one of tiles that multiply bn_tail of their bn columns
  if (v->bn_tail > 0 && v->bn > 0) rounds = (double)v->grid / (double)slots - 1.0 + (double)v->bn_tail / v->bn + 0.05;
  if (v->stream_k) {
    // every CU gets the same number of K steps: the tile count over the CU count, no ragged last round. But the
    // shares start at arbitrary K offsets, so the work-groups of an XCD no longer walk through K together and
    // stop sharing operand panels in its L2 (measured: about 1.6x the time per K step), each piece refills
    // the pipeline, and each shared tile costs its contributors the store acknowledgement, the ticket and a
    // load round trip, one after the other
    rounds = 1.6 * (double)((pr->M + v->bm - 1) / v->bm) * (double)((pr->N + v->bn - 1) / v->bn) / (double)hw->cus;
    fused_tail_us = 12.0;
  }
  const double per_cu = rounds * (double)co_resident;            // work-groups one CU works through
  const double us = per_cu * (ktiles * ktile + fill + tile_end + exchange) / mhz;
  const double ws_us = v->split_k > 1 ? 2.0 * v->split_k * 4.0 * pr->M * (double)pr->N / (hw->hbm_gbs_peak * 1e3) : 0.0;
  // HBM floor: about three quarters of the peak rate when at least 32 KB per CU are in flight
  // (prefetched tiles of all co-resident work-groups), in proportion below that
  double inflight = (double)co_resident * (v->stages - 1) * stage_bytes / 32768.0;
  if (inflight > 1.0) inflight = 1.0;
  // launch, first tile from HBM and drain: about 3.6 us per launch
  // K order rotated by XCD: measured 2-4 % faster on 2048^3, between equal and 10 % faster on
  // 4096 x 11008 x 4096 depending on the kernel and the chip: proposed first, the plain order right behind
  // (the eight-wave 256 x 128 and 128 x 256 tiles were 0-8 % slower with it on five other shapes)
  const double rot = !v->k_rotate ? 1.0 : ((long)v->bm * v->bn == 32768 && wg_waves == 8) ? 1.02 : 0.98;
  // B given as [N][K] behind a separate transposing pass: one more launch that reads and writes all of B
  const double pretrans_us = (pr->op == TF_OP_GEMM_EPILOGUE && pr->trans_b && !v->trans_b)
                                 ? 3.0 + 4.0 * (double)pr->K * pr->N / (0.6 * hw->hbm_gbs_peak * 1e3) : 0.0;
  // tiles dealt round-robin over the XCDs (offered for one row of tiles): every row of B is then pulled through all
  // eight L2s at once, which streams about a tenth faster than a contiguous run of columns per XCD
  // (and a K tile of 128 streams 3-13 % slower than one of 64, the same kernel otherwise: 16 x 8192 x 8192 29.6 against
  // 27.4 us, 1 x 4096 x 11008 21.4 / 18.9, 8 x 4096 x 4096 12.3 / 11.3, 16 x 4096 x 11008 22.0 / 20.5, 4 x 11008 x 4096
  // 21.6 / 20.8, 32 x 8192 x 4096 18.5 / 17.9. Over 40 skinny problems whose pick the factor moves, the picks were 3.8,
  // 4.0 and 4.5 % behind the best of them with 1.08, 1.09 and 1.12; 1.08 and 1.09 part on two problems in 900)
  // (not where B is [N][K] and each work-group reads rows of its own: over 24 skinny problems whose pick that moves,
  // picks in runs were 10 % faster than the round-robin ones, e.g. 32 x 8576 x 3840 20.1 against 24.2 us)
  const double spread = (v->xcd_swizzle || v->trans_b ? 1.0 : 0.9) * (bk > 64 ? 1.09 : 1.0);
  return fmax(us * rot, (hbm_us + ws_us) / (0.75 * inflight) * spread) + 3.6 + reduce_us + fused_tail_us + pretrans_us;
}

// What ranks the tile kernels beside the constants above. Those were fitted when every tile kernel ran 32x32x16 MFMAs and fetched
// whole K tiles ahead; what the kernels have gained since differs by kind (128 x 128 tiles of 2 x 4 waves 0 to 2 %, 256 x 128
// and 128 x 256 ones 2 to 5, 192 x 256 ones with a ragged K 11, the others 0), and so did what the constants were off before.
//  * Eight-wave 128 x 256 tiles, also in slices, lead those of 256 x 128: rows of 512 bytes instead of 256 (1500 x 4096 x 4096 with
//    B as [N][K] 47.4 against 50.8 us, 1559 x 4096 x 3328 42.8 / 47.7, 487 x 10200 x 1688 26.2 / 28.8).
//  * 64 x 64 tiles where K is short (845 x 5568 x 256 8.8 against 10.0 us, 101 x 7552 x 832 6.9 / 7.8). The whole K counts, a slice's
//    would pick alike in 716 problems; so would leaving out the register-staged and the pre-transposed ones.
//  * Sixteen slices behind a second kernel, whose partial tiles cost more than predicted (300 x 448 x 14016 in 128 x 128 tiles
//    19.1 us, with eight in 64 x 128 16.4).
//  * Rows staged in whole lines, against three buffers: 5 % ([N][K] 12 %) from 16 K tiles a slice on; with fewer the two are level
//    (12 to 15 tiles: 1.01 over 58 launches, [N][K] 0.98 over 43; from 48 on 0.91 and 0.78).
// Over 451 drawn problems (M above 32) the picks are 1.6 % behind the fastest variant, 4.3 % without the four factors; without the
// first 2.0, the second 2.0, the third 2.1, the fourth 2.9. They are not in what decides which problems are small
// (base_predict_us).
extern "C" double tf_predict_us(const tf_problem_desc* pr, const tf_hw* hw, const tf_variant_desc* v) {
  double us = tf::base_predict_us(pr, hw, v);
  if (v->kind != TF_KIND_MFMA_LDS || pr->op != TF_OP_GEMM_EPILOGUE) return us;
  if (v->bm == 128 && v->bn == 256 && v->waves_m * v->waves_n == 8) us *= 0.95;
  if (v->bm == 64 && v->bn == 64) us *= 1.0 - 0.2 * exp(-(pr->K / 64.0) / 12.0);
  if (v->split_k >= 16 && !v->fused_reduce) us *= 1.08;
  if (v->direct_to_lds == 3) {
    const bool few = cdiv(cdiv(pr->K, 64), v->split_k) < 16;
    us *= v->trans_b ? (few ? 0.97 : 0.88) : few ? 1.0 : 0.95;
  }
  return us;
}

// ------------------------------------------------------------------ Proposal
static bool matches_hint(int bn, const tf_hw* hw, const tf_variant_desc* b, const tf_variant_desc* v) {
  const double fill_b = tf_grid_fill(hw, b), fill_v = tf_grid_fill(hw, v);
  const long area_b = (long)b->bm * b->bn, area_v = (long)v->bm * v->bn;
  switch (bn) {
    case TF_BN_UNDERFILLED:   // more, smaller units of work
      return fill_v > fill_b + 1e-9;
    case TF_BN_HBM:           // more bytes in flight
      return v->stages > b->stages || v->split_k > b->split_k || (v->direct_to_lds && !b->direct_to_lds) ||
             v->grid > b->grid;
    case TF_BN_MFMA:          // only quantisation and LDS traffic per MFMA are left
      return area_v >= area_b && fill_v >= fill_b - 1e-9;
    case TF_BN_LDS_CONFLICT:  // other staging path or other tile shape
      return !v->direct_to_lds != !b->direct_to_lds || v->bn != b->bn;
    case TF_BN_OCCUPANCY:     // fewer registers / less LDS per work-group
      return area_v < area_b || (area_v == area_b && v->lds_bytes < b->lds_bytes);
    case TF_BN_LATENCY:       // deeper staging (more buffers, or a longer K tile: fewer hand-overs), or bigger tiles to amortise it
      return v->stages > b->stages || v->bk > b->bk || (v->direct_to_lds && !b->direct_to_lds) || area_v > area_b;
    default:
      return true;
  }
}

// The kernels that the hints speak of: tiles staged through LDS, with one wave or several to a share of K.
static bool hinted(const tf_variant_desc* v) { return is_tile_kernel(v) || tf::is_kshare(v); }

extern "C" int32_t tf_proposal_from(const tf_hw* hw, const tf_variant_desc* family, const double* predicted_us,
                                    int32_t n, const uint8_t* tried, int32_t base_id, int32_t bottleneck) {
  if (!hw || !family || !predicted_us || !tried || n <= 0) return -1;
  const tf_variant_desc* base = (base_id >= 0 && base_id < n) ? &family[base_id] : nullptr;
  const bool use_hint = base && hinted(base) && bottleneck != TF_BN_UNKNOWN;
  int best = -1, best_any = -1;
  for (int i = 0; i < n; ++i) {
    if (tried[i]) continue;
    if (best_any < 0 || predicted_us[i] < predicted_us[best_any]) best_any = i;
    if (use_hint && hinted(&family[i]) && matches_hint(bottleneck, hw, base, &family[i])) {
      if (best < 0 || predicted_us[i] < predicted_us[best]) best = i;
    }
  }
  return best >= 0 ? best : best_any;
}

// A tile kernel and the TF_KIND_MFMA_LDS_ANY variant made of it are one launch wherever both run.
static bool same_launch(const tf_variant_desc* a, const tf_variant_desc* b) {
  return a->bm == b->bm && a->bn == b->bn && a->bk == b->bk && a->waves_m == b->waves_m && a->waves_n == b->waves_n &&
         a->waves_k == b->waves_k && a->stages == b->stages && a->split_k == b->split_k && a->direct_to_lds == b->direct_to_lds &&
         a->a_bypass_lds == b->a_bypass_lds && a->trans_b == b->trans_b && a->stream_k == b->stream_k && a->bn_tail == b->bn_tail &&
         a->k_rotate == b->k_rotate && a->xcd_swizzle == b->xcd_swizzle && a->workspace_bytes == b->workspace_bytes;
}

// Slices of a tile kernel behind a second kernel.
static bool second_kernel(const tf_variant_desc* v) {
  return v->kind == TF_KIND_MFMA_LDS && v->split_k > 1 && !v->fused_reduce && v->workspace_bytes > 0;
}

// The static pick of a problem that is not small, `first` being the variant with the smallest prediction. The predictions of slices
// behind a second kernel are of the time when their partial tiles stayed in the L2s; they pass them by now and take less, but for tiles
// of few rows, whose streams of B each slice begins anew: 3.8 us and a twentieth of the exchange less, 5 % less with sixteen
// slices, 13 % more at up to 32 rows (fitted to the fastest of 900 drawn problems). Whether there are slices at all, and so a workspace
// that calls side by side must not share, is left as it was. What has slices anyhow moves where the second kernel is predicted 5 % faster
// than another tile or streaming kernel, 16 % than one whose waves share K, whose predictions are within 10 % for large tiles
// and off by up to 20 for small ones; and where its workspace is no larger than the first choice's or the library's own buffer
// (it is two to eight times the first choice's: tf.h says so to callers with a buffer of their own).
// us, before / after: 170 x 648 x 14936 23.4 / 15.6, 322 x 504 x 7528 with B as [N][K] 17.9 / 12.3, 72 x 1576 x 7032 18.2 / 11.2. Of 900 drawn
// problems whose pick has slices 107 move, 14 % faster on average; one loses more than 3 (69 x 616 x 16176 [N][K] 3.3). That fit was
// made while partial tiles inside a launch went out non-temporal, which they no longer do (up to 6 % faster, and wrong once in a run of all tests);
// with both kinds of kernel as they are now 60 other moves take 0.83 of the time, one loses more than 3 % (38 x 1568 x 8192 11.3 / 12.2).
// It stands here and not in tf_predict_us because what the loop tries after its first round goes by that, and is measured.
static int with_second_kernel(const tf_problem_desc* pr, const tf_hw* hw, const tf_variant_desc* family, int n, const double* pred,
                              const uint8_t* out, int first) {
  if (pr->op != TF_OP_GEMM_EPILOGUE || family[first].split_k <= 1) return first;
  auto price = [&](int i) {
    const tf_variant_desc& v = family[i];
    if (!second_kernel(&v)) return pred[i];
    const double exchange = (v.split_k + 0.5) * 4.0 * pr->M * (double)pr->N / (0.686 * hw->hbm_gbs_peak * 1e3);
    return (pred[i] * (v.split_k >= 16 ? 1.0 / 1.08 : 1.0) - 3.8 - 0.05 * exchange) * (v.split_k >= 16 ? 1.03 : 1.0) * (pr->M <= 32 ? 1.13 : 1.0);
  };
  const int64_t own = tf_static_scratch_bytes(), room = family[first].workspace_bytes > own ? family[first].workspace_bytes : own;
  int best = -1;
  for (int i = 0; i < n; ++i)
    if (!out[i] && second_kernel(&family[i]) && family[i].workspace_bytes <= room && (best < 0 || price(i) < price(best))) best = i;
  return best >= 0 && price(best) < (tf::is_kshare(&family[first]) ? 0.84 : 0.95) * price(first) ? best : first;
}

extern "C" int32_t tf_proposal(const tf_problem_desc* prob, const tf_hw* hw, const tf_variant_desc* family,
                               int32_t n, const uint8_t* tried, int32_t base_id, int32_t bottleneck) {
  if (!prob || !hw || !family || !tried || n <= 0) return -1;
  double* pred = new double[n];
  uint8_t* out = new uint8_t[n];          // what is not proposed this time
  int small = -1;                         // the variant that marks a small problem
  bool first = true, tiles = false;
  for (int i = 0; i < n; ++i) {
    pred[i] = tf_predict_us(prob, hw, &family[i]);
    out[i] = tried[i];
    if (family[i].kind == TF_KIND_MFMA_LDS_ANY && !tf::is_kshare(&family[i])) small = i;
    tiles |= family[i].kind == TF_KIND_MFMA_LDS;
    if (i > 0 && tried[i]) first = false;
  }
  if (first && (small >= 0 || !tiles)) {
    // the static pick of a small problem (which may be too small for any tile): what takes any pointer and needs no workspace
    for (int i = 0; i < n; ++i)
      if (family[i].kind == TF_KIND_MFMA_LDS || family[i].kind == TF_KIND_MFMA_STREAM || family[i].kind == TF_KIND_MFMA_KSHARE) out[i] = 1;
  } else if (small >= 0) {
    // later rounds: the tile kernel under one of its two ids
    for (int i = 0; i < n; ++i)
      if (i == small ? !tried[i] : tried[small] && family[i].kind == TF_KIND_MFMA_LDS && same_launch(&family[i], &family[small])) out[i] = 1;
  }
  int r = tf_proposal_from(hw, family, pred, n, out, base_id, bottleneck);
  if (first && small < 0 && tiles && r >= 0) r = with_second_kernel(prob, hw, family, n, pred, out, r);
  delete[] pred;
  delete[] out;
  return r;
}

// ------------------------------------------------------------------ Algorithm 1
namespace tf {

tf_status run_loop(const tf_problem_desc* prob, const tf_hw* hw, const tf_variant_desc* family, int32_t n,
                   const int32_t* launches, const tf_theta* theta, profile_fn profile, void* user, int32_t* best_variant, tf_report* best,
                   tf_report* round_log, int32_t log_cap, int32_t* n_log) {
  if (!prob || !hw || !family || n <= 0 || !theta || !profile || !best_variant || !best || !round_log || !n_log)
    return TF_E_INVALID;
  if (log_cap < 1 + theta->max_rounds) return TF_E_RANGE;
  uint8_t* tried = new uint8_t[n]();
  // K* <- K, R* <- R : the baseline kernel is variant 0
  tf_report R;
  tf_status st = profile(user, 0, &R);
  if (st != TF_OK || R.status != TF_OK) { delete[] tried; return st != TF_OK ? st : (tf_status)R.status; }
  R.bottleneck = tf_refine_hint(nullptr, &R, hw);
  tried[0] = 1;
  int nl = 0;
  round_log[nl++] = R;
  tf_report Rstar = R;
  int kstar = 0, kcur = 0, bottleneck = TF_BN_UNKNOWN;   // first proposal: the static one-shot pick
  int stall = 0;
  for (int round = 1; round <= theta->max_rounds; ++round) {
    int cand = tf_proposal(prob, hw, family, n, tried, kcur, bottleneck);
    while (cand >= 0 && launches && launches[cand] < 0) {        // not on these operands: the next one
      tried[cand] = 1;
      cand = tf_proposal(prob, hw, family, n, tried, kcur, bottleneck);
    }
    if (cand < 0) break;                          // family exhausted
    tried[cand] = 1;
    if (launches)
      for (int i = 0; i < n; ++i)
        if (launches[i] == launches[cand]) tried[i] = 1;
    tf_report Rc;
    st = profile(user, cand, &Rc);                // BuildRun + parity gate + Profile
    if (st != TF_OK) { Rc.status = st; Rc.variant_id = cand; }
    Rc.bottleneck = tf_refine_hint(&R, &Rc, hw);
    round_log[nl++] = Rc;
    const int dec = tf_arbiter(&Rc, &Rstar, theta, kstar == 0, stall, round);
    if (dec == TF_DEC_ACCEPT) { kstar = cand; Rstar = Rc; stall = 0; }
    else ++stall;
    if (dec == TF_DEC_FINISH) break;
    // K <- RefineHint(K, R, R'): an accepted candidate becomes the kernel the next proposal
    // starts from; otherwise the next proposal starts again from K*. Either way the newest
    // valid diagnosis gives the direction.
    kcur = (dec == TF_DEC_ACCEPT) ? cand : kstar;
    if (launches) kcur = launches[kcur];          // (the kernel that the diagnosis is about)
    bottleneck = (Rc.status == TF_OK && Rc.t_med_us > 0.0) ? Rc.bottleneck : Rstar.bottleneck;
    R = Rc;
  }
  *best_variant = kstar;
  *best = Rstar;
  *n_log = nl;
  delete[] tried;
  return TF_OK;
}

}  // namespace tf

// Algorithm 1 over pre-made reports (reports[i] is what Profile would return for variant i):
// the loop without a GPU, for tests and for replaying recorded profiles.
struct SimCtx { const tf_report* reports; int n; };
static tf_status sim_profile(void* user, int32_t id, tf_report* out) {
  const SimCtx* c = (const SimCtx*)user;
  if (id < 0 || id >= c->n) return TF_E_INVALID;
  *out = c->reports[id];
  out->variant_id = id;
  return TF_OK;
}

extern "C" tf_status tf_tune_replay(const tf_problem_desc* prob, const tf_hw* hw, const tf_variant_desc* family,
                                    const tf_report* reports, int32_t n, const tf_theta* theta,
                                    int32_t* best_variant, tf_report* best, tf_report* round_log,
                                    int32_t log_cap, int32_t* n_log) {
  if (!reports) return TF_E_INVALID;
  SimCtx c{reports, n};
  return tf::run_loop(prob, hw, family, n, nullptr, theta, sim_profile, &c, best_variant, best, round_log, log_cap, n_log);
}
