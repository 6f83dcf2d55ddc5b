// Internal: the loop driver shared by tf_tune (profiles on the GPU) and tf_tune_replay
// (reads pre-made reports).
#pragma once
#include "tf.h"

namespace tf {
constexpr int KSHARE_TWO_TILES_KB = 40;    // two K tiles in a ring of a cut where the rings of a CU have no more in flight without the second
constexpr int KSHARE_CUT_MARK = 64;    // what a launch of cut tiles asks for beyond its rings: a descriptor tells by it which of two kernels it means
// A variant of the kernels whose waves share K: of a small problem, the ones without slices are listed as
// TF_KIND_MFMA_LDS_ANY (no other tile kernel has a single wave per k group and several groups).
inline bool is_kshare(const tf_variant_desc* v) {
  return v->kind == TF_KIND_MFMA_KSHARE || (v->kind == TF_KIND_MFMA_LDS_ANY && v->waves_m == 1 && v->waves_n == 1 && v->waves_k > 1);
}

// What a launch of such a variant takes for a tile: eights of rows and of columns (of a [K][N] B always all of them), and how
// many K tiles a wave's ring holds.
struct KshareShape {
  int groups_a, groups_b, stages;
  long tiles_m, tiles_n;
  int lds_bytes;
  double us, whole_us;     // predicted time of the launch, and of one of whole tiles
  bool is_cut;
};
inline bool kshare_is_cut(const tf_variant_desc* v) { return v->lds_bytes % 1024 == KSHARE_CUT_MARK; }
KshareShape kshare_shape(const tf_problem_desc* pr, const tf_hw* hw, const tf_variant_desc* v);

// Profile callback: BuildRun + parity gate + Profile of variant `id` into *out.
typedef tf_status (*profile_fn)(void* user, int32_t id, tf_report* out);

// launches: per variant, the variant that runs in its place on the caller's operands, or -1 where those are refused
// (null: every variant runs as itself). The loop proposes no refused variant and no launch twice.
tf_status run_loop(const tf_problem_desc* prob, const tf_hw* hw, const tf_variant_desc* family, int32_t n,
                   const int32_t* launches, const tf_theta* theta, profile_fn profile, void* user, int32_t* best_variant, tf_report* best,
                   tf_report* round_log, int32_t log_cap, int32_t* n_log);
// tf_predict_us without the factors that only rank the tile kernels: what decides which problems are small.
double base_predict_us(const tf_problem_desc* pr, const tf_hw* hw, const tf_variant_desc* v);

}  // namespace tf
