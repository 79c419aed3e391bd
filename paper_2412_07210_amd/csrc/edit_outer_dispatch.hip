// Launchers of the outer-step kernels by worker count K: each call finds the
// kernel set of K's range (one object of edit_outer_kernels.hip per range)
// and forwards to it.  Host code only.
#include "edit_outer_internal.h"
#include "lds_cap.h"

namespace edit {
namespace {

const KernelSet* kernels_for(int K) {
#define EDIT_RANGE(first, last) \
  if (K >= (first) && K <= (last)) return EDIT_KERNEL_SET_FN(first)(K);
  EDIT_K_RANGES(EDIT_RANGE)
#undef EDIT_RANGE
  return nullptr;
}

}  // namespace

hipError_t launch_gram(int K, bool bf16, const UnitDesc* unit, int count, int max_blocks, hipStream_t stream) {
  const KernelSet* s = kernels_for(K);
  return s ? s->gram(bf16, unit, count, max_blocks, stream) : hipErrorInvalidValue;
}

hipError_t launch_decide(int K, const UnitDesc* unit, int count, const DecideParams& prm, hipStream_t stream) {
  const KernelSet* s = kernels_for(K);
  return s ? s->decide(unit, count, prm, stream) : hipErrorInvalidValue;
}

hipError_t launch_small_step(int K, bool bf16, const UnitDesc* unit, int count, const DecideParams& prm, double lr,
                             double rho, hipStream_t stream) {
  const KernelSet* s = kernels_for(K);
  return s ? s->small_step(bf16, unit, count, prm, lr, rho, stream) : hipErrorInvalidValue;
}

int batch_units(int K) {
  const KernelSet* s = kernels_for(K);
  return s ? s->batch_units : 1;
}

hipError_t launch_gram_reduce(int K, const double* partials, int rows, double* gram, hipStream_t stream) {
  const KernelSet* s = kernels_for(K);
  return s ? s->gram_reduce(partials, rows, gram, stream) : hipErrorInvalidValue;
}

hipError_t launch_decide_gram(int K, const double* gram, UnitRecord* rec, const DecideParams& prm,
                              hipStream_t stream) {
  const KernelSet* s = kernels_for(K);
  return s ? s->decide_gram(gram, rec, prm, stream) : hipErrorInvalidValue;
}

hipError_t launch_update(int K, bool bf16, const UnitDesc* unit, int count, int lds, double lr, double rho,
                         hipStream_t stream) {
  const KernelSet* s = kernels_for(K);
  return s ? s->update(bf16, unit, count, lds, lr, rho, stream) : hipErrorInvalidValue;
}

// The update pass streams 2K + 4 buffers at once (K + 2 read, K + 2
// written), and the HBM serves that mix faster with fewer of its waves in
// flight than its registers allow.  Blocks resident per CU, us a step or
// round on one box at 4, 5, 6, 8 and uncapped: K = 8 bf16, two of 51.4M
// 1,132, 1,132, 1,144, 1,165 and 1,195; K = 8 fp32, three of 12.8M 722, 706,
// 703, 707 and 768; K = 16 bf16, 51.4M 1,053, 1,031, 1,035, 1,053 and 1,069;
// K = 4 bf16, four of 12.8M 392, 373, 369, 374 and 378; K = 24 bf16, 20M 668,
// 662, 662, 665 and 664; K = 32 bf16, 9.4M 471, 461, 459, 458 and 457.
// (128-thread blocks at K = 8 were slower at every count.)  With few workers
// a block has fewer loads in flight (K + 2 with fp32 replicas, K + 4 with
// bf16) and more blocks are needed; at 5, 8, 16 and uncapped: K = 1 fp32,
// 28.3M 183, 163, 145 and 148; K = 2 bf16, 28.3M 163, 158, 153 and 153; K = 3
// fp32, 12.8M 130, 119, 118 and 119; K = 4 fp32, nine of 2.9M 309, 284, 289
// and 294.
constexpr int update_pass_blocks_per_cu(int K, bool bf16) {
  if (K <= 2) return 16;
  return K <= 4 && !bf16 ? 8 : 5;
}

// The one-pass kernel streams the same 2K + 4 buffers as the update pass, in
// one-wave blocks, two 16-byte vectors per thread with bf16 replicas up to
// K = 16 and one otherwise (one took 474-484 us per 51.4M bf16 unit at K = 8
// against 435: each block's closing reduction and partial row then cover half
// as much data).  Resident blocks per CU, us a round on one box at 4, 5, 6, 7,
// 8 and uncapped: bf16 K = 2, two of 28.3M 288, 276, 272, 271, 272 and 278;
// K = 3, three of 12.8M 219, 213, 213, 214, 217 and 221; K = 4, four of 12.8M
// 316, 313, 314, 320, 324 and 334; K = 5, three of 28.3M 560, 560, 565, 570,
// 574 and 601; K = 8, four of 28.3M 971, 981, 993, 1,003, 1,010 and 1,018;
// K = 12, three of 12.8M 456, 460, 465, 467, 468 and 468; K = 24, two of 9M
// 391, 399, 402, 406, 406 and 406.  fp32 K = 3, three of 12.8M 371, 321, 296,
// 285, 279 and 310; K = 5, three of 5M 176, 168, 166, 165, 167 and 176; K = 8,
// four of 12.8M 789, 725, 702, 697, 703 and 780; K = 12, three of 5M 304, 306,
// 312, 316, 317 and 323; K = 32, two of 4M 413, 418, 418, 421, 415 and 415.
constexpr int one_pass_blocks_per_cu(int K, bool bf16) {  // 0: uncapped
  if (K <= 2) return 0;
  if (!bf16) return K <= 8 ? 7 : 4;
  return K <= 4 ? 5 : 4;
}

// the kernel's block sums red[K+1]
constexpr int one_pass_static_lds(int K) { return static_cast<int>(sizeof(double)) * (K + 1); }

constexpr bool caps_hold() {
  for (int K = 1; K <= kMaxK; ++K)
    for (int bf16 = 0; bf16 < 2; ++bf16) {
      const int up = update_pass_blocks_per_cu(K, bf16), one = one_pass_blocks_per_cu(K, bf16);
      const int own = one_pass_static_lds(K);
      if (lds_blocks(lds_for_blocks(up, 0, kLdsPerCu), kLdsPerCu) != up) return false;
      if (one > 0 && lds_blocks(lds_for_blocks(one, own, kLdsPerCu) + own, kLdsPerCu) != one) return false;
    }
  return true;
}
static_assert(caps_hold(), "the reserved LDS lets exactly the named number of blocks run on a CU");

int update_pass_lds(int K, bool bf16, int lds_per_cu) {
  return lds_for_blocks(update_pass_blocks_per_cu(K, bf16), 0, lds_per_cu);
}

int one_pass_lds(int K, bool bf16, int lds_per_cu) {
  const int blocks = one_pass_blocks_per_cu(K, bf16);
  return blocks > 0 ? lds_for_blocks(blocks, one_pass_static_lds(K), lds_per_cu) : 0;
}

int fused_vectors_per_thread(int K, bool bf16) {
  const KernelSet* s = kernels_for(K);
  return s ? (bf16 ? s->fused_vectors_bf16 : s->fused_vectors_f32) : 1;
}

hipError_t launch_fused_mean(int K, bool bf16, int rows, int lds, float* theta, float* mom, void* const* reps,
                             double* partials, int64_t n, double lr, double rho,
                             hipStream_t stream) {
  const KernelSet* s = kernels_for(K);
  return s ? s->fused_mean(bf16, rows, lds, theta, mom, reps, partials, n, lr, rho, stream)
           : hipErrorInvalidValue;
}

hipError_t launch_fused_finish(int K, const FinishDesc* unit, int count, int sliced, hipStream_t stream) {
  const KernelSet* s = kernels_for(K);
  return s ? s->fused_finish(unit, count, sliced, stream) : hipErrorInvalidValue;
}

hipError_t launch_pattern_probe(int K, bool bf16, int blocks, int lds, float* theta, float* mom, void* const* reps,
                                int64_t n, hipStream_t stream) {
  const KernelSet* s = kernels_for(K);
  return s ? s->pattern_probe(bf16, blocks, lds, theta, mom, reps, n, stream) : hipErrorInvalidValue;
}

}  // namespace edit
