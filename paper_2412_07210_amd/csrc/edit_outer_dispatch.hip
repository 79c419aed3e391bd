// Launchers of the outer-step kernels by worker count K: each call finds the
// kernel set of K's range (one object of edit_outer_kernels.hip per range)
// and forwards to it.  Host code only.
#include "edit_outer_internal.h"

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
// flight than its registers allow.  Sweeps on one box (alternating runs,
// 1B round at K = 8 bf16): 128-thread blocks, 8 per CU (the register
// limit) 14.31-14.36 ms, 4 per CU 13.91-14.01, 3 per CU 13.84-13.87;
// one-wave blocks, 6 per CU 13.56-13.60 ms, against 13.60-13.68 at 4 or 5,
// 13.72-13.73 at 7 and 14.00-14.02 at 8.  Six one-wave blocks per CU also
// gave the shortest 350M, 7B half-shard and A-EDiT K = 16 rounds.  With few
// workers a block has fewer loads in flight (K + 2 with fp32 replicas, K + 4
// with bf16) and more blocks are needed; measured on one box at 6, 8 and 16
// blocks per CU: K = 1 fp32, 28.3M elements 200, 180 and 162 us a step; K = 2
// bf16, nine of 28.3M 1,443, 1,442 and 1,371; K = 2 fp32, 5.8M 63, 59 and 59;
// K = 4 fp32, nine of 2.9M 323, 295 and 303; but K = 4 bf16, nine of 12.8M
// 839, 862 and 850, K = 3 bf16, 51.4M 325, 329 and 331, K = 6 fp32, 12.8M
// 200, 200 and 203.
int update_pass_blocks_per_cu(int K, bool bf16) {
  if (K <= 2) return 16;
  return K <= 4 && !bf16 ? 8 : 6;
}

int update_pass_lds(int K, bool bf16, int lds_per_cu) {
  // the largest multiple of 256 bytes that still lets that many blocks fit
  return lds_per_cu > 0 ? (lds_per_cu / update_pass_blocks_per_cu(K, bf16)) & ~255 : 0;
}

int fused_vectors_per_thread(int K, bool bf16) {
  const KernelSet* s = kernels_for(K);
  return s ? (bf16 ? s->fused_vectors_bf16 : s->fused_vectors_f32) : 1;
}

// The one-pass kernel streams the same 2K + 4 buffers as the update pass, in
// one-wave blocks, two 16-byte vectors per thread with bf16 replicas up to
// K = 16 and one otherwise (one took 474-484 us per 51.4M bf16 unit at K = 8
// against 435: each block's closing reduction and partial row then cover half
// as much data).  Resident blocks per CU, us per round on one box at the
// cap's best and uncapped: K = 8 bf16, four of 28.3M 968 at five, 982 at six,
// 1,025; K = 8 fp32, four of 12.8M 690 at eight, 713 at six, 788; K = 16
// fp32, three of 5M 383 at five, 453; K = 16 bf16, two of 9.4M 301 and 310;
// K = 24 bf16 406 at five, 441; K = 4 bf16, four of 12.8M 323 at six, 338;
// K = 4 fp32, six of 2.9M 180 at eight, 183; K = 2 no gain at any.
int one_pass_lds(int K, bool bf16, int lds_per_cu) {
  const int blocks = K <= 2 ? 0 : (!bf16 && K <= 8 ? 8 : (K <= 4 ? 6 : 5));
  return blocks > 0 && lds_per_cu > 0 ? (lds_per_cu / blocks) & ~255 : 0;
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
