// Internal declarations shared by the kernels and the host runtime of
// libedit_outer.so.  Not part of the public ABI (include/edit_outer.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "edit_outer.h"

namespace edit {

constexpr int kRowVectors = 256;     // 16-byte vectors per Gram partial row, at least (up to one row per CU)
constexpr int kUpdateThreads = 64;   // threads per block of the update pass (one wave)
constexpr int kCopyThreads = 256;     // threads per block of the copy probe
constexpr int kFusedThreads = 64;    // threads per block of the one-pass mean step (one wave)
constexpr int kMaxK = EDIT_MAX_K;
constexpr int kMaxPairs = kMaxK * (kMaxK + 1) / 2;

// Device-resident state and decision of one sync unit.  Written by the
// decision kernel, read by the update pass and copied out by state_get.
struct alignas(16) UnitRecord {
  double mu[kMaxK];         // EMA mean of G_j (Eq. 1)
  double sigma[kMaxK];      // EMA std of G_j (Eq. 1)
  double norm[kMaxK];       // G_j of the last step
  double weight[kMaxK];     // w_j of the last step
  double synced_norm;       // ||Delta_bar||
  double clip_coef;         // beta
  int64_t round;            // completed rounds of this unit
  double coef[kMaxK];       // beta * w_j, consumed by the update pass
  int32_t src[kMaxK];       // worker whose data the update pass loads for slot j
  int32_t rollback;         // 1: every worker flagged, reset replicas only
  int32_t use_deltas;       // 0: no worker has a non-zero coefficient
  int32_t z_tested;
  int32_t stepped;          // at least one step or state_set happened
  uint8_t anomalous[kMaxK];
};

// A unit whose one-pass record a launch makes.
struct FinishDesc {
  const double* partials;  // [rows][K+1]
  double* sums;            // [kFoldSlices][K+1], written by the fold launch (sliced units only)
  UnitRecord* rec;
  int32_t rows;
  int32_t slice;  // rows per slice that the fold launch sums first (1: none)
};
constexpr int kFoldSlices = 64;      // at most, per unit
constexpr int kMaxFinishUnits = 64;  // units of one record launch

struct DecideParams {
  double alpha, delta, phi, eps;
  int64_t warmup;
  uint32_t flags;
};

// One unit of a launch; a launch takes a batch of them.
constexpr int kMaxBatchUnits = 16;  // half of it above K = 16
struct UnitDesc {
  float* theta;
  float* mom;
  void* const* reps;   // host array of K device pointers (read at launch)
  int64_t n;
  int64_t cut;         // Gram pass up to K = 8: first element read through the cache
  double* partials;    // [rows][K(K+1)/2]
  UnitRecord* rec;
  int32_t rows;        // blocks (= partial rows) of the Gram pass
  int32_t update_blocks;
};

// A unit whose decision one block takes.
struct DecideDesc {
  const double* partials;
  UnitRecord* rec;
  int32_t rows;
};

// The kernels specialised for one K, behind plain function pointers.  The
// kernels file is compiled once per range of K below (the ranges' template
// instantiations then compile in parallel); the object of the range that
// starts at F exports EDIT_KERNEL_SET_FN(F)(K), which returns the set of a K
// in its range and nullptr otherwise.
#define EDIT_K_RANGES(X) X(1, 8) X(9, 16) X(17, 24) X(25, 32)
#define EDIT_KERNEL_SET_FN2(first) kernel_set_from_##first
#define EDIT_KERNEL_SET_FN(first) EDIT_KERNEL_SET_FN2(first)

struct KernelSet {
  hipError_t (*gram)(bool bf16, const UnitDesc* unit, int count, int max_blocks, hipStream_t stream);
  hipError_t (*decide)(const UnitDesc* unit, int count, const DecideParams& prm, hipStream_t stream);
  hipError_t (*small_step)(bool bf16, const UnitDesc* unit, int count, const DecideParams& prm, double lr,
                           double rho, hipStream_t stream);
  hipError_t (*gram_reduce)(const double* partials, int rows, double* gram, hipStream_t stream);
  hipError_t (*decide_gram)(const double* gram, UnitRecord* rec, const DecideParams& prm, hipStream_t stream);
  hipError_t (*update)(bool bf16, const UnitDesc* unit, int count, int lds, double lr, double rho,
                       hipStream_t stream);
  hipError_t (*fused_mean)(bool bf16, int rows, int lds, float* theta, float* mom, void* const* reps,
                           double* partials, int64_t n, double lr, double rho, hipStream_t stream);
  hipError_t (*fused_finish)(const FinishDesc* unit, int count, int sliced, hipStream_t stream);
  hipError_t (*pattern_probe)(bool bf16, int blocks, int lds, float* theta, float* mom, void* const* reps,
                              int64_t n, hipStream_t stream);
  int batch_units;
  int fused_vectors_bf16, fused_vectors_f32;
};

#define EDIT_DECLARE_SET(first, last) const KernelSet* EDIT_KERNEL_SET_FN(first)(int K);
EDIT_K_RANGES(EDIT_DECLARE_SET)
#undef EDIT_DECLARE_SET

// Launchers (edit_outer_dispatch.hip, through the kernel sets).  All enqueue
// on `stream` and return the launch status (hipErrorInvalidValue for a K
// outside 1..EDIT_MAX_K); none synchronises.
// Each takes a batch of 1 to batch_units(K) units.  The Gram pass: one
// partial row per item, `max_blocks` (one per CU) persistent blocks.
hipError_t launch_gram(int K, bool bf16, const UnitDesc* unit, int count, int max_blocks, hipStream_t stream);
// The decisions from the partial rows.
hipError_t launch_decide(int K, const UnitDesc* unit, int count, const DecideParams& prm, hipStream_t stream);
// Whole steps of units of one partial row, a block each.
hipError_t launch_small_step(int K, bool bf16, const UnitDesc* unit, int count, const DecideParams& prm, double lr,
                             double rho, hipStream_t stream);
int batch_units(int K);
// The fixed-order sum of the partials as a K(K+1)/2 vector in device memory.
hipError_t launch_gram_reduce(int K, const double* partials, int rows, double* gram,
                              hipStream_t stream);
// The decision from a device-resident Gram vector.
hipError_t launch_decide_gram(int K, const double* gram, UnitRecord* rec, const DecideParams& prm,
                              hipStream_t stream);
// The update pass; `lds` bytes of dynamic LDS per block (used by nothing)
// cap its resident blocks per CU (update_pass_lds).
hipError_t launch_update(int K, bool bf16, const UnitDesc* unit, int count, int lds, double lr, double rho,
                         hipStream_t stream);
// The dynamic LDS per block that caps the update pass's resident blocks, given
// the CU's LDS bytes.
int update_pass_lds(int K, bool bf16, int lds_per_cu);
// One-pass mean step (no penalty components): `rows` blocks of
// fused_vectors_per_thread(K, bf16) * kFusedThreads vectors each, leaving
// rows x (K+1) norm partials (each block's K+1 sums contiguous); then one
// block per unit turns them into its record.
int fused_vectors_per_thread(int K, bool bf16);
// `lds`: dynamic LDS per block capping its resident blocks per CU
// (one_pass_lds), as for the update pass.
int one_pass_lds(int K, bool bf16, int lds_per_cu);
hipError_t launch_fused_mean(int K, bool bf16, int rows, int lds, float* theta, float* mom,
                             void* const* reps, double* partials, int64_t n,
                             double lr, double rho, hipStream_t stream);
// The records of 1 to kMaxFinishUnits units, of which the first `sliced` have
// slices to sum first.
hipError_t launch_fused_finish(int K, const FinishDesc* unit, int count, int sliced, hipStream_t stream);
hipError_t launch_copy(void* dst, const void* src, int64_t nbytes, int blocks,
                       hipStream_t stream);
// The update pass's loads and stores (whole vectors only) with no arithmetic.
hipError_t launch_pattern_probe(int K, bool bf16, int blocks, int lds, float* theta, float* mom, void* const* reps,
                                int64_t n, hipStream_t stream);

inline int num_pairs(int K) { return K * (K + 1) / 2; }

}  // namespace edit
