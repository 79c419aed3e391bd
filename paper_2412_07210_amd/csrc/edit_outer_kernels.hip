// Device kernels of the EDiT outer synchronization step for gfx950.
//
// One step of a batch of sync units (one unit, or several small ones of a
// round) is three launches on one stream:
//
//   gram   streams theta and the K replicas once and accumulates, per block,
//          the upper triangle of the Gram matrix  Gram_jk = <Delta_j, Delta_k>
//          of the pseudo gradients Delta_j = r_j - theta (Sec. 3.2).  The
//          diagonal gives the module norms G_j; the off-diagonal terms give
//          ||sum_j w_j Delta_j||^2 = w^T Gram w, so the clip factor of Eq. 4
//          is known before the update pass and the step needs two streaming
//          passes instead of three.
//   decide one block per unit: fixed-order reduction of the per-block
//          partials, then one wave (worker j in lane j) takes the decision:
//          EMA z-test and update (Eq. 1), rollback test, softmax weights
//          (Eq. 2), Gbar and beta (Eq. 4), coefficients beta*w_j.
//   update streams theta, b and the replicas of the workers with a non-zero
//          coefficient, forms Delta_hat = sum_j beta w_j Delta_j (Eq. 3, 5),
//          applies Nesterov momentum and writes theta, b and all K replicas.
//
// Storage is fp32 (theta, b) and fp32/bf16 (replicas); arithmetic is fp64
// from the exact pseudo gradients on, rounded once when stored.
//
// The passes are HBM-bound (2-4 flop per byte at K = 8).  Lanes move 16-byte
// vectors (global_load_dwordx4).  The Gram pass runs a persistent grid of one
// block per CU (strided over the unit), so the chip streams one contiguous
// window of every buffer at a time and the decision reduces one partial row
// per CU; each lane double-buffers its vectors (the loads of trip t+1 are in
// flight while trip t is computed), so the fp64 work hides under the memory
// latency.  Above K = 8 the Gram is a rank-n update on the fp64 matrix cores
// (v_mfma_f64_4x4x4f64 tiles), which the VALU could not hold in registers.
// The update pass, which writes as much as it reads, instead gives each
// thread one vector and lets the block dispatcher order the traffic.
//
// The update pass follows its own Gram pass with only the decision between
// them, so it finds the end of its input in the 256 MB Infinity Cache: the
// Gram pass reads that end through the cache (everything before it
// non-temporally) and the update pass takes its blocks from the end.
//
// Also here: the step of units of one Gram block in one block
// (small_step_kernel; the bodies of the Gram and update passes are the
// fragments gram_rows_valu.inc, gram_rows_mfma.inc and update_vector_at.inc,
// shared with the kernels above), the Gram export/import of a sharded module
// (gram_reduce_kernel, decide_gram_kernel), the one-pass mean step used when
// no penalty component is on (fused_mean_kernel, fused_finish_kernel), and a
// plain copy kernel for bandwidth and counter calibration.  Reductions go
// wave -> LDS -> per-block partial -> one block in a fixed order, so results
// are bitwise reproducible.
#include "edit_outer_internal.h"

#include <algorithm>

// Compiled once per range of worker counts (EDIT_K_RANGES); the build passes
// the range's first and last K.
#if !defined(EDIT_K_FIRST) || !defined(EDIT_K_LAST)
#error "compile with -DEDIT_K_FIRST=<first K> -DEDIT_K_LAST=<last K> of one of EDIT_K_RANGES"
#endif

namespace edit {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));

// Cache policy of the streaming kernels: each pass touches every byte once;
// non-temporal accesses measured ~15% faster for the VALU Gram pass and ~5%
// for the update pass.  The matrix-core Gram pass, bound by issue, reads
// through the cache.
constexpr bool kNTMfma = false;
constexpr bool kNT2 = true;

template <int K>
struct ConstPtrs {
  const void* p[K];
};
template <int K>
struct MutPtrs {
  void* p[K];
};

template <bool BF16>
struct Vec {
  static constexpr int VE = BF16 ? 8 : 4;  // elements per 16-byte replica vector
};

// 16-byte global accesses; NT marks them non-temporal (streaming) in the cache.
template <bool NT, typename T>
__device__ __forceinline__ T ld16(const T* p) {
  if constexpr (NT)
    return __builtin_nontemporal_load(p);
  else
    return *p;
}
template <bool NT, typename T>
__device__ __forceinline__ void st16(T* p, T v) {
  if constexpr (NT)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// Element e of a 16-byte replica vector, widened to fp32 (exact).
template <bool BF16>
__device__ __forceinline__ float element(const u32x4& raw, int e) {
  if constexpr (BF16) {
    const uint32_t word = raw[e >> 1];
    return __uint_as_float((e & 1) ? (word & 0xffff0000u) : (word << 16));
  } else {
    return __uint_as_float(raw[e]);
  }
}

template <bool BF16>
__device__ __forceinline__ float load_scalar(const void* base, int64_t i) {
  if constexpr (BF16) {
    const uint16_t h = reinterpret_cast<const uint16_t*>(base)[i];
    return __uint_as_float(static_cast<uint32_t>(h) << 16);
  } else {
    return reinterpret_cast<const float*>(base)[i];
  }
}

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const float2_t f = {a, b};
  const bf16x2_t h = __builtin_convertvector(f, bf16x2_t);  // v_cvt_pk_bf16_f32, RNE
  return __builtin_bit_cast(uint32_t, h);
}

template <bool BF16>
__device__ __forceinline__ void store_scalar(void* base, int64_t i, float x) {
  if constexpr (BF16) {
    reinterpret_cast<uint16_t*>(base)[i] = static_cast<uint16_t>(pack_bf16x2(x, 0.f) & 0xffffu);
  } else {
    reinterpret_cast<float*>(base)[i] = x;
  }
}

// fp32 values [v*VE, v*VE+VE) of a theta/momentum buffer.
template <int VE, bool NT>
__device__ __forceinline__ void load_f32(const float* p, int64_t v, float (&x)[VE]) {
  const f32x4* q = reinterpret_cast<const f32x4*>(p) + v * (VE / 4);
#pragma unroll
  for (int h = 0; h < VE / 4; ++h) {
    const f32x4 t = ld16<NT>(q + h);
#pragma unroll
    for (int c = 0; c < 4; ++c) x[4 * h + c] = t[c];
  }
}

template <int VE, bool NT>
__device__ __forceinline__ void store_f32(float* p, int64_t v, const float (&x)[VE]) {
  f32x4* q = reinterpret_cast<f32x4*>(p) + v * (VE / 4);
#pragma unroll
  for (int h = 0; h < VE / 4; ++h) {
    f32x4 t;
#pragma unroll
    for (int c = 0; c < 4; ++c) t[c] = x[4 * h + c];
    st16<NT>(q + h, t);
  }
}

// VE fp32 values -> one 16-byte replica vector.
template <bool BF16>
__device__ __forceinline__ u32x4 pack(const float (&x)[Vec<BF16>::VE]) {
  u32x4 r;
  if constexpr (BF16) {
#pragma unroll
    for (int c = 0; c < 4; ++c) r[c] = pack_bf16x2(x[2 * c], x[2 * c + 1]);
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) r[c] = __float_as_uint(x[c]);
  }
  return r;
}

// Element e of a replica vector minus theta, in fp64: the pseudo gradient of
// that element, exact for fp32/bf16 inputs whose exponents differ by < 29.
template <bool BF16>
__device__ __forceinline__ double delta64(const u32x4& raw, int e, float th) {
  return static_cast<double>(element<BF16>(raw, e)) - static_cast<double>(th);
}

// A field of a unit record read by the update pass: from LDS where the block
// has just made the record (the single-block step), otherwise from a record
// that an earlier launch wrote, constant for this one and read as such, by
// scalar loads.  As plain loads beside stores that the compiler cannot tell
// apart from it, the fields came by vector loads and every replica pointer
// was chosen per lane (K = 16 update pass 750 us against 680 with scalar
// loads, K = 8 415 against 409).
template <bool kInLds, typename T>
__device__ __forceinline__ T rec_load(const T* p) {
  if constexpr (kInLds)
    return *p;
  else
    return *reinterpret_cast<const __attribute__((address_space(4))) T*>(reinterpret_cast<uintptr_t>(p));
}

// Sum over the 64 lanes of a wave, fixed butterfly order (same in every lane).
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
  return x;
}

// Two doubles a, b exchanged between the halves of every 2B lanes (B = 32 or
// 16): x takes the lower halves of a and of b, y the upper halves.
template <int B>
__device__ __forceinline__ void swap_halves(double a, double b, double& x, double& y) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const unsigned alo = __double2loint(a), ahi = __double2hiint(a);
  const unsigned blo = __double2loint(b), bhi = __double2hiint(b);
  u32x2 lo, hi;
  if constexpr (B == 32) {
    lo = __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
    hi = __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
  } else {
    lo = __builtin_amdgcn_permlane16_swap(alo, blo, false, false);
    hi = __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false);
  }
  x = __hiloint2double(hi[0], lo[0]);
  y = __hiloint2double(hi[1], lo[1]);
}

// A double from another lane of the 16-lane row (DPP control CTRL).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double a) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(a), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(a), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// The sums over a wave's 64 lanes of M values at once (M <= 64): each step
// adds two lanes' values and leaves half of the values in either half of the
// lanes, so that after six steps every lane holds one finished sum, the one
// that index(lane) names (a sum that several lanes name has the same bits in
// all of them).  36 values take about 150 vector instructions and no LDS
// access, where a butterfly per value takes 432 LDS permutes per wave: at
// K = 8 that closing reduction was most of the Gram pass's fixed cost (on
// 2,048 bf16 elements the pass took 11.3 us with it and takes 4.8 us with
// this one; 1,024 fp32 elements at K = 4: 5.0 and 3.0).  The order of the
// additions is fixed, so results are reproducible.
template <int B, int M>
struct WaveSums {
  static_assert(M >= 1 && M <= 64, "one sum per lane at most");
  static constexpr int H = (M + 1) / 2;
  static __device__ __forceinline__ double sum(const double (&x)[M], int lane) {
    double y[H];
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double p = x[2 * i], q = x[2 * i + 1 < M ? 2 * i + 1 : 2 * i];  // an odd last value pairs with itself
      if constexpr (B >= 16) {
        double a, b;
        swap_halves<B>(p, q, a, b);
        y[i] = a + b;
      } else {
        // partner lanes: rotate by 8, mirror of 8, the quad's xor 2 and xor 1
        constexpr int kCtrl = B == 8 ? 0x128 : B == 4 ? 0x141 : B == 2 ? 0x4E : 0xB1;
        const bool up = (lane & B) != 0;
        const double send = up ? p : q, keep = up ? q : p;
        y[i] = keep + dpp_move<kCtrl>(send);
      }
    }
    if constexpr (B > 1)
      return WaveSums<B / 2, H>::sum(y, lane);
    else
      return y[0];
  }
  static __device__ __forceinline__ int index(int lane) {
    int i = 0;
    if constexpr (B > 1) i = WaveSums<B / 2, H>::index(lane);
    i = 2 * i + ((lane & B) ? 1 : 0);
    return i < M - 1 ? i : M - 1;
  }
};

__device__ __forceinline__ int pair_index(int K, int j, int k) {  // j <= k
  return j * K - (j * (j - 1)) / 2 + (k - j);
}

// ------------------------------------------------------------- decision

constexpr int kDecideThreads = 1024;  // one block; wide so the partial loads overlap

// Reduce a unit's partial rows [rows][NP] in a fixed order into gram[NP]
// (shared memory).  Thread t reads the flat array at t, t + S, t + 2S, ...
// with S a multiple of NP within the block, so it always reads
// column t % NP and a wave's loads are contiguous; the S threads' sums are
// then added per column in thread order, by one thread per column, so at
// most 32 threads share a column: with as many as fit the block, K = 1 and 2
// added 1,023 and 340 terms one after the other (a step of 65,536 fp32
// elements at K = 1 29.0 us, of 300,000 at K = 2 21.2; now 17.0 and 16.0).
// The rows were just written by every XCD's blocks, so the loads come from
// the Infinity Cache or HBM and the reduction is latency-bound: all of a
// thread's loads for 256 rows are in flight at once up to K = 16, 48 at a
// time above.  As [NP][rows], whose loads touched a cache line per lane, over
// up to 1,023 rows the decision kernel took 9.2 us at K = 4 (1.05M fp32 elements; now 4.0), 6.8 at K = 8
// (4.7) and 79 at K = 32 (27, bound by one CU reading 1.1 MB).
template <int K>
__device__ void reduce_partials(const double* partials, int rows, double* gram, double* scratch) {
  constexpr int NP = K * (K + 1) / 2;
  constexpr int T = kDecideThreads / NP < 32 ? kDecideThreads / NP : 32;  // threads per column
  constexpr int S = NP * T;
  constexpr int kAll = (256 + T - 1) / T;
  constexpr int U = kAll < 48 ? kAll : 48;
  const int t = threadIdx.x;
  if (t < S) {
    const int total = rows * NP;
    double acc = 0.0;
    for (int i = t; i < total; i += S * U) {
      double x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int at = i + u * S;
        x[u] = at < total ? __builtin_nontemporal_load(partials + at) : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) acc += x[u];
    }
    scratch[t] = acc;
  }
  __syncthreads();
  if (t < NP) {
    double g = scratch[t];
#pragma unroll
    for (int k = 1; k < T; ++k) g += scratch[k * NP + t];
    gram[t] = g;
  }
}

// The state a decision starts from: round counter and each worker's EMA
// pair, loaded by the deciding wave before the partial reduction so that
// their latency hides behind it.
struct DecideState {
  int64_t round;
  double mu, sigma;  // of the lane's worker (lane < K)
};

template <int K>
__device__ __forceinline__ DecideState load_decide_state(const UnitRecord* rec) {
  const int lane = threadIdx.x & 63;
  DecideState st{rec->round, 0.0, 0.0};
  if (lane < K) {
    st.mu = rec->mu[lane];
    st.sigma = rec->sigma[lane];
  }
  return st;
}

// The decision of one step from the unit's Gram matrix, taken by one wave:
// worker j's norm, z-test, EMA update and softmax term live in lane j; the
// cross-lane steps (min, sums, first contributing worker) are fixed-order
// butterflies and ballots, so the result is reproducible bit for bit.
template <int K>
__device__ void decide(const double* gram, UnitRecord* rec, const DecideParams& prm,
                       const DecideState& st) {
  const int lane = threadIdx.x & 63;
  const bool ae = prm.flags & EDIT_AE;
  const bool wa = prm.flags & EDIT_WA;
  const bool gc = prm.flags & EDIT_GC;
  const int64_t t = st.round;
  const bool z_test = ae && t >= prm.warmup;
  const bool mine = lane < K;

  // Norms and anomaly elimination (Sec. 3.2): the z-test z = (G - mu)/sigma > delta
  // is taken as G - mu > delta*sigma against the state before this round; a
  // non-finite norm is always flagged.  Eq. 1 then updates the unflagged.
  double G = 0.0;
  bool bad = true;
  if (mine) {
    G = sqrt(gram[pair_index(K, lane, lane)]);
    bad = !isfinite(G);
    const double mu0 = st.mu;
    const double sg0 = st.sigma;
    if (z_test && !bad) bad = (G - mu0) > prm.delta * sg0;
    rec->norm[lane] = G;
    rec->anomalous[lane] = bad ? 1 : 0;
    if (ae && !bad) {
      const double mu = prm.alpha * G + (1.0 - prm.alpha) * mu0;
      const double dev = G - mu;
      rec->sigma[lane] = sqrt((1.0 - prm.alpha) * sg0 * sg0 + prm.alpha * dev * dev);
      rec->mu[lane] = mu;
    }
  }
  const bool ok = mine && !bad;
  const int n_ok = __popcll(__ballot(ok));

  double w = 0.0, gbar = 0.0, beta = 0.0;
  if (n_ok > 0) {
    if (wa) {  // Eq. 2 as a softmax of -G over the unflagged workers, shifted by min G
      double g0 = ok ? G : INFINITY;
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) g0 = fmin(g0, __shfl_xor(g0, m, 64));
      const double e = ok ? exp(-(G - g0)) : 0.0;
      w = e / wave_sum(e);
    } else {
      w = ok ? 1.0 / n_ok : 0.0;
    }
    // ||sum_j w_j Delta_j||^2 = sum_jk w_j w_k Gram_jk (Eq. 3-4); every lane
    // takes part in every shuffle (uniform trip count).
    double q = 0.0;
#pragma unroll
    for (int it = 0; it < (K * K + 63) / 64; ++it) {
      const int pk = lane + 64 * it;
      const int pkc = pk < K * K ? pk : 0;
      const int j = pkc / K, k = pkc % K;
      const double wj = __shfl(w, j, 64);
      const double wk = __shfl(w, k, 64);
      const double g = j <= k ? gram[pair_index(K, j, k)] : gram[pair_index(K, k, j)];
      // flagged workers have w = 0 and may have non-finite Gram entries
      if (pk < K * K && wj != 0.0 && wk != 0.0) q += wj * wk * g;
    }
    gbar = sqrt(fmax(wave_sum(q), 0.0));
    beta = gc ? fmin(prm.phi / (gbar + prm.eps), 1.0) : 1.0;
  }

  // The update pass loads slot j from worker src[j]: itself when it
  // contributes, otherwise a contributing worker (a cache hit, and never the
  // data of a flagged worker, which may hold NaN).
  const double c = beta * w;
  const unsigned long long nz = __ballot(mine && c != 0.0);
  const int first = nz ? __ffsll(static_cast<long long>(nz)) - 1 : -1;
  if (mine) {
    rec->weight[lane] = w;
    rec->coef[lane] = c;
    rec->src[lane] = (c != 0.0 || first < 0) ? lane : first;
  }
  if (lane == 0) {
    rec->use_deltas = first >= 0 ? 1 : 0;
    rec->rollback = n_ok == 0 ? 1 : 0;
    rec->synced_norm = gbar;
    rec->clip_coef = beta;
    rec->z_tested = z_test ? 1 : 0;
    rec->stepped = 1;
    rec->round = t + 1;
  }
}

// ------------------------------------------------------------- Gram pass

// Threads per block of the Gram pass.  The MFMA version runs one block per
// CU holding all its resident waves (3 per SIMD up to K = 16, 2 above, where
// the 21 to 36 accumulator tiles and the double-buffered vectors of eight
// worker groups need up to 256 VGPRs per lane), so the block reduction
// combines them and the decision reduces one partial row per CU.  The VALU
// version runs one 256-thread block per CU: four waves with two trips of
// loads each already keep more bytes in flight than HBM needs (K = 8 bf16,
// 51.4M elements: 150 us at one block per CU, 151 at two; 1.05M: 7.4 and
// 9.0; K = 4 fp32 at 12.8M: 40.6 and 40.2, at 2.9M 11.2 and 11.7).
template <int K>
constexpr int gram_threads() {
  return K <= 8 ? 256 : (K <= 16 ? 768 : 512);
}

// Gram contributions of one 16-byte vector of every replica.
template <int K, bool BF16>
__device__ __forceinline__ void gram_vector(double (&acc)[K * (K + 1) / 2], const u32x4 (&raw)[K],
                                            const float (&th)[Vec<BF16>::VE]) {
#pragma unroll
  for (int e = 0; e < Vec<BF16>::VE; ++e) {
    double d[K];
#pragma unroll
    for (int j = 0; j < K; ++j) d[j] = delta64<BF16>(raw[j], e, th[e]);
    int p = 0;
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
      for (int k = j; k < K; ++k, ++p) acc[p] = fma(d[j], d[k], acc[p]);
  }
}

// theta and every replica at vector v (< nvec).  Unguarded: the caller
// clamps v, so that no load sits under a lane mask; a masked load makes the
// compiler wait for the next trip's loads before computing this one.
template <int K, bool BF16, bool NT>
__device__ __forceinline__ void load_gram(const float* theta, const ConstPtrs<K>& reps, int64_t v,
                                           float (&th)[Vec<BF16>::VE], u32x4 (&raw)[K]) {
  load_f32<Vec<BF16>::VE, NT>(theta, v, th);
#pragma unroll
  for (int j = 0; j < K; ++j) raw[j] = ld16<NT>(reinterpret_cast<const u32x4*>(reps.p[j]) + v);
}

// Where each unit of a batch begins in the launch's items or blocks (unused
// places hold INT32_MAX).  The array lies together in the kernel arguments,
// so a block finds its unit from one wide scalar load.
template <int U>
struct FirstOf {
  int32_t at[U];
  __device__ __forceinline__ int unit_of(int x) const {
    int w = 0;
#pragma unroll
    for (int i = 1; i < U; ++i) w += at[i] <= x ? 1 : 0;
    return w;
  }
};

// One unit of a Gram launch.
template <int K>
struct GramUnit {
  const float* theta;
  ConstPtrs<K> reps;
  int64_t nvec;
  int64_t n;
  int64_t cut;       // first vector read through the cache (VALU pass)
  double* partials;  // [rows][K(K+1)/2]
  int32_t rows;
};

// The units of a Gram launch.  Its work items are the units' partial rows in
// unit order; block b takes items b, b + gridDim.x, ...
template <int K, int U>
struct GramBatch {
  FirstOf<U> first;  // items
  GramUnit<K> u[U];
  int32_t items;
};

template <int K, bool BF16, int U>
__global__ __launch_bounds__(gram_threads<K>(), 2) void gram_kernel(GramBatch<K, U> batch) {
  static_assert(K <= 8, "VALU Gram pass covers K <= 8");
  constexpr int NP = K * (K + 1) / 2;
  constexpr int VE = Vec<BF16>::VE;
#pragma unroll 1
  for (int it = blockIdx.x; it < batch.items; it += gridDim.x) {
    const int w = batch.first.unit_of(it);
    const GramUnit<K>& unit = batch.u[w];
    const float* __restrict__ theta = unit.theta;
    ConstPtrs<K> reps;
#pragma unroll
    for (int j = 0; j < K; ++j) reps.p[j] = unit.reps.p[j];
    const int64_t nvec = unit.nvec, n = unit.n, cut = unit.cut;
    const int rows = unit.rows, b = it - batch.first.at[w];
    double* __restrict__ row_out = unit.partials + static_cast<int64_t>(b) * NP;
#include "gram_rows_valu.inc"
    if (U == 1) break;
    __syncthreads();  // red[] is read before the next item writes it
  }
}

// The Gram pass for 8 < K <= 32: the Gram matrix sum_i d_i d_i^T over the unit's
// elements is a rank-n update, and with K(K+1)/2 = 136 to 528 fp64 sums per
// lane a VALU version runs out of registers.  It runs on the fp64 matrix
// cores as v_mfma_f64_4x4x4f64, four independent 4x4x4 products per wave
// instruction (blocks b = 0..3).  The workers form G = ceil(K/4) groups of
// four and the Gram matrix 4x4 tiles (I, J); only the G(G+1)/2 tiles with
// I <= J are formed (10 of 16 at K = 16, 36 of 64 at K = 32): 160 products
// per element at K = 16 where the 16x16x4 instruction forms all 256, and
// this one also sustains a higher share of the fp64 matrix peak.  On gfx950 the fp64 matrix work and the fp64
// vector work of the deltas (widening, subtracting theta) do not overlap,
// so the pass is bound by their sum rather than by HBM.
//
// Operand layout of the instruction on gfx950 (checked with a one-hot
// probe): lane l holds A[i][k] and B[k][j] of block b with i = j = l % 4,
// b = (l / 4) % 4, k = l / 16, and the result D[i][j] of block b sits in
// lane j + 4b + 16i.  So the four lanes of a quad q = l / 4 share (b, k):
// they take one element, lane c = l % 4 holding the pseudo gradients of
// workers c, c+4, c+8, c+12 of it, and for tile (I, J) a lane passes its
// group-I value as A and its group-J value as B.  Each instruction adds the
// products of 16 elements (one per quad) into the tile, block b summing the
// quads b, b+4, b+8, b+12; the blocks are added at the end.

// Vector slots per lane per loop trip of the matrix-core pass (two, or
// loads two trips ahead, measured no faster and need 512-thread blocks).
constexpr int kMfmaSlots = 1;
// Load buffers per lane in the matrix-core pass's loop: two (the next trip's
// loads in flight while one is computed).  With every load unmasked, three
// buffers and 1024-thread blocks measured within 1% of this at K = 16 (A/B
// on one box): the pass is not waiting on memory latency.  Its matrix-core
// and vector instructions share one issue port and take its time.
template <int K>
constexpr int kMfmaDepth() {
  return 2;
}

template <int K>
struct Tiles4 {
  static constexpr int G = (K + 3) / 4;      // worker groups of four
  static constexpr int T = G * (G + 1) / 2;  // tiles (I, J), I <= J
};

// One vector slot of a quad: the whole theta vector (every lane of the quad
// loads it; the L1 serves the repeats, which measured faster than loading a
// quarter per lane and broadcasting it by DPP moves, eight more vector
// instructions per slot) and lane c's groups' replica vectors.
template <int G, bool BF16>
struct Quad4 {
  static constexpr int TH = Vec<BF16>::VE;
  u32x4 raw[G];
  float th[TH];
};

// Vector v (< nvec) of theta and of this lane's replicas (rep[g] is worker
// 4g + lane % 4).  Lanes of workers >= K (act false, only in the last group
// when K is not a multiple of 4) feed zeros.  No bounds guard: the caller
// clamps v, so that no load sits under a lane mask and the loads of later
// trips stay in flight.
template <int G, bool BF16, bool NT>
__device__ __forceinline__ void load_quad4(const float* theta, const void* const (&rep)[G],
                                           const bool (&act)[G], int64_t v, Quad4<G, BF16>& q) {
  load_f32<Vec<BF16>::VE, NT>(theta, v, q.th);
#pragma unroll
  for (int g = 0; g < G; ++g)
    q.raw[g] = act[g] ? ld16<NT>(reinterpret_cast<const u32x4*>(rep[g]) + v) : u32x4{0u, 0u, 0u, 0u};
}

// A quad whose vector lies past the unit's end contributes nothing.
template <int G, bool BF16>
__device__ __forceinline__ void zero_quad4(Quad4<G, BF16>& q) {
#pragma unroll
  for (int g = 0; g < G; ++g) q.raw[g] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
  for (int t = 0; t < Quad4<G, BF16>::TH; ++t) q.th[t] = 0.f;
}

// The Gram tiles of one vector slot: for each of its VE elements, the
// lane's group deltas (exact, fp64) go into every tile (I, J), I <= J.
template <int K, bool BF16>
__device__ __forceinline__ void gram_quad4(double (&acc)[Tiles4<K>::T], const u32x4 (&raw)[Tiles4<K>::G],
                                           const float (&th)[Vec<BF16>::VE], const bool (&act)[Tiles4<K>::G]) {
  constexpr int G = Tiles4<K>::G;
#pragma unroll
  for (int e = 0; e < Vec<BF16>::VE; ++e) {
    double d[G];
#pragma unroll
    for (int g = 0; g < G; ++g) d[g] = act[g] ? delta64<BF16>(raw[g], e, th[e]) : 0.0;
    int t = 0;
#pragma unroll
    for (int I = 0; I < G; ++I)
#pragma unroll
      for (int J = I; J < G; ++J, ++t) acc[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(d[I], d[J], acc[t], 0, 0, 0);
  }
}

template <int K, bool BF16, bool NT, int U>
__global__ __launch_bounds__(gram_threads<K>()) void gram_mfma_kernel(GramBatch<K, U> batch) {
  static_assert(K > 8 && K <= 32, "MFMA Gram pass covers 8 < K <= 32");
  constexpr int NP = K * (K + 1) / 2;
  constexpr int VE = Vec<BF16>::VE;
  constexpr int kDepth = kMfmaDepth<K>();
#pragma unroll 1
  for (int it = blockIdx.x; it < batch.items; it += gridDim.x) {
    const int w = batch.first.unit_of(it);
    const GramUnit<K>& unit = batch.u[w];
    const float* __restrict__ theta = unit.theta;
    ConstPtrs<K> reps;
#pragma unroll
    for (int j = 0; j < K; ++j) reps.p[j] = unit.reps.p[j];
    const int64_t nvec = unit.nvec, n = unit.n;
    const int rows = unit.rows, b = it - batch.first.at[w];
    double* __restrict__ row_out = unit.partials + static_cast<int64_t>(b) * NP;
#include "gram_rows_mfma.inc"
    if (U == 1) break;
    __syncthreads();  // gsh[] is read before the next item writes it
  }
}

// ---------------------------------------------------------------- decide

// The units of a decision launch, one block each.
template <int U>
struct DecideBatch {
  DecideDesc u[U];
};

template <int K, int U>
__global__ __launch_bounds__(kDecideThreads) void decide_kernel(DecideBatch<U> batch, DecideParams prm) {
  __shared__ double gram[K * (K + 1) / 2];
  __shared__ double scratch[kDecideThreads];
  const DecideDesc& unit = batch.u[U == 1 ? 0 : blockIdx.x];
  UnitRecord* rec = unit.rec;
  const DecideState st = load_decide_state<K>(rec);
  reduce_partials<K>(unit.partials, unit.rows, gram, scratch);
  __syncthreads();
  if (threadIdx.x < 64) decide<K>(gram, rec, prm, st);
}

// The Gram of one unit as a plain vector (upper triangle, row by row): the
// decision kernel's own fixed-order reduction, written out instead of
// decided on, so that the shards of one module can add their Grams before a
// shared decision.
template <int K>
__global__ __launch_bounds__(kDecideThreads) void gram_reduce_kernel(const double* __restrict__ partials,
                                                                     int rows,
                                                                     double* __restrict__ gram_out) {
  __shared__ double gram[K * (K + 1) / 2];
  __shared__ double scratch[kDecideThreads];
  reduce_partials<K>(partials, rows, gram, scratch);
  __syncthreads();
  for (int p = threadIdx.x; p < K * (K + 1) / 2; p += kDecideThreads) gram_out[p] = gram[p];
}

// The decision from a Gram supplied by the caller (one wave).
template <int K>
__global__ __launch_bounds__(64) void decide_gram_kernel(const double* __restrict__ gram_in,
                                                         UnitRecord* __restrict__ rec,
                                                         DecideParams prm) {
  __shared__ double gram[K * (K + 1) / 2];
  const DecideState st = load_decide_state<K>(rec);
  for (int p = threadIdx.x; p < K * (K + 1) / 2; p += 64) gram[p] = gram_in[p];
  __syncthreads();
  decide<K>(gram, rec, prm, st);
}

// ----------------------------------------------------------- update pass

// theta' and b' of one element, in fp64 from fp32 inputs (rounded once on store):
//   Delta_hat = sum_j c_j (r_j - theta), c_j = beta w_j      (Eq. 3, 5)
//   g = -Delta_hat;  b' = rho b + g;  theta' = theta - nu (g + rho b')
__device__ __forceinline__ void nesterov(double dhat, float th, float b, double lr, double rho,
                                         float& th_out, float& b_out) {
  const double g = -dhat;
  const double bn = fma(rho, static_cast<double>(b), g);
  th_out = static_cast<float>(static_cast<double>(th) - lr * fma(rho, bn, g));
  b_out = static_cast<float>(bn);
}

// theta, b and the contributing replicas at vector v (nothing past the end).
template <int K, bool BF16, bool NT>
__device__ __forceinline__ void load_update(const float* theta, const float* mom,
                                           const u32x4* const (&src)[K], bool use, int64_t v,
                                           int64_t nvec, float (&th)[Vec<BF16>::VE],
                                           float (&b)[Vec<BF16>::VE], u32x4 (&raw)[K]) {
  if (v < nvec) {
    load_f32<Vec<BF16>::VE, NT>(theta, v, th);
    load_f32<Vec<BF16>::VE, NT>(mom, v, b);
    if (use) {
#pragma unroll
      for (int j = 0; j < K; ++j) raw[j] = ld16<NT>(src[j] + v);
    }
  }
}

// The update of one vector: weighted average, Nesterov, write-back.
template <int K, bool BF16, bool NT>
__device__ __forceinline__ void update_vector(float* theta, float* mom, const MutPtrs<K>& reps,
                                              const double (&c)[K], bool use, int64_t v,
                                              const float (&th)[Vec<BF16>::VE],
                                              const float (&b)[Vec<BF16>::VE],
                                              const u32x4 (&raw)[K], double lr, double rho) {
  constexpr int VE = Vec<BF16>::VE;
  double acc[VE];
#pragma unroll
  for (int e = 0; e < VE; ++e) acc[e] = 0.0;
  if (use) {
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
      for (int e = 0; e < VE; ++e) acc[e] = fma(c[j], delta64<BF16>(raw[j], e, th[e]), acc[e]);
  }
  float tn[VE], bn[VE];
#pragma unroll
  for (int e = 0; e < VE; ++e) nesterov(acc[e], th[e], b[e], lr, rho, tn[e], bn[e]);
  store_f32<VE, NT>(theta, v, tn);
  store_f32<VE, NT>(mom, v, bn);
  const u32x4 out = pack<BF16>(tn);
#pragma unroll
  for (int j = 0; j < K; ++j) st16<NT>(reinterpret_cast<u32x4*>(reps.p[j]) + v, out);
}

// One 16-byte vector of every buffer per thread, one one-wave block per 64
// vectors (a flat grid): the hardware dispatcher then keeps the in-flight
// window of each of the 2K+4 streams short and ordered (measured 5.5 TB/s
// here against 4.9 TB/s for a persistent grid-stride loop).  The launch
// reserves dynamic LDS so that few blocks at a time run on a CU
// (update_pass_blocks_per_cu): fewer waves in flight serve this traffic
// faster.  Blocks are taken from the unit's end; forward order measured the
// same.
template <int K>
struct UpdateUnit {
  float* theta;
  float* mom;
  MutPtrs<K> reps;
  const UnitRecord* rec;
  int64_t nvec;
  int64_t n;
  int32_t blocks;
};

template <int K, int U>
struct UpdateBatch {
  FirstOf<U> first;  // blocks
  UpdateUnit<K> u[U];
  double lr, rho;
};

template <int K, bool BF16, bool NT, int U>
__global__ __launch_bounds__(kUpdateThreads) void update_kernel(UpdateBatch<K, U> batch) {
  constexpr int VE = Vec<BF16>::VE;
  const int blk = static_cast<int>(gridDim.x - 1 - blockIdx.x);  // from the batch's end
  const int w = batch.first.unit_of(blk);
  const int own = blk - batch.first.at[w];  // the unit's block
  const UpdateUnit<K>& unit = batch.u[w];
  float* __restrict__ theta = unit.theta;
  float* __restrict__ mom = unit.mom;
  const MutPtrs<K>& rep_args = unit.reps;
  MutPtrs<K> reps;
#pragma unroll
  for (int j = 0; j < K; ++j) reps.p[j] = rep_args.p[j];
  const UnitRecord* __restrict__ rec = unit.rec;
  const int64_t nvec = unit.nvec, n = unit.n;
  const double lr = batch.lr, rho = batch.rho;
  const int64_t v = static_cast<int64_t>(own) * kUpdateThreads + threadIdx.x;
  const int64_t tail = nvec * VE + threadIdx.x;
  const bool do_tail = own == unit.blocks - 1 && tail < n;
  constexpr bool kRecInLds = false;  // written by the decision of an earlier launch

#include "update_vector_at.inc"
}

// The access pattern of the update pass with no arithmetic: the same grid, block
// order and 16-byte accesses, reading theta, b and all K replicas and
// writing them all back (XOR with `flip`, zero at run time, keeps every
// store), so its time is what this traffic costs with nothing computed.
// Used to calibrate the update pass against its own pattern, not by the method.
template <int K, bool BF16, bool NT>
__global__ __launch_bounds__(kUpdateThreads) void update_pattern_probe_kernel(float* __restrict__ theta,
                                                                            float* __restrict__ mom,
                                                                            MutPtrs<K> reps, int64_t nvec,
                                                                            uint32_t flip) {
  const int64_t v = static_cast<int64_t>(gridDim.x - 1 - blockIdx.x) * kUpdateThreads + threadIdx.x;
  if (v >= nvec) return;
  constexpr int H = Vec<BF16>::VE / 4;  // 16-byte vectors of theta (and of b) per replica vector
  u32x4 t[H], b[H], r[K];
  u32x4* tp = reinterpret_cast<u32x4*>(theta) + v * H;
  u32x4* bp = reinterpret_cast<u32x4*>(mom) + v * H;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    t[h] = ld16<NT>(tp + h);
    b[h] = ld16<NT>(bp + h);
  }
#pragma unroll
  for (int j = 0; j < K; ++j) r[j] = ld16<NT>(reinterpret_cast<const u32x4*>(reps.p[j]) + v);
#pragma unroll
  for (int h = 0; h < H; ++h) {
    st16<NT>(tp + h, t[h] ^ flip);
    st16<NT>(bp + h, b[h] ^ flip);
  }
#pragma unroll
  for (int j = 0; j < K; ++j) st16<NT>(reinterpret_cast<u32x4*>(reps.p[j]) + v, r[j] ^ flip);
}

// ------------------------------------------------------ single-block units

// A unit whose Gram pass is one block (at most 256 vectors) can be stepped
// whole by one block: its Gram row, the decision and the update pass, one
// after the other, in one launch instead of three.  A launch takes up to
// batch_units<K>() such units, a block each.  The block runs the code of the
// three launches (the Gram pass with one row, the decision, the update with
// one vector per thread), included from the same fragments, so the results
// are the same bit for bit.  The row and the record stay in LDS: the block
// copies the record in while its first loads are in flight, decides on it
// there, and copies it back at the end.
template <int K>
struct SmallUnit {
  float* theta;
  float* mom;
  MutPtrs<K> reps;
  UnitRecord* rec;
  int64_t n;
};

template <int K, int U>
struct SmallBatch {
  SmallUnit<K> u[U];
  double lr, rho;
};

template <int K, bool BF16, int U>
__global__ __launch_bounds__(gram_threads<K>()) void small_step_kernel(SmallBatch<K, U> batch, DecideParams prm) {
  constexpr int NP = K * (K + 1) / 2;
  constexpr int VE = Vec<BF16>::VE;
  static_assert(sizeof(UnitRecord) % 16 == 0, "the record is copied in 16-byte vectors");
  constexpr int kRecVectors = sizeof(UnitRecord) / 16;  // at most one per thread
  static_assert(kRecVectors <= gram_threads<K>(), "one vector of the record per thread");
  __shared__ double gram[NP];
  __shared__ UnitRecord record;
  const SmallUnit<K>& su = batch.u[U == 1 ? 0 : blockIdx.x];
  const int64_t n = su.n;
  const int64_t nvec = n / VE;
  if (threadIdx.x < kRecVectors)
    reinterpret_cast<u32x4*>(&record)[threadIdx.x] = reinterpret_cast<const u32x4*>(su.rec)[threadIdx.x];
  {  // the Gram pass: the unit's only row
    const float* __restrict__ theta = su.theta;
    ConstPtrs<K> reps;
#pragma unroll
    for (int j = 0; j < K; ++j) reps.p[j] = su.reps.p[j];
    double* row_out = gram;
    const int b = 0, rows = 1;
    if constexpr (K > 8) {
      constexpr bool NT = kNTMfma;
      constexpr int kDepth = 1;  // two trips at most: a second buffer only makes the code longer
#include "gram_rows_mfma.inc"
    } else {
      const int64_t cut = 0;
#include "gram_rows_valu.inc"
    }
  }
  __syncthreads();
  if (threadIdx.x < 64) decide<K>(gram, &record, prm, load_decide_state<K>(&record));
  __syncthreads();
  if (threadIdx.x < kRecVectors)
    reinterpret_cast<u32x4*>(su.rec)[threadIdx.x] = reinterpret_cast<const u32x4*>(&record)[threadIdx.x];
  {  // the update: one vector per thread (nvec <= 256 <= the block's threads)
    constexpr bool NT = kNT2;
    float* __restrict__ theta = su.theta;
    float* __restrict__ mom = su.mom;
    const MutPtrs<K>& rep_args = su.reps;
    MutPtrs<K> reps;
#pragma unroll
    for (int j = 0; j < K; ++j) reps.p[j] = rep_args.p[j];
    const UnitRecord* rec = &record;
    const double lr = batch.lr, rho = batch.rho;
    const int64_t v = threadIdx.x;
    const int64_t tail = nvec * VE + threadIdx.x;
    const bool do_tail = tail < n;
    constexpr bool kRecInLds = true;
#include "update_vector_at.inc"
  }
}

// ------------------------------------------------------ one-pass mean step

// With every penalty component off (the plain DiLoCo outer step, the paper's
// "w/o ALL" ablation), the weights are 1/K whatever the norms are, so the
// average, Nesterov and the write-back need no earlier pass: one kernel reads
// theta, b and the K replicas once and writes theta', b' and the replicas.
// The norms G_j and ||Delta_bar|| are still summed on the way (per-block
// partials, reduced by fused_finish_kernel) for the step's record.  A block owns V*kFusedThreads
// consecutive vectors; a thread loads its V vectors of every buffer before
// computing, so V*(K+2) 16-byte loads are in flight per thread (V = 2 for
// bf16 replicas measured best here: one vector leaves the block's closing
// reduction exposed, four cost occupancy).
template <int K, bool BF16, bool NT, int V>
__global__ __launch_bounds__(kFusedThreads) void fused_mean_kernel(float* __restrict__ theta,
                                                                   float* __restrict__ mom,
                                                                   MutPtrs<K> reps,
                                                                   double* __restrict__ partials,
                                                                   int64_t nvec, int64_t n,
                                                                   double lr, double rho) {
  constexpr int VE = Vec<BF16>::VE;
  constexpr double inv_k = 1.0 / K;
  const int b = blockIdx.x;
  double sq[K + 1];  // sum of Delta_j^2 per worker, then of Delta_bar^2
#pragma unroll
  for (int p = 0; p <= K; ++p) sq[p] = 0.0;

  {
    const int64_t base = static_cast<int64_t>(b) * V * kFusedThreads + threadIdx.x;
    float th[V][VE], bm[V][VE];
    u32x4 raw[V][K];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int64_t v = base + u * kFusedThreads;
      if (v < nvec) {
        load_f32<VE, NT>(theta, v, th[u]);
        load_f32<VE, NT>(mom, v, bm[u]);
#pragma unroll
        for (int j = 0; j < K; ++j) raw[u][j] = ld16<NT>(reinterpret_cast<const u32x4*>(reps.p[j]) + v);
      }
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int64_t v = base + u * kFusedThreads;
      if (v < nvec) {
        float tn[VE], bn[VE];
#pragma unroll
        for (int e = 0; e < VE; ++e) {
          double sum = 0.0;
#pragma unroll
          for (int j = 0; j < K; ++j) {
            const double d = delta64<BF16>(raw[u][j], e, th[u][e]);
            sq[j] = fma(d, d, sq[j]);
            sum += d;
          }
          const double dbar = sum * inv_k;  // Eq. 3 with w_j = 1/K
          sq[K] = fma(dbar, dbar, sq[K]);
          nesterov(dbar, th[u][e], bm[u][e], lr, rho, tn[e], bn[e]);
        }
        store_f32<VE, NT>(theta, v, tn);
        store_f32<VE, NT>(mom, v, bn);
        const u32x4 out = pack<BF16>(tn);
#pragma unroll
        for (int j = 0; j < K; ++j) st16<NT>(reinterpret_cast<u32x4*>(reps.p[j]) + v, out);
      }
    }
  }
  const int64_t tail = nvec * VE + threadIdx.x;  // the last n - nvec*VE elements
  if (b == 0 && tail < n) {
    const float t0 = theta[tail];
    double sum = 0.0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const double d = static_cast<double>(load_scalar<BF16>(reps.p[j], tail)) - static_cast<double>(t0);
      sq[j] = fma(d, d, sq[j]);
      sum += d;
    }
    const double dbar = sum * inv_k;
    sq[K] = fma(dbar, dbar, sq[K]);
    float tn, bn;
    nesterov(dbar, t0, mom[tail], lr, rho, tn, bn);
    theta[tail] = tn;
    mom[tail] = bn;
#pragma unroll
    for (int j = 0; j < K; ++j) store_scalar<BF16>(reps.p[j], tail, tn);
  }

  // block sums in a fixed order: the wave's, then the waves in order
  constexpr int kWaves = kFusedThreads / 64;
  __shared__ double red[kWaves][K + 1];
  {
    const int lane = threadIdx.x & 63;
    const double t = WaveSums<32, K + 1>::sum(sq, lane);
    red[threadIdx.x >> 6][WaveSums<32, K + 1>::index(lane)] = t;
  }
  __syncthreads();
  if (threadIdx.x <= K) {  // the block's K + 1 sums, contiguous
    double t = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) t += red[w][threadIdx.x];
    partials[static_cast<int64_t>(b) * (K + 1) + threadIdx.x] = t;
  }
}

// The sums over `count` rows [count][K+1], per column in a fixed order, in
// tot[K+1] (shared memory).  Thread t always reads column t % NV and a
// wave's loads are contiguous; U loads per thread are in flight at a time,
// and the threads' sums are added per column in thread order.
template <int K>
__device__ __forceinline__ void sum_rows(const double* rows, int count, double* part, double* tot) {
  constexpr int NV = K + 1;
  constexpr int T = kDecideThreads / NV;  // rows read at a time
  constexpr int U = 8;
  const int t = threadIdx.x, c = t % NV;
  double s = 0.0;
  if (t < NV * T) {
    for (int r = t / NV; r < count; r += T * U) {
      double v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int at = r + u * T;
        v[u] = at < count ? rows[static_cast<int64_t>(at) * NV + c] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) s += v[u];
    }
  }
  part[t] = s;
  __syncthreads();
  if (t < NV) {
    double x = 0.0;
    for (int k = t; k < NV * T; k += NV) x += part[k];
    tot[t] = x;
  }
}

// The units of a record launch, those with slices first.
template <int U>
struct FinishBatch {
  FinishDesc u[U];
};

// Large one-pass units: block (s, u) sums slice s of unit u's rows into row s
// of its slice sums, so that the one block that makes the unit's record has
// at most kFoldSlices rows to read.  The partial rows stay as they are.  By itself that block read every row of a
// 28.3M-element unit (27,651 of nine sums) at the rate of one CU: 36 us for
// a round's units, where the two launches take 8.8 and 6.8.
template <int K, int U>
__global__ __launch_bounds__(kDecideThreads) void fused_fold_kernel(FinishBatch<U> batch) {
  const FinishDesc& unit = batch.u[U == 1 ? 0 : blockIdx.y];
  const int r0 = blockIdx.x * unit.slice;
  if (r0 >= unit.rows) return;  // block-uniform
  __shared__ double part[kDecideThreads];
  __shared__ double tot[K + 1];
  sum_rows<K>(unit.partials + static_cast<int64_t>(r0) * (K + 1), min(unit.slice, unit.rows - r0), part, tot);
  if (threadIdx.x < K + 1) unit.sums[blockIdx.x * (K + 1) + threadIdx.x] = tot[threadIdx.x];
}

// The records of one-pass steps: G_j and ||Delta_bar|| from each unit's
// partial rows or slice sums (in a fixed order), w_j = 1/K, beta = 1.  One
// block per unit, so a round can take all its units' reductions in one launch
// after its last fused pass; only the units stepped are listed, since others
// of the handle may be in flight on another stream.  Nothing is masked in
// this mode: a non-finite replica shows up as a non-finite G_j (and in
// theta).
template <int K, int U>
__global__ __launch_bounds__(kDecideThreads) void fused_finish_kernel(FinishBatch<U> batch) {
  const FinishDesc& unit = batch.u[U == 1 ? 0 : blockIdx.x];
  UnitRecord* rec = unit.rec;
  __shared__ double part[kDecideThreads];
  __shared__ double tot[K + 1];
  if (unit.slice > 1)
    sum_rows<K>(unit.sums, (unit.rows + unit.slice - 1) / unit.slice, part, tot);
  else
    sum_rows<K>(unit.partials, unit.rows, part, tot);
  __syncthreads();
  if (threadIdx.x < K) {
    rec->norm[threadIdx.x] = sqrt(tot[threadIdx.x]);
    rec->weight[threadIdx.x] = 1.0 / K;
    rec->coef[threadIdx.x] = 1.0 / K;
    rec->src[threadIdx.x] = threadIdx.x;
    rec->anomalous[threadIdx.x] = 0;
  }
  if (threadIdx.x == 0) {
    rec->synced_norm = sqrt(tot[K]);
    rec->clip_coef = 1.0;
    rec->use_deltas = 1;
    rec->rollback = 0;
    rec->z_tested = 0;
    rec->stepped = 1;
    rec->round = rec->round + 1;
  }
}

// ------------------------------------------------------------ copy probe

template <int U, bool NT>
__global__ __launch_bounds__(kCopyThreads) void copy_kernel(u32x4* __restrict__ dst,
                                                       const u32x4* __restrict__ src,
                                                       int64_t nvec) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kCopyThreads;
  for (int64_t v = static_cast<int64_t>(blockIdx.x) * kCopyThreads + threadIdx.x; v < nvec; v += stride * U) {
    u32x4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u == 0 || v + u * stride < nvec) x[u] = ld16<NT>(src + v + u * stride);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u == 0 || v + u * stride < nvec) st16<NT>(dst + v + u * stride, x[u]);
  }
}

}  // namespace

// ------------------------------------------------------------ launchers

namespace {

// Units of one launch (a batch of a round), bounded by the 4 KiB of kernel
// arguments; a batch of one has kernels of its own, without the unit search.
template <int K>
constexpr int batch_units() {
  return K <= 16 ? kMaxBatchUnits : kMaxBatchUnits / 2;
}

template <int K, bool BF16, int U>
hipError_t gram_launch_u(const UnitDesc* unit, int count, int max_blocks, hipStream_t stream) {
  GramBatch<K, U> batch{};
  std::fill_n(batch.first.at, U, INT32_MAX);
  for (int i = 0; i < count; ++i) {
    const UnitDesc& d = unit[i];
    GramUnit<K>& g = batch.u[i];
    g.theta = d.theta;
    for (int j = 0; j < K; ++j) g.reps.p[j] = d.n > 0 ? d.reps[j] : nullptr;
    g.nvec = d.n / Vec<BF16>::VE;
    g.n = d.n;
    g.cut = d.cut / Vec<BF16>::VE;
    g.partials = d.partials;
    g.rows = d.rows;
    batch.first.at[i] = batch.items;
    batch.items += d.rows;
  }
  const int blocks = U == 1 ? batch.items : std::min(batch.items, max_blocks);
  if constexpr (K <= 8)
    hipLaunchKernelGGL((gram_kernel<K, BF16, U>), dim3(blocks), dim3(gram_threads<K>()), 0, stream, batch);
  else
    hipLaunchKernelGGL((gram_mfma_kernel<K, BF16, kNTMfma, U>), dim3(blocks), dim3(gram_threads<K>()), 0, stream,
                       batch);
  return hipGetLastError();
}

template <int K, bool BF16>
hipError_t gram_launch(const UnitDesc* unit, int count, int max_blocks, hipStream_t stream) {
  if (count < 1 || count > batch_units<K>()) return hipErrorInvalidValue;
  return count == 1 ? gram_launch_u<K, BF16, 1>(unit, count, max_blocks, stream)
                    : gram_launch_u<K, BF16, batch_units<K>()>(unit, count, max_blocks, stream);
}

template <int K, bool BF16, int U>
hipError_t small_step_launch_u(const UnitDesc* unit, int count, const DecideParams& prm, double lr, double rho,
                               hipStream_t stream) {
  SmallBatch<K, U> batch{};
  batch.lr = lr;
  batch.rho = rho;
  for (int i = 0; i < count; ++i) {
    const UnitDesc& d = unit[i];
    batch.u[i].theta = d.theta;
    batch.u[i].mom = d.mom;
    for (int j = 0; j < K; ++j) batch.u[i].reps.p[j] = d.n > 0 ? d.reps[j] : nullptr;
    batch.u[i].rec = d.rec;
    batch.u[i].n = d.n;
  }
  hipLaunchKernelGGL((small_step_kernel<K, BF16, U>), dim3(count), dim3(gram_threads<K>()), 0, stream, batch, prm);
  return hipGetLastError();
}

template <int K, bool BF16>
hipError_t small_step_launch(const UnitDesc* unit, int count, const DecideParams& prm, double lr, double rho,
                             hipStream_t stream) {
  if (count < 1 || count > batch_units<K>()) return hipErrorInvalidValue;
  return count == 1 ? small_step_launch_u<K, BF16, 1>(unit, count, prm, lr, rho, stream)
                    : small_step_launch_u<K, BF16, batch_units<K>()>(unit, count, prm, lr, rho, stream);
}

template <int K, int U>
hipError_t decide_launch_u(const UnitDesc* unit, int count, const DecideParams& prm, hipStream_t stream) {
  DecideBatch<U> batch{};
  for (int i = 0; i < count; ++i) batch.u[i] = {unit[i].partials, unit[i].rec, unit[i].rows};
  hipLaunchKernelGGL((decide_kernel<K, U>), dim3(count), dim3(kDecideThreads), 0, stream, batch, prm);
  return hipGetLastError();
}

template <int K>
hipError_t decide_launch(const UnitDesc* unit, int count, const DecideParams& prm, hipStream_t stream) {
  if (count < 1 || count > batch_units<K>()) return hipErrorInvalidValue;
  return count == 1 ? decide_launch_u<K, 1>(unit, count, prm, stream)
                    : decide_launch_u<K, batch_units<K>()>(unit, count, prm, stream);
}

template <int K>
hipError_t gram_reduce_launch(const double* partials, int rows, double* gram, hipStream_t stream) {
  hipLaunchKernelGGL((gram_reduce_kernel<K>), dim3(1), dim3(kDecideThreads), 0, stream, partials, rows,
                     gram);
  return hipGetLastError();
}

template <int K>
hipError_t decide_gram_launch(const double* gram, UnitRecord* rec, const DecideParams& prm,
                              hipStream_t stream) {
  hipLaunchKernelGGL((decide_gram_kernel<K>), dim3(1), dim3(64), 0, stream, gram, rec, prm);
  return hipGetLastError();
}

template <int K, bool BF16>
hipError_t pattern_probe_launch(int blocks, int lds, float* theta, float* mom, void* const* reps, int64_t n,
                                hipStream_t stream) {
  MutPtrs<K> rp;
  for (int j = 0; j < K; ++j) rp.p[j] = reps[j];
  const int64_t nvec = n / Vec<BF16>::VE;
  hipLaunchKernelGGL((update_pattern_probe_kernel<K, BF16, kNT2>), dim3(blocks), dim3(kUpdateThreads), lds, stream,
                     theta, mom, rp, nvec, 0u);
  return hipGetLastError();
}

template <int K, bool BF16, int U>
hipError_t update_launch_u(const UnitDesc* unit, int count, int lds, double lr, double rho, hipStream_t stream) {
  UpdateBatch<K, U> batch{};
  std::fill_n(batch.first.at, U, INT32_MAX);
  batch.lr = lr;
  batch.rho = rho;
  int blocks = 0;
  for (int i = 0; i < count; ++i) {
    const UnitDesc& d = unit[i];
    UpdateUnit<K>& u = batch.u[i];
    u.theta = d.theta;
    u.mom = d.mom;
    for (int j = 0; j < K; ++j) u.reps.p[j] = d.n > 0 ? d.reps[j] : nullptr;
    u.rec = d.rec;
    u.nvec = d.n / Vec<BF16>::VE;
    u.n = d.n;
    batch.first.at[i] = blocks;
    u.blocks = d.update_blocks;
    if (d.update_blocks > INT32_MAX - blocks) return hipErrorInvalidValue;
    blocks += d.update_blocks;
  }
  hipLaunchKernelGGL((update_kernel<K, BF16, kNT2, U>), dim3(blocks), dim3(kUpdateThreads), lds, stream, batch);
  return hipGetLastError();
}

template <int K, bool BF16>
hipError_t update_launch(const UnitDesc* unit, int count, int lds, double lr, double rho, hipStream_t stream) {
  if (count < 1 || count > batch_units<K>()) return hipErrorInvalidValue;
  return count == 1 ? update_launch_u<K, BF16, 1>(unit, count, lds, lr, rho, stream)
                    : update_launch_u<K, BF16, batch_units<K>()>(unit, count, lds, lr, rho, stream);
}

// Vectors per thread of the one-pass kernel (measured: two 16-byte vectors
// of bf16 replicas, one of fp32; one above K = 16, where two would hold
// 2K 16-byte registers of replica data per lane).
template <int K, bool BF16>
constexpr int fused_v() {
  return BF16 && K <= 16 ? 2 : 1;
}

template <int K, bool BF16>
hipError_t fused_mean_launch(int rows, int lds, float* theta, float* mom, void* const* reps, double* partials,
                             int64_t n, double lr, double rho, hipStream_t stream) {
  MutPtrs<K> rp;
  for (int j = 0; j < K; ++j) rp.p[j] = reps[j];
  const int64_t nvec = n / Vec<BF16>::VE;
  hipLaunchKernelGGL((fused_mean_kernel<K, BF16, kNT2, fused_v<K, BF16>()>), dim3(rows), dim3(kFusedThreads),
                     lds, stream, theta, mom, rp, partials, nvec, n, lr, rho);
  return hipGetLastError();
}

template <int K, int U>
hipError_t fused_finish_launch_u(const FinishDesc* unit, int count, int sliced, hipStream_t stream) {
  FinishBatch<U> batch{};
  std::copy_n(unit, count, batch.u);
  if (sliced > 0) {
    hipLaunchKernelGGL((fused_fold_kernel<K, U>), dim3(kFoldSlices, sliced), dim3(kDecideThreads), 0, stream, batch);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((fused_finish_kernel<K, U>), dim3(count), dim3(kDecideThreads), 0, stream, batch);
  return hipGetLastError();
}

template <int K>
hipError_t fused_finish_launch(const FinishDesc* unit, int count, int sliced, hipStream_t stream) {
  if (count < 1 || count > kMaxFinishUnits || sliced < 0 || sliced > count) return hipErrorInvalidValue;
  return count == 1 ? fused_finish_launch_u<K, 1>(unit, count, sliced, stream)
                    : fused_finish_launch_u<K, kMaxFinishUnits>(unit, count, sliced, stream);
}

template <int K>
struct Launchers {
  static hipError_t gram(bool bf16, const UnitDesc* unit, int count, int max_blocks, hipStream_t stream) {
    return bf16 ? gram_launch<K, true>(unit, count, max_blocks, stream)
                : gram_launch<K, false>(unit, count, max_blocks, stream);
  }
  static hipError_t small_step(bool bf16, const UnitDesc* unit, int count, const DecideParams& prm, double lr,
                               double rho, hipStream_t stream) {
    return bf16 ? small_step_launch<K, true>(unit, count, prm, lr, rho, stream)
                : small_step_launch<K, false>(unit, count, prm, lr, rho, stream);
  }
  static hipError_t update(bool bf16, const UnitDesc* unit, int count, int lds, double lr, double rho,
                           hipStream_t stream) {
    return bf16 ? update_launch<K, true>(unit, count, lds, lr, rho, stream)
                : update_launch<K, false>(unit, count, lds, lr, rho, stream);
  }
  static hipError_t pattern_probe(bool bf16, int blocks, int lds, float* theta, float* mom, void* const* reps,
                                  int64_t n, hipStream_t stream) {
    return bf16 ? pattern_probe_launch<K, true>(blocks, lds, theta, mom, reps, n, stream)
                : pattern_probe_launch<K, false>(blocks, lds, theta, mom, reps, n, stream);
  }
  static hipError_t fused_mean(bool bf16, int rows, int lds, float* theta, float* mom, void* const* reps,
                               double* partials, int64_t n, double lr, double rho,
                               hipStream_t stream) {
    return bf16 ? fused_mean_launch<K, true>(rows, lds, theta, mom, reps, partials, n, lr, rho, stream)
                : fused_mean_launch<K, false>(rows, lds, theta, mom, reps, partials, n, lr, rho, stream);
  }
};

// The set of K, or nullptr when K lies outside this object's range (the
// discarded branch instantiates nothing).
template <int K>
const KernelSet* set_if_in_range() {
  if constexpr (K >= EDIT_K_FIRST && K <= EDIT_K_LAST) {
    static constexpr KernelSet set{
        &Launchers<K>::gram,   &decide_launch<K>,          &Launchers<K>::small_step, &gram_reduce_launch<K>,
        &decide_gram_launch<K>, &Launchers<K>::update,      &Launchers<K>::fused_mean, &fused_finish_launch<K>,
        &Launchers<K>::pattern_probe, batch_units<K>(), fused_v<K, true>(), fused_v<K, false>()};
    return &set;
  } else {
    return nullptr;
  }
}

}  // namespace

#define EDIT_FOR_EACH_K(X)                                                                       \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17)   \
  X(18) X(19) X(20) X(21) X(22) X(23) X(24) X(25) X(26) X(27) X(28) X(29) X(30) X(31) X(32)

const KernelSet* EDIT_KERNEL_SET_FN(EDIT_K_FIRST)(int K) {
  switch (K) {
#define EDIT_CASE(KK) \
  case KK:            \
    return set_if_in_range<KK>();
    EDIT_FOR_EACH_K(EDIT_CASE)
#undef EDIT_CASE
    default:
      return nullptr;
  }
}

#if EDIT_K_FIRST == 1  // the copy probe is compiled into one object only
constexpr int kUnrollCopy = 1;
constexpr bool kNTCopy = false;

hipError_t launch_copy(void* dst, const void* src, int64_t nbytes, int blocks, hipStream_t stream) {
  hipLaunchKernelGGL((copy_kernel<kUnrollCopy, kNTCopy>), dim3(blocks), dim3(kCopyThreads), 0, stream,
                     reinterpret_cast<u32x4*>(dst), reinterpret_cast<const u32x4*>(src), nbytes / 16);
  return hipGetLastError();
}
#endif

}  // namespace edit
