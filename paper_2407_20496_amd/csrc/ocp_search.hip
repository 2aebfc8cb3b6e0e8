// Output-channel permutation search of gyro-permutation (arXiv 2407.20496, Section 4.1 Eq. 2 and
// Section 4.2): the output channels are re-distributed over the tiles of V channels so that
// column-vector pruning removes as little saliency as possible.  One iteration:
//   sampling   : the same number n of channels leaves every tile (positions given by the caller);
//   clustering : the T n sampled channels are grouped into T clusters of n (given by the caller; by
//                default every tile's own samples -- the balanced K-means of the paper is not part
//                of this file);
//   cost       : Eq. 4, cost[i][j] = saliency vector pruning removes from tile i's remaining channels
//                plus cluster j = the sum of the K - Kv smallest column scores, a score being
//                (sum over the remaining channels) + (sum over the cluster's channels) in binary64;
//   assignment : clusters -> tiles at minimal total cost (the solver of the tile-wise search);
//   apply      : the channels of cluster assign[i] fill the positions tile i vacated, in order.
// Indices read from the caller's arrays (positions, cluster items, channels) are clamped into range
// before use, so malformed input gives a meaningless order but no access out of bounds.
#include "hinm_internal.h"
#include "wave_reduce.h"

namespace hinm {
namespace {

constexpr int kThreads = 256;

template <int DT>
__device__ __forceinline__ double saliency_at(const uint16_t* W, const float* rho, size_t idx) {
  return rho ? (double)rho[idx] : (double)__builtin_fabsf(bits_to_float<DT>(W[idx]));
}

__device__ __forceinline__ int clamp_index(int x, int n) { return x < 0 ? 0 : (x >= n ? n - 1 : x); }

// base[t][k] = sum over the positions of tile t that stay (ascending position) of the saliency in
// column k; cluster[t][k] = the same over the channels of cluster t (cluster order).  The rows' numbers are looked up once a
// workgroup and sixteen rows are requested before the first is added: with one row at a time, each behind its look-up and
// the one before, 96 tiles of 32 rows and 768 columns took 13.9 us, 6.6 here (16384 x 16384, V = 128 365 -> 237, magnitudes of W
// 312 -> 115).  Which of the two is read is settled outside the loops: chosen at every read, each read of W waited for the one
// before (16384 x 16384 317 us, 512 tiles of 32 rows, 2048 columns 36 against 21).  LDS for what the tile has and no more: with room
// for 4096 rows a unit held four workgroups (256 tiles of 32 rows, 8192 columns 72 us, 57 here; W 139 and 39).
constexpr int kSumRows = 16;
inline size_t ocp_sums_lds_bytes(int V, int n) { return (size_t)V * 5 + (size_t)n * 4; }
template <int DT>
__global__ __launch_bounds__(kThreads) void ocp_sums_kernel(const uint16_t* __restrict__ W,
                                                            const float* __restrict__ rho,
                                                            const int32_t* __restrict__ row_order,
                                                            const int32_t* __restrict__ samples,
                                                            const int32_t* __restrict__ clusters,
                                                            double* __restrict__ base, double* __restrict__ cluster,
                                                            int T, int K, int V, int n) {
  extern __shared__ int32_t sums_lds[];  // ocp_sums_lds_bytes
  int32_t* const row_of = sums_lds;
  int32_t* const come_row = row_of + V;
  uint8_t* const leaves = reinterpret_cast<uint8_t*>(come_row + n);
  const int t = blockIdx.x;
  for (int p = threadIdx.x; p < V; p += kThreads) {
    leaves[p] = 0;
    row_of[p] = clamp_index(row_order[(size_t)t * V + p], T * V);
  }
  for (int e = threadIdx.x; e < n; e += kThreads) {
    const int q = clusters ? clamp_index(clusters[(size_t)t * n + e], T * n) : t * n + e;
    const int tq = q / n, eq = q % n;
    come_row[e] = clamp_index(row_order[(size_t)tq * V + clamp_index(samples[(size_t)tq * n + eq], V)], T * V);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < n; e += kThreads) leaves[clamp_index(samples[(size_t)t * n + e], V)] = 1;
  __syncthreads();
  const int k = blockIdx.y * kThreads + threadIdx.x;
  if (k >= K) return;
  double stay = 0.0, come = 0.0;
  auto add_rows = [&](auto load, auto saliency) {
    for (int p0 = 0; p0 < V; p0 += kSumRows) {
      decltype(load(0)) x[kSumRows];
#pragma unroll
      for (int r = 0; r < kSumRows; ++r) x[r] = load(row_of[min(p0 + r, V - 1)]);
#pragma unroll
      for (int r = 0; r < kSumRows; ++r)
        if (p0 + r < V && !leaves[p0 + r]) stay += saliency(x[r]);
    }
    for (int e0 = 0; e0 < n; e0 += 4) {
      decltype(load(0)) x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = load(come_row[min(e0 + r, n - 1)]);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (e0 + r < n) come += saliency(x[r]);
    }
  };
  if (rho) add_rows([&](int row) { return rho[(size_t)row * K + k]; }, [](float x) { return (double)x; });
  else
    add_rows([&](int row) { return W[(size_t)row * K + k]; },
             [](uint16_t x) { return (double)__builtin_fabsf(bits_to_float<DT>(x)); });
  base[(size_t)t * K + k] = stay;
  cluster[(size_t)t * K + k] = come;
}

__device__ __forceinline__ unsigned long long ordered_key(double x) {
  const unsigned long long bits = (unsigned long long)__double_as_longlong(x);
  return (bits >> 63) ? ~bits : (bits | (1ull << 63));
}
__device__ __forceinline__ double key_value(unsigned long long key) {
  const unsigned long long bits = (key >> 63) ? (key & ~(1ull << 63)) : ~key;
  return __longlong_as_double((long long)bits);
}

// Workgroup-wide sum of one int per thread.  Three counters are used in rotation: every call clears
// the counter of the next call before its own barrier, when every thread has long left the call
// that read it last.
__device__ __forceinline__ int block_count(int local, int* counters, int call) {
  local = wave_sum(local);
  if (threadIdx.x == 0) counters[(call + 1) % 3] = 0;
  if ((threadIdx.x & 63) == 0) atomicAdd(&counters[call % 3], local);
  __syncthreads();
  return counters[call % 3];
}

// One workgroup per (tile i, cluster j): the K column scores live in registers (KPT per thread) as
// order-preserving 64-bit keys, split into two 32-bit words.  The Kv-th largest key is found bit by
// bit with 64 workgroup-wide counting passes -- 32 on the high words, then 32 on the low words of
// the keys whose high word equals the threshold's (the others have their low word cleared, and a
// candidate always has a bit set) -- so every pass is one full-rate 32-bit compare and one add per
// key.  A candidate with exactly Kv keys at or above it separates them: no further bit changes the sum,
// and without ties that takes some 20 passes instead of 65 (each is a barrier and an LDS round trip:
// 48 x 48 pairs of 768 columns 35.6 -> 21.5 us).  Then everything below the threshold, plus the surplus of
// scores equal to it, is summed.
template <int KPT>
__global__ __launch_bounds__(kThreads) void ocp_cost_kernel(const double* __restrict__ base,
                                                            const double* __restrict__ cluster,
                                                            double* __restrict__ cost, int T, int K, int Kv) {
  __shared__ int counters[3];
  __shared__ double wave_sum_f64[kThreads / 64];
  const int j = blockIdx.x, i = blockIdx.y;
  const double* b = base + (size_t)i * K;
  const double* c = cluster + (size_t)j * K;
  uint32_t hi[KPT], lo[KPT];
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    const int k = q * kThreads + threadIdx.x;
    const unsigned long long key = (k < K) ? ordered_key(b[k] + c[k]) : 0ull;  // key 0: never counted below
    hi[q] = (uint32_t)(key >> 32);
    lo[q] = (uint32_t)key;
  }
  if (threadIdx.x < 3) counters[threadIdx.x] = 0;
  __syncthreads();
  int call = 0;
  int count = 0;
  uint32_t tau_hi = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = tau_hi | (1u << bit);
    int local = 0;
#pragma unroll
    for (int q = 0; q < KPT; ++q) local += (hi[q] >= cand) ? 1 : 0;
    count = block_count(local, counters, call++);
    if (count >= Kv) tau_hi = cand;
    if (count == Kv) break;
  }
  const bool separated = count == Kv;
  // keys above the threshold's high word always count; those below never do
  uint32_t tau_lo = 0;
  if (!separated) {
    int above_hi = 0;
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      above_hi += (hi[q] > tau_hi) ? 1 : 0;
      lo[q] = (hi[q] == tau_hi) ? lo[q] : 0u;  // in place: the last pass reads the scores again
    }
    const int need = Kv - block_count(above_hi, counters, call++);  // >= 1 by the choice of tau_hi
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t cand = tau_lo | (1u << bit);
      int local = 0;
#pragma unroll
      for (int q = 0; q < KPT; ++q) local += (lo[q] >= cand) ? 1 : 0;
      const int enough = block_count(local, counters, call++);
      if (enough >= need) tau_lo = cand;
      if (enough == need) break;
    }
  }
  // the Kv-th largest key, or a bound below it and above the next one
  const unsigned long long tau = ((unsigned long long)tau_hi << 32) | tau_lo;
  int above = 0, equal = 0;
  double below = 0.0;
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    const int k = q * kThreads + threadIdx.x;
    if (k < K) {
      const unsigned long long key = ordered_key(b[k] + c[k]);
      above += key > tau ? 1 : 0;
      equal += key == tau ? 1 : 0;
      if (key < tau) below += key_value(key);
    }
  }
  const int n_above = block_count(above, counters, call++);
  const int n_equal = block_count(equal, counters, call++);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) below += __shfl_xor(below, off);
  if ((threadIdx.x & 63) == 0) wave_sum_f64[threadIdx.x >> 6] = below;
  __syncthreads();
  if (threadIdx.x == 0) {
    double total = 0.0;
    for (int w = 0; w < kThreads / 64; ++w) total += wave_sum_f64[w];
    const int pruned_equal = n_equal - (Kv - n_above);  // scores equal to the threshold that do not survive
    if (pruned_equal > 0) total += (double)pruned_equal * key_value(tau);
    cost[(size_t)i * T + j] = total;
  }
}

// The same for up to 1024 columns, one wave per pair of tile and cluster: a pass counts with one compare a key whose lane mask
// is counted by scalar instructions, and there is no barrier in it.  48 x 48 pairs of 768 columns 21.5 us with a workgroup a
// pair, 13.7 here.
template <int KPT>
__global__ __launch_bounds__(kThreads) void ocp_cost_wave_kernel(const double* __restrict__ base,
                                                                 const double* __restrict__ cluster,
                                                                 double* __restrict__ cost, int T, int K, int Kv) {
  const int lane = threadIdx.x & 63;
  const int pair = __builtin_amdgcn_readfirstlane(blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6));
  if (pair >= T * T) return;
  const int i = pair / T, j = pair % T;
  const double* b = base + (size_t)i * K;
  const double* c = cluster + (size_t)j * K;
  double score[KPT];
  uint32_t hi[KPT];
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    const int k = min(q * 64 + lane, K - 1);
    score[q] = b[k] + c[k];
  }
#pragma unroll
  for (int q = 0; q < KPT; ++q) hi[q] = q * 64 + lane < K ? (uint32_t)(ordered_key(score[q]) >> 32) : 0u;
  int count = 0;
  uint32_t tau_hi = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = tau_hi | (1u << bit);
    count = 0;
#pragma unroll
    for (int q = 0; q < KPT; ++q) count += __popcll(__ballot(hi[q] >= cand));
    if (count >= Kv) tau_hi = cand;
    if (count == Kv) break;
  }
  uint32_t tau_lo = 0;
  if (count != Kv) {  // the low words of the keys that share the threshold's high word
    int need = Kv;
    uint32_t lo[KPT];
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      need -= __popcll(__ballot(hi[q] > tau_hi));
      lo[q] = hi[q] == tau_hi && q * 64 + lane < K ? (uint32_t)ordered_key(score[q]) : 0u;
    }
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t cand = tau_lo | (1u << bit);
      int enough = 0;
#pragma unroll
      for (int q = 0; q < KPT; ++q) enough += __popcll(__ballot(lo[q] >= cand));
      if (enough >= need) tau_lo = cand;
      if (enough == need) break;
    }
  }
  const unsigned long long tau = ((unsigned long long)tau_hi << 32) | tau_lo;
  int above = 0, equal = 0;
  double below = 0.0;
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    const bool there = q * 64 + lane < K;
    const unsigned long long key = ordered_key(score[q]);
    above += __popcll(__ballot(there && key > tau));
    equal += __popcll(__ballot(there && key == tau));
    if (there && key < tau) below += score[q];
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) below += __shfl_xor(below, off);
  if (lane == 0) {
    const int pruned_equal = equal - (Kv - above);  // scores equal to the threshold that do not survive
    if (pruned_equal > 0) below += (double)pruned_equal * key_value(tau);
    cost[(size_t)i * T + j] = below;
  }
}

// The same with whole 64-bit keys and 64 passes of 64-bit compares (a quarter of the 32-bit rate): with
// 64 keys per thread the split form needs more registers than it saves time (measured 2.5 ms against
// 1.8 ms on a 16384-column layer), so the widest configuration keeps this form.
template <int KPT>
__global__ __launch_bounds__(kThreads) void ocp_cost_wide_kernel(const double* __restrict__ base,
                                                            const double* __restrict__ cluster,
                                                            double* __restrict__ cost, int T, int K, int Kv) {
  __shared__ int counters[3];
  __shared__ double wave_sum_f64[kThreads / 64];
  const int j = blockIdx.x, i = blockIdx.y;
  const double* b = base + (size_t)i * K;
  const double* c = cluster + (size_t)j * K;
  unsigned long long key[KPT];
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    const int k = q * kThreads + threadIdx.x;
    key[q] = (k < K) ? ordered_key(b[k] + c[k]) : 0ull;  // key 0 is below every real score's key
  }
  if (threadIdx.x < 3) counters[threadIdx.x] = 0;
  __syncthreads();
  int call = 0;
  unsigned long long tau = 0ull;  // becomes the Kv-th largest key, or a bound below it and above the next one
  for (int bit = 63; bit >= 0; --bit) {
    const unsigned long long cand = tau | (1ull << bit);
    int local = 0;
#pragma unroll
    for (int q = 0; q < KPT; ++q) local += (key[q] >= cand) ? 1 : 0;
    const int count = block_count(local, counters, call++);
    if (count >= Kv) tau = cand;
    if (count == Kv) break;
  }
  int above = 0, equal = 0;
  double below = 0.0;
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    const int k = q * kThreads + threadIdx.x;
    if (k < K) {
      above += key[q] > tau ? 1 : 0;
      equal += key[q] == tau ? 1 : 0;
      if (key[q] < tau) below += key_value(key[q]);
    }
  }
  const int n_above = block_count(above, counters, call++);
  const int n_equal = block_count(equal, counters, call++);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) below += __shfl_xor(below, off);
  if ((threadIdx.x & 63) == 0) wave_sum_f64[threadIdx.x >> 6] = below;
  __syncthreads();
  if (threadIdx.x == 0) {
    double total = 0.0;
    for (int w = 0; w < kThreads / 64; ++w) total += wave_sum_f64[w];
    const int pruned_equal = n_equal - (Kv - n_above);  // scores equal to the threshold that do not survive
    if (pruned_equal > 0) total += (double)pruned_equal * key_value(tau);
    cost[(size_t)i * T + j] = total;
  }
}

// moved[i][e] = the channel of cluster assign[i], item e; block 0 also reports the total cost.
__global__ __launch_bounds__(kThreads) void ocp_moved_kernel(const double* __restrict__ cost,
                                                             const int32_t* __restrict__ assign,
                                                             const int32_t* __restrict__ row_order,
                                                             const int32_t* __restrict__ samples,
                                                             const int32_t* __restrict__ clusters,
                                                             int32_t* __restrict__ moved, double* __restrict__ objective,
                                                             int T, int V, int n) {
  __shared__ double picked[kThreads];
  const int i = blockIdx.x;
  const int j = clamp_index(assign[i], T);
  for (int e = threadIdx.x; e < n; e += kThreads) {
    const int q = clusters ? clamp_index(clusters[(size_t)j * n + e], T * n) : j * n + e;
    const int tq = q / n, eq = q % n;
    moved[(size_t)i * n + e] = row_order[(size_t)tq * V + clamp_index(samples[(size_t)tq * n + eq], V)];
  }
  if (objective && i == 0) {  // tiles in ascending order, looked up by all threads
    double total = 0.0;
    for (int r0 = 0; r0 < T; r0 += kThreads) {
      const int r = r0 + threadIdx.x;
      __syncthreads();
      picked[threadIdx.x] = r < T ? cost[(size_t)r * T + clamp_index(assign[r], T)] : 0.0;
      __syncthreads();
      if (threadIdx.x == 0) {
        const int count = min(kThreads, T - r0);
#pragma unroll 8
        for (int e = 0; e < count; ++e) total += picked[e];
      }
    }
    if (threadIdx.x == 0) *objective = total;
  }
}

__global__ __launch_bounds__(kThreads) void ocp_write_kernel(const int32_t* __restrict__ moved,
                                                             const int32_t* __restrict__ samples,
                                                             int32_t* __restrict__ row_order, int V, int n) {
  const int i = blockIdx.x;
  for (int e = threadIdx.x; e < n; e += kThreads)
    row_order[(size_t)i * V + clamp_index(samples[(size_t)i * n + e], V)] = moved[(size_t)i * n + e];
}

// ---------------------------------------------------------------------------------------------
// Clustering phase (Section 4.2 names balanced K-means without detail; this is one reading): the
// T n sampled channels are the points, their saliency rows the features; T clusters of exactly n
// points.  A round = squared Euclidean distances in binary64 (columns in ascending order, separate
// multiply and add), a minimal-cost assignment of the points to the T n (cluster, slot) pairs, and
// centroids = sum of the members in ascending item order, divided by n.
// ---------------------------------------------------------------------------------------------
template <int DT>
__global__ __launch_bounds__(kThreads) void km_features_kernel(const uint16_t* __restrict__ W,
                                                               const float* __restrict__ rho,
                                                               const int32_t* __restrict__ row_order,
                                                               const int32_t* __restrict__ samples,
                                                               float* __restrict__ F, int T, int K, int V, int n) {
  const int q = blockIdx.x;
  const int k = blockIdx.y * kThreads + threadIdx.x;
  if (k >= K) return;
  const int t = q / n, e = q % n;
  const size_t row = (size_t)clamp_index(row_order[(size_t)t * V + clamp_index(samples[(size_t)t * n + e], V)], T * V);
  F[(size_t)q * K + k] = (float)saliency_at<DT>(W, rho, row * K + k);
}

__global__ __launch_bounds__(kThreads) void km_init_kernel(const float* __restrict__ F, double* __restrict__ C, int K,
                                                           int n) {
  const int c = blockIdx.x;
  const int k = blockIdx.y * kThreads + threadIdx.x;
  if (k < K) C[(size_t)c * K + k] = (double)F[(size_t)c * n * K + k];
}

// d[q][c] for 64 clusters (one a lane) and one point a wave.  A chain of K steps per pair is the definition (the
// rounding of every step is pinned), so the chains have to run on operands that are at hand: 32 columns of the
// centroids at a time go through LDS (two pieces in turn, the next one requested ahead; rows padded to an odd number of
// doubles: no bank conflicts), and a piece of a point's features is held by 32 lanes, each read from its lane as a scalar.
// 384 points x 48 clusters x 768 columns: 76 us with one column of a different centroid row per lane and step, 26.5 us with
// the features as scalar loads (they share a counter with the LDS reads, which makes every one wait for all), 21.0 here.
constexpr int kDistColumns = 32;
__global__ __launch_bounds__(kThreads) void km_distance_kernel(const float* __restrict__ F,
                                                               const double* __restrict__ C,
                                                               double* __restrict__ dist, int T, int K, int points) {
#pragma clang fp contract(off)  // product and sum are rounded separately: that rounding is part of the definition
  __shared__ double tile[2][64][kDistColumns + 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c0 = blockIdx.y * 64;
  const int q = blockIdx.x * (kThreads / 64) + wave;
  const int column = threadIdx.x % kDistColumns, row = threadIdx.x / kDistColumns;
  const float* const f = F + (size_t)min(q, points - 1) * K;
  double acc = 0.0;
  constexpr int kRows = kThreads / kDistColumns;  // of a piece, at a time
  constexpr int kPieces = 64 / kRows;
  double ahead[kPieces];
  float f_ahead;
  auto request = [&](int k0) {
    const int k = min(k0 + column, K - 1);
#pragma unroll
    for (int r = 0; r < kPieces; ++r) ahead[r] = C[(size_t)min(c0 + row + r * kRows, T - 1) * K + k];
    f_ahead = f[k];  // (column is the lane's, too)
  };
  auto put = [&](int at) {
#pragma unroll
    for (int r = 0; r < kPieces; ++r) tile[at][row + r * kRows][column] = ahead[r];
  };
  request(0);
  put(0);
  int at = 0;
  for (int k0 = 0; k0 < K; k0 += kDistColumns) {
    const double mine = (double)f_ahead;
    __syncthreads();  // this piece is there, and nobody reads the one before it
    if (k0 + kDistColumns < K) request(k0 + kDistColumns);
    auto square = [&](double cen, int k) {
      const double x = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(mine), k),
                                        __builtin_amdgcn_readlane(__double2loint(mine), k));
      const double diff = x - cen;
      return diff * diff;
    };
    if (k0 + kDistColumns <= K) {
      // the squares of the next four columns between the sums of these: a lone wave issues in order
      constexpr int kAhead = 4;
      double cen[2 * kAhead], sq[2][kAhead];
#pragma unroll
      for (int e = 0; e < 2 * kAhead; ++e) cen[e] = tile[at][lane][e];
#pragma unroll
      for (int e = 0; e < kAhead; ++e) sq[0][e] = square(cen[e], e);
#pragma unroll
      for (int k = 0; k < kDistColumns; k += kAhead) {
        const int now = (k / kAhead) & 1;
        double after[kAhead];
#pragma unroll
        for (int e = 0; e < kAhead; ++e)
          if (k + 2 * kAhead < kDistColumns) after[e] = tile[at][lane][k + 2 * kAhead + e];
#pragma unroll
        for (int e = 0; e < kAhead; ++e) {
          acc = acc + sq[now][e];
          if (k + kAhead < kDistColumns) sq[now ^ 1][e] = square(cen[kAhead + e], k + kAhead + e);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int e = 0; e < kAhead; ++e) cen[kAhead + e] = after[e];
      }
    } else {
      for (int k = 0; k < K - k0; ++k) acc = acc + square(tile[at][lane][k], k);
    }
    at ^= 1;
    if (k0 + kDistColumns < K) put(at);
  }
  if (c0 + lane < T && q < points) dist[(size_t)q * T + c0 + lane] = acc;
}

// The same with two points a wave, for more than three workgroups a unit of the kernel above: there instructions count, and features
// as scalar loads cost none.  256 x 4 points to 256 clusters, 2048 columns 131 us above, 125 here, 512 x 2 to 512 244 and 209; but 192 x
// 5 to 192 (720 workgroups above) 105 and 125, 128 x 8 to 128 78 and 119.
constexpr int kManyColumns = 64, kManyPoints = 2;
__global__ __launch_bounds__(kThreads) void km_distance_many_kernel(const float* __restrict__ F,
                                                                    const double* __restrict__ C,
                                                                    double* __restrict__ dist, int T, int K, int points) {
#pragma clang fp contract(off)  // product and sum are rounded separately: that rounding is part of the definition
  __shared__ double tile[64][kManyColumns + 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c0 = blockIdx.y * 64;
  const int q0 = (blockIdx.x * (kThreads / 64) + wave) * kManyPoints;
  const float* f[kManyPoints];
  double acc[kManyPoints];
#pragma unroll
  for (int p = 0; p < kManyPoints; ++p) {
    f[p] = F + (size_t)min(q0 + p, points - 1) * K;
    acc[p] = 0.0;
  }
  constexpr int kPieces = 64 / (kThreads / 64);
  double ahead[kPieces];
  auto request = [&](int k0) {
    const int k_lane = min(k0 + lane, K - 1);
#pragma unroll
    for (int r = 0; r < kPieces; ++r)
      ahead[r] = C[(size_t)min(c0 + wave + r * (kThreads / 64), T - 1) * K + k_lane];
  };
  request(0);
  for (int k0 = 0; k0 < K; k0 += kManyColumns) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPieces; ++r) tile[wave + r * (kThreads / 64)][lane] = ahead[r];
    __syncthreads();
    if (k0 + kManyColumns < K) request(k0 + kManyColumns);
    const int count = min(kManyColumns, K - k0);
    if (count == kManyColumns) {
#pragma unroll 16
      for (int k = 0; k < kManyColumns; ++k) {
        const double cen = tile[lane][k];
#pragma unroll
        for (int p = 0; p < kManyPoints; ++p) {
          const double diff = (double)f[p][k0 + k] - cen;
          const double sq = diff * diff;
          acc[p] = acc[p] + sq;
        }
      }
    } else {
      for (int k = 0; k < count; ++k) {
        const double cen = tile[lane][k];
#pragma unroll
        for (int p = 0; p < kManyPoints; ++p) {
          const double diff = (double)f[p][k0 + k] - cen;
          const double sq = diff * diff;
          acc[p] = acc[p] + sq;
        }
      }
    }
  }
  if (c0 + lane < T) {
#pragma unroll
    for (int p = 0; p < kManyPoints; ++p)
      if (q0 + p < points) dist[(size_t)(q0 + p) * T + c0 + lane] = acc[p];
  }
}

// New centroids and cluster lists from the assignment (point q belongs to cluster assign[q] / n): every workgroup
// finds its cluster's members, in ascending item order, with one pass over the assignment and then reads their
// features only.  Block (0, 0) also reports the sum of the distances of the points to the centroids they were
// assigned to.
__global__ __launch_bounds__(kThreads) void km_update_kernel(const float* __restrict__ F,
                                                             const int32_t* __restrict__ assign,
                                                             const double* __restrict__ dist, double* __restrict__ C,
                                                             int32_t* __restrict__ clusters,
                                                             double* __restrict__ objective, int T, int K, int n) {
  __shared__ int members[kIcpMaxPartitions];
  __shared__ int wave_count[kThreads / 64];
  const int c = blockIdx.x;
  const int k = blockIdx.y * kThreads + threadIdx.x;
  const int points = T * n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int filled = 0;
  for (int q0 = 0; q0 < points; q0 += kThreads) {
    const int q = q0 + threadIdx.x;
    const bool in = q < points && clamp_index(assign[q], points) / n == c;
    const unsigned long long mask = __ballot(in);
    if (lane == 0) wave_count[wave] = __popcll(mask);
    __syncthreads();
    int at = filled + __popcll(mask & ((1ull << lane) - 1ull));
    for (int w = 0; w < kThreads / 64; ++w) {
      if (w < wave) at += wave_count[w];
      filled += wave_count[w];
    }
    if (in) members[at] = q;
    __syncthreads();
  }
  if (k < K) {
    double acc = 0.0;
#pragma unroll 4
    for (int e = 0; e < filled; ++e) acc += (double)F[(size_t)members[e] * K + k];
    C[(size_t)c * K + k] = acc / (double)n;
  }
  if (blockIdx.y == 0)
    for (int e = threadIdx.x; e < n; e += kThreads)
      clusters[(size_t)c * n + e] = e < filled ? members[e] : c * n + e;  // the latter only after a malformed assignment
  if (objective && c == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    double total = 0.0;
    for (int q = 0; q < points; ++q) total += dist[(size_t)q * T + clamp_index(assign[q], points) / n];
    *objective = total;
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

KmeansWorkspace kmeans_workspace_layout(const hinm_shape& s, int n_samples) {
  const size_t T = s.M / s.V, points = T * (size_t)n_samples;
  KmeansWorkspace w;
  size_t off = 0;
  w.features = off; off += align256(points * s.K * sizeof(float));
  w.dist = off;     off += align256(points * T * sizeof(double));
  w.assign = off;   off += align256(points * sizeof(int32_t));
  w.total_bytes = off;
  return w;
}

hipError_t launch_ocp_cluster(const KmeansArgs& a, hipStream_t stream) {
  const hinm_shape& s = a.s;
  const int T = s.M / s.V, n = a.n_samples, points = T * n;
  const KmeansWorkspace w = kmeans_workspace_layout(s, n);
  uint8_t* ws = static_cast<uint8_t*>(a.workspace);
  float* F = reinterpret_cast<float*>(ws + w.features);
  double* dist = reinterpret_cast<double*>(ws + w.dist);
  int32_t* assign = reinterpret_cast<int32_t*>(ws + w.assign);
  const uint16_t* Wb = static_cast<const uint16_t*>(a.W);
  const int k_blocks = (s.K + kThreads - 1) / kThreads;
  if (s.dtype == HINM_F16)
    km_features_kernel<HINM_F16><<<dim3(points, k_blocks), kThreads, 0, stream>>>(Wb, a.rho, a.row_order, a.samples, F, T,
                                                                                   s.K, s.V, n);
  else
    km_features_kernel<HINM_BF16><<<dim3(points, k_blocks), kThreads, 0, stream>>>(Wb, a.rho, a.row_order, a.samples, F,
                                                                                    T, s.K, s.V, n);
  if (a.init_centroids) km_init_kernel<<<dim3(T, k_blocks), kThreads, 0, stream>>>(F, a.centroids, s.K, n);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  for (int r = 0; r < a.rounds; ++r) {
    constexpr int kWaves = kThreads / 64;
    const int cluster_blocks = (T + 63) / 64;
    const int ones = (points + kWaves - 1) / kWaves;
    if (ones * cluster_blocks <= 3 * 256)
      km_distance_kernel<<<dim3(ones, cluster_blocks), kThreads, 0, stream>>>(F, a.centroids, dist, T, s.K, points);
    else
      km_distance_many_kernel<<<dim3((ones + kManyPoints - 1) / kManyPoints, cluster_blocks), kThreads, 0, stream>>>(
          F, a.centroids, dist, T, s.K, points);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_assignment(dist, assign, 1, points, T, stream);
    if (e != hipSuccess) return e;
    km_update_kernel<<<dim3(T, k_blocks), kThreads, 0, stream>>>(F, assign, dist, a.centroids, a.clusters,
                                                                 a.objective ? a.objective + r : nullptr, T, s.K, n);
  }
  return hipGetLastError();
}

OcpWorkspace ocp_workspace_layout(const hinm_shape& s, int n_samples) {
  const size_t T = s.M / s.V;
  OcpWorkspace w;
  size_t off = 0;
  w.base = off;    off += align256(T * s.K * sizeof(double));
  w.cluster = off; off += align256(T * s.K * sizeof(double));
  w.cost = off;    off += align256(T * T * sizeof(double));
  w.assign = off;  off += align256(T * sizeof(int32_t));
  w.moved = off;   off += align256(T * (size_t)n_samples * sizeof(int32_t));
  w.total_bytes = off;
  return w;
}

hipError_t launch_ocp_search(const OcpArgs& a, hipStream_t stream) {
  const hinm_shape& s = a.s;
  const int T = s.M / s.V, n = a.n_samples;
  const OcpWorkspace w = ocp_workspace_layout(s, n);
  uint8_t* ws = static_cast<uint8_t*>(a.workspace);
  double* base = reinterpret_cast<double*>(ws + w.base);
  double* cluster = reinterpret_cast<double*>(ws + w.cluster);
  double* cost = reinterpret_cast<double*>(ws + w.cost);
  int32_t* assign = reinterpret_cast<int32_t*>(ws + w.assign);
  int32_t* moved = reinterpret_cast<int32_t*>(ws + w.moved);
  const uint16_t* Wb = static_cast<const uint16_t*>(a.W);
  const dim3 sums_grid(T, (s.K + kThreads - 1) / kThreads);
  const size_t sums_lds = ocp_sums_lds_bytes(s.V, n);
  const dim3 cost_grid(T, T);
  for (int it = 0; it < a.iters; ++it) {
    const int32_t* smp = a.samples + (size_t)it * T * n;
    const int32_t* cl = a.clusters ? a.clusters + (size_t)it * T * n : nullptr;
    if (s.dtype == HINM_F16)
      ocp_sums_kernel<HINM_F16><<<sums_grid, kThreads, sums_lds, stream>>>(Wb, a.rho, a.row_order, smp, cl, base, cluster, T,
                                                                     s.K, s.V, n);
    else
      ocp_sums_kernel<HINM_BF16><<<sums_grid, kThreads, sums_lds, stream>>>(Wb, a.rho, a.row_order, smp, cl, base, cluster, T,
                                                                      s.K, s.V, n);
    const int pair_blocks = (T * T + kThreads / 64 - 1) / (kThreads / 64);
    if (s.K <= 512) ocp_cost_wave_kernel<8><<<pair_blocks, kThreads, 0, stream>>>(base, cluster, cost, T, s.K, s.Kv);
    else if (s.K <= 1024) ocp_cost_wave_kernel<16><<<pair_blocks, kThreads, 0, stream>>>(base, cluster, cost, T, s.K, s.Kv);
    else if (s.K <= 16 * kThreads) ocp_cost_kernel<16><<<cost_grid, kThreads, 0, stream>>>(base, cluster, cost, T, s.K, s.Kv);
    else ocp_cost_wide_kernel<64><<<cost_grid, kThreads, 0, stream>>>(base, cluster, cost, T, s.K, s.Kv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_assignment(cost, assign, 1, T, T, stream);
    if (e != hipSuccess) return e;
    ocp_moved_kernel<<<T, kThreads, 0, stream>>>(cost, assign, a.row_order, smp, cl, moved,
                                                 a.objective ? a.objective + it : nullptr, T, s.V, n);
    ocp_write_kernel<<<T, kThreads, 0, stream>>>(moved, smp, a.row_order, s.V, n);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace hinm
