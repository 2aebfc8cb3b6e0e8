// Tile-wise input-channel permutation search of gyro-permutation (arXiv 2407.20496, Section 4.1
// Eq. 3 and Section 4.2): the kept column vectors of every tile are re-arranged so that the 2:4 step
// prunes as little saliency as possible.  Every four consecutive kept vectors form one partition.
// One iteration, per tile:
//   sampling   : one vector per partition, chosen by the caller (`samples`);
//   cost       : Eq. 4, cost[i][j] = saliency the 2:4 step prunes in partition i when the slot it
//                vacated holds sample j = sum over rows of the two smallest of four values, added in
//                binary64 in ascending row order.  With (m1, m2) the two smallest of partition i's
//                three remaining values this is sum_r m1 + min(sample_j, m2): a (min, +) contraction
//                over the V rows, the data-parallel part of the search;
//   assignment : samples -> partitions minimising the total cost (shortest augmenting paths with row
//                and column potentials, one wave per tile: assignment.hip);
//   apply      : every sample moves into the slot its partition vacated.
// The arrangement is tracked as a permutation of the slots of the incoming vector index, so the
// saliencies are gathered from W (or rho) only once.
#include "hinm_internal.h"

namespace hinm {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxP = kIcpMaxPartitions;
// block of the cost matrix per workgroup: 64 samples (one a lane) x 16 partitions (four a wave), 64 rows at a time
constexpr int kCostSamples = 64;
constexpr int kCostPartitionsPerWave = 4;
constexpr int kCostPartitions = kCostPartitionsPerWave * (kThreads / 64);
constexpr int kCostRows = 64;

// G[t][r][slot] = saliency of W[tV + r][vec_idx[t][slot]]: the caller's rho, or |w|; order = identity
template <int DT>
__global__ __launch_bounds__(kThreads) void icp_gather_kernel(const uint16_t* __restrict__ W,
                                                              const float* __restrict__ rho,
                                                              const int32_t* __restrict__ vec_idx,
                                                              float* __restrict__ G, int32_t* __restrict__ order,
                                                              int K, int V, int Kv) {
  const int t = blockIdx.x, r = blockIdx.y;
  const size_t row = (size_t)t * V + r;
  const int32_t* vi = vec_idx + (size_t)t * Kv;
  float* g = G + row * Kv;
  for (int s = threadIdx.x; s < Kv; s += kThreads) {
    const int c = vi[s];
    g[s] = rho ? rho[row * K + c] : __builtin_fabsf(bits_to_float<DT>(W[row * K + c]));
    if (r == 0) order[(size_t)t * Kv + s] = s;
  }
}

// Per row and partition: the sampled value, and the two smallest of the three remaining ones.
__global__ __launch_bounds__(kThreads) void icp_split_kernel(const float* __restrict__ G,
                                                             const int32_t* __restrict__ order,
                                                             const uint8_t* __restrict__ samples,
                                                             float* __restrict__ S, float* __restrict__ M1,
                                                             float* __restrict__ M2, int V, int Kv) {
  const int t = blockIdx.x, r = blockIdx.y;
  const int P = Kv / 4;
  const size_t row = (size_t)t * V + r;
  const float* g = G + row * Kv;
  const int32_t* ord = order + (size_t)t * Kv;
  const uint8_t* smp = samples + (size_t)t * P;
  for (int i = threadIdx.x; i < P; i += kThreads) {
    const int pick = smp[i] & 3;
    float v[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) v[m] = g[ord[4 * i + m]];
    const float s = pick == 0 ? v[0] : pick == 1 ? v[1] : pick == 2 ? v[2] : v[3];
    // the two smallest of the three that stay: the sampled one is lifted out of the way
#pragma unroll
    for (int m = 0; m < 4; ++m) v[m] = (m == pick) ? __builtin_inff() : v[m];
    const float lo01 = __builtin_fminf(v[0], v[1]), hi01 = __builtin_fmaxf(v[0], v[1]);
    const float lo23 = __builtin_fminf(v[2], v[3]), hi23 = __builtin_fmaxf(v[2], v[3]);
    const float m1 = __builtin_fminf(lo01, lo23);
    const float m2 = __builtin_fminf(__builtin_fmaxf(lo01, lo23), __builtin_fminf(hi01, hi23));
    S[row * P + i] = s;
    M1[row * P + i] = m1;
    M2[row * P + i] = m2;
  }
}

// cost[t][i][j] = sum_r (double) m1[r][i] + (double) min(s[r][j], m2[r][i]), rows ascending.
// A chain of V rows per entry, whose additions take four clocks a wave: the rows have to be at hand.  64 of them go
// through LDS in one burst of loads (m1 converted on the way), then a wave reads one sample a lane and four broadcast
// partitions per row.  48 tiles of 64 rows and 96 partitions: 53 us with the operands of every row loaded from L2 as
// the chain reached them and 160 of 256 lanes beyond the last sample; 15.9 us here.
__global__ __launch_bounds__(kThreads) void icp_cost_kernel(const float* __restrict__ S, const float* __restrict__ M1,
                                                            const float* __restrict__ M2, double* __restrict__ cost,
                                                            int V, int P) {
  __shared__ float s_rows[kCostRows][kCostSamples];
  __shared__ __attribute__((aligned(16))) double m1_rows[kCostRows][kCostPartitions];
  __shared__ __attribute__((aligned(16))) float m2_rows[kCostRows][kCostPartitions];
  const int t = blockIdx.z;
  const int i0 = blockIdx.y * kCostPartitions;
  const int j0 = blockIdx.x * kCostSamples;
  const int lane = threadIdx.x & 63;
  const int mine = (threadIdx.x >> 6) * kCostPartitionsPerWave;  // this wave's partitions of the block
  const float* s_t = S + (size_t)t * V * P;
  const float* m1_t = M1 + (size_t)t * V * P;
  const float* m2_t = M2 + (size_t)t * V * P;
  double acc[kCostPartitionsPerWave];
#pragma unroll
  for (int e = 0; e < kCostPartitionsPerWave; ++e) acc[e] = 0.0;
  for (int r0 = 0; r0 < V; r0 += kCostRows) {
    // rows beyond the tile and samples and partitions beyond P repeat the last one; what they give is not used
    constexpr int kSamplePieces = kCostRows * kCostSamples / kThreads;
    constexpr int kPartitionPieces = kCostRows * kCostPartitions / kThreads;
    float sv[kSamplePieces], m1v[kPartitionPieces], m2v[kPartitionPieces];
#pragma unroll
    for (int q = 0; q < kSamplePieces; ++q) {
      const int at = q * kThreads + threadIdx.x;
      sv[q] = s_t[(size_t)min(r0 + at / kCostSamples, V - 1) * P + min(j0 + at % kCostSamples, P - 1)];
    }
#pragma unroll
    for (int q = 0; q < kPartitionPieces; ++q) {
      const int at = q * kThreads + threadIdx.x;
      const size_t from = (size_t)min(r0 + at / kCostPartitions, V - 1) * P + min(i0 + at % kCostPartitions, P - 1);
      m1v[q] = m1_t[from];
      m2v[q] = m2_t[from];
    }
    if (r0 > 0) __syncthreads();
#pragma unroll
    for (int q = 0; q < kSamplePieces; ++q) (&s_rows[0][0])[q * kThreads + threadIdx.x] = sv[q];
#pragma unroll
    for (int q = 0; q < kPartitionPieces; ++q) {
      (&m1_rows[0][0])[q * kThreads + threadIdx.x] = (double)m1v[q];
      (&m2_rows[0][0])[q * kThreads + threadIdx.x] = m2v[q];
    }
    __syncthreads();
    const int rows = min(kCostRows, V - r0);
#pragma unroll 8
    for (int r = 0; r < rows; ++r) {
      const float s = s_rows[r][lane];
#pragma unroll
      for (int e = 0; e < kCostPartitionsPerWave; ++e)
        acc[e] += m1_rows[r][mine + e] + (double)__builtin_fminf(s, m2_rows[r][mine + e]);
    }
  }
  if (j0 + lane < P) {
#pragma unroll
    for (int e = 0; e < kCostPartitionsPerWave; ++e)
      if (i0 + mine + e < P) cost[((size_t)t * P + i0 + mine + e) * P + j0 + lane] = acc[e];
  }
}

// Moves sample assign[i] into the slot partition i vacated, and reports the total cost of the
// assignment (partitions added in ascending order).
__global__ __launch_bounds__(kThreads) void icp_apply_kernel(const double* __restrict__ cost,
                                                             const int32_t* __restrict__ assign,
                                                             const uint8_t* __restrict__ samples,
                                                             int32_t* __restrict__ order,
                                                             double* __restrict__ objective, int Kv) {
  __shared__ int32_t moved[kMaxP];
  __shared__ double picked[kMaxP];
  const int t = blockIdx.x;
  const int P = Kv / 4;
  const int32_t* asg = assign + (size_t)t * P;
  const uint8_t* smp = samples + (size_t)t * P;
  int32_t* ord = order + (size_t)t * Kv;
  for (int i = threadIdx.x; i < P; i += kThreads) {
    int j = asg[i];
    j = (j >= 0 && j < P) ? j : i;
    moved[i] = ord[4 * j + (smp[j] & 3)];
    picked[i] = cost[((size_t)t * P + i) * P + j];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < P; i += kThreads) ord[4 * i + (smp[i] & 3)] = moved[i];
  if (objective && threadIdx.x == 0) {
    double total = 0.0;
    for (int i = 0; i < P; ++i) total += picked[i];
    objective[t] = total;
  }
}

// vec_idx[t][pos] = (incoming vec_idx)[t][order[t][pos]], in place through LDS.
__global__ __launch_bounds__(kThreads) void icp_finish_kernel(const int32_t* __restrict__ order,
                                                              int32_t* __restrict__ vec_idx, int Kv) {
  __shared__ int32_t cols[4 * kMaxP];
  const int t = blockIdx.x;
  int32_t* vi = vec_idx + (size_t)t * Kv;
  const int32_t* ord = order + (size_t)t * Kv;
  for (int s = threadIdx.x; s < Kv; s += kThreads) cols[s] = vi[s];
  __syncthreads();
  for (int s = threadIdx.x; s < Kv; s += kThreads) {
    const int o = ord[s];
    vi[s] = cols[(o >= 0 && o < Kv) ? o : s];
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

IcpWorkspace icp_workspace_layout(const hinm_shape& s) {
  const size_t T = s.M / s.V, P = s.Kv / 4;
  IcpWorkspace w;
  size_t off = 0;
  w.gathered = off; off += align256((size_t)s.M * s.Kv * sizeof(float));
  w.order = off;    off += align256(T * s.Kv * sizeof(int32_t));
  w.sample = off;   off += align256((size_t)s.M * P * sizeof(float));
  w.min1 = off;     off += align256((size_t)s.M * P * sizeof(float));
  w.min2 = off;     off += align256((size_t)s.M * P * sizeof(float));
  w.cost = off;     off += align256(T * P * P * sizeof(double));
  w.assign = off;   off += align256(T * P * sizeof(int32_t));
  w.total_bytes = off;
  return w;
}

hipError_t launch_icp_search(const IcpArgs& a, hipStream_t stream) {
  const hinm_shape& s = a.s;
  const int T = s.M / s.V, P = s.Kv / 4;
  const IcpWorkspace w = icp_workspace_layout(s);
  uint8_t* base = static_cast<uint8_t*>(a.workspace);
  float* G = reinterpret_cast<float*>(base + w.gathered);
  int32_t* order = reinterpret_cast<int32_t*>(base + w.order);
  float* S = reinterpret_cast<float*>(base + w.sample);
  float* M1 = reinterpret_cast<float*>(base + w.min1);
  float* M2 = reinterpret_cast<float*>(base + w.min2);
  double* cost = reinterpret_cast<double*>(base + w.cost);
  int32_t* assign = reinterpret_cast<int32_t*>(base + w.assign);
  const uint16_t* Wb = static_cast<const uint16_t*>(a.W);
  const dim3 rows_grid(T, s.V);
  if (s.dtype == HINM_F16)
    icp_gather_kernel<HINM_F16><<<rows_grid, kThreads, 0, stream>>>(Wb, a.rho, a.vec_idx, G, order, s.K, s.V, s.Kv);
  else
    icp_gather_kernel<HINM_BF16><<<rows_grid, kThreads, 0, stream>>>(Wb, a.rho, a.vec_idx, G, order, s.K, s.V, s.Kv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 cost_grid((P + kCostSamples - 1) / kCostSamples, (P + kCostPartitions - 1) / kCostPartitions, T);
  for (int it = 0; it < a.iters; ++it) {
    const uint8_t* smp = a.samples + (size_t)it * T * P;
    icp_split_kernel<<<rows_grid, kThreads, 0, stream>>>(G, order, smp, S, M1, M2, s.V, s.Kv);
    icp_cost_kernel<<<cost_grid, kThreads, 0, stream>>>(S, M1, M2, cost, s.V, P);
    e = launch_assignment(cost, assign, T, P, P, stream);
    if (e != hipSuccess) return e;
    icp_apply_kernel<<<T, kThreads, 0, stream>>>(cost, assign, smp, order,
                                                 a.objective ? a.objective + (size_t)it * T : nullptr, s.Kv);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  icp_finish_kernel<<<T, kThreads, 0, stream>>>(order, a.vec_idx, s.Kv);
  return hipGetLastError();
}

}  // namespace hinm
