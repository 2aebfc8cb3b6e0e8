// Exact minimal-cost assignment for the permutation searches (arXiv 2407.20496, Section 4.2: samples to partitions,
// clusters to tiles, and the size-constrained clustering step): n rows to m columns of capacity cap = n / m each, costs
// in binary64.
//
// The exact part is shortest augmenting paths with column potentials v: one dependent chain of "scan a row, take the
// minimum", whose cost is its length times the latency of a link.  Both are kept small:
//   start  : any v is a valid start, a good one leaves few rows without a column.  A fixed number of rounds moves all
//            potentials at once: with o[i][j] = the best reduced cost of row i outside column j, column j moves half
//            way to the midpoint between its cap-th and (cap + 1)-th smallest (cost[i][j] - v[j]) - o[i][j] (damped
//            max-product message passing; the midpoint is where exactly cap rows prefer the column).  This part is
//            parallel over the matrix and runs on the whole workgroup.  Rows then take the column of their minimum
//            while it has room.  On the 96 x 96 problems of the tile-wise search 2 to 6 rows stay free, on
//            384 points x 48 clusters of 8 about 5 (60 and 300 from plain column and row minima).
//   paths  : for the free rows, on one wave that holds column 64 c + lane in register c: no barrier and no shared
//            minimum in a link; a row arrives with one read per 64 columns from LDS (matrices up to some 150 KB) or
//            L2, and the minimum over the lanes is six data-parallel-primitive moves on the high words of the costs
//            (the low words only where those tie).
// With capacities the matrix is n x m instead of n x n with every column repeated.
// Measured per call, against one augmenting-path search per row from column minima on two to four waves: 48 problems
// of 96 x 96 1.10 -> 0.104 ms, 384 and 192 points to 48 clusters (n x n before) 16.6 -> 0.15 ms on average, one of
// 48 x 48 0.365 -> 0.040 ms, 64 of 512 x 512 (four iterations of the tile-wise search on 4096 x 4096) 161 -> 16 ms.
// Every loop is bounded by the problem's size.  Costs may be of any finite size below 1e300: a row's smallest cost is
// taken off the row first (a constant of a row changes no choice, but next to one of 1e39 the other rows' costs would
// be rounded away), and the start, which works in single precision, scales what is left by the power of two of
// its largest entry.  An infinite or undefined cost is a pair that cannot be taken; problems without an
// assignment of finite pairs end in the identity.
#include "hinm_internal.h"
#include "wave_reduce.h"

namespace hinm {
namespace {

constexpr int kStartRounds = 12;  // 384 x 48: path steps 62 after 10 rounds, 96 x 96: 30 .. 70 after 10, 15 .. 30 after 20
constexpr double kInf = 1e300;  // distance of a column that is closed; costs are below
constexpr double kFar = 5e299;  // distance of a column that cannot be reached yet
constexpr int kLdsBytes = 160 * 1024;

// lane that holds the smallest x (the lowest of several), wave-uniform
__device__ __forceinline__ int wave_argmin_lane(double x) {
  const int hi = __double2hiint(x);
  const int sign = hi >> 31;
  const int key = hi ^ (sign & 0x7fffffff);  // orders doubles by their high words
  const int least = wave_min(key);
  unsigned long long at = __ballot(key == least);
  if (at & (at - 1)) {  // several lanes share the high word: the low words decide
    const int low = (int)(((unsigned)__double2loint(x) ^ (unsigned)sign) ^ 0x80000000u);  // unsigned order as signed
    const int low_key = key == least ? low : 0x7fffffff;
    const int least_low = wave_min(low_key);
    at &= __ballot(low_key == least_low);
  }
  return __builtin_ctzll(at);
}
__device__ __forceinline__ double read_lane(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                          __builtin_amdgcn_readlane(__double2loint(x), lane));
}
// the value that belongs to column j
template <int CPL>
__device__ __forceinline__ int at_column(const int (&a)[CPL], int j) {
  int r = a[0];
#pragma unroll
  for (int c = 1; c < CPL; ++c) r = (j >> 6) == c ? a[c] : r;
  return __builtin_amdgcn_readlane(r, j & 63);
}
template <int CPL>
__device__ __forceinline__ double at_column(const double (&a)[CPL], int j) {
  double r = a[0];
#pragma unroll
  for (int c = 1; c < CPL; ++c) r = (j >> 6) == c ? a[c] : r;
  return read_lane(r, j & 63);
}
template <int CPL>
__device__ __forceinline__ void set_column(int (&a)[CPL], int j, int lane, int value) {
#pragma unroll
  for (int c = 0; c < CPL; ++c) a[c] = (64 * c + lane == j) ? value : a[c];
}

// order-preserving integer key of a float, and back
__device__ __forceinline__ int float_key(float x) {
  const int b = __float_as_int(x);
  return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float key_float(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7fffffff)); }

struct __attribute__((aligned(16))) RowBest {
  float best;  // reduced cost of the row's best column (single precision: only the start uses it),
  float gap;   // how much worse its second best is,
  int col;     // and which column it is
  int unused;
};

struct AssignLds {  // byte offsets into dynamic LDS
  int cost, v, rows, base, filled, work, row_col, list, members, total;
};
__host__ __device__ inline AssignLds assign_lds(int n, int m, int threads, bool with_cost) {
  AssignLds l;
  int off = 0;
  l.rows = off;     off += n * (int)sizeof(RowBest);
  l.cost = off;     off += with_cost ? n * m * 8 : 0;
  l.base = off;     off += with_cost ? 0 : n * 8;  // what is taken off every row (a matrix in LDS has it taken off)
  l.v = off;        off += m * 8;
  l.work = off;                     // start: two floats per (row group, column); afterwards:
  l.row_col = off;                  // column of every row, -1 = free
  l.list = l.row_col + n * 4;       // free rows
  l.members = l.list + n * 4;       // rows of every column, by slot
  const int groups = threads / m > 0 ? threads / m : 1;
  const int start = groups * m * 8, paths = 3 * n * 4;
  off += start > paths ? start : paths;
  l.filled = off;   off += m * 4;
  l.total = off;
  return l;
}

// CAPACITY false: m == n, cap == 1.
template <int CPL, int THREADS, bool IN_LDS, bool CAPACITY>
__global__ __launch_bounds__(THREADS) void assign_kernel(const double* __restrict__ cost, int32_t* __restrict__ assign,
                                                         int n, int m, int cap) {
  constexpr int WAVES = THREADS / 64;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const AssignLds L = assign_lds(n, m, THREADS, IN_LDS);
  double* col_v = reinterpret_cast<double*>(lds + L.v);
  RowBest* rows = reinterpret_cast<RowBest*>(lds + L.rows);
  double* base = reinterpret_cast<double*>(lds + L.base);
  int* filled = reinterpret_cast<int*>(lds + L.filled);
  float2* smallest = reinterpret_cast<float2*>(lds + L.work);
  int* row_col = reinterpret_cast<int*>(lds + L.row_col);
  int* list = reinterpret_cast<int*>(lds + L.list);
  int* members = reinterpret_cast<int*>(lds + L.members);
  const double* global_cost = cost + (size_t)blockIdx.x * n * m;
  double* lds_cost = reinterpret_cast<double*>(lds + L.cost);
  int32_t* out = assign + (size_t)blockIdx.x * n;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto row_of = [&](int i) -> const double* { return (IN_LDS ? lds_cost : global_cost) + (size_t)i * m; };
  auto base_of = [&](int i) { return IN_LDS ? 0.0 : base[i]; };

  // ---- start: the whole workgroup ------------------------------------------------------------------
  const int groups = THREADS / m > 0 ? THREADS / m : 1;  // row groups that share a column
  const int group = tid / m;                             // (m > THREADS: one group, several columns a thread)
  if constexpr (IN_LDS) {
#pragma unroll 4
    for (int e = tid; e < n * m; e += THREADS) lds_cost[e] = global_cost[e];
  }
  for (int j = tid; j < m; j += THREADS) col_v[j] = 0.0;
  if (tid == 0) filled[0] = 0;
  __syncthreads();
  // the smallest cost of every row is taken off it (two rows at a time, their chains overlap); filled[0] = high word of
  // the largest finite cost that is left
  int largest = 0;
  for (int i0 = wave; i0 < n; i0 += 2 * WAVES) {
    double x[2][CPL], least[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double* r = row_of(min(i0 + h * WAVES, n - 1));
      least[h] = kInf;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        x[h][c] = r[min(64 * c + lane, m - 1)];
        least[h] = x[h][c] < least[h] ? x[h][c] : least[h];
      }
    }
    const int at0 = wave_argmin_lane(least[0]), at1 = wave_argmin_lane(least[1]);
    least[0] = read_lane(least[0], at0);
    least[1] = read_lane(least[1], at1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = i0 + h * WAVES;
      if (i >= n) break;  // (another wave's row)
      const double off = least[h] > -kInf && least[h] < kInf ? least[h] : 0.0;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        x[h][c] -= off;
        if (__builtin_fabs(x[h][c]) < kInf) largest = max(largest, __double2hiint(x[h][c]) & 0x7fffffff);
        if constexpr (IN_LDS) {
          if (64 * c + lane < m) lds_cost[(size_t)i * m + 64 * c + lane] = x[h][c];
        }
      }
      if constexpr (!IN_LDS) {
        if (lane == 0) base[i] = off;
      }
    }
  }
  largest = -wave_min(-largest);
  if (lane == 0) atomicMax(&filled[0], largest);
  __syncthreads();
  // powers of two: costs times `scale` are below 2, and the start's potentials are of scaled costs
  const int exponent = max(filled[0] >> 20, 1);
  const double scale = __hiloint2double((2046 - exponent) << 20, 0), unscale = __hiloint2double(exponent << 20, 0);
  auto scaled = [&](int i, double cost_ij, double vj) {
    return __builtin_fma(IN_LDS ? cost_ij : cost_ij - base[i], scale, -vj);
  };

  // best and second best column of every row; two rows at a time, their chains overlap
  auto scan_rows = [&]() {
    for (int i0 = wave; i0 < n; i0 += 2 * WAVES) {
      const int i1 = min(i0 + WAVES, n - 1);
      int k1[2], k2[2], c1[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int i = h ? i1 : i0;
        const double* r = row_of(i);
        k1[h] = k2[h] = 0x7fffffff;
        c1[h] = 0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const int j = min(64 * c + lane, m - 1);
          const int x = float_key((float)scaled(i, r[j], col_v[j]));
          const int key = 64 * c + lane < m ? x : 0x7fffffff;
          const bool first = key < k1[h];
          k2[h] = first ? k1[h] : min(k2[h], key);
          k1[h] = first ? key : k1[h];
          c1[h] = first ? c : c1[h];
        }
      }
      int least[2], at[2], second[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        least[h] = wave_min(k1[h]);
        at[h] = __builtin_ctzll(__ballot(k1[h] == least[h]));
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) second[h] = wave_min(lane == at[h] ? k2[h] : k1[h]);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (lane == at[h]) {
          const float u1 = key_float(least[h]), u2 = key_float(second[h]);
          // a row without a finite cost moves no potential; one with a single one claims its column, within bounds
          const bool any = __builtin_fabsf(u1) < 1e30f;
          rows[h ? i1 : i0] = RowBest{any ? u1 : -3e38f, any ? fminf(u2 - u1, 4.f) : 0.f, 64 * c1[h] + at[h], 0};
        }
    }
    __syncthreads();
  };
  if (m > 1) {
    for (int round = 0; round < kStartRounds; ++round) {
      scan_rows();
      if (group < groups) {
        for (int j = (m > THREADS) ? tid : tid - group * m; j < m; j += (m > THREADS) ? THREADS : m) {
          const double vj = col_v[j];
          float s1 = 3e38f, s2 = 3e38f;
#pragma unroll 4
          for (int i = group; i < n; i += groups) {
            const RowBest rb = rows[i];
            const float g = (float)(scaled(i, row_of(i)[j], vj) - (double)rb.best) - (rb.col == j ? rb.gap : 0.f);
            s2 = fminf(s2, fmaxf(s1, g));
            s1 = fminf(s1, g);
          }
          smallest[group * m + j] = make_float2(s1, s2);
        }
      }
      __syncthreads();
      if constexpr (CAPACITY) {
        // one wave per column; of every row group the two smallest values are known, which nearly always holds
        // the cap + 1 smallest of all (groups >= cap), and a start needs no more
        const int values = 2 * groups;
        const float* s = reinterpret_cast<const float*>(smallest);
        for (int j = wave; j < m; j += WAVES) {
          const auto value = [&](int e) {
            return e < values ? float_key(s[2 * ((e >> 1) * m + j) + (e & 1)]) : 0x7fffffff;
          };
          // cap-th smallest, bit by bit over the unsigned order of the keys, and the one after it
          unsigned prefix = 0;
          int next = 0x7fffffff;
          if (values <= 64) {
            const int key = value(lane);
            for (int bit = 31; bit >= 0; --bit) {
              const unsigned cand = prefix | (1u << bit);  // how many lie below it?
              if (__popcll(__ballot(((unsigned)key ^ 0x80000000u) < cand)) < cap) prefix = cand;
            }
            if (key > (int)(prefix ^ 0x80000000u)) next = key;
          } else {  // few columns
            for (int bit = 31; bit >= 0; --bit) {
              const unsigned cand = prefix | (1u << bit);
              int below = 0;
              for (int e = lane; e < ((values + 63) & ~63); e += 64)
                below += __popcll(__ballot(((unsigned)value(e) ^ 0x80000000u) < cand));
              if (below < cap) prefix = cand;
            }
            for (int e = lane; e < values; e += 64) {
              const int key = value(e);
              if (key > (int)(prefix ^ 0x80000000u)) next = min(next, key);
            }
          }
          const int kth = (int)(prefix ^ 0x80000000u);
          next = wave_min(next);
          const float lo = key_float(kth), hi = next == 0x7fffffff ? lo : key_float(next);
          if (lane == 0 && lo < 1e38f && hi < 1e38f) col_v[j] += 0.25 * ((double)lo + (double)hi);
        }
      } else {
        for (int j = tid; j < m; j += THREADS) {
          float s1 = 3e38f, s2 = 3e38f;
          for (int g = 0; g < groups; ++g) {
            const float2 s = smallest[g * m + j];
            s2 = fminf(fminf(s2, s.y), fmaxf(s1, s.x));
            s1 = fminf(s1, s.x);
          }
          if (s2 < 1e38f) col_v[j] += 0.25 * ((double)s1 + (double)s2);
        }
      }
      __syncthreads();
    }
  }
  for (int j = tid; j < m; j += THREADS) col_v[j] *= unscale;
  __syncthreads();
  for (int i = wave; i < n; i += WAVES) {  // now exactly
    const double* r = row_of(i);
    const double off = base_of(i);
    double least = kInf;
    int least_c = 0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int j = min(64 * c + lane, m - 1);
      const double x = 64 * c + lane < m ? (IN_LDS ? r[j] : r[j] - off) - col_v[j] : kInf;
      const bool less = x < least;
      least = less ? x : least;
      least_c = less ? c : least_c;
    }
    const int at = wave_argmin_lane(least);
    if (lane == at) rows[i].col = least < kFar ? 64 * least_c + at : -1;
  }
  __syncthreads();
  // every row sits in its best column while there is room, lower rows first
  for (int i = tid; i < n; i += THREADS) row_col[i] = -1;
  __syncthreads();
  for (int j = tid; j < m; j += THREADS) {
    int count = 0;
    for (int i = 0; i < n && count < cap; ++i)
      if (rows[i].col == j) {
        members[j * cap + count++] = i;
        row_col[i] = j;
      }
    filled[j] = count;
  }
  __syncthreads();
  if (wave != 0) return;  // no barrier below

  // ---- paths: one wave, column 64 c + lane in register c ---------------------------------------------
  double v[CPL];
  int y[CPL];  // capacity 1: the column's row or -1; capacities: how many rows the column holds
  int col[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int j = 64 * c + lane;
    col[c] = min(j, m - 1);
    v[c] = j < m ? col_v[j] : 0.0;
    const int count = j < m ? filled[col[c]] : 0;
    y[c] = CAPACITY ? count : (count ? members[col[c]] : -1);
  }
  int n_free = 0;
  for (int i0 = 0; i0 < n; i0 += 64) {
    const bool is_free = i0 + lane < n && row_col[min(i0 + lane, n - 1)] < 0;
    const unsigned long long mask = __ballot(is_free);
    if (is_free) list[n_free + __popcll(mask & ((1ull << lane) - 1ull))] = i0 + lane;
    n_free += __popcll(mask);
  }
  auto reduced_row = [&](int i, double (&x)[CPL]) {
    const double* r = row_of(i);
    const double off = base_of(i);
#pragma unroll
    for (int c = 0; c < CPL; ++c) x[c] = r[col[c]];
#pragma unroll
    for (int c = 0; c < CPL; ++c) x[c] = (IN_LDS ? x[c] : x[c] - off) - v[c];
  };
  bool failed = false;
  for (int k = 0; k < n_free && !failed; ++k) {
    const int start = __builtin_amdgcn_readfirstlane(list[k]);
    double d[CPL];     // shortest distance to every column that has not been scanned,
    double open[CPL];  // the same with kInf where it has
    int pred[CPL];
    reduced_row(start, d);
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      pred[c] = start;
      // columns that do not exist are closed; one that costs infinitely much from here may be reached through others
      d[c] = 64 * c + lane < m ? __builtin_fmin(d[c], kFar) : kInf;
      open[c] = d[c];
    }
    int end = -1;
    double reach = 0.0;
    for (int step = 0; step < m; ++step) {  // every pass but the last closes one more column
      double least = open[0];
      int least_c = 0;
#pragma unroll
      for (int c = 1; c < CPL; ++c) {
        const bool less = open[c] < least;
        least = less ? open[c] : least;
        least_c = less ? c : least_c;
      }
      const int at = wave_argmin_lane(least);
      reach = read_lane(least, at);
      if (!(reach < kFar)) break;
      const int at_c = CPL == 1 ? 0 : __builtin_amdgcn_readlane(least_c, at);
      const int j1 = 64 * at_c + at;
      const int held = at_column(y, j1);
      if (CAPACITY ? held < cap : held < 0) {
        end = j1;
        break;
      }
#pragma unroll
      for (int c = 0; c < CPL; ++c) open[c] = (c == at_c && lane == at) ? kInf : open[c];
      auto relax = [&](int i, const double (&x)[CPL]) {
        const double h = at_column(x, j1) - reach;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const double through = x[c] - h;
          const bool better = through < open[c] && open[c] < kInf;
          open[c] = better ? through : open[c];
          d[c] = better ? through : d[c];
          pred[c] = better ? i : pred[c];
        }
      };
      if constexpr (CAPACITY) {
        const int* who = members + j1 * cap;
        int e = 0;
        for (; e + 4 <= cap; e += 4) {  // four rows in flight
          int i4[4];
          double x4[4][CPL];
#pragma unroll
          for (int q = 0; q < 4; ++q) i4[q] = __builtin_amdgcn_readfirstlane(who[e + q]);
#pragma unroll
          for (int q = 0; q < 4; ++q) reduced_row(i4[q], x4[q]);
#pragma unroll
          for (int q = 0; q < 4; ++q) relax(i4[q], x4[q]);
        }
        for (; e < cap; ++e) {
          const int i = __builtin_amdgcn_readfirstlane(who[e]);
          double x[CPL];
          reduced_row(i, x);
          relax(i, x);
        }
      } else {
        double x[CPL];
        reduced_row(held, x);
        relax(held, x);
      }
    }
    if (end < 0) {
      failed = true;
      break;
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c)  // scanned columns only
      if (d[c] < open[c]) v[c] += d[c] - reach;
    // shift the rows along the path
    int j = end;
    int slot = 0;
    if constexpr (CAPACITY) {
      slot = at_column(y, end);
      set_column(y, end, lane, slot + 1);
    }
    for (int guard = 0; guard <= m; ++guard) {
      const int i = at_column(pred, j);
      const int from = __builtin_amdgcn_readfirstlane(row_col[i]);
      row_col[i] = j;
      if constexpr (CAPACITY) {
        int freed = 0;
        if (i != start) {
          const int* who = members + from * cap;
          for (int e = 0; e < cap; ++e)
            if (__builtin_amdgcn_readfirstlane(who[e]) == i) freed = e;
        }
        members[j * cap + slot] = i;
        slot = freed;
      } else {
        set_column(y, j, lane, i);
      }
      if (i == start) break;
      j = from;
    }
  }
  if (failed) {
    for (int i = lane; i < n; i += 64) out[i] = i;
  } else if constexpr (CAPACITY) {
    for (int e = lane; e < n; e += 64) out[members[e]] = e;
  } else {
    for (int i = lane; i < n; i += 64) out[i] = row_col[i];
  }
}

template <int CPL, bool IN_LDS, bool CAPACITY>
hipError_t launch_cfg(const double* cost, int32_t* assign, int problems, int n, int m, int cap, hipStream_t stream) {
  constexpr int THREADS = CPL <= 4 ? 1024 : 512;  // 128 / 256 registers a lane: the paths need a dozen per column
  constexpr auto kernel = assign_kernel<CPL, THREADS, IN_LDS, CAPACITY>;
  if (hipError_t e = raise_lds_limit<kernel>(kLdsBytes); e != hipSuccess) return e;
  kernel<<<problems, THREADS, assign_lds(n, m, THREADS, IN_LDS).total, stream>>>(cost, assign, n, m, cap);
  return hipGetLastError();
}

template <bool CAPACITY>
hipError_t launch(const double* cost, int32_t* assign, int problems, int n, int m, int cap, hipStream_t stream) {
  if (m <= 256 && assign_lds(n, m, 1024, true).total <= kLdsBytes) {
    if (m <= 64) return launch_cfg<1, true, CAPACITY>(cost, assign, problems, n, m, cap, stream);
    if (m <= 128) return launch_cfg<2, true, CAPACITY>(cost, assign, problems, n, m, cap, stream);
    return launch_cfg<4, true, CAPACITY>(cost, assign, problems, n, m, cap, stream);  // at most some 135 x 135
  }
  if (m <= 64) return launch_cfg<1, false, CAPACITY>(cost, assign, problems, n, m, cap, stream);
  if (m <= 128) return launch_cfg<2, false, CAPACITY>(cost, assign, problems, n, m, cap, stream);
  if (m <= 256) return launch_cfg<4, false, CAPACITY>(cost, assign, problems, n, m, cap, stream);
  if (m <= 512) return launch_cfg<8, false, CAPACITY>(cost, assign, problems, n, m, cap, stream);
  if constexpr (!CAPACITY) return launch_cfg<16, false, false>(cost, assign, problems, n, m, cap, stream);
  return hipErrorInvalidValue;  // capacities of two and more leave at most kIcpMaxPartitions / 2 columns
}

}  // namespace

hipError_t launch_assignment(const double* cost, int32_t* assign, int problems, int n, int m, hipStream_t stream) {
  const int cap = n / m;
  return cap == 1 ? launch<false>(cost, assign, problems, n, m, 1, stream)
                  : launch<true>(cost, assign, problems, n, m, cap, stream);
}

}  // namespace hinm
