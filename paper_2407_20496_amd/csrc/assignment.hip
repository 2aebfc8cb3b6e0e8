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
//            while it has room.  On 96 x 96 problems of the tile-wise search 2 to 6 rows stayed free, on 384 points x
//            48 clusters of 8 about 5 (60 and 300 from plain column and row minima), before these sizes had a kernel
//            of their own, below.
//   paths  : for the free rows, on one wave that holds column 64 c + lane in register c: no barrier and no shared
//            minimum in a link; a row arrives with one read per 64 columns from LDS (matrices up to some 150 KB) or
//            L2, and the minimum over the lanes is six data-parallel-primitive moves on the high words of the costs
//            (the low words only where those tie).
// With capacities the matrix is n x m instead of n x n with every column repeated.
// Measured, against one augmenting-path search per row from column minima on two to four waves: 64 problems of 512 x 512
// (four iterations of the tile-wise search on 4096 x 4096) 161 -> 15 ms, 12 with `row_paths` (129 to 512 columns of one row
// each 1.09 to 1.21 times).
// Every loop is bounded by the problem's size.  Costs may be of any finite size below 1e300: a row's smallest cost is
// taken off the row first (a constant of a row changes no choice, but next to one of 1e39 the other rows' costs would
// be rounded away), and the start, which works in single precision, scales what is left by the power of two of
// its largest entry.  An infinite or undefined cost is a pair that cannot be taken; problems without an
// assignment of finite pairs end in the identity.
#include "hinm_internal.h"
#include "wave_reduce.h"

namespace hinm {
namespace {

constexpr int kStartRounds = 12;  // (chosen on 384 x 48: path steps 62 after 10 rounds; 96 x 96: 30 .. 70 after 10, 15 .. 30 after 20)
constexpr double kInf = 1e300;  // distance of a column that is closed; costs are below
constexpr double kFar = 5e299;  // distance of a column that cannot be reached yet
constexpr int kFarHigh = 0x7e27e43c, kInfHigh = 0x7e37e43c;  // their high words
constexpr int kClosedHigh = (int)0xffe00000;  // of a potential far below every cost
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

// The column nearest to the tree of a path among those still open: lane `at`, register `c`; false if none can be reached.
// Distances are not negative (but for rounding: the sign of those that are does not order them among each other), so their
// high words order them as integers and the low words decide only where those tie.
template <int CPL>
__device__ __forceinline__ bool nearest_column(const double (&open)[CPL], double& reach, int& at, int& c) {
  double least = open[0];
  int least_c = 0;
  unsigned long long upper = 0;
  if constexpr (CPL == 2) {
    const bool less = open[1] < open[0];
    upper = __ballot(less);
    least = less ? open[1] : least;
  } else {
#pragma unroll
    for (int k = 1; k < CPL; ++k) {
      const bool less = open[k] < least;
      least = less ? open[k] : least;
      least_c = less ? k : least_c;
    }
  }
  const int key = __double2hiint(least);
  const int high = wave_min(key);
  unsigned long long where = __ballot(key == high);
  if (__builtin_expect((where & (where - 1)) != 0, 0)) {
    const int low = __double2loint(least) ^ (int)0x80000000;  // unsigned order as signed
    const int low_key = key == high ? low : 0x7fffffff;
    where &= __ballot(low_key == wave_min(low_key));
  }
  at = __builtin_ctzll(where);
  reach = read_lane(least, at);
  c = CPL == 1 ? 0 : CPL == 2 ? (int)(upper >> at) & 1 : __builtin_amdgcn_readlane(least_c, at);
  return high < kFarHigh;
}

// A column leaves the open ones: its distance is kept, and no later link of the path can reach it again (its entry less the
// working potential is beyond every distance).  High words are enough for the latter two.
template <int CPL>
__device__ __forceinline__ void close_column(double (&open)[CPL], double (&work)[CPL], double (&d)[CPL], double reach, int j) {
#pragma unroll
  for (int k = 0; k < CPL; ++k) {
    const bool here = 64 * k + (int)(threadIdx.x & 63) == j;
    open[k] = __hiloint2double(here ? kInfHigh : __double2hiint(open[k]), __double2loint(open[k]));
    work[k] = __hiloint2double(here ? kClosedHigh : __double2hiint(work[k]), __double2loint(work[k]));
    d[k] = here ? reach : d[k];
  }
}
template <int CPL>
__device__ __forceinline__ void move_potentials(double (&v)[CPL], const double (&work)[CPL], const double (&d)[CPL], double reach) {
#pragma unroll
  for (int c = 0; c < CPL; ++c)
    if (__double2hiint(work[c]) == kClosedHigh) v[c] += d[c] - reach;
}

// Distances from a free row to the columns, its nearest at 0; false if it has none.
template <int CPL>
__device__ __forceinline__ bool start_path(const double (&row)[CPL], const double (&v)[CPL], int m, double (&open)[CPL],
                                           double (&work)[CPL], double (&d)[CPL]) {
  const int lane = threadIdx.x & 63;
  double least = kFar;
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    open[c] = row[c] - v[c];
    if (64 * c + lane < m) least = open[c] < least ? open[c] : least;
    work[c] = 64 * c + lane < m ? v[c] : __hiloint2double(kClosedHigh, 0);
    d[c] = 0.0;
  }
  least = read_lane(least, wave_argmin_lane(least));
#pragma unroll
  for (int c = 0; c < CPL; ++c)  // columns that do not exist are closed; one that costs infinitely much from here may be
    open[c] = 64 * c + lane < m ? __builtin_fmin(open[c] - least, kFar) : kInf;  // reached through others
  return least < kFar;
}

// Paths of the free rows where a column takes one row, on one wave: column 64 c + lane in register c.  entry(i, j): what row i
// costs in column j, less a constant of the row.  What the row of a column pays there (`own`) stays in registers, so that a link
// waits for one read and does nothing else behind it than compare.
template <int CPL, class Entry>
__device__ __forceinline__ bool row_paths(Entry entry, const double* col_v, const int* filled, const int* members,
                                          const int* list, int n_free, int* row_col, int m) {
  const int lane = threadIdx.x & 63;
  double v[CPL], own[CPL];
  int y[CPL];  // the column's row or -1
  int col[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int j = 64 * c + lane;
    col[c] = min(j, m - 1);
    v[c] = j < m ? col_v[j] : 0.0;
    y[c] = j < m && filled[col[c]] ? members[col[c]] : -1;
    own[c] = entry(max(y[c], 0), col[c]);
  }
  for (int k = 0; k < n_free; ++k) {
    const int start = __builtin_amdgcn_readfirstlane(list[k]);
    double row[CPL], open[CPL], work[CPL], d[CPL], held_at[CPL];
    int pred[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      row[c] = entry(start, col[c]);
      held_at[c] = own[c] - v[c];
      pred[c] = start;
    }
    if (!start_path(row, v, m, open, work, d)) return false;
    int end = -1;
    double reach = 0.0;
    for (int link = 0; link < m; ++link) {  // every pass but the last closes one more column
      int at, at_c;
      if (__builtin_expect(!nearest_column(open, reach, at, at_c), 0)) break;
      const int j1 = 64 * at_c + at;
      const int held = at_column(y, j1);
      if (__builtin_expect(held < 0, 0)) {
        end = j1;
        break;
      }
      double x[CPL];
#pragma unroll
      for (int c = 0; c < CPL; ++c) x[c] = entry(held, col[c]);
      const double h = at_column(held_at, j1) - reach;
      close_column(open, work, d, reach, j1);
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const double through = (x[c] - work[c]) - h;
        const bool better = through < open[c];
        open[c] = better ? through : open[c];
        pred[c] = better ? held : pred[c];
      }
    }
    if (end < 0) return false;
    move_potentials(v, work, d, reach);
    // shift the rows along the path
    int j = end;
    for (int guard = 0; guard <= m; ++guard) {
      const int i = at_column(pred, j);
      const int from = __builtin_amdgcn_readfirstlane(row_col[i]);
      row_col[i] = j;
      set_column(y, j, lane, i);
      const double pays = entry(i, j);
#pragma unroll
      for (int c = 0; c < CPL; ++c) own[c] = (64 * c + lane == j) ? pays : own[c];
      if (i == start) break;
      j = from;
    }
  }
  return true;
}

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
  int n_free = 0;
  for (int i0 = 0; i0 < n; i0 += 64) {
    const bool is_free = i0 + lane < n && row_col[min(i0 + lane, n - 1)] < 0;
    const unsigned long long mask = __ballot(is_free);
    if (is_free) list[n_free + __popcll(mask & ((1ull << lane) - 1ull))] = i0 + lane;
    n_free += __popcll(mask);
  }
  bool failed = false;
  // `row_paths` keeps two more values a column, which sixteen columns a lane leave no registers for: 64 spilled ones in the chain of
  // links took 31 ms against 19.6 (4 problems of 1024 x 1024; of 600 x 600 9.4 against 6.6).
  if constexpr (!CAPACITY && CPL <= 8) {
    failed = !row_paths<CPL>([&](int i, int j) { return row_of(i)[j] - base_of(i); }, col_v, filled, members, list, n_free,
                             row_col, m);
    for (int i = lane; i < n; i += 64) out[i] = failed ? i : row_col[i];
    return;
  }
  double v[CPL];
  int y[CPL];  // how many rows the column holds; where it takes one, that row or -1
  int col[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int j = 64 * c + lane;
    col[c] = min(j, m - 1);
    v[c] = j < m ? col_v[j] : 0.0;
    const int count = j < m ? filled[col[c]] : 0;
    y[c] = CAPACITY ? count : (count ? members[col[c]] : -1);
  }
  auto reduced_row = [&](int i, double (&x)[CPL]) {
    const double* r = row_of(i);
    const double off = base_of(i);
#pragma unroll
    for (int c = 0; c < CPL; ++c) x[c] = r[col[c]];
#pragma unroll
    for (int c = 0; c < CPL; ++c) x[c] = (IN_LDS ? x[c] : x[c] - off) - v[c];
  };
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

// ---- the same for problems whose matrix fits the workgroup's registers, or nearly -------------------------------------
//
// What bounds the general kernel on these is the start: a row comes from LDS twice a round, one wave a row, with three
// reductions over 64 lanes behind each other.  Here the matrix stays in registers, in single precision: eight lanes a row
// (column lane % 8 + 8 c in register c), 128 rows at a time, so that a row's two smallest take three moves inside a row of lanes,
// and a column's candidates leave a wave after two more.  The potentials begin at the columns' means and move 0.8 of the way
// to the midpoint: after 5 rounds as many rows are left as after 12 of half the way from zero.  The rounds end as soon as
// no column is asked for by more rows than it takes: centroids that are means of their points leave nothing to do.
// With capacities a path only ever needs, for every pair of full columns, the least that moving a row of the one to
// the other costs: that m x m matrix is worked out by the whole workgroup, held in LDS, and only the columns of a path are
// worked out again after it.  A link of a path is one read instead of `cap`.
// Per call, against the general kernel (3072 x 768, V = 64, us): 48 problems of 96 x 96 105 -> 62; 384, 192 and 96 points to 48
// clusters 148 -> 24 on average, 35 to 53 the first round of a clustering, 7 to 15 the second; 48 x 48 45 -> 18.  The forms for 49 to 96
// columns of up to 256 and 384 rows have 24 and 36 entries a thread and spill 43 and 98 registers; still, first and second round: 256
// points to 64 clusters 190 -> 88 and 170 -> 31, 384 to 64 334 -> 121 and 255 -> 50, 384 to 96 462 -> 142 and 334 -> 50.  512 points (438
// and 313 to 64 clusters) are the general kernel's.  What is left is the chain of the paths, some 700 clocks a link with two
// columns a lane, 450 with one, and 3300 to 8500 clocks a round.

constexpr int kTileThreads = 1024;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kTileLanes = 8;                                    // of a row
constexpr int kTileRows = kTileThreads / kTileLanes;             // at a time
constexpr int kTileRounds = 5;
constexpr int kTileMaxCap = 12;  // of a column's candidates two of every twelve rows are looked at
constexpr float kTileFar = 1e30f;  // a pair that cannot be taken; scaled costs are below 2
constexpr float kTileAny = 1e29f;

struct TileLds {  // byte offsets into dynamic LDS
  int cost, step, who, v, vf, count, largest, row_col, best, list, members, filled, changed, partial, total;
};
template <int TC, bool CAPACITY>
__host__ __device__ inline TileLds tile_lds(int n, int m) {
  TileLds l;
  int off = 0;
  l.cost = l.step = off;                                         // costs; capacities: what moving a row costs, and
  off += (CAPACITY ? m * m : n * m) * 8;
  l.v = off;        off += m * 8;
  l.partial = off;  off += kTileWaves * (CAPACITY ? 2 : 1) * (TC * kTileLanes + 1) * 8;
  l.vf = off;       off += TC * kTileLanes * 4;
  l.count = off;    off += 2 * TC * kTileLanes * 4;
  l.largest = off;  off += 8;
  l.row_col = off;  off += n * 4;
  l.best = off;     off += n * 4;
  l.list = off;     off += n * 4;
  l.members = off;  off += n * 4;
  l.filled = off;   off += m * 4;
  l.changed = off;  off += (m + 4) * 4;
  l.who = off;      off += CAPACITY ? m * m * 2 : 0;             // which row it is
  l.total = (off + 15) & ~15;
  return l;
}

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true));
}
// lane ^ 1, lane ^ 2, the other four of eight (once those agree), lane ^ 8
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppXor8 = 0x128;

// Minimum as a median: one instruction, where fminf first quiets operands that come from another lane.
__device__ __forceinline__ float least_of(float x, float y) { return __builtin_amdgcn_fmed3f(x, y, -__builtin_inff()); }
// two smallest of (s1 <= s2) and (t1 <= t2)
__device__ __forceinline__ void merge_two(float& s1, float& s2, float t1, float t2) {
  s2 = least_of(__builtin_amdgcn_fmed3f(s1, s2, t1), t2);
  s1 = least_of(s1, t1);
}
template <int CTRL>
__device__ __forceinline__ void merge_two_dpp(float& s1, float& s2) {
  merge_two(s1, s2, dpp<CTRL>(s1), dpp<CTRL>(s2));
}
__device__ __forceinline__ void swap32(float& a, float& b) {  // upper half of a <-> lower half of b
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(float& a, float& b) {  // odd rows of 16 lanes of a <-> even rows of b
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

__device__ __forceinline__ float read_lane(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// The value of lane ^ D.
template <int D>
__device__ __forceinline__ float across(float x) {
  if constexpr (D == 1) return dpp<kDppXor1>(x);
  if constexpr (D == 2) return dpp<kDppXor2>(x);
  if constexpr (D == 4) {  // four lanes down in the lower fours of eight, four up in the upper ones
    const int down = __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x104, 0xf, 0x5, false);
    return __int_as_float(__builtin_amdgcn_update_dpp(down, __float_as_int(x), 0x114, 0xf, 0xa, false));
  }
  if constexpr (D == 8) return dpp<kDppXor8>(x);
  float a = x, b = x;
  if constexpr (D == 16) swap16(a, b);
  else swap32(a, b);
  return (threadIdx.x & D) ? a : b;
}

// Q times 64 values, one a lane, ascending over the lanes (bitonic; the Q sorts hide each other's latency).  Counting passes
// over the bits of a key took twice as long: their scalar instructions depend on each other.
template <int K, int D, int Q>
__device__ __forceinline__ void sort_pass(float (&x)[Q], const uint32_t (&sign)[7]) {
  // minus infinity: the smaller value stays here
  const float end = __uint_as_float(0xff800000u ^ sign[__builtin_ctz(D)] ^ sign[__builtin_ctz(K)]);
#pragma unroll
  for (int q = 0; q < Q; ++q) x[q] = __builtin_amdgcn_fmed3f(x[q], across<D>(x[q]), end);
  if constexpr (D > 1) sort_pass<K, D / 2>(x, sign);
  else if constexpr (K < 64) sort_pass<2 * K, K>(x, sign);
}
template <int Q>
__device__ __forceinline__ void wave_sort(float (&x)[Q]) {
  uint32_t sign[7];  // of every bit of the lane's number
#pragma unroll
  for (int bit = 0; bit < 7; ++bit) sign[bit] = bit < 6 ? (threadIdx.x << (31 - bit)) & 0x80000000u : 0u;
  // (worked out here: 21 words kept over the rounds are spilled)
  asm volatile("" : "+v"(sign[0]), "+v"(sign[1]), "+v"(sign[2]), "+v"(sign[3]), "+v"(sign[4]), "+v"(sign[5]));
  sort_pass<2, 1>(x, sign);
}

// Rows take the column of their minimum (`best`, -1 = none) while it has room, lower rows first; the others are listed.
// One wave.  Returns how many are left.
__device__ __forceinline__ int fill_columns(const int* best, int* row_col, int* filled, int* members, int* list, int n, int cap) {
  const int lane = threadIdx.x & 63;
  const unsigned long long lower = (1ull << lane) - 1ull;
  int n_free = 0;
  for (int i0 = 0; i0 < n; i0 += 64) {
    const int i = i0 + lane;
    const int j = i < n ? best[i] : -1;
    unsigned long long same = __ballot(j >= 0);  // lanes of the same column
#pragma unroll
    for (int bit = 0; bit < 7; ++bit) {
      const bool set = (j >> bit) & 1;
      const unsigned long long mask = __ballot(set);
      same &= set ? mask : ~mask;
    }
    const int before = j >= 0 ? filled[j] : cap;
    const int slot = before + __popcll(same & lower);
    const bool sits = slot < cap;
    if (sits) members[j * cap + slot] = i;
    if (j >= 0 && (same >> lane) == 1ull) filled[j] = min(slot + 1, cap);  // the column's last lane
    if (i < n) row_col[i] = sits ? j : -1;
    const bool is_free = i < n && !sits;
    const unsigned long long mask = __ballot(is_free);
    if (is_free) list[n_free + __popcll(mask & lower)] = i;
    n_free += __popcll(mask);
  }
  return n_free;
}

// Start of a problem of at most TR * 128 rows and TC * 8 columns: everything up to `fill_columns`.  Without capacities the
// matrix is left in LDS, less the smallest cost of every row.
template <int TR, int TC, bool CAPACITY>
__device__ __forceinline__ void tile_start(const double* __restrict__ cost, uint8_t* lds, const TileLds& L, int n, int m, int cap) {
  constexpr int COLUMNS = TC * kTileLanes;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane & (kTileLanes - 1);
  const int r0 = tid >> 3;  // row of the thread, of every kTileRows
  double* const lds_cost = reinterpret_cast<double*>(lds + L.cost);
  double* const v = reinterpret_cast<double*>(lds + L.v);
  float* const vf = reinterpret_cast<float*>(lds + L.vf);
  int* const count = reinterpret_cast<int*>(lds + L.count);
  int* const largest_at = reinterpret_cast<int*>(lds + L.largest);
  int* const best = reinterpret_cast<int*>(lds + L.best);
  int* const filled = reinterpret_cast<int*>(lds + L.filled);
  constexpr int kGroupStride = COLUMNS + 1;  // float2: the candidates of a column are read from all banks
  float2* const partial = reinterpret_cast<float2*>(lds + L.partial);

  // A second time from L2 where the costs themselves do not fit beside the scaled ones.
  constexpr bool KEEP = TR * TC <= 16;
  double x[KEEP ? TR : 1][TC], off[TR];
  auto cost_at = [&](int i, int j) {  // 32-bit offsets from one address
    return *reinterpret_cast<const double*>(reinterpret_cast<const uint8_t*>(cost) + (uint32_t)(i * m + j) * 8u);
  };
  auto one_at_a_time = [] {
    if constexpr (!KEEP) __builtin_amdgcn_sched_barrier(0);
  };
  auto load_row = [&](int k) {
    one_at_a_time();
    const int i = min(r0 + k * kTileRows, n - 1);
#pragma unroll
    for (int c = 0; c < TC; ++c) x[KEEP ? k : 0][c] = cost_at(i, min(lc + kTileLanes * c, m - 1));
  };
  if constexpr (KEEP) {
#pragma unroll
    for (int k = 0; k < TR; ++k) load_row(k);
  }
  for (int j = tid; j < COLUMNS; j += kTileThreads) {
    count[j] = count[COLUMNS + j] = 0;
    if (j < m) filled[j] = 0;
  }
  if (tid == 0) *largest_at = 0;
  int largest = 0;
#pragma unroll
  for (int k = 0; k < TR; ++k) {
    if constexpr (!KEEP) load_row(k);
    double (&row)[TC] = x[KEEP ? k : 0];
    double least = kInf;
#pragma unroll
    for (int c = 0; c < TC; ++c) least = row[c] < least ? row[c] : least;
    double other = dpp<kDppXor1>(least);
    least = other < least ? other : least;
    other = dpp<kDppXor2>(least);
    least = other < least ? other : least;
    other = dpp<kDppHalfMirror>(least);
    least = other < least ? other : least;
    off[k] = least > -kInf && least < kInf ? least : 0.0;
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      row[c] -= off[k];
      if (__builtin_fabs(row[c]) < kInf) largest = max(largest, __double2hiint(row[c]) & 0x7fffffff);
    }
  }
  largest = -wave_min(-largest);
  __syncthreads();
  if (lane == 0) atomicMax(largest_at, largest);
  __syncthreads();
  // powers of two: costs times `scale` are below 2, and the start's potentials are of scaled costs
  const int exponent = max(*largest_at >> 20, 1);
  const double scale = __hiloint2double((2046 - exponent) << 20, 0), unscale = __hiloint2double(exponent << 20, 0);
  float cf[TR][TC];
#pragma unroll
  for (int k = 0; k < TR; ++k) {
    const int i = r0 + k * kTileRows;
    if constexpr (!KEEP) load_row(k);
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      const int j = lc + kTileLanes * c;
      const bool there = i < n && j < m;
      const double left = KEEP ? x[KEEP ? k : 0][c] : x[0][c] - off[k];
      cf[k][c] = there && __builtin_fabs(left) < kInf ? (float)(left * scale) : kTileFar;
      if constexpr (!CAPACITY) {
        if (there) lds_cost[i * m + j] = left;
      }
    }
  }

  // The potentials begin at the columns' means: what a column costs every row more than others do is out of the way at
  // once (a centroid's own norm), which the rounds would take four to find.
  constexpr int H = TC / 2;  // over a wave's rows half of the columns end up in each half of the wave
  {
    float sum[TC];
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      sum[c] = 0.f;
#pragma unroll
      for (int k = 0; k < TR; ++k) sum[c] += r0 + k * kTileRows < n ? fminf(cf[k][c], 2.f) : 0.f;
    }
#pragma unroll
    for (int c = 0; c < H; ++c) {
      swap32(sum[c], sum[c + H]);
      float t = sum[c] += sum[c + H];
      swap16(sum[c], t);
      sum[c] += t;
      sum[c] += dpp<kDppXor8>(sum[c]);
      if ((lane & 31) < 8) partial[wave * kGroupStride + lc + kTileLanes * (lane < 32 ? c : c + H)].x = sum[c];
    }
    __syncthreads();
    if (tid < COLUMNS) {
      float total = 0.f;
#pragma unroll
      for (int w = 0; w < kTileWaves; ++w) total += partial[w * kGroupStride + tid].x;
      vf[tid] = total / (float)n;
    }
    __syncthreads();
  }
  for (int round = 0; round < kTileRounds; ++round) {
    float u[TC];
#pragma unroll
    for (int c = 0; c < TC; ++c) u[c] = vf[lc + kTileLanes * c];
    // An entry's claim on its column is its reduced cost less the best of its row outside the column.
    float y[TC];
    float s1[TC], s2[TC];
#pragma unroll
    for (int c = 0; c < TC; ++c) s1[c] = s2[c] = 3e38f;
    int* const asked = count + (round == 0 ? 0 : COLUMNS);
    const bool looks = round == 0 || round == kTileRounds / 2;  // whether the rounds can end
#pragma unroll
    for (int k = 0; k < TR; ++k) {
      float b1 = 3e38f, b2 = 3e38f;
#pragma unroll
      for (int c = 0; c < TC; ++c) {
        y[c] = cf[k][c] - u[c];
        b2 = __builtin_amdgcn_fmed3f(b1, b2, y[c]);
        b1 = least_of(b1, y[c]);
      }
      const float mine = b1;
      merge_two_dpp<kDppXor1>(b1, b2);
      merge_two_dpp<kDppXor2>(b1, b2);
      merge_two_dpp<kDppHalfMirror>(b1, b2);
      // a row without a finite cost moves no potential; one with a single one claims its column, within bounds
      const bool any = b1 < kTileAny;
      if (looks && any && mine == b1) {
        int at = 0;
#pragma unroll
        for (int c = 1; c < TC; ++c) at = y[c] == b1 ? c : at;
        atomicAdd(&asked[lc + kTileLanes * at], 1);
      }
      const float first = any ? b1 : -3e38f, second = any ? b1 + fminf(b2 - b1, 4.f) : -3e38f;
#pragma unroll
      for (int c = 0; c < TC; ++c) {
        const float claim = y[c] - (y[c] == b1 ? second : first);
        s2[c] = __builtin_amdgcn_fmed3f(s1[c], s2[c], claim);
        s1[c] = least_of(s1[c], claim);
      }
    }
#pragma unroll
    for (int c = 0; c < H; ++c) {
      swap32(s1[c], s1[c + H]);
      swap32(s2[c], s2[c + H]);
      merge_two(s1[c], s2[c], s1[c + H], s2[c + H]);
      float t1 = s1[c], t2 = s2[c];
      swap16(s1[c], t1);
      swap16(s2[c], t2);
      merge_two(s1[c], s2[c], t1, t2);
      if constexpr (!CAPACITY) merge_two_dpp<kDppXor8>(s1[c], s2[c]);
      const int j = lc + kTileLanes * (lane < 32 ? c : c + H);
      if ((lane & 31) < (CAPACITY ? 16 : 8))
        partial[(CAPACITY ? 2 * wave + ((lane >> 3) & 1) : wave) * kGroupStride + j] = make_float2(s1[c], s2[c]);
    }
    __syncthreads();
    if (looks) {
      bool too_many = false;
      for (int j = lane; j < COLUMNS; j += 64) too_many = too_many || asked[j] > cap;
      if (__ballot(too_many) == 0) break;  // every row has its best column
    }
    if constexpr (CAPACITY) {
      // One wave per column, several at once: of every twelve rows the two smallest are known, which nearly always holds the
      // cap-th smallest of all and the one after it.
      constexpr int Q = (COLUMNS + kTileWaves - 1) / kTileWaves;
      float x[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int j = min(wave + q * kTileWaves, COLUMNS - 1);
        x[q] = reinterpret_cast<const float*>(partial + (lane >> 1) * kGroupStride + j)[lane & 1];
      }
      wave_sort(x);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int j = wave + q * kTileWaves;
        const float lo = read_lane(x[q], cap - 1), hi = read_lane(x[q], cap);
        if (lane == 0 && j < m && hi < kTileAny) vf[j] += 0.4f * (lo + hi);
      }
    } else if (tid < m) {
      float t1 = 3e38f, t2 = 3e38f;
#pragma unroll
      for (int w = 0; w < kTileWaves; ++w) {
        const float2 s = partial[w * kGroupStride + tid];
        merge_two(t1, t2, s.x, s.y);
      }
      if (t2 < kTileAny) vf[tid] += 0.4f * (t1 + t2);
    }
    __syncthreads();
  }
  if (tid < m) v[tid] = (double)vf[tid] * unscale;
  __syncthreads();
  // now exactly
#pragma unroll
  for (int k = 0; k < TR; ++k) {
    const int i = r0 + k * kTileRows;
    const int row = min(i, n - 1);
    one_at_a_time();
    double least = kInf;
    int at = 0;
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      const int j = lc + kTileLanes * c;
      const int jj = min(j, m - 1);
      const double y = (CAPACITY ? cost_at(row, jj) - off[k] : lds_cost[row * m + jj]) - v[jj];
      const bool less = y < least && j < m;
      least = less ? y : least;
      at = less ? j : at;
    }
    auto take = [&](double y, int j) {
      const bool less = y < least || (y == least && j < at);
      least = less ? y : least;
      at = less ? j : at;
    };
    take(dpp<kDppXor1>(least), __builtin_amdgcn_mov_dpp(at, kDppXor1, 0xf, 0xf, true));
    take(dpp<kDppXor2>(least), __builtin_amdgcn_mov_dpp(at, kDppXor2, 0xf, 0xf, true));
    take(dpp<kDppHalfMirror>(least), __builtin_amdgcn_mov_dpp(at, kDppHalfMirror, 0xf, 0xf, true));
    if (lc == 0 && i < n) best[i] = least < kFar ? at : -1;
  }
  __syncthreads();
}

// Paths of the free rows where a column takes `cap` rows, 64 c + lane in register c.  `step` and `who`: for every column
// that holds rows the least that moving one of them to another column costs, and which row that is.
template <int CPL>
__device__ __forceinline__ bool capacity_paths(const double* __restrict__ cost, uint8_t* lds, const TileLds& L, int n, int m,
                                               int cap) {
  double* const step = reinterpret_cast<double*>(lds + L.step);
  uint16_t* const who = reinterpret_cast<uint16_t*>(lds + L.who);
  const double* const start_v = reinterpret_cast<const double*>(lds + L.v);
  int* const row_col = reinterpret_cast<int*>(lds + L.row_col);
  int* const list = reinterpret_cast<int*>(lds + L.list);
  int* const members = reinterpret_cast<int*>(lds + L.members);
  int* const filled = reinterpret_cast<int*>(lds + L.filled);
  int* const changed = reinterpret_cast<int*>(lds + L.changed);  // columns; [m] how many, [m + 1] free rows, [m + 2] failed
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int col[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) col[c] = min(64 * c + lane, m - 1);
  auto work_out = [&](int j) {  // one wave
    const int rows = __builtin_amdgcn_readfirstlane(filled[j]);
    double least[CPL];
    int least_row[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      least[c] = kInf;
      least_row[c] = 0;
    }
    for (int e0 = 0; e0 < rows; e0 += 8) {  // eight rows in flight
      double x[8][CPL];
      int i[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        i[e] = __builtin_amdgcn_readfirstlane(members[j * cap + min(e0 + e, rows - 1)]);
#pragma unroll
        for (int c = 0; c < CPL; ++c) x[e][c] = cost[(size_t)i[e] * m + col[c]];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double from = at_column(x[e], j);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const double y = x[e][c] - from;
          const bool less = y < least[c];
          least[c] = less ? y : least[c];
          least_row[c] = less ? i[e] : least_row[c];
        }
      }
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c)
      if (64 * c + lane < m) {
        step[j * m + col[c]] = least[c];
        who[j * m + col[c]] = (uint16_t)least_row[c];
      }
  };
  const int n_free = __builtin_amdgcn_readfirstlane(changed[m + 1]);
  if (n_free > 0)
    for (int j = wave; j < m; j += kTileWaves) work_out(j);
  __syncthreads();
  double v[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) v[c] = 64 * c + lane < m ? start_v[col[c]] : 0.0;
  for (int k = 0; k < n_free; ++k) {
    if (wave == 0) {
      const int start = __builtin_amdgcn_readfirstlane(list[k]);
      double row[CPL], open[CPL], work[CPL], d[CPL];
      int pred[CPL], y[CPL];
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        row[c] = cost[(size_t)start * m + col[c]];
        pred[c] = start;
        y[c] = 64 * c + lane < m ? filled[col[c]] : 0;
      }
      {  // less a constant of the row: its smallest cost
        double base = kInf;
#pragma unroll
        for (int c = 0; c < CPL; ++c) base = row[c] < base ? row[c] : base;
        base = read_lane(base, wave_argmin_lane(base));
        base = base > -kInf && base < kInf ? base : 0.0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) row[c] -= base;
      }
      int end = -1;
      double reach = 0.0;
      if (start_path(row, v, m, open, work, d)) {
        for (int link = 0; link < m; ++link) {  // every pass but the last closes one more column
          int at, at_c;
          if (__builtin_expect(!nearest_column(open, reach, at, at_c), 0)) break;
          const int j1 = 64 * at_c + at;
          double x[CPL];
          int mover[CPL];
#pragma unroll
          for (int c = 0; c < CPL; ++c) {
            x[c] = step[j1 * m + col[c]];
            mover[c] = who[j1 * m + col[c]];
          }
          if (__builtin_expect(at_column(y, j1) < cap, 0)) {
            end = j1;
            break;
          }
          const double h = at_column(v, j1) + reach;
          close_column(open, work, d, reach, j1);
#pragma unroll
          for (int c = 0; c < CPL; ++c) {
            const double through = (x[c] - work[c]) + h;
            const bool better = through < open[c];
            open[c] = better ? through : open[c];
            pred[c] = better ? mover[c] : pred[c];
          }
        }
      }
      int touched = 0;
      if (end >= 0) {
        move_potentials(v, work, d, reach);
        // shift the rows along the path
        int j = end;
        int slot = at_column(y, end);
        if (lane == 0) filled[end] = slot + 1;
        for (int guard = 0; guard <= m; ++guard) {
          const int i = at_column(pred, j);
          const int from = __builtin_amdgcn_readfirstlane(row_col[i]);
          int freed = 0;
          if (i != start) freed = __builtin_ctzll(__ballot(members[from * cap + min(lane, cap - 1)] == i));
          if (lane == 0) {
            row_col[i] = j;
            members[j * cap + slot] = i;
            changed[touched] = j;
          }
          ++touched;
          slot = freed;
          if (i == start || touched == m) break;
          j = from;
        }
      }
      if (lane == 0) {
        changed[m] = touched;
        if (end < 0) changed[m + 2] = 1;
      }
    }
    __syncthreads();
    if (changed[m + 2]) return false;
    const int touched = changed[m];
    if (k + 1 < n_free)
      for (int e = wave; e < touched; e += kTileWaves) work_out(__builtin_amdgcn_readfirstlane(changed[e]));
    __syncthreads();
  }
  return true;
}

template <int CPL, int TR, int TC, bool CAPACITY>
__global__ __launch_bounds__(kTileThreads) void assign_tile_kernel(const double* __restrict__ cost, int32_t* __restrict__ assign,
                                                                   int n, int m, int cap) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const TileLds L = tile_lds<TC, CAPACITY>(n, m);
  cost += (size_t)blockIdx.x * n * m;
  assign += (size_t)blockIdx.x * n;
  tile_start<TR, TC, CAPACITY>(cost, lds, L, n, m, cap);
  const int* const best = reinterpret_cast<const int*>(lds + L.best);
  int* const row_col = reinterpret_cast<int*>(lds + L.row_col);
  int* const list = reinterpret_cast<int*>(lds + L.list);
  int* const members = reinterpret_cast<int*>(lds + L.members);
  int* const filled = reinterpret_cast<int*>(lds + L.filled);
  int* const changed = reinterpret_cast<int*>(lds + L.changed);
  const int tid = threadIdx.x;
  int n_free = 0;
  if (tid < 64) {
    n_free = fill_columns(best, row_col, filled, members, list, n, cap);
    if (tid == 0) {
      changed[m + 1] = n_free;
      changed[m + 2] = 0;
    }
  }
  if constexpr (CAPACITY) {
    __syncthreads();
    const bool found = capacity_paths<CPL>(cost, lds, L, n, m, cap);
    for (int e = tid; e < n; e += kTileThreads) {
      if (found) assign[members[e]] = e;
      else assign[e] = e;
    }
  } else {
    if (tid >= 64) return;
    const double* const matrix = reinterpret_cast<const double*>(lds + L.cost);
    const bool found = row_paths<CPL>([&](int i, int j) { return matrix[i * m + j]; }, reinterpret_cast<const double*>(lds + L.v),
                                      filled, members, list, n_free, row_col, m);
    for (int i = tid; i < n; i += 64) assign[i] = found ? row_col[i] : i;
  }
}

template <int CPL, int TR, int TC, bool CAPACITY>
hipError_t launch_tile(const double* cost, int32_t* assign, int problems, int n, int m, int cap, hipStream_t stream) {
  constexpr auto kernel = assign_tile_kernel<CPL, TR, TC, CAPACITY>;
  if (hipError_t e = raise_lds_limit<kernel>(kLdsBytes); e != hipSuccess) return e;
  kernel<<<problems, kTileThreads, (tile_lds<TC, CAPACITY>(n, m).total), stream>>>(cost, assign, n, m, cap);
  return hipGetLastError();
}

// Matrices of up to 36 entries a thread (of up to 16 without capacities, and 132 KB in LDS); larger ones were not tried.
bool tile_holds(int n, int m, int cap) {
  return cap == 1 ? m <= 128 : n <= 3 * kTileRows && m <= 96 && cap <= kTileMaxCap;
}

hipError_t launch_tiles(const double* cost, int32_t* assign, int problems, int n, int m, int cap, hipStream_t stream) {
  if (cap == 1) {
    if (m <= 48) return launch_tile<1, 1, 6, false>(cost, assign, problems, n, m, cap, stream);
    if (m <= 64) return launch_tile<1, 1, 8, false>(cost, assign, problems, n, m, cap, stream);
    if (m <= 96) return launch_tile<2, 1, 12, false>(cost, assign, problems, n, m, cap, stream);
    return launch_tile<2, 1, 16, false>(cost, assign, problems, n, m, cap, stream);
  }
  if (m <= 48) {
    if (n <= kTileRows) return launch_tile<1, 1, 6, true>(cost, assign, problems, n, m, cap, stream);
    if (n <= 2 * kTileRows) return launch_tile<1, 2, 6, true>(cost, assign, problems, n, m, cap, stream);
    return launch_tile<1, 3, 6, true>(cost, assign, problems, n, m, cap, stream);
  }
  if (n <= 2 * kTileRows) return launch_tile<2, 2, 12, true>(cost, assign, problems, n, m, cap, stream);
  return launch_tile<2, 3, 12, true>(cost, assign, problems, n, m, cap, stream);
}

template <int CPL, bool IN_LDS, bool CAPACITY>
hipError_t launch_cfg(const double* cost, int32_t* assign, int problems, int n, int m, int cap, hipStream_t stream) {
  constexpr int THREADS = CPL <= 4 ? 1024 : 512;  // 128 / 256 registers a lane: the paths need a dozen per column
  constexpr auto kernel = assign_kernel<CPL, THREADS, IN_LDS, CAPACITY>;
  if (hipError_t e = raise_lds_limit<kernel>(kLdsBytes); e != hipSuccess) return e;
  kernel<<<problems, THREADS, assign_lds(n, m, THREADS, IN_LDS).total, stream>>>(cost, assign, n, m, cap);
  return hipGetLastError();
}

// Problems that `tile_holds` leaves: with one row a column those have more than 128 columns.
template <bool CAPACITY>
hipError_t launch(const double* cost, int32_t* assign, int problems, int n, int m, int cap, hipStream_t stream) {
  const bool in_lds = assign_lds(n, m, 1024, true).total <= kLdsBytes;
  if constexpr (CAPACITY) {
    if (m <= 64) return (in_lds ? launch_cfg<1, true, true> : launch_cfg<1, false, true>)(cost, assign, problems, n, m, cap, stream);
    if (m <= 128) return (in_lds ? launch_cfg<2, true, true> : launch_cfg<2, false, true>)(cost, assign, problems, n, m, cap, stream);
  } else {
    if (in_lds) return launch_cfg<4, true, false>(cost, assign, problems, n, m, cap, stream);  // at most some 135 x 135
  }
  if (m <= 256) return launch_cfg<4, false, CAPACITY>(cost, assign, problems, n, m, cap, stream);
  if (m <= 512) return launch_cfg<8, false, CAPACITY>(cost, assign, problems, n, m, cap, stream);
  if constexpr (!CAPACITY) return launch_cfg<16, false, false>(cost, assign, problems, n, m, cap, stream);
  return hipErrorInvalidValue;  // capacities of two and more leave at most kIcpMaxPartitions / 2 columns
}

}  // namespace

hipError_t launch_assignment(const double* cost, int32_t* assign, int problems, int n, int m, hipStream_t stream) {
  const int cap = n / m;
  if (tile_holds(n, m, cap)) return launch_tiles(cost, assign, problems, n, m, cap, stream);
  return cap == 1 ? launch<false>(cost, assign, problems, n, m, 1, stream)
                  : launch<true>(cost, assign, problems, n, m, cap, stream);
}

}  // namespace hinm
