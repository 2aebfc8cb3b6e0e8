// HiNM product for few columns from the device-tuned layer form, 16 output channels per workgroup
// (arXiv 2407.20496, Section 3.2; layout in prepared_layout.h).
//
// spmm_skinny_prepared_kernel gives every workgroup a 32-row block of a tile; a layer with few tiles
// (4096 rows at V = 128: 128 blocks) then leaves half of the 256 compute units idle.  This kernel
// halves the granularity: one workgroup owns 16 rows and a block of 16 columns and uses the 16x16x64
// sparse MFMA, whose A operand for lane (row i, lane group q) is exactly the 16 bytes the prepared
// block holds for lane 32 (q % 2) + i of substep q / 2 -- so the prepared form is read in place, four
// contiguous 256-byte segments per step.  Otherwise it works like the canonical-array kernel for few
// columns: the waves split the tile's steps into contiguous ranges, every wave issues all loads of a
// batch of steps before it uses the first, gathered rows pass through a private LDS slab and come
// back transposed, and the per-wave partial tiles are added in a fixed order through LDS.
#include "hinm_internal.h"
#include "mfma_types.h"
#include "prepared_layout.h"
#include "direct_lds.h"
#include "column_pieces.h"

namespace hinm {
namespace {

constexpr int kRows = 16;   // rows per workgroup
constexpr int kCols = 16;   // columns per workgroup
constexpr int kStep = 64;   // kept columns per MFMA
// private LDS slab of one wave: 64 rows x 16 columns, 8-row blocks padded so that the four lane
// groups of a transposing read fall on different banks
constexpr int kSlabBytes = 8 * 384;
constexpr int kXLdsMaxBytes = 48 * 1024;    // XMODE 3: the input vector in LDS, up to 24568 elements,
template <int NW>
constexpr int x_pieces = (kXLdsMaxBytes / 16 + NW * 64 - 1) / (NW * 64);  // ... and 16-byte pieces of it per thread

__device__ __forceinline__ int slab_row_offset(int row) { return row * 32 + (row >> 3) * 128; }

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// B operand of one step from the wave's slab: slots 8 h + 4 u .. + 3 of lane group q hold rows
// 32 h + 8 q + 4 u + (0..3) at column i; inside a 16-lane group lane i addresses row (i / 4) and
// columns 4 (i % 4) .. + 3.
__device__ __forceinline__ u32x8 read_b_operand(const uint8_t* slab, int i, int q) {
  u32x8 b;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = 32 * h + 8 * q + 4 * u + (i >> 2);
      const u32x2 v = lds_read_tr16(slab + slab_row_offset(row) + (i & 3) * 8);
      b[(2 * h + u) * 2] = v.x;
      b[(2 * h + u) * 2 + 1] = v.y;
    }
  return b;
}

// XMODE: 1 = rows are 16-byte aligned (ld % 8 == 0; columns beyond N
// are computed on whatever the padding holds and never stored), 2 = N == 1, 3 = N == 1 with the input vector staged in LDS (a 64-lane gather of 2-byte
// elements from global memory costs the address unit one cycle per lane; the vector is small, so the
// workgroup copies it whole, requested before everything else, and picks from LDS), 4 = 16 columns with all K
// input rows resident in LDS (32 bytes each, copied once per workgroup with direct-to-LDS loads: rows
// scattered by the input-channel order otherwise cost a whole 128-byte line each on the way from L2).
// KB = steps whose loads are issued together.  RBW = 1: the workgroup owns 16 rows; RBW = 2: both halves of a
// 32-row block, which share the gathered input rows; RBW = 4: two neighbouring 32-row blocks of one tile (V % 64 == 0).
// CB = 16-column blocks per workgroup (XMODE 1 only): with two or four, a step's weights, gather entries and
// cache lines of input rows serve 32 or 64 columns.
template <int DT, int NW, int XMODE, int KB, int RBW, int CB = 1>
__global__ __launch_bounds__(NW * 64) void spmm_rows16_prepared_kernel(
    const uint8_t* __restrict__ prep_blocks, const int32_t* __restrict__ gather, const int32_t* __restrict__ out_rows,
    const uint8_t* __restrict__ zeros, const uint16_t* __restrict__ X, int64_t ldx, void* __restrict__ Y, int64_t ldy,
    int V, int RB, int S64, int N, int K, bool relu, bool out_f32) {
  // a wave's slab holds its gathered rows, later its partial tiles (a kilobyte per 16 rows)
  constexpr int kTiles = RBW * CB;  // 16 x 16 output tiles of the workgroup
  constexpr int kSlab = (XMODE != 4 && kTiles * kRows * kCols * 4 > kSlabBytes) ? kTiles * kRows * kCols * 4 : kSlabBytes;
  __shared__ __attribute__((aligned(16))) uint8_t slab_all[NW * kSlab];
  extern __shared__ __attribute__((aligned(16))) uint16_t x_lds[];  // XMODE 3: K elements + 8 zeros; 4: K rows + a zero row
  static_assert(RBW == 1 || RBW == 2 || RBW == 4, "half a 32-row block, one, or two neighbours");
  static_assert(CB == 1 || ((CB == 2 || CB == 4) && XMODE == 1), "several column blocks only with paired-lane vector loads");
  uint8_t* x_bytes = reinterpret_cast<uint8_t*>(x_lds);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = blockIdx.x * (kRows * RBW);  // first row of the layer handled here
  const int t = row0 / V;
  const int rb32 = (row0 % V) / 32;     // 32-row block of the prepared form that holds these rows
  const int hf = (row0 % 32) / 16;      // ... and which half of it (0 when the workgroup owns both)
  const int n0 = blockIdx.y * (kCols * CB);
  const int per_wave = (S64 + NW - 1) / NW;
  const int s_begin = wave * per_wave;
  const int s_end = min(S64, s_begin + per_wave);  // this wave's contiguous range of steps (all steps are full: padded)

  uint8_t* slab = slab_all + wave * kSlab;
  const int i = lane & 15;   // A row / B column inside the block
  const int q = lane >> 4;   // lane group: groups 4 q .. 4 q + 3 of the step = substep q / 2, quad q % 2
  // this lane's 16 bytes inside a (tile, step, row block) block of the prepared form, and its index word
  const int lane32 = 32 * (q & 1) + 16 * hf + i;
  const uint8_t* a_lane = prep_blocks + ((size_t)t * S64 * RB + rb32) * kPrepBlockBytes + (q >> 1) * 1024 + lane32 * 16;
  const uint8_t* idx_lane = prep_blocks + ((size_t)t * S64 * RB + rb32) * kPrepBlockBytes + kPrepIdxOffset + lane32 * 4;
  const size_t step_stride = (size_t)RB * kPrepBlockBytes;
  const int32_t* gt = gather + (size_t)t * S64 * 64;

  // output rows of the epilogue, fetched early: element e = threadIdx.x + k * blockDim.x
  constexpr int kOutPerThread = (kTiles * kRows * kCols + NW * 64 - 1) / (NW * 64);
  int64_t out_row[kOutPerThread];
#pragma unroll
  for (int k = 0; k < kOutPerThread; ++k) {
    const int e = min((int)threadIdx.x + k * NW * 64, kTiles * kRows * kCols - 1);
    const int row = (e / kCols) % (RBW * kRows);  // element e: column block, then row, then column
    out_row[k] = out_rows[row0 + row];
  }

  f32x4 acc[CB][RBW];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) acc[cb][rb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // XMODE 3: this thread's 16-byte pieces of the input vector (requested now, written to LDS after the first
  // batch of weight loads has been issued); every wave passes the barrier exactly once
  u32x4 x_mine[x_pieces<NW>];
  bool x_staged = XMODE != 3 && XMODE != 4;
  if constexpr (XMODE == 3) {
#pragma unroll
    for (int r = 0; r < x_pieces<NW>; ++r) {
      if (r * NW * 64 >= K / 8) break;
      const int piece = min((int)threadIdx.x + r * NW * 64, K / 8 - 1);  // beyond the vector: its last piece again
      x_mine[r] = reinterpret_cast<const u32x4*>(X)[piece];
    }
  }
  // XMODE 4: wave-wide copies of 32 rows x 32 bytes (lane l: row l / 2, half l % 2), requested before everything
  // else; rows past K repeat the last row and are never addressed; the zero row sits behind the last copy
  const int x_copies = (K + 31) / 32;
  const int x_zero_row = 32 * x_copies;
  if constexpr (XMODE == 4) {
    for (int j = wave; j < x_copies; j += NW) {
      const int r = min(32 * j + (lane >> 1), K - 1);
      copy16_to_lds(X + (size_t)r * ldx + n0 + 8 * (lane & 1), x_bytes + (size_t)j * 1024);
    }
    if (threadIdx.x < 8) reinterpret_cast<uint32_t*>(x_bytes + (size_t)x_zero_row * 32)[threadIdx.x] = 0u;
  }
  auto stage_x = [&]() {
    if constexpr (XMODE == 4) {
      wait_copies_outstanding<0>();  // this wave's copies (and its other loads) have landed
      __syncthreads();               // ... and everyone's
    }
    if constexpr (XMODE == 3) {
#pragma unroll
      for (int r = 0; r < x_pieces<NW>; ++r) {
        const int piece = (int)threadIdx.x + r * NW * 64;
        if (piece < K / 8) reinterpret_cast<u32x4*>(x_lds)[piece] = x_mine[r];
      }
      if (threadIdx.x < 8) x_lds[K + threadIdx.x] = 0;  // where padded kept columns read
      __syncthreads();
    }
    x_staged = true;
  };

  // XMODE 1: whether this lane's 16-byte piece of column block cb holds any of the N columns
  bool piece_there[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) piece_there[cb] = piece_inside(n0 + kCols * cb + 8 * (lane & 1), N);
  for (int sb = s_begin; sb < s_end; sb += KB) {
    u32x4 a_reg[KB][RBW];
    int idx_reg[KB][RBW];
    int col[KB];
    u32x4 b_lo[KB][CB], b_hi[KB][CB];
    // Loads come back in issue order: the gather-table entries go first, the bulk weight stream is issued
    // behind them, and the input rows are requested as soon as their indices are known and arrive while the
    // weights are still streaming.  (Steps past the wave's range are clamped to its last step and zeroed
    // before use.)
    // phase 1: gather-table entries (vector index composed with the input-channel order; -1 = padding)
#pragma unroll
    for (int u = 0; u < KB; ++u) col[u] = gt[kStep * min(sb + u, s_end - 1) + lane];
    __builtin_amdgcn_sched_barrier(0);
    // phase 2: stored values and NM nibbles, 16 bytes + one index word per lane and step
#pragma unroll
    for (int u = 0; u < KB; ++u) {
      const size_t off = (size_t)min(sb + u, s_end - 1) * step_stride;
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb) {  // the second half sits 16 lanes further in the block
        // 16-row block rb: half rb % 2 of 32-row block rb / 2 (the second half sits 16 lanes further); the
        // weights are read once, so they are kept from displacing the input rows and tables in the caches
        const size_t blk = (size_t)(rb >> 1) * kPrepBlockBytes;
        a_reg[u][rb] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(a_lane + off + blk + (rb & 1) * 256));
        const uint32_t word = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(idx_lane + off + blk + (rb & 1) * 64));
        idx_reg[u][rb] = (int)((q >> 1) ? (word >> 16) : (word & 0xFFFFu));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!x_staged) stage_x();
    // phase 3: input rows, 16 columns wide
#pragma unroll
    for (int u = 0; u < KB; ++u) {
      const uint16_t* xr = (col[u] >= 0) ? X + (size_t)col[u] * ldx + n0 : reinterpret_cast<const uint16_t*>(zeros);
      if constexpr (XMODE == 4) {
        const uint8_t* xl = x_bytes + (size_t)(col[u] >= 0 ? col[u] : x_zero_row) * 32;
        b_lo[u][0] = *reinterpret_cast<const u32x4*>(xl);
        b_hi[u][0] = *reinterpret_cast<const u32x4*>(xl + 16);
      } else if constexpr (XMODE == 3) {
        b_lo[u][0] = u32x4{(uint32_t)x_lds[col[u] >= 0 ? col[u] : K], 0, 0, 0};
        b_hi[u][0] = u32x4{0, 0, 0, 0};
      } else if constexpr (XMODE == 1) {
        // Lanes 2 j and 2 j + 1 fetch the two 16-byte halves of one row (rows j and 32 + j of the step):
        // neighbouring lanes then fall into one cache line, which halves the tag look-ups that a gather of
        // rows scattered by the input-channel order costs.
        const int c_lo = __builtin_amdgcn_ds_bpermute((lane >> 1) * 4, col[u]);
        const int c_hi = __builtin_amdgcn_ds_bpermute((32 + (lane >> 1)) * 4, col[u]);
        // (a piece of a ragged last block that holds none of the N columns may lie past the end of X: the zero row is
        // read instead; what the last piece holds beyond N never reaches a stored column)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          const uint16_t* r_lo = (c_lo >= 0 && piece_there[cb]) ? X + (size_t)c_lo * ldx + n0 + kCols * cb : reinterpret_cast<const uint16_t*>(zeros);
          const uint16_t* r_hi = (c_hi >= 0 && piece_there[cb]) ? X + (size_t)c_hi * ldx + n0 + kCols * cb : reinterpret_cast<const uint16_t*>(zeros);
          b_lo[u][cb] = *reinterpret_cast<const u32x4*>(r_lo + 8 * (lane & 1));
          b_hi[u][cb] = *reinterpret_cast<const u32x4*>(r_hi + 8 * (lane & 1));
        }
      } else {
        b_lo[u][0] = u32x4{(uint32_t)xr[0], 0, 0, 0};
        b_hi[u][0] = u32x4{0, 0, 0, 0};
      }
    }
    // phase 4: multiply
#pragma unroll
    for (int u = 0; u < KB; ++u) {
      const bool live = sb + u < s_end;  // wave-uniform
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        if constexpr (XMODE == 1) {  // half rows: see the loads
          *reinterpret_cast<u32x4*>(slab + slab_row_offset(lane >> 1) + 16 * (lane & 1)) = b_lo[u][cb];
          *reinterpret_cast<u32x4*>(slab + slab_row_offset(32 + (lane >> 1)) + 16 * (lane & 1)) = b_hi[u][cb];
        } else {
          uint8_t* wr = slab + slab_row_offset(lane);
          *reinterpret_cast<u32x4*>(wr) = b_lo[u][cb];
          *reinterpret_cast<u32x4*>(wr + 16) = b_hi[u][cb];
        }
        wave_sync_lds();
        u32x8 b = read_b_operand(slab, i, q);
        if (!live) b = u32x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int rb = 0; rb < RBW; ++rb) {
          const u32x4 a = live ? a_reg[u][rb] : u32x4{0, 0, 0, 0};
          acc[cb][rb] = smfmac_16x16x64<DT, 0>(a, b, acc[cb][rb], idx_reg[u][rb]);
        }
        wave_sync_lds();
      }
    }
  }

  if (!x_staged) stage_x();  // a wave without steps still owes the barrier

  // ---- fixed-order reduction over the waves, epilogue ---------------------------------------
  // D layout: lane holds column lane % 16, rows 4 * (lane / 16) + reg.
  // (the slab is free now; its first kilobytes take this wave's partial tiles)
  wave_sync_lds();
  // XMODE 4: the partial tiles (a kilobyte each) go where the input rows were, once nobody reads them
  constexpr int kPartialStride = (XMODE == 4) ? kTiles * kRows * kCols * 4 : kSlab;
  if constexpr (XMODE == 4) __syncthreads();
  uint8_t* partial_all = (XMODE == 4) ? x_bytes : slab_all;
  float* partial = reinterpret_cast<float*>(partial_all + wave * kPartialStride);
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
      for (int reg = 0; reg < 4; ++reg) partial[(16 * (cb * RBW + rb) + 4 * q + reg) * kCols + i] = acc[cb][rb][reg];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOutPerThread; ++k) {
    const int e = threadIdx.x + k * NW * 64;
    if (e < kTiles * kRows * kCols) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) sum += reinterpret_cast<const float*>(partial_all + w * kPartialStride)[e];
      if (relu) sum = sum > 0.f ? sum : 0.f;
      const int c = kCols * (e / (RBW * kRows * kCols)) + e % kCols;
      if (n0 + c < N) {
        if (out_f32) static_cast<float*>(Y)[out_row[k] * ldy + n0 + c] = sum;
        else static_cast<uint16_t*>(Y)[out_row[k] * ldy + n0 + c] = float_to_bits<DT>(sum);
      }
    }
  }
}

template <int DT, int NW, int XMODE, int KB, int RBW, int CB = 1>
void launch_form(const PreparedArgs& a, const PreparedLayout& L, int grid_y, size_t lds, hipStream_t stream) {
  if (a.plan) {
    plan_record(a.plan, "spmm_rows16_prepared_kernel<DT=%d,NW=%d,XMODE=%d,KB=%d,RBW=%d,CB=%d> grid=%dx%d block=%d", DT, NW, XMODE,
                KB, RBW, CB, a.s.M / (kRows * RBW), grid_y, NW * 64);
    return;
  }
  const uint8_t* base = static_cast<const uint8_t*>(a.prepared);
  spmm_rows16_prepared_kernel<DT, NW, XMODE, KB, RBW, CB><<<dim3(a.s.M / (kRows * RBW), grid_y), NW * 64, lds, stream>>>(
      base + L.a_offset, reinterpret_cast<const int32_t*>(base + L.gather_offset),
      reinterpret_cast<const int32_t*>(base + L.pi_out_offset), base + L.zero_offset, static_cast<const uint16_t*>(a.X), a.ldx,
      a.Y, a.ldy, a.s.V, L.RB, L.S, a.N, a.s.K, a.relu, a.out_f32);
}

template <int DT, int NW, int KB, int RBW>
void launch_one_column(const PreparedArgs& a, const PreparedLayout& L, hipStream_t stream) {
  if constexpr (KB == 3 || (NW == 8 && KB >= 4)) {  // (the others never have more than four steps a wave)
    // staging the input vector pays once a wave gathers for more than four steps (4096 x 11008 at 50 %:
    // 10.4 -> 9.9 us; with four steps per wave and 688 workgroups it costs 0.8 us instead), with any vector that fits (us, not
    // staged -> staged on eight waves: 6656 x 17920, 140 steps 31.5 -> 17.2, 9216 x 20000, 157 steps 46.5 -> 27.0, 5120 x 24560,
    // 192 steps 43.3 -> 20.4, 8192 x 20480, 40 steps 7.9 -> 7.6; sixteen waves with batches of six, staged: 22.9, 33.3, 24.0 and 11.7)
    const size_t x_bytes = ((size_t)a.s.K + 8) * 2;
    const bool stage = a.ldx == 1 && a.s.K % 8 == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15u) == 0 &&
                       x_bytes <= (size_t)kXLdsMaxBytes && L.S > 4 * NW;
    if (stage) {
      // slabs (static) plus the vector (dynamic) can exceed the default 64 KB of a workgroup
      if (!a.plan && raise_lds_limit<spmm_rows16_prepared_kernel<DT, NW, 3, KB, RBW>>(kXLdsMaxBytes) != hipSuccess)
        return;  // the error stays pending and is reported by the caller's hipGetLastError
      launch_form<DT, NW, 3, KB, RBW>(a, L, 1, x_bytes, stream);
      return;
    }
  }
  launch_form<DT, NW, 2, KB, RBW>(a, L, 1, 0, stream);
}

// Several columns: rows of X start on 16-byte boundaries (the calls ask for it), vector loads for every block, the ragged last
// one included.
template <int DT, int NW, int KB, int RBW>
void launch_columns(const PreparedArgs& a, const PreparedLayout& L, int blocks_per_wg, hipStream_t stream) {
  const int col_blocks = (a.N + kCols - 1) / kCols;
  if constexpr (NW <= 8 && KB == 4) {  // (sixteen waves leave 128 registers per lane: not enough for several blocks)
    // (batches of two steps: four blocks of input rows per step)
    if (blocks_per_wg == 4) return launch_form<DT, NW, 1, 2, RBW, 4>(a, L, (col_blocks + 3) / 4, 0, stream);
    if (blocks_per_wg == 2) return launch_form<DT, NW, 1, KB, RBW, 2>(a, L, (col_blocks + 1) / 2, 0, stream);
  }
  launch_form<DT, NW, 1, KB, RBW>(a, L, col_blocks, 0, stream);
}

// The layer's input rows resident in LDS (XMODE 4): 16 columns, 64 rows per workgroup.
inline size_t resident_lds_bytes(int K) { return (size_t)((K + 31) / 32) * 1024 + 32; }
// The same region later takes the waves' partial tiles (four 16 x 16 fp32 tiles = 4096 bytes per wave), which
// for short input vectors is the larger of the two.
inline size_t resident_dynamic_lds_bytes(int K, int NW) {
  const size_t partials = (size_t)NW * 4 * kRows * kCols * 4;
  return resident_lds_bytes(K) > partials ? resident_lds_bytes(K) : partials;
}

template <int DT, int NW>
void launch_resident(const PreparedArgs& a, const PreparedLayout& L, hipStream_t stream) {
  constexpr auto kernel = spmm_rows16_prepared_kernel<DT, NW, 4, 4, 4>;
  if (a.plan) {
    plan_record(a.plan, "spmm_rows16_prepared_kernel<DT=%d,NW=%d,XMODE=4,KB=4,RBW=4,CB=1> grid=%dx1 block=%d lds=%d", DT,
                NW, a.s.M / 64, NW * 64, (int)resident_dynamic_lds_bytes(a.s.K, NW));
    return;
  }
  if (raise_lds_limit<kernel>(160 * 1024 - NW * kSlabBytes) != hipSuccess)
    return;  // the error stays pending and is reported by the caller's hipGetLastError
  const uint8_t* base = static_cast<const uint8_t*>(a.prepared);
  kernel<<<dim3(a.s.M / 64, 1), NW * 64, resident_dynamic_lds_bytes(a.s.K, NW), stream>>>(
      base + L.a_offset, reinterpret_cast<const int32_t*>(base + L.gather_offset),
      reinterpret_cast<const int32_t*>(base + L.pi_out_offset), base + L.zero_offset,
      static_cast<const uint16_t*>(a.X), a.ldx, a.Y, a.ldy, a.s.V, L.RB, L.S, a.N, a.s.K, a.relu, a.out_f32);
}

// Launch shape beyond the template choice by N: 16-row blocks per workgroup, waves, column blocks per workgroup.
struct Rows16Plan {
  int rbw;
  int nw;
  int blocks_per_wg;  // 16-column blocks: 1, 2 or 4
  int kb;             // steps of a batch
};

// Waves and batch with one column block.  A wave's steps pass through its slab one after the other and every step of a batch is
// code to fetch and registers to hold, so short layers take a wave a step (four at least, which share the epilogue; one column
// has little to hide, eight steps on four waves do), and up to 48 steps a wave's steps are one batch (two with 41 to 48 steps of one
// column; a wave has as many steps as the others or fewer, and what a batch has beyond them is multiplied by zero).  Against one
// to sixteen waves with batches of four and six, geometric means over 130 drawn layers with up to 16 columns: 1.19 up to four
// steps, 1.15 up to eight, 1.1 up to sixteen unless several workgroups of eight waves share a unit (6528 x 7512, 15 steps, N = 16, 408
// workgroups 0.91), 1.07 up to 24, 1.05 up to 40.  Beyond (us, weights from memory): one column, 41 to 48 steps, batches of three
// against one of six on ten layers 0.77 to 0.90 of the time (11008 x 5632, 44 steps 9.8 and 12.8); 49 to 56 steps are one batch
// on sixteen waves, which are ahead while the workgroups fit the units in one round (1600 x 6256, 49 steps 5.49 and 5.81; 8000 x
// 6400, 50 steps 11.2 and 9.5) and as long as their gathers find the vector nearby (eight waves stage it: 0.97 times over 24
// layers of twice the kept columns, 1.03 with three times, 9408 and more, 1.12 with four: 1024 x 14336, 56 steps 7.00 and 5.89);
// with 57 to 64 steps eight are (2464 x 8064 6.84 -> 6.51, 8192 x 8192 13.5 -> 10.2); 86 steps 10.0 -> 8.8, 5120 x 13824, 108
// steps, 320 workgroups 21.6 -> 13.0 (sixteen waves 14.6).  With more columns sixteen waves are ahead throughout (60 layers with
// 49 to 64 steps; 4992 x 6512, N = 4 13.6 and 15.3), in batches of six up to 96 steps (4096 x 11008, N = 16 11.9 and 14.0) and
// beyond 128, where four make three of them (30 layers, 1.03 times; 2112 x 10872, N = 2 21.1 and 22.4), of four between (97 to 128
// steps, 16 layers 1.22 times; 3072 x 16384, 128 steps, N = 16 19.6 -> 16.3).
void one_block_waves(Rows16Plan& p, int S, int K, int N, int64_t wgs) {
  if (S <= 4) p.nw = 4, p.kb = 1;
  else if (S <= 8 && N == 1) p.nw = 4, p.kb = 2;
  else if (S > 12 && S <= 16 && wgs > 256) p.nw = 4, p.kb = 4;
  else if (S > 40 && S <= 48 && N == 1) p.nw = 8, p.kb = 3;
  else if (S <= 48) p.nw = 8, p.kb = (S + 7) / 8;
  else if (S <= 64) p.nw = N == 1 && (S > 56 || K > 9216 || wgs > 256) ? 8 : 16, p.kb = 4;
  else if (N == 1) p.nw = wgs <= 256 ? 16 : 8, p.kb = 3;
  else p.nw = 16, p.kb = S <= 96 || S > 128 ? 6 : 4;
}

Rows16Plan plan_rows16(const PreparedArgs& a) {
  const PreparedLayout L = prepared_layout(a.s);
  Rows16Plan p;
  // Several 16-row blocks in one workgroup share the gathered input rows: both halves of a 32-row block when
  // the grid then still holds 256 workgroups (column blocks count: 4096 x 4096 at N = 128 22.8 -> 17.1 us; one column: 16384 x
  // 4096, 32 steps 10.0 -> 8.8, 13824 x 5120, 40 steps 12.1 -> 9.5), two
  // neighbouring 32-row blocks under the same condition on layers of at least 2048 rows and beyond one column
  // block (-> 13.0 us; 8192 x 8192 at N = 128 62.8 -> 47.8 us; with fewer rows the shorter grid loses: 768 x 3072
  // at N = 384 9.2 -> 12.0 us).
  const int64_t col_blocks = (a.N + kCols - 1) / kCols;
  const bool quad = a.N > kCols && a.s.V % 64 == 0 && a.s.M >= 2048 && (a.s.M / 64) * col_blocks >= 256;
  // One batch of eight waves, one column: everything is requested at once either way, and blocks of 16 rows are kept where they spread
  // more evenly over the units.  From memory 25 layers of 8448 to 12288 rows with 25 to 32 steps 0.98 to 1.06 times (11008 x 4096, 32
  // steps 8.9 -> 8.5 us; 8448 rows, 30 steps 8.2 -> 7.8), from the memory-side cache 0.90 to 1.01 (8.5 and 8.7): a layer is one of many.
  // With 13 to 24 steps both are nearer to level (0.98 to 1.06 and 0.93 to 1.01; 11008 rows, 24 steps 7.3 and 7.1) and the line
  // leaves them; beyond 32 the blocks of 16 lose either way (from memory 0.87 to 0.99).
  const int64_t halves = a.s.M / 16;
  const bool spread = a.N == 1 && L.S > 24 && L.S <= 32 && (halves / 2 + 255) / 256 * 2 > (halves + 255) / 256;
  const bool both = (a.s.M / 32) * col_blocks >= 256 && !spread;
  p.rbw = quad ? 4 : both ? 2 : 1;
  p.blocks_per_wg = 1;
  const int64_t row_wgs = a.s.M / (kRows * p.rbw);
  if (a.N <= kCols) {
    one_block_waves(p, L.S, a.s.K, a.N, row_wgs);
    return p;
  }
  // One batch per wave where possible (every load of the wave in flight at once): waves x batch >= steps ...
  const int nw_steps = L.S <= 4 ? 1 : L.S <= 16 ? 4 : L.S <= 32 ? 8 : 16;
  p.nw = nw_steps;
  // ... but no more waves than the chip can hold at once: with many workgroups (several column blocks, or
  // a tall layer) the parallelism is already there, and fewer waves per workgroup mean fewer partial tiles
  // to sum and more of each wave's own loads in flight one after another (4096 x 4096 at N = 128, 2048
  // workgroups: 32.8 us with eight waves, 22.7 us with one).  About eight waves per compute unit in total.
  //
  // Two or four column blocks per workgroup: a step's weights, gather entries and the 128-byte cache lines of
  // its input rows then serve 32 or 64 columns (11008 x 4096 at N = 128 42.3 -> 31.1 -> 24.8 us, 8192 x 8192
  // at N = 256 89.5 -> 69.3 -> 45.0 us).  It needs a grid that still covers most of the chip (160 workgroups;
  // with 96..159 it measured slower: 4096 x 4096 at N = 64, 128 workgroups left, 7.9 -> 9.5 us) and at least
  // eight steps (from there on never slower under that condition; 8192 x 1024 with 512 kept columns at
  // N = 256: 17.7 -> 13.5 us).
  if (a.ldx % 8 == 0 && L.S >= 8) {
    if (col_blocks >= 3 && row_wgs * ((col_blocks + 3) / 4) >= 160) p.blocks_per_wg = 4;
    else if (row_wgs * ((col_blocks + 1) / 2) >= 160) p.blocks_per_wg = 2;
  }
  const int64_t wgs = row_wgs * ((col_blocks + p.blocks_per_wg - 1) / p.blocks_per_wg);
  while (p.nw > 1 && wgs * p.nw > 2048) p.nw >>= 1;
  if (p.blocks_per_wg > 1 && p.nw > 8) {  // sixteen waves leave too few registers for several blocks
    p.blocks_per_wg = 1;
    p.nw = nw_steps;
    while (p.nw > 1 && row_wgs * col_blocks * p.nw > 2048) p.nw >>= 1;
  }
  p.kb = p.nw == 16 && L.S > 64 ? 6 : 4;
  // Short layers as with one column block while that makes no more than eight waves a unit (1.09 to 1.26 times).
  if (p.blocks_per_wg == 1 && L.S <= 16) {
    Rows16Plan q = p;
    one_block_waves(q, L.S, a.s.K, a.N, row_wgs * col_blocks);
    if (row_wgs * col_blocks * q.nw <= 2048) p = q;
  }
  return p;
}

// The forms that `plan_rows16` chooses: four 16-row blocks only beyond 16 columns, and then eight waves at most.
template <int DT, int RBW>
void launch_waves(const PreparedArgs& a, const Rows16Plan& plan, hipStream_t stream) {
  const PreparedLayout L = prepared_layout(a.s);
  const int blocks = plan.blocks_per_wg, form = plan.nw * 8 + plan.kb;
  if constexpr (RBW <= 2) {
    if (a.N == 1) {
      switch (form) {
        case 4 * 8 + 1: return launch_one_column<DT, 4, 1, RBW>(a, L, stream);
        case 4 * 8 + 2: return launch_one_column<DT, 4, 2, RBW>(a, L, stream);
        case 4 * 8 + 4: return launch_one_column<DT, 4, 4, RBW>(a, L, stream);
        case 8 * 8 + 2: return launch_one_column<DT, 8, 2, RBW>(a, L, stream);
        case 8 * 8 + 3: return launch_one_column<DT, 8, 3, RBW>(a, L, stream);
        case 8 * 8 + 4: return launch_one_column<DT, 8, 4, RBW>(a, L, stream);
        case 8 * 8 + 5: return launch_one_column<DT, 8, 5, RBW>(a, L, stream);
        case 16 * 8 + 4: return launch_one_column<DT, 16, 4, RBW>(a, L, stream);
        default: return launch_one_column<DT, 16, 3, RBW>(a, L, stream);
      }
    }
    switch (form) {
      case 8 * 8 + 3: return launch_columns<DT, 8, 3, RBW>(a, L, 1, stream);
      case 8 * 8 + 5: return launch_columns<DT, 8, 5, RBW>(a, L, 1, stream);
      case 8 * 8 + 6: return launch_columns<DT, 8, 6, RBW>(a, L, 1, stream);
      case 16 * 8 + 4: return launch_columns<DT, 16, 4, RBW>(a, L, 1, stream);
      case 16 * 8 + 6: return launch_columns<DT, 16, 6, RBW>(a, L, 1, stream);
      default: break;
    }
  }
  switch (form) {
    case 1 * 8 + 4: return launch_columns<DT, 1, 4, RBW>(a, L, blocks, stream);
    case 2 * 8 + 4: return launch_columns<DT, 2, 4, RBW>(a, L, blocks, stream);
    case 4 * 8 + 1: return launch_columns<DT, 4, 1, RBW>(a, L, 1, stream);
    case 4 * 8 + 4: return launch_columns<DT, 4, 4, RBW>(a, L, blocks, stream);
    case 8 * 8 + 1: return launch_columns<DT, 8, 1, RBW>(a, L, 1, stream);
    case 8 * 8 + 2: return launch_columns<DT, 8, 2, RBW>(a, L, 1, stream);
    default: return launch_columns<DT, 8, 4, RBW>(a, L, blocks, stream);
  }
}

template <int DT>
void launch_dt(const PreparedArgs& a, hipStream_t stream) {
  // 16 columns and a layer whose input fits in LDS beside the slabs: no gather from global memory at all.
  // Each workgroup then owns 64 rows, so the layer needs enough of them to keep most of the chip streaming,
  // and copying the 32 K bytes of input has to be small beside the workgroup's weights (11008 x 4096:
  // 12.4 -> 10.3 us with 2048 kept columns, 7.4 -> 7.9 us with 1024).
  const PreparedLayout L = prepared_layout(a.s);
  if (spmm_rows16_resident_supported(a) && (a.tile_variant == 19 || spmm_rows16_resident_preferred(a))) {
    if (L.S <= 16) launch_resident<DT, 4>(a, L, stream);
    else launch_resident<DT, 8>(a, L, stream);
    return;
  }
  const Rows16Plan plan = plan_rows16(a);
  if (plan.rbw == 4) launch_waves<DT, 4>(a, plan, stream);
  else if (plan.rbw == 2) launch_waves<DT, 2>(a, plan, stream);
  else launch_waves<DT, 1>(a, plan, stream);
}

}  // namespace

int spmm_rows16_prepared_blocks_per_wg(const PreparedArgs& a) { return plan_rows16(a).blocks_per_wg; }

bool spmm_rows16_resident_supported(const PreparedArgs& a) {
  const PreparedLayout L = prepared_layout(a.s);
  if (a.N != 16 || a.ldx % 8 != 0 || (reinterpret_cast<uintptr_t>(a.X) & 15u) != 0) return false;
  if (a.s.V % 64 != 0 || L.S > 32 || a.tile_variant == 11) return false;
  const int NW = L.S <= 16 ? 4 : 8;
  return resident_dynamic_lds_bytes(a.s.K, NW) + (size_t)NW * kSlabBytes <= 160 * 1024;
}

bool spmm_rows16_resident_preferred(const PreparedArgs& a) {
  return spmm_rows16_resident_supported(a) && a.s.M / 64 >= 160 && prepared_layout(a.s).S > 16;
}

int64_t spmm_rows16_prepared_workgroups(const PreparedArgs& a) {
  const Rows16Plan p = plan_rows16(a);
  const int64_t col_blocks = (a.N + kCols - 1) / kCols;
  return a.s.M / (kRows * p.rbw) * ((col_blocks + p.blocks_per_wg - 1) / p.blocks_per_wg);
}

hipError_t launch_spmm_rows16_prepared(const PreparedArgs& a, hipStream_t stream) {
  if (a.s.dtype == HINM_F16) launch_dt<HINM_F16>(a, stream);
  else launch_dt<HINM_BF16>(a, stream);
  if (a.plan) return hipSuccess;  // a dry run launched nothing
  return hipGetLastError();
}

}  // namespace hinm
