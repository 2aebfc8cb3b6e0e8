// HiNM product for few columns (decode-like shapes) and for V = 16 tiles
// (arXiv 2407.20496, Section 3.2: input rows are fetched through the vector index, here composed
// with pi_in on the fly; output rows are stored through pi_out).
//
// The work is bound by streaming the packed weights once from HBM.  One workgroup owns 16 rows of
// one tile and a block of 16 columns; its waves split the tile's kept columns into contiguous
// ranges of 64-column steps and each wave runs on its own: it streams its rows' stored values and
// NM nibbles straight into the A operand of the 16x16x64 sparse MFMA, gathers its 64 input rows
// (16 columns wide) into a private LDS slab, reads them back transposed as the B operand, and
// accumulates in fp32.  All global loads of a batch of steps are issued before the first is used
// (weights first, then the index chain vec_idx -> pi_in -> X), without branches, so that every wave
// keeps several kilobytes in flight.  The per-wave partial tiles are summed in a fixed order
// through LDS, so results do not depend on timing.
#include "hinm_internal.h"
#include "mfma_types.h"
#include "column_pieces.h"

namespace hinm {
namespace {

constexpr int kRows = 16;   // rows per workgroup
constexpr int kCols = 16;   // columns per workgroup
constexpr int kStep = 64;   // kept columns per MFMA
// private LDS slab of one wave: 64 rows x 16 columns, 8-row blocks padded so that the four lane
// groups of a transposing read fall on different banks
constexpr int kSlabBytes = 8 * 384;

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

// XMODE: 1 = rows are 16-byte aligned (ld % 8 == 0; columns beyond N are computed on whatever their piece holds and
// never stored), 2 = N == 1.  KB = steps whose loads are issued together.  RBW = 16-row blocks per
// workgroup (they share the gathered B operand).
template <int DT, int NW, int XMODE, int KB, int RBW>
__global__ __launch_bounds__(NW * 64) void spmm_skinny_kernel(
    const uint16_t* __restrict__ vals, const uint8_t* __restrict__ nm_idx, const int32_t* __restrict__ vec_idx,
    const int32_t* __restrict__ pi_in, const int32_t* __restrict__ pi_out, const uint16_t* __restrict__ X,
    int64_t ldx, void* __restrict__ Y, int64_t ldy, int V, int Kv, int N, bool relu, bool out_f32) {
  __shared__ __attribute__((aligned(16))) uint8_t slab_all[NW * kSlabBytes];
  static_assert(RBW * kRows * kCols * 4 <= kSlabBytes, "partial tiles must fit the slab");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = blockIdx.x * (kRows * RBW);  // first row of W handled here
  const int t = row0 / V;
  const int n0 = blockIdx.y * kCols;
  const int full_steps = Kv / kStep;                       // steps with all 64 columns present
  const int steps = (Kv + kStep - 1) / kStep;
  const int per_wave = (full_steps + NW - 1) / NW;
  const int s_begin = wave * per_wave;
  const int s_end = min(full_steps, s_begin + per_wave);   // this wave's contiguous range of full steps

  uint8_t* slab = slab_all + wave * kSlabBytes;
  const int i = lane & 15;   // A row / B column inside the block
  const int q = lane >> 4;   // lane group
  const uint16_t* vrow = vals + (size_t)(row0 + i) * (Kv / 2);
  const uint8_t* nrow = nm_idx + (size_t)(row0 + i) * (Kv / 8);
  const size_t vblock = (size_t)kRows * (Kv / 2);  // distance between the 16-row blocks
  const size_t nblock = (size_t)kRows * (Kv / 8);
  const int32_t* vi = vec_idx + (size_t)t * Kv;
  const bool nm_pairs_aligned = ((Kv / 8) & 1) == 0;

  // output rows of the epilogue, fetched early: element e = threadIdx.x + k * blockDim.x
  constexpr int kOutPerThread = (RBW * kRows * kCols + NW * 64 - 1) / (NW * 64);
  int64_t out_row[kOutPerThread];
#pragma unroll
  for (int k = 0; k < kOutPerThread; ++k) {
    const int e = threadIdx.x + k * NW * 64;
    const int row = min(e / kCols, RBW * kRows - 1);
    out_row[k] = pi_out ? pi_out[row0 + row] : (row0 + row);
  }

  f32x4 acc[RBW];
#pragma unroll
  for (int rb = 0; rb < RBW; ++rb) acc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- the ragged last step (Kv % 64 != 0) belongs to the last wave: guarded loads, requested before everything else
  // and multiplied at the end (the index chain behind the other steps instead: 12.5 against 8.5 us on 192 x 528, V = 16,
  // Kv = 264, N = 220, together with vector loads for ragged columns)
  const bool has_tail = steps > full_steps && wave == NW - 1;
  u32x4 tail_lo = {0, 0, 0, 0}, tail_hi = {0, 0, 0, 0}, tail_a[RBW];
  int tail_idx[RBW];
  auto load_tail = [&]() {
    const int g0 = 16 * full_steps + 4 * q;  // this lane's four groups, all, half or none of them there (Kv % 8 == 0)
    const int j = kStep * full_steps + lane;
    int c = j < Kv ? vi[j] : -1;
    if (c >= 0 && pi_in) c = pi_in[c];
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) {
      tail_a[rb] = u32x4{0, 0, 0, 0};
      tail_idx[rb] = 0;
      const uint16_t* vp = vrow + rb * vblock + 2 * g0;
      const uint8_t* np = nrow + rb * nblock + (g0 >> 1);
      if (g0 + 4 <= Kv / 4) {
        tail_a[rb] = *reinterpret_cast<const u32x4_a4*>(vp);
        tail_idx[rb] = (int)np[0] | ((int)np[1] << 8);
      } else if (g0 + 2 <= Kv / 4) {
        const u32x2 half = *reinterpret_cast<const u32x2_a4*>(vp);
        tail_a[rb] = u32x4{half.x, half.y, 0, 0};
        tail_idx[rb] = (int)np[0];
      }
    }
    if (c >= 0) {
      const uint16_t* xr = X + (size_t)c * ldx + n0;
      if constexpr (XMODE == 1) {
        tail_lo = *reinterpret_cast<const u32x4*>(xr);
        if (piece_inside(n0 + 8, N)) tail_hi = *reinterpret_cast<const u32x4*>(xr + 8);
      } else {
        tail_lo = u32x4{(uint32_t)xr[0], 0, 0, 0};
      }
    }
  };
  if (RBW == 1 && has_tail) load_tail();  // (two row blocks leave no registers for it)
  // this lane's half of a row's 16 columns
  const int piece = half_offset(n0, lane & 1, N);

  for (int sb = s_begin; sb < s_end; sb += KB) {
    u32x4 a_reg[KB][RBW];
    int idx_reg[KB][RBW];
    int col[KB];
    u32x4 b_lo[KB], b_hi[KB];
    // Loads come back in issue order, so the short index chain vec_idx -> pi_in goes first and the
    // bulk weight stream is issued behind it; the input rows are requested as soon as their indices
    // are known and arrive while the weights are still streaming.  (Steps past the wave's range
    // are clamped to its last step and zeroed before use.)
    // phase 1: vector-index entries, then the input-channel order
#pragma unroll
    for (int u = 0; u < KB; ++u) col[u] = vi[kStep * min(sb + u, s_end - 1) + lane];
    if (pi_in) {
#pragma unroll
      for (int u = 0; u < KB; ++u) col[u] = pi_in[col[u]];
    }
    __builtin_amdgcn_sched_barrier(0);
    // phase 2: stored values and NM nibbles
#pragma unroll
    for (int u = 0; u < KB; ++u) {
      const int s = min(sb + u, s_end - 1);
      const int g0 = 16 * s + 4 * q;  // this lane's four groups
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb) {
        a_reg[u][rb] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_a4*>(vrow + rb * vblock + 2 * g0));  // read once
        const uint8_t* np = nrow + rb * nblock + (g0 >> 1);
        if (nm_pairs_aligned) idx_reg[u][rb] = *reinterpret_cast<const uint16_t*>(np);
        else idx_reg[u][rb] = (int)np[0] | ((int)np[1] << 8);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // phase 3: input rows, 16 columns wide
#pragma unroll
    for (int u = 0; u < KB; ++u) {
      const uint16_t* xr = X + (size_t)col[u] * ldx + n0;
      if constexpr (XMODE == 1) {
        // Lanes 2 j and 2 j + 1 fetch the two 16-byte halves of one row (rows j and 32 + j of the step):
        // neighbouring lanes then fall into one cache line, which halves the tag look-ups that a gather of
        // rows scattered by the input-channel order costs.
        const int c_lo = __builtin_amdgcn_ds_bpermute((lane >> 1) * 4, col[u]);
        const int c_hi = __builtin_amdgcn_ds_bpermute((32 + (lane >> 1)) * 4, col[u]);
        b_lo[u] = *reinterpret_cast<const u32x4*>(X + (size_t)c_lo * ldx + n0 + piece);
        b_hi[u] = *reinterpret_cast<const u32x4*>(X + (size_t)c_hi * ldx + n0 + piece);
      } else {
        b_lo[u] = u32x4{(uint32_t)xr[0], 0, 0, 0};
        b_hi[u] = u32x4{0, 0, 0, 0};
      }
    }
    // phase 4: multiply
#pragma unroll
    for (int u = 0; u < KB; ++u) {
      const bool live = sb + u < s_end;  // wave-uniform
      if constexpr (XMODE == 1) {  // half rows: see the loads
        *reinterpret_cast<u32x4*>(slab + slab_row_offset(lane >> 1) + 16 * (lane & 1)) = b_lo[u];
        *reinterpret_cast<u32x4*>(slab + slab_row_offset(32 + (lane >> 1)) + 16 * (lane & 1)) = b_hi[u];
      } else {
        uint8_t* wr = slab + slab_row_offset(lane);
        *reinterpret_cast<u32x4*>(wr) = b_lo[u];
        *reinterpret_cast<u32x4*>(wr + 16) = b_hi[u];
      }
      wave_sync_lds();
      u32x8 b = read_b_operand(slab, i, q);
      if (!live) b = u32x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int rb = 0; rb < RBW; ++rb) {
        const u32x4 a = live ? a_reg[u][rb] : u32x4{0, 0, 0, 0};
        acc[rb] = smfmac_16x16x64<DT, 0>(a, b, acc[rb], idx_reg[u][rb]);
      }
      wave_sync_lds();
    }
  }

  if (has_tail) {
    if (RBW > 1) load_tail();
    uint8_t* wr = slab + slab_row_offset(lane);
    *reinterpret_cast<u32x4*>(wr) = tail_lo;
    *reinterpret_cast<u32x4*>(wr + 16) = tail_hi;
    wave_sync_lds();
    const u32x8 b = read_b_operand(slab, i, q);
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) acc[rb] = smfmac_16x16x64<DT, 0>(tail_a[rb], b, acc[rb], tail_idx[rb]);
  }

  // ---- fixed-order reduction over the waves, epilogue ---------------------------------------
  // D layout: lane holds column lane % 16, rows 4 * (lane / 16) + reg.
  // (the slab is free now; its first kilobytes take this wave's partial tiles)
  wave_sync_lds();
  float* partial = reinterpret_cast<float*>(slab);
#pragma unroll
  for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
    for (int reg = 0; reg < 4; ++reg) partial[(16 * rb + 4 * q + reg) * kCols + i] = acc[rb][reg];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOutPerThread; ++k) {
    const int e = threadIdx.x + k * NW * 64;
    if (e < RBW * kRows * kCols) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) sum += reinterpret_cast<const float*>(slab_all + w * kSlabBytes)[e];
      if (relu) sum = sum > 0.f ? sum : 0.f;
      const int c = e % kCols;
      if (n0 + c < N) {
        if (out_f32) static_cast<float*>(Y)[out_row[k] * ldy + n0 + c] = sum;
        else static_cast<uint16_t*>(Y)[out_row[k] * ldy + n0 + c] = float_to_bits<DT>(sum);
      }
    }
  }
}

template <int DT, int NW, int KB, int RBW>
void launch_modes(const SpmmArgs& a, hipStream_t stream) {
  auto v = static_cast<const uint16_t*>(a.vals);
  auto x = static_cast<const uint16_t*>(a.X);
  const int col_blocks = (a.N + kCols - 1) / kCols;
  auto launch = [&](auto kernel) {
    kernel<<<dim3(a.s.M / (kRows * RBW), col_blocks), NW * 64, 0, stream>>>(
        v, a.nm_idx, a.vec_idx, a.pi_in, a.pi_out, x, a.ldx, a.Y, a.ldy, a.s.V, a.s.Kv, a.N, a.relu, a.out_f32);
  };
  if (a.N == 1) launch(spmm_skinny_kernel<DT, NW, 2, KB, RBW>);
  else launch(spmm_skinny_kernel<DT, NW, 1, KB, RBW>);  // N > 1: every caller's ldx is a multiple of 8
}

template <int DT, int RBW>
void launch_waves(const SpmmArgs& a, hipStream_t stream) {
  const int full_steps = a.s.Kv / kStep;
  // One batch per wave (every load of the wave in flight at once): waves x batch >= steps.  A wave's steps pass through its
  // slab one after the other and every step of a batch is code to fetch, so short layers take a wave a step, and four waves at
  // least, which share the epilogue: 256 x 256, V = 16, Kv = 128, N = 64 3.21 us with one wave and batches of four, 2.67 with two
  // waves, 2.36 with four.  Geometric means over 130 drawn layers: 1.36 up to two steps, 1.3 up to four, 1.17 up to eight (one
  // column: four waves, 1.15 against 1.13) and, with batches of two, 1.08 up to twelve (13 to 16 steps 0.95 to 1.09).  Up to 32
  // steps sixteen waves with batches of two are ahead with one column (1.09; 0.96 with up to 16), except at 25 to 28 (0.94 to 1.02 on 16
  // layers, weights from memory: 12544 x 3584, V = 16 13.1 us on eight, 14.0 on sixteen).  Grids do not change the
  // order: 16-row tiles with up to 36080 workgroups 1.01 to 1.6 times up to eight steps (3200 x 896, 7 steps, N = 2764 190 -> 118
  // us), 1.05 to 1.14 up to twelve.
  if (full_steps <= 4) launch_modes<DT, 4, 1, RBW>(a, stream);
  else if (full_steps <= 8 && a.N == 1) launch_modes<DT, 4, 2, RBW>(a, stream);
  else if (full_steps <= 8) launch_modes<DT, 8, 1, RBW>(a, stream);
  else if (full_steps <= 12) launch_modes<DT, 8, 2, RBW>(a, stream);
  else if (full_steps <= 16) launch_modes<DT, 4, 4, RBW>(a, stream);
  else if (full_steps <= 32 && a.N == 1 && (full_steps <= 24 || full_steps > 28)) launch_modes<DT, 16, 2, RBW>(a, stream);
  else if (full_steps <= 32) launch_modes<DT, 8, 4, RBW>(a, stream);
  // Sixteen waves with batches of three, weights from memory, against eight with six (batches of two and four are slower than
  // either): 768 x 5000, 36 steps, N = 1 6.63 -> 5.90 us, 4480 x 5200, V = 32, 40 steps 12.6 -> 12.1, 896 x 4300, 33 steps, N = 11
  // 7.49 -> 6.85, 256 x 6000, V = 16, 40 steps, N = 40 10.5 -> 9.2; but 1024 x 6000, V = 32, 46 steps, N = 9 9.92 -> 10.49.
  else if (full_steps <= 48 && (full_steps <= 40 || a.N > kCols)) launch_modes<DT, 16, 3, RBW>(a, stream);
  else if (full_steps <= 48) launch_modes<DT, 8, 6, RBW>(a, stream);
  else if (full_steps <= 64) launch_modes<DT, 16, 4, RBW>(a, stream);
  else launch_modes<DT, 16, 6, RBW>(a, stream);
}

}  // namespace

bool spmm_skinny_supported(const SpmmArgs& a) {
  return a.s.V % 16 == 0 && (a.N + 15) / 16 <= 65535;
}

hipError_t launch_spmm_skinny(const SpmmArgs& a, hipStream_t stream) {
  // Two 16-row blocks per workgroup share the gathered input rows; used when there are enough
  // rows that the grid still fills the chip in one round.
  const bool two = (a.s.V % 32 == 0) && (a.s.M / 32 >= 320);
  if (a.s.dtype == HINM_F16) {
    if (two) launch_waves<HINM_F16, 2>(a, stream);
    else launch_waves<HINM_F16, 1>(a, stream);
  } else {
    if (two) launch_waves<HINM_BF16, 2>(a, stream);
    else launch_waves<HINM_BF16, 1>(a, stream);
  }
  return hipGetLastError();
}

}  // namespace hinm
