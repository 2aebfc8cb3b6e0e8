// Epilogue shared by the tile kernels whose waves each hold all V = 32 * RB rows of the tile for WC of the
// workgroup's NB columns in 32x32 MFMA accumulators (arXiv 2407.20496, Section 3.2: the tile's result goes to the
// output channels named by the output-channel order; Section 5.3: re-ordering at no run-time cost).
//   fp32 accumulators -> optional ReLU -> either fp32 straight from the registers, or rounded to the 16-bit
//   storage type, staged through LDS so that every output row leaves as one
//   contiguous segment, written with non-temporal 16-byte stores (the ragged tail element by element).
#pragma once

#include "hinm_internal.h"
#include "mfma_types.h"

namespace hinm {

// acc[rb][cb][e]: D layout of the 32x32 MFMA, lane holds column lane % 32, rows 8 * (e / 4) + 4 * (lane / 32) + e % 4
// of row block rb, 32-column block cb of the wave.  `out_row_of(row)` names the row of Y for row `row` of the tile.

// Bytes between two staged rows: NB columns and 64 bytes more, so that the four pieces of 64 bytes that a half-wave of
// stage_block writes (two rows) and the 16-byte reads of a row fall on different banks.
template <int NB>
constexpr int kStageStride = NB * 2 + 64;

// v > 0 ? v : +0, and 0 for NaN: the median of v, 0 and infinity, one instruction (written as a comparison the compiler
// takes two, one of them for signalling NaN).
__device__ __forceinline__ float relu_f32(float v) { return __builtin_amdgcn_fmed3f(v, 0.f, __builtin_inff()); }

// One 32x32 block of results into the staging area: `block` is the staged address of its first row and column.  A lane
// holds one column, and writing its 16 values by themselves (ds_write_b16, 11 clocks each with every wave of a 128 x 512
// workgroup writing) took 4 to 7 us of a workgroup's life, as much as four 64-row stages of the k loop.  Neighbouring
// lanes exchange halves first (even lane: row e, odd lane: row e + 1, two columns each), which halves the writes and
// makes them 32 bits wide: 11100 -> 4700 clocks.
template <int DT, int STRIDE>
__device__ __forceinline__ void stage_block(const f32x16& acc, uint8_t* block, bool relu) {
  const int lane = threadIdx.x & 63;
  const uint32_t pick = (lane & 1) ? 0x03020706u : 0x05040100u;  // halves of (neighbour, own) that make this lane's word
  uint8_t* const dst = block + (4 * (lane >> 5) + (lane & 1)) * STRIDE + (lane & 30) * 2;
  auto put = [&](int e, float v0, float v1) {
    const uint32_t own = floats_to_bits<DT>(v0, v1);
    const uint32_t neighbour = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xf, 0xf, true);  // lane ^ 1
    *reinterpret_cast<uint32_t*>(dst + (8 * (e >> 2) + (e & 3)) * STRIDE) = __builtin_amdgcn_perm(neighbour, own, pick);
  };
  if (relu) {
#pragma unroll
    for (int e = 0; e < 16; e += 2) put(e, relu_f32(acc[e]), relu_f32(acc[e + 1]));
  } else {
#pragma unroll
    for (int e = 0; e < 16; e += 2) put(e, acc[e], acc[e + 1]);
  }
}

// The first `left` (1 .. 7) of a lane's eight values to the end of a row, as one store each of four, two and one of them:
// element by element, in a loop that picks halves of words, this took 8 us of a workgroup of 128 rows (512 x 1192, V = 128,
// Kv = 592, N = 311 21.5 -> 14.0 us with 512-column rings; panel kernel, 4416 x 536, V = 64, N = 4119 34.6 -> 30.4).
__device__ __forceinline__ void store_row_end(uint16_t* dst, u32x4 v, int left) {
  if (left & 4) *reinterpret_cast<u32x2*>(dst) = u32x2{v.x, v.y};
  const uint32_t pair = (left & 4) ? v.z : v.x;
  if (left & 2) *reinterpret_cast<uint32_t*>(dst + (left & 4)) = pair;
  const uint32_t last = (left & 2) ? ((left & 4) ? v.w : v.y) : pair;
  if (left & 1) dst[left & 6] = (uint16_t)last;
}

// Writes `rows` staged rows to Y, every row as one contiguous segment.  The rows' numbers are requested before the first
// one is used.  The caller has passed the barrier behind the staging.
template <int ROWS, int NB, int THREADS, class OutRow>
__device__ __forceinline__ void store_staged_rows(const uint8_t* lds, void* Y, int64_t ldy, int N, int n0, OutRow out_row_of) {
  constexpr int LANES_PER_ROW = NB / 8;
  constexpr int PASS = THREADS / LANES_PER_ROW;  // rows at a time
  constexpr int PASSES = (ROWS + PASS - 1) / PASS;
  constexpr int BATCH = PASSES < 8 ? PASSES : 8;
  const int tid = threadIdx.x;
  const int chunk = tid % LANES_PER_ROW;
  const int first = tid / LANES_PER_ROW;
  const int n = n0 + chunk * 8;
  if (n >= N) return;
  uint16_t* const Yh = static_cast<uint16_t*>(Y) + n;
  const bool whole = n + 8 <= N;
#pragma unroll
  for (int b = 0; b < PASSES; b += BATCH) {
    int64_t out[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int row = first + (b + i) * PASS;
      out[i] = row < ROWS ? out_row_of(row) : 0;
    }
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int row = first + (b + i) * PASS;
      if (row >= ROWS) break;
      const u32x4 v = *reinterpret_cast<const u32x4*>(lds + row * kStageStride<NB> + chunk * 16);
      uint16_t* dst = Yh + out[i] * ldy;
      if (whole) {
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
      } else {
        store_row_end(dst, v, N - n);
      }
    }
  }
}

// The caller guarantees nothing: the barrier that ends the k loop's use of LDS is taken here.
template <int DT, int RB, int CBS, int NB, int WC, int THREADS, class OutRow>
__device__ __forceinline__ void store_tile_rows(const f32x16 (&acc)[RB][CBS], uint8_t* lds, void* Y, int64_t ldy, int N,
                                                int n0, bool relu, bool out_f32, OutRow out_row_of) {
  constexpr int V = 32 * RB;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i32 = lane & 31;
  const int qh = lane >> 5;
  if (out_f32) {
    float* Yf = static_cast<float*>(Y);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int64_t out_row = out_row_of(32 * rb + 8 * (e >> 2) + 4 * qh + (e & 3));
#pragma unroll
        for (int cb = 0; cb < CBS; ++cb) {
          const int n = n0 + wave * WC + cb * 32 + i32;
          float v = acc[rb][cb][e];
          if (relu) v = v > 0.f ? v : 0.f;
          if (n < N) Yf[out_row * ldy + n] = v;
        }
      }
    return;
  }
  __builtin_amdgcn_s_barrier();  // every wave is done reading the stages
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < CBS; ++cb)
      stage_block<DT, kStageStride<NB>>(acc[rb][cb], lds + 32 * rb * kStageStride<NB> + (wave * WC + cb * 32) * 2, relu);
  __syncthreads();
  store_staged_rows<V, NB, THREADS>(lds, Y, ldy, N, n0, out_row_of);
}

}  // namespace hinm
