// hinm_prepare: canonical packed arrays + channel orders -> device-tuned form (see prepared_layout.h).
// A pure re-ordering: arXiv 2407.20496, Section 3.2 has the channel orders settled offline and the
// vector indices rewritten to match; this is that offline step, done on the GPU.
#include "hinm_internal.h"
#include "prepared_layout.h"

namespace hinm {
namespace {

constexpr int kThreads = 256;
constexpr int kStepsPerWave = 2;                                  // 128 bytes of every row: whole cache lines
constexpr int kStepsPerBlock = kStepsPerWave * (kThreads / 64);

typedef uint32_t quad_a8 __attribute__((ext_vector_type(4), aligned(8)));  // rows of stored values start on 8 bytes
typedef uint32_t quad __attribute__((ext_vector_type(4)));

// One launch: workgroups below n_block_wgs re-order stored values and NM nibbles, the others write the tables.
//
// A wave owns one 32-row block of a tile for two neighbouring steps: lane (row i, lane group qa) loads the 16 bytes of
// its four groups per substep as they stand in the canonical array and stores them in lane order, a kilobyte per
// instruction.  Bound by memory and by cache lines per load (a load touches 32 rows): 11008 x 4096 with 2048 kept columns (25 MB in, 25 MB out) took 35 us with 2-byte loads and
// steps in different workgroups and another 5 us for the tables, 13.6 us in one launch here.
// WIDE: vals is 8-byte aligned.  WHOLE: no padded groups, and a step's eight nibble bytes of a row are aligned.
template <bool WIDE, bool WHOLE>
__global__ __launch_bounds__(kThreads) void prepare_kernel(
    const uint16_t* __restrict__ vals, const uint8_t* __restrict__ nm_idx, const int32_t* __restrict__ vec_idx,
    const int32_t* __restrict__ pi_in, const int32_t* __restrict__ pi_out, uint8_t* __restrict__ out,
    int32_t* __restrict__ gather, int32_t* __restrict__ out_rows, uint32_t* __restrict__ zeros,
    uint32_t* __restrict__ panel, int V, int Kv, int RB, int S, int T, int Kp, int M, int K, int64_t n_block_wgs) {
  if ((int64_t)blockIdx.x < n_block_wgs) {
    const int step_blocks = (S + kStepsPerBlock - 1) / kStepsPerBlock;
    const int sb = (int)(blockIdx.x % step_blocks);
    const int64_t tr = blockIdx.x / step_blocks;
    const int rb = (int)(tr % RB), t = (int)(tr / RB);
    const int lane = threadIdx.x & 63;
    const int qa = lane >> 5;
    const int row = t * V + 32 * rb + (lane & 31);
    const int groups = Kv / 4;
    const uint16_t* vr = vals + (size_t)row * (Kv / 2);
    const uint8_t* nr = nm_idx + (size_t)row * (Kv / 8);
#pragma unroll
    for (int u = 0; u < kStepsPerWave; ++u) {
      const int s = sb * kStepsPerBlock + (int)(threadIdx.x >> 6) * kStepsPerWave + u;
      if (s >= S) return;
      uint8_t* blk = out + (((size_t)t * S + s) * RB + rb) * kPrepBlockBytes;
      uint32_t idx_word = 0;
      uint2 step_nibbles;  // WHOLE: of all sixteen groups of the row
      if constexpr (WHOLE) step_nibbles = *reinterpret_cast<const uint2*>(nr + 8 * s);
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        const int g0 = 16 * s + 8 * sub + 4 * qa;
        quad v = {0u, 0u, 0u, 0u};
        uint32_t nibbles = 0x4444u;  // padded groups: value 0, positions 0 and 1
        if (WHOLE || g0 + 4 <= groups) {
          if constexpr (WIDE) {
            v = *reinterpret_cast<const quad_a8*>(vr + 2 * g0);
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = (uint32_t)vr[2 * (g0 + k)] | ((uint32_t)vr[2 * (g0 + k) + 1] << 16);
          }
          if constexpr (WHOLE) nibbles = ((sub ? step_nibbles.y : step_nibbles.x) >> (16 * qa)) & 0xFFFFu;
          else nibbles = (uint32_t)nr[g0 / 2] | ((uint32_t)nr[g0 / 2 + 1] << 8);
        } else {
          // the last kept columns: groups come in pairs (Kv is a multiple of 8), so 0 or 2 of these 4 exist
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int g = g0 + k;
            if (g < groups) {
              v[k] = (uint32_t)vr[2 * g] | ((uint32_t)vr[2 * g + 1] << 16);
              nibbles = (nibbles & ~(0xFu << (4 * k))) | (((uint32_t)(nr[g >> 1] >> (4 * (g & 1))) & 0xFu) << (4 * k));
            }
          }
        }
        *reinterpret_cast<quad*>(blk + sub * 1024 + lane * 16) = v;
        idx_word |= nibbles << (16 * sub);
      }
      *reinterpret_cast<uint32_t*>(blk + kPrepIdxOffset + lane * 4) = idx_word;
    }
    return;
  }
  const int64_t id = ((int64_t)blockIdx.x - n_block_wgs) * kThreads + threadIdx.x;
  if (id < (int64_t)T * Kp) {
    const int t = (int)(id / Kp), j = (int)(id % Kp);
    int g = -1;
    if (j < Kv) {
      g = vec_idx[(size_t)t * Kv + j];
      if (pi_in) g = pi_in[g];
    }
    gather[id] = g;
    panel[id] = panel_entry_of_row(g, K);
  }
  if (id < M) out_rows[id] = pi_out ? pi_out[id] : (int32_t)id;
  if (id < kPrepZeroBytes / 4) zeros[id] = 0;
}

}  // namespace

hipError_t launch_prepare(const hinm_shape& s, const void* vals, const uint8_t* nm_idx, const int32_t* vec_idx,
                          const int32_t* pi_in, const int32_t* pi_out, void* prepared, hipStream_t stream) {
  const PreparedLayout L = prepared_layout(s);
  uint8_t* base = static_cast<uint8_t*>(prepared);
  const int64_t block_wgs = (int64_t)L.T * L.RB * ((L.S + kStepsPerBlock - 1) / kStepsPerBlock);
  int64_t n = (int64_t)L.T * L.Kp;
  if (n < s.M) n = s.M;
  if (n < kPrepZeroBytes / 4) n = kPrepZeroBytes / 4;
  const int64_t table_wgs = (n + kThreads - 1) / kThreads;
  auto launch = [&](auto kernel) {
    kernel<<<(unsigned)(block_wgs + table_wgs), kThreads, 0, stream>>>(
        static_cast<const uint16_t*>(vals), nm_idx, vec_idx, pi_in, pi_out, base + L.a_offset,
        reinterpret_cast<int32_t*>(base + L.gather_offset), reinterpret_cast<int32_t*>(base + L.pi_out_offset),
        reinterpret_cast<uint32_t*>(base + L.zero_offset), reinterpret_cast<uint32_t*>(base + L.panel_offset), s.V, s.Kv,
        L.RB, L.S, L.T, L.Kp, s.M, s.K, block_wgs);
  };
  const bool wide = (reinterpret_cast<uintptr_t>(vals) & 7u) == 0;
  const bool whole = s.Kv % 64 == 0 && (reinterpret_cast<uintptr_t>(nm_idx) & 7u) == 0;
  if (wide && whole) launch(prepare_kernel<true, true>);
  else if (wide) launch(prepare_kernel<true, false>);
  else launch(prepare_kernel<false, false>);
  return hipGetLastError();
}

}  // namespace hinm
