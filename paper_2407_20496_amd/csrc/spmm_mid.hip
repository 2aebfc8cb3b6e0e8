// HiNM product for a moderate number of columns: too many for the decoding kernels, too few workgroups for the tile
// kernels (arXiv 2407.20496, Section 3.2; layout of the device-tuned form in prepared_layout.h).
//
// One workgroup owns 32 RB rows of a tile and 32 CB columns; its waves split the tile's 64-column steps between them
// and never meet before the end: every wave keeps a private two-slot ring of gathered input rows in LDS, filled by
// direct-to-LDS copies, and takes the stored values straight into registers.  So no wave waits for another's data, every
// wave has one step's worth of requests in flight, and the row blocks of a tile share the gathered rows (which the 16-row
// kernel fetches again for every 64 rows).  The partial
// tiles of the waves are added through LDS in a fixed order, two row blocks at a time.
//
// Bound: the latency of a wave's step while there is one workgroup per compute unit (0.14 to 0.26 us per 64-column
// step by block size), the gathered rows on their way from L2 when there are several (up to 20 TB/s over the chip).
// Prepared form, 11008 x 4096 at 50 %: N = 64 15.3 -> 10.4 us, N = 100 28.0 -> 16.6, N = 256 35.4 -> 20.5;
// 4096 x 11008 at 50 %: N = 512 74 -> 37, N = 1024 86 -> 58.  Packed arrays, which had a 16-column and a 256-column
// kernel and nothing in between: 4096 x 4096 at 50 %, V = 64, N = 32 30.9 -> 8.4 us, N = 256 30.9 -> 13.1; kept columns
// that are no multiple of 64 on the way (5376 x 5584, Kv = 2792, N = 12: 79 -> 11; 4224 x 7120, Kv = 888, N = 3797:
// 820 -> 95).
#include "hinm_internal.h"
#include "mfma_types.h"
#include "prepared_layout.h"
#include "direct_lds.h"

#include <type_traits>

namespace hinm {
namespace {

enum { kFromPrepared = 0, kFromCanonical = 1, kFromVectors = 2 };  // vectors: a layer before its 2:4 step

struct MidSource {
  const uint8_t* blocks;     // prepared: the blocks of the layer; canonical: stored values [M][Kv/2];
                             // vectors: [M][Kv]
  const uint8_t* nm_idx;     // canonical only
  const int32_t* gather;     // prepared: gather table [T][Kp]; else vector index [T][Kv]
  const int32_t* pi_in;      // not prepared; may be NULL
  const int32_t* out_rows;   // not prepared: may be NULL
  const uint8_t* zeros;      // prepared only: where padded kept columns read (else kZeroRow)
};

// What the columns past Kv of a ragged last step read; never written.
__device__ __attribute__((aligned(256))) uint8_t kZeroRow[256];

struct MidShape {
  int V, Kv, steps, N, col_blocks, work, work_per_xcd;
  bool columns_last;  // a die's share walks the row groups of one column block before the next block
  bool relu, out_f32;
};

template <int RB, int CB, int NW>
struct MidCfg {
  static constexpr int ROW_BYTES = CB * 64;            // one gathered row: 32 CB columns
  static constexpr int SLOT_BYTES = 64 * ROW_BYTES;    // one step's rows
  static constexpr int LANES_PER_ROW = CB * 4;
  static constexpr int ROWS_PER_COPY = 64 / LANES_PER_ROW;
  static constexpr int COPIES = 64 / ROWS_PER_COPY;
  static constexpr int PR = RB < 2 ? RB : 2;           // row blocks reduced together
  static constexpr int ROUNDS = RB / PR;
  static constexpr int PARTIAL_BYTES = PR * 32 * CB * 32 * 4;
  static constexpr int WAVE_BYTES = 2 * SLOT_BYTES;
  static_assert(PARTIAL_BYTES <= WAVE_BYTES, "a wave's partial tiles take the place of its ring");
  static constexpr int LDS_BYTES = NW * WAVE_BYTES;
  static constexpr int ITEMS = PR * 32 * CB * 8;       // groups of four output columns of one round
  static constexpr int PER_THREAD = (ITEMS + NW * 64 - 1) / (NW * 64);
};

// The 32-byte units of row r sit at unit ^ mid_swizzle(r): the rows r .. r + 3 of a transposing read then cover
// all banks once (64-byte rows do so by themselves).
template <int CB>
__device__ __forceinline__ int mid_swizzle(int r) {
  return CB == 1 ? 0 : CB == 2 ? (r & 2) : ((r & 3) << 1);
}

__device__ __forceinline__ uint32_t load_u16(const uint8_t* p) {
  uint16_t v;
  __builtin_memcpy(&v, p, 2);
  return v;
}

// B operands of one 32-column substep: transposing reads of the rows at the given offsets, issued as raw instructions
// (the compiler would hold them until every copy in flight had landed) and waited for in the same block, so that no
// register is touched before its data is there.
template <int R0, int R1, int R2, int R3>
__device__ __forceinline__ void read_rows(uint32_t at, u32x8& b) {
  static_assert(R3 < 65536, "DS offset field is 16 bits");
  u32x2 v0, v1, v2, v3;
  asm volatile(
      "ds_read_b64_tr_b16 %0, %4 offset:%5\n\t"
      "ds_read_b64_tr_b16 %1, %4 offset:%6\n\t"
      "ds_read_b64_tr_b16 %2, %4 offset:%7\n\t"
      "ds_read_b64_tr_b16 %3, %4 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v0), "=&v"(v1), "=&v"(v2), "=&v"(v3)
      : "v"(at), "n"(R0), "n"(R1), "n"(R2), "n"(R3));
  b = u32x8{v0.x, v0.y, v1.x, v1.y, v2.x, v2.y, v3.x, v3.y};
}
template <int R0, int R1, int R2, int R3>
__device__ __forceinline__ void read_rows(uint32_t at0, uint32_t at1, u32x8& b0, u32x8& b1) {
  static_assert(R3 < 65536, "DS offset field is 16 bits");
  u32x2 v0, v1, v2, v3, w0, w1, w2, w3;
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8 offset:%10\n\t"
      "ds_read_b64_tr_b16 %1, %8 offset:%11\n\t"
      "ds_read_b64_tr_b16 %2, %8 offset:%12\n\t"
      "ds_read_b64_tr_b16 %3, %8 offset:%13\n\t"
      "ds_read_b64_tr_b16 %4, %9 offset:%10\n\t"
      "ds_read_b64_tr_b16 %5, %9 offset:%11\n\t"
      "ds_read_b64_tr_b16 %6, %9 offset:%12\n\t"
      "ds_read_b64_tr_b16 %7, %9 offset:%13\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v0), "=&v"(v1), "=&v"(v2), "=&v"(v3), "=&v"(w0), "=&v"(w1), "=&v"(w2), "=&v"(w3)
      : "v"(at0), "v"(at1), "n"(R0), "n"(R1), "n"(R2), "n"(R3));
  b0 = u32x8{v0.x, v0.y, v1.x, v1.y, v2.x, v2.y, v3.x, v3.y};
  b1 = u32x8{w0.x, w0.y, w1.x, w1.y, w2.x, w2.y, w3.x, w3.y};
}

template <int DT, int SRC, int RB, int CB, int NW>
__global__ __launch_bounds__(NW * 64) void spmm_mid_kernel(MidSource src, const uint16_t* __restrict__ X, int64_t ldx,
                                                           void* __restrict__ Y, int64_t ldy, MidShape p) {
  using C = MidCfg<RB, CB, NW>;
  extern __shared__ __attribute__((aligned(256))) uint8_t lds[];
  // workgroups are dealt to the eight dies in turn: every die takes a contiguous range of the work
  const int w = (int)(blockIdx.x & 7) * p.work_per_xcd + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= p.work_per_xcd || w >= p.work) return;
  const int row_groups = p.work / p.col_blocks;
  const int group = p.columns_last ? w % row_groups : w / p.col_blocks;
  const int n0 = (p.columns_last ? w / row_groups : w % p.col_blocks) * (32 * CB);
  const int row0 = group * (32 * RB);
  const int t = row0 / p.V;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i32 = lane & 31, qh = lane >> 5, i16 = lane & 15;
  const int steps = p.steps;
  const int mine = wave < steps ? (steps - wave + NW - 1) / NW : 0;  // steps wave, wave + NW, ...
  uint8_t* ring = lds + wave * C::WAVE_BYTES;
  const uint32_t ring_addr = (uint32_t)(uintptr_t)(lds_void_t*)ring;

  // rows of Y this thread will store, requested early
  int out_row[C::ROUNDS][C::PER_THREAD];
#pragma unroll
  for (int r = 0; r < C::ROUNDS; ++r)
#pragma unroll
    for (int k = 0; k < C::PER_THREAD; ++k) {
      const int item = min((int)threadIdx.x + k * NW * 64, C::ITEMS - 1);
      const int row = row0 + r * 32 * C::PR + item / (CB * 8);
      out_row[r][k] = src.out_rows ? src.out_rows[row] : row;
    }

  // ---- gathered rows ---------------------------------------------------------------------------------
  const int32_t* table = src.gather + (size_t)t * (SRC == kFromPrepared ? steps * 64 : p.Kv);
  auto load_entry = [&](int j) {
    const int at = (wave + min(j, mine - 1) * NW) * 64 + lane;
    if constexpr (SRC == kFromPrepared) return table[at];  // padded to whole steps with -1
    const int v = table[min(at, p.Kv - 1)];
    return at < p.Kv ? v : -1;
  };
  auto translate = [&](int v) {
    if (SRC == kFromPrepared || !src.pi_in) return v;
    const int c = src.pi_in[max(v, 0)];
    return v >= 0 ? c : -1;
  };
  const int piece = lane % C::LANES_PER_ROW;  // this lane's place in a row: 16 bytes
  const int granule = (((piece >> 1) ^ mid_swizzle<CB>(lane / C::LANES_PER_ROW)) << 1) | (piece & 1);
  // pieces at or beyond column N read the block's first columns instead: what they feed is never stored
  const uint32_t piece_off = (n0 + granule * 8 < p.N) ? granule * 16u : 0u;
  const uint8_t* x_lane = reinterpret_cast<const uint8_t*>(X + n0) + piece_off;
  const uint8_t* zero_lane = (SRC == kFromPrepared ? src.zeros : kZeroRow) + piece_off;
  const int64_t row_stride = ldx * 2;
  auto issue_rows = [&](int slot, int entry) {
#pragma unroll
    for (int k = 0; k < C::COPIES; ++k) {
      const int c = __builtin_amdgcn_ds_bpermute((C::ROWS_PER_COPY * k + lane / C::LANES_PER_ROW) * 4, entry);
      copy16_to_lds(c >= 0 ? x_lane + (int64_t)c * row_stride : zero_lane, ring + slot * C::SLOT_BYTES + k * 1024);
    }
  };

  // ---- stored values ---------------------------------------------------------------------------------
  struct Weights {
    u32x4 a[RB][SRC == kFromVectors ? 4 : 2];
    uint32_t idx[RB][SRC == kFromCanonical ? 2 : 1];
  };
  const int rb_total = p.V / 32;
  const uint8_t* a_lane;
  const uint8_t* nm_lane = nullptr;
  if constexpr (SRC == kFromPrepared) {
    a_lane = src.blocks + ((size_t)t * steps * rb_total + (row0 % p.V) / 32) * kPrepBlockBytes + lane * 16;
    nm_lane = src.blocks + ((size_t)t * steps * rb_total + (row0 % p.V) / 32) * kPrepBlockBytes + kPrepIdxOffset + lane * 4;
  } else if constexpr (SRC == kFromVectors) {
    a_lane = src.blocks + (size_t)(row0 + i32) * p.Kv * 2 + qh * 16;
  } else {
    a_lane = src.blocks + (size_t)(row0 + i32) * p.Kv + qh * 16;         // Kv / 2 values of two bytes per row
    nm_lane = src.nm_idx + (size_t)(row0 + i32) * (p.Kv / 8) + qh * 2;
  }
  auto load_weights = [&](int j, Weights& wt) {
    const int s = wave + j * NW;
    if constexpr (SRC == kFromPrepared) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const size_t off = ((size_t)s * rb_total + rb) * kPrepBlockBytes;
        wt.a[rb][0] = *reinterpret_cast<const u32x4*>(a_lane + off);
        wt.a[rb][1] = *reinterpret_cast<const u32x4*>(a_lane + off + 1024);
        wt.idx[rb][0] = *reinterpret_cast<const uint32_t*>(nm_lane + off);
      }
    } else if constexpr (SRC == kFromVectors) {  // 16-byte pieces, all of one or nothing there (Kv % 8 == 0)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint8_t* a = a_lane + (size_t)rb * 64 * p.Kv + (size_t)s * 128 + q * 32;
          const bool there = s * 64 + q * 16 + qh * 8 < p.Kv;
          wt.a[rb][q] = *reinterpret_cast<const u32x4*>(there ? a : a_lane - qh * 16);
          if (!there) wt.a[rb][q] = u32x4{0, 0, 0, 0};
        }
    } else if ((s + 1) * 64 <= p.Kv) {  // rows are only 8-byte aligned, their nibbles not at all
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          wt.a[rb][q] = *reinterpret_cast<const u32x4_a4*>(a_lane + (size_t)rb * 32 * p.Kv + (size_t)s * 64 + q * 32);
          wt.idx[rb][q] = load_u16(nm_lane + (size_t)rb * 32 * (p.Kv / 8) + (size_t)s * 8 + q * 4);
        }
    } else {  // the ragged last step: Kv % 8 == 0, so a lane has all, half or none of its four groups
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          wt.a[rb][q] = u32x4{0, 0, 0, 0};
          wt.idx[rb][q] = 0;
          const uint8_t* a = a_lane + (size_t)rb * 32 * p.Kv + (size_t)s * 64 + q * 32;
          const uint8_t* nm = nm_lane + (size_t)rb * 32 * (p.Kv / 8) + (size_t)s * 8 + q * 4;
          const int groups = p.Kv / 4 - (16 * s + 8 * q + 4 * qh);
          if (groups >= 4) {
            wt.a[rb][q] = *reinterpret_cast<const u32x4_a4*>(a);
            wt.idx[rb][q] = load_u16(nm);
          } else if (groups >= 2) {
            const u32x2 half = *reinterpret_cast<const u32x2_a4*>(a);
            wt.a[rb][q] = u32x4{half.x, half.y, 0, 0};
            wt.idx[rb][q] = *nm;
          }
        }
    }
  };

  // ---- one step --------------------------------------------------------------------------------------
  uint32_t b_off[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
    b_off[cb] = ring_addr + (8 * qh + (i16 >> 2)) * C::ROW_BYTES +
                (((cb * 2 + (i32 >> 4)) ^ mid_swizzle<CB>(i16 >> 2)) * 32) + (i16 & 3) * 8;
  f32x16 acc[RB][CB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[rb][cb][e] = 0.f;
  // B slots 8 h + 4 u .. + 3 of lane group qh <- rows 16 h + 8 qh + 4 u + (0..3) of the 32-column substep
  auto multiply_sub = [&](int slot, const Weights& wt, auto sub_tag) {
    constexpr int Q = decltype(sub_tag)::value;
    constexpr int R0 = (Q * 32 + 0) * C::ROW_BYTES, R1 = (Q * 32 + 4) * C::ROW_BYTES, R2 = (Q * 32 + 16) * C::ROW_BYTES,
                  R3 = (Q * 32 + 20) * C::ROW_BYTES;
    u32x8 b[CB];
    if constexpr (CB == 1) {
      read_rows<R0, R1, R2, R3>(b_off[0] + slot * C::SLOT_BYTES, b[0]);
    } else {
#pragma unroll
      for (int cb = 0; cb < CB; cb += 2)
        read_rows<R0, R1, R2, R3>(b_off[cb] + slot * C::SLOT_BYTES, b_off[cb + 1] + slot * C::SLOT_BYTES, b[cb], b[cb + 1]);
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        if constexpr (SRC == kFromVectors) {
          acc[rb][cb] = mfma_32x32x16<DT>(wt.a[rb][2 * Q], u32x4{b[cb][0], b[cb][1], b[cb][2], b[cb][3]}, acc[rb][cb]);
          acc[rb][cb] = mfma_32x32x16<DT>(wt.a[rb][2 * Q + 1], u32x4{b[cb][4], b[cb][5], b[cb][6], b[cb][7]}, acc[rb][cb]);
        } else if constexpr (SRC == kFromPrepared)
          acc[rb][cb] = smfmac_32x32x32<DT, Q>(wt.a[rb][Q], b[cb], acc[rb][cb], (int)wt.idx[rb][0]);
        else
          acc[rb][cb] = smfmac_32x32x32<DT, 0>(wt.a[rb][Q], b[cb], acc[rb][cb], (int)wt.idx[rb][Q]);
      }
  };
  auto multiply = [&](int slot, const Weights& wt) {
    multiply_sub(slot, wt, std::integral_constant<int, 0>{});
    multiply_sub(slot, wt, std::integral_constant<int, 1>{});
    asm volatile("" ::: "memory");  // the slot is free: its reads have returned
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- the wave's steps --------------------------------------------------------------------------------
  if (mine > 0) {
    Weights w0, w1;
    int vec1 = load_entry(1);  // rows of step j + 1; with a table to translate through, its entries of j + 2
    int row_now = translate(load_entry(0));
    int row_next = translate(vec1);
    int vec_next = SRC != kFromPrepared ? load_entry(2) : 0;
    load_weights(0, w0);
    issue_rows(0, row_now);
    // Step j: request the rows of j + 1, request its weights, multiply.  The row numbers of j + 1 were loaded behind the rows
    // and weights of j, and a register whose value is needed while direct copies are in flight makes the compiler wait for
    // everything requested: that wait, at the head of the step, is where the rows and weights of j land, and the one
    // below is there for their order only.  Row numbers through LDS, with no such wait, were 1 to 6 % faster on the
    // prepared form and up to 8 % slower on the packed arrays.
    auto step = [&](int j, int slot, const Weights& cur, Weights& next) {
      issue_rows(slot ^ 1, row_next);
      __builtin_amdgcn_sched_barrier(0);
      wait_copies_outstanding<C::COPIES>();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (SRC != kFromPrepared) {
        row_next = translate(vec_next);
        vec_next = load_entry(j + 3);
      } else {
        row_next = load_entry(j + 2);
      }
      load_weights(j + 1, next);
      __builtin_amdgcn_sched_barrier(0);
      multiply(slot, cur);
    };
    int j = 0;
    for (; j + 2 < mine; j += 2) {
      step(j, 0, w0, w1);
      step(j + 1, 1, w1, w0);
    }
    if (j + 1 < mine) {
      step(j, 0, w0, w1);
      wait_copies_outstanding<0>();
      __builtin_amdgcn_sched_barrier(0);
      multiply(1, w1);
    } else {
      wait_copies_outstanding<0>();
      __builtin_amdgcn_sched_barrier(0);
      multiply(0, w0);
    }
  }

  // ---- sum over the waves, epilogue --------------------------------------------------------------------
  // a lane holds column l % 32, rows 8 (reg / 4) + 4 (l / 32) + reg % 4 of a 32 x 32 block
  constexpr int kCols = 32 * CB;
#pragma unroll
  for (int r = 0; r < C::ROUNDS; ++r) {
    if (r > 0) __syncthreads();
    float* partial = reinterpret_cast<float*>(ring);
#pragma unroll
    for (int pb = 0; pb < C::PR; ++pb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          partial[(32 * pb + 8 * (e >> 2) + 4 * qh + (e & 3)) * kCols + 32 * cb + i32] = acc[r * C::PR + pb][cb][e];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < C::PER_THREAD; ++k) {
      const int item = threadIdx.x + k * NW * 64;
      if (item >= C::ITEMS) break;
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < NW; ++v) sum += *reinterpret_cast<const f32x4*>(lds + v * C::WAVE_BYTES + item * 16);
      if (p.relu) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] = sum[e] > 0.f ? sum[e] : 0.f;
      }
      const int n = n0 + (item % (CB * 8)) * 4;
      const int64_t at = (int64_t)out_row[r][k] * ldy + n;
      if (p.out_f32) {
        float* y = static_cast<float*>(Y) + at;
        if (n + 4 <= p.N) {
          __builtin_nontemporal_store(sum, reinterpret_cast<f32x4*>(y));
        } else {
          for (int e = 0; e < 4; ++e)
            if (n + e < p.N) y[e] = sum[e];
        }
      } else {
        uint16_t* y = static_cast<uint16_t*>(Y) + at;
        if (n + 4 <= p.N) {
          const u32x2 bits = {(uint32_t)float_to_bits<DT>(sum[0]) | (uint32_t)float_to_bits<DT>(sum[1]) << 16,
                              (uint32_t)float_to_bits<DT>(sum[2]) | (uint32_t)float_to_bits<DT>(sum[3]) << 16};
          __builtin_nontemporal_store(bits, reinterpret_cast<u32x2*>(y));
        } else {
          for (int e = 0; e < 4; ++e)
            if (n + e < p.N) y[e] = float_to_bits<DT>(sum[e]);
        }
      }
    }
  }
}

struct MidCall {
  MidSource src;
  int M, K, V, Kv, N;
  const uint16_t* X;
  int64_t ldx;
  void* Y;
  int64_t ldy;
  bool relu, out_f32;
  LaunchPlan* plan;
};

// An input that a die's L2 (4 MB) holds is shared by all column blocks there; a larger one is taken block by block.
bool columns_last(int K, int N) { return (double)K * N * 2 > 3.0e6; }

template <int DT, int SRC, int RB, int CB, int NW>
hipError_t launch_cfg(const MidCall& c, hipStream_t stream) {
  using C = MidCfg<RB, CB, NW>;
  MidShape p;
  p.V = c.V;
  p.Kv = c.Kv;
  p.steps = (c.Kv + 63) / 64;
  p.N = c.N;
  p.col_blocks = (c.N + 32 * CB - 1) / (32 * CB);
  p.work = c.M / (32 * RB) * p.col_blocks;
  p.work_per_xcd = (p.work + 7) / 8;
  p.columns_last = columns_last(c.K, c.N);
  p.relu = c.relu;
  p.out_f32 = c.out_f32;
  constexpr auto kernel = spmm_mid_kernel<DT, SRC, RB, CB, NW>;
  if (c.plan) {
    plan_record(c.plan, "spmm_mid_kernel<DT=%d,SRC=%d,RB=%d,CB=%d,NW=%d> grid=%d block=%d lds=%d", DT, SRC, RB, CB, NW,
                p.work_per_xcd * 8, NW * 64, C::LDS_BYTES);
    return hipSuccess;
  }
  if (hipError_t e = raise_lds_limit<kernel>(C::LDS_BYTES); e != hipSuccess) return e;
  kernel<<<dim3((unsigned)p.work_per_xcd * 8), NW * 64, C::LDS_BYTES, stream>>>(c.src, c.X, c.ldx, c.Y, c.ldy, p);
  return hipGetLastError();
}

// ---- which block per workgroup, how many waves ------------------------------------------------------------
struct MidPlan {
  int rb, cb, nw;
};

// The largest block of which about 150 exist (a block that is alone on its compute unit runs 2 + 0.14 S us with 32
// x 32 outputs and eight waves, 2.6 + 0.19 S with 64 x 64, S = 64-column steps; 64 x 64 blocks read 3/8 fewer bytes
// per output than 64 x 32 ones).  64 x 64 blocks from 129 on: split in two they would be more than 256 of 128 KB of
// LDS each, a second round (3072 x 8192 at 50 %, N = 160, 144 blocks: 14.2 against 20.9 us; 2304 x 4096, N = 256
// 8.2 and 11.5).  Beyond 256 blocks of 64 x 64 several share a unit: four waves each leave room for two, two waves
// for four (11008 x 4096 at 50 %, N = 256, 688 blocks: 20.5 us with two waves, 22.3 with four, 23.3 with eight;
// 16384 x 4096, N = 128, 512 blocks: 21.3, 15.5, 17.7).  Twice the block instead is worth it on long passes where
// 150 to 256 of them exist: 128 rows in the prepared form (4096 x 11008 at 50 %, N = 512: 37.3 against 41.3 us;
// with 16 steps 11.2 against 10.0), 128 columns on the packed arrays, whose rows of values cost a cache line each
// and step (4096 x 4096, N = 512: 19.1 against 24.3; with 8 steps 10.1 against 9.2).  For the same reason the
// packed arrays take 32-row blocks with 64 columns before 64-row blocks with 32 (8192 x 4096, N = 24: 11.0 and
// 14.6).
MidPlan plan_mid(int M, int V, int Kv, int N, bool canonical) {
  const int S = (Kv + 63) / 64;
  const int64_t rows = M / 32;
  const int64_t b2 = (N + 63) / 64, b4 = (N + 127) / 128;
  const bool two = (V / 32) % 2 == 0, four = (V / 32) % 4 == 0;
  auto fills = [](int64_t blocks) { return blocks >= 150 && blocks <= 256; };
  if (N <= 32) {
    if (two && !canonical && rows / 2 >= 150) return {2, 1, 8};
    return {1, 1, S <= 4 ? 4 : 8};
  }
  if (two) {
    const int64_t blocks = rows / 2 * b2;
    if (blocks > 512) return {2, 2, 2};
    if (blocks > 256) {
      if (canonical && S >= 16 && fills(rows / 2 * b4)) return {2, 4, 4};
      if (!canonical && four && S >= 32 && fills(rows / 4 * b2)) return {4, 2, 4};
      return {2, 2, 4};
    }
    if (blocks > 128) return {2, 2, 8};
  }
  const int64_t blocks = rows * b2;  // 32 x 64; V % 64 != 0 has nothing larger
  if (blocks > 512) return {1, 2, 2};
  if (blocks > 256) return {1, 2, S >= 16 ? 8 : 4};
  if (blocks >= 150) return {1, 2, 8};
  return {1, 1, S <= 4 ? 4 : 8};
}

// 64 x 64 blocks (32 x 64 where V % 64 != 0): what the choice against the tile kernels goes by.
int64_t plain_blocks(int M, int V, int N) {
  return (int64_t)(M / ((V / 32) % 2 == 0 ? 64 : 32)) * ((N + 63) / 64);
}

template <int DT, int SRC>
hipError_t launch_planned(const MidCall& c, hipStream_t stream) {
  const MidPlan m = plan_mid(c.M, c.V, c.Kv, c.N, SRC != kFromPrepared);
  if constexpr (SRC == kFromPrepared) {
    if (m.rb == 4) return launch_cfg<DT, SRC, 4, 2, 4>(c, stream);
    if (m.rb == 2 && m.cb == 1) return launch_cfg<DT, SRC, 2, 1, 8>(c, stream);
  } else {
    if (m.cb == 4) return launch_cfg<DT, SRC, 2, 4, 4>(c, stream);
  }
  if (m.rb == 2) {
    if (m.nw == 2) return launch_cfg<DT, SRC, 2, 2, 2>(c, stream);
    if (m.nw == 4) return launch_cfg<DT, SRC, 2, 2, 4>(c, stream);
    return launch_cfg<DT, SRC, 2, 2, 8>(c, stream);
  }
  if (m.cb == 2) {
    if (m.nw == 2) return launch_cfg<DT, SRC, 1, 2, 2>(c, stream);
    if (m.nw == 4) return launch_cfg<DT, SRC, 1, 2, 4>(c, stream);
    return launch_cfg<DT, SRC, 1, 2, 8>(c, stream);
  }
  if (m.nw == 4) return launch_cfg<DT, SRC, 1, 1, 4>(c, stream);
  return launch_cfg<DT, SRC, 1, 1, 8>(c, stream);
}

}  // namespace

// Against the 16-row kernels, up to 128 columns.  A layer is one of many in a model, so its values come from memory, not
// from the 256 MB cache that a layer called over and over stays in: both were timed, over some 500 (layer, N) pairs.  Below,
// "a / b -> c / d us" is the 16-row kernel and then this one, with buffers rotated past that cache / from it.  A compute
// unit fetches from memory at a bounded rate (neither more waves per workgroup nor requests further ahead change it), so
// what counts there is how many units take part and for how many rounds.
//   2 .. 4 columns: this one on tall layers (9600 rows and more).  Against the 16-row kernel's form with both halves of a 32-row
//     block it is ahead from 49 steps on (7 layers 0.84 to 0.95 of the time from memory, 0.57 to 0.62 from the cache), level from
//     memory between 14 and 48 steps (0.91 to 1.12) and ahead from the cache (0.67 to 1.01: 14208 x 12032, 47 steps, N = 4 17.1 / 16.4 ->
//     17.6 / 11.8); up to twelve steps it is behind (26 layers 1.05 to 1.38 of the time from memory, 0.92 to 1.23 from the cache:
//     11008 x 1280, 10 steps, N = 4 4.9 -> 6.7 from memory), which the line does not go by.
//   5 .. 16: that kernel is ahead where its workgroups fit the chip in one round (4096 x 11008 at 50 %, N = 16: 13.7 / 12.1 ->
//     17.5 / 8.8; 4096 x 4096: 6.3 / 4.9 -> 8.5 / 5.1; 8192 x 8192, Kv = 2048: 8.2 / 6.5 -> 9.6 / 6.2), this one with a second
//     round (5120 x 5120: 13.4 / 11.7 -> 10.1 / 5.9; 7296 x 13240, N = 15: 37.9 / 34.7 -> 22.8 / 14.9) unless its workgroups have
//     four waves and share units (up to 16 steps), and not against its form with the input in LDS (11008 x 4096, N = 16:
//     9.7 / 8.4 -> 11.1 / 6.4).
//   17 .. 64: this one from 150 blocks of 32 x 32 on (11008 x 4096, N = 32: 11.4 / 9.9 -> 11.0 / 6.2); below it where both are
//     short, where the other's last round is no more than 3/4 full (2176 x 10488, Kv = 2624, N = 32 1.06 / 1.7 times), where
//     it needs sixteen waves (4096 x 11008, Kv = 2752, N = 32: 10.3 / 9.0 -> 10.3 / 5.5) or two batches per wave; else the
//     16-row kernel (2048 x 8192, V = 32, Kv = 2048, N = 32: 5.9 / 4.9 -> 8.3 / 4.5; 768 x 3072 at 50 %: 4.9 / 3.6 -> 6.4 / 4.0).
//     These examples are of the 16-row kernel before its layers of up to sixteen steps took a wave a step.  With those, 22 drawn
//     layers of up to 16 steps that come here: up to seven steps 0.70 to 1.29 of its time, eight to 16 steps 0.72 to 1.11 (from
//     memory: 1280 rows, 4 steps, N = 40 3.0 there, 3.9 here; 10560 rows, 1 step, N = 64 6.2 and 4.4).
//   65 .. 128: that kernel on the smallest layers (512 x 7048, Kv = 1760, N = 100: 5.7 / 4.6 -> 7.2 / 4.8).
static bool beats_rows16(const PreparedArgs& a) {
  const int S = (a.s.Kv + 63) / 64;
  const int64_t blocks = (int64_t)(a.s.M / 32) * ((a.N + 31) / 32);
  const int64_t others = spmm_rows16_prepared_workgroups(a);
  const bool tall = a.s.V % 64 == 0 && a.s.M / 64 >= 150;
  if (a.N <= 4) return tall;
  if (a.N <= 16)
    return !spmm_rows16_resident_preferred(a) && others > 256 && (tall ? S >= 16 : a.N > 8 && S > 16);
  if (a.N <= 64)
    return blocks >= 150 || (S <= 8 && a.N > 24) || S > 96 || (S > 32 && blocks >= 96) ||
           (blocks >= 64 && others * 4 <= 3 * 256 * ((others + 255) / 256));
  return a.N > 128 || S <= 8 || S > 32 || blocks > 64;
}

// Many columns belong to the kernels with larger blocks, which gather less.  Beyond this line the private rings of
// spmm_rings.hip serve them all, and within it where they are estimated ahead by a margin (of the examples the rings
// have taken 8192 x 4096, N = 512 18.0 us; 1728 x 6480 19.3; 4096 x 4096, N = 1024 18.2; 7872 x 1248 9.2; 14400 x 824
// 6.2; 16384 x 4096 18.3; 9088 x 1928 stays here).  It was drawn against the staged tile kernel, whose times the
// examples give: at four workgroups per unit (4096 x 11008 at 50 %, N = 1024, 1024 blocks: 58 against 86 us there;
// 11008 x 4096, N = 300, 860 blocks: 25 and 38; N = 400, 1204 blocks: 44 and 36; 1024 x 1024, N = 1666, 432 blocks:
// 7.7 and 13.0; 512 x 5904, N = 3488, 440 blocks: 24 and 42), at three with V % 64 != 0.  Where the tile kernel has
// one round of 64-row tiles, which is a short one, it is at three for inputs that are taken one column block at a
// time (8192 x 8192, Kv = 2048, N = 384, 768 blocks: 24.4 and 26.2; N = 448 28.4 and 26.4; 8192 x 4096, N = 512 32.6
// and 25.7; 1728 x 6480, N = 2168, 918 blocks: 25.1 and 22.5) unless two of them at a time leave no slot of a unit
// empty (4096 x 4096, N = 1024, 1024 blocks: 24.5 and 25.8) and for passes of up to 16 steps (7872 x 1248, Kv = 624,
// N = 417, 861 blocks: 12.2 and 10.7), at two for up to four steps (14400 x 824, Kv = 208, N = 224, 900 blocks: 7.8
// and 6.2); else at four (16384 x 4096, N = 256, 1024 blocks: 24.2 and 26.6; 9088 x 1928, Kv = 960, N = 394, 994
// blocks and a second round of tiles: 15.4 and 21.3).
bool spmm_mid_prepared_preferred(const PreparedArgs& a) {
  if (a.N == 1 || a.ldx % 8 != 0 || a.ldy % 8 != 0) return false;
  if (a.N <= 128 && !beats_rows16(a)) return false;
  if (a.N <= 64) return true;
  const int64_t blocks = plain_blocks(a.s.M, a.s.V, a.N);
  int64_t line = a.s.V % 64 == 0 ? 1024 : 768;
  if (a.s.V == 64 && (int64_t)(a.s.M / 64) * ((a.N + 255) / 256) <= 256) {
    const bool shared = a.s.M <= 4096 && blocks > 960;  // two column blocks of a die share its reads of the weights
    line = a.s.Kv <= 256 ? 512 : a.s.Kv <= 1024 || (columns_last(a.s.K, a.N) && !shared) ? 768 : 1024;
  }
  return blocks <= line;
}

// Fitted to 300 random layers with 65 to 4000 columns (error 10 %).
double spmm_mid_prepared_us(const PreparedArgs& a) {
  const double steps = (a.s.Kv + 63) / 64;
  const double units = (double)plain_blocks(a.s.M, a.s.V, a.N) / 256;  // rounds of blocks
  return a.s.V % 64 == 0 ? 3.5 + 0.046 * steps + units * (0.175 * steps + 0.72) : 3.25 + 0.050 * steps + units * (0.162 * steps + 0.06);
}

hipError_t launch_spmm_mid_prepared(const PreparedArgs& a, hipStream_t stream) {
  const PreparedLayout L = prepared_layout(a.s);
  const uint8_t* base = static_cast<const uint8_t*>(a.prepared);
  const MidCall c{{base + L.a_offset, nullptr, reinterpret_cast<const int32_t*>(base + L.gather_offset), nullptr,
                   reinterpret_cast<const int32_t*>(base + L.pi_out_offset), base + L.zero_offset},
                  a.s.M, a.s.K, a.s.V, a.s.Kv, a.N, static_cast<const uint16_t*>(a.X), a.ldx, a.Y, a.ldy, a.relu,
                  a.out_f32, a.plan};
  return a.s.dtype == HINM_F16 ? launch_planned<HINM_F16, kFromPrepared>(c, stream)
                               : launch_planned<HINM_BF16, kFromPrepared>(c, stream);
}

// Up to 16 columns the 16-row kernel is ahead where its workgroups fit the chip in one round and its waves have no more
// than one batch of steps or so (as above, "from memory / from the cache", that kernel -> this one: 4096 x 4096 at 50 %, N = 16
// 7.9 / 6.0 -> 11.9 / 8.1 us; 2048 x 8192, V = 32, Kv = 2048, N = 2 7.4 / 5.4 -> 11.6 / 7.6; with 320 workgroups, 5120 x 5120,
// Kv = 1280, N = 9 11.0 / 9.5 -> 9.7 / 6.4; with 109 steps, 832 x 13960, Kv = 6976, N = 9 25.4 / 21.4 -> 28.5 / 15.5).
// Against the tile kernel the line lies at 640 blocks (8192 x 4096 at 50 %, N = 300, 640 blocks: 31 against 39 us;
// 4096 x 4096, N = 1024, 1024 blocks: 41 against 33); that kernel's fast form needs whole 64-column steps, without them this one
// is the better at any size.
bool spmm_mid_canonical_preferred(const SpmmArgs& a) {
  if (a.s.V % 32 != 0 || a.N == 1 || a.ldx % 8 != 0 || a.ldy % 8 != 0) return false;
  const int64_t blocks = plain_blocks(a.s.M, a.s.V, a.N);
  if (blocks >= (1 << 28)) return false;
  if (a.N <= 16 && a.s.M / 16 <= 256 && a.s.Kv <= 4096) return false;
  return a.N <= 64 || a.s.Kv % 64 != 0 || blocks <= 640;
}

hipError_t launch_spmm_mid_canonical(const SpmmArgs& a, hipStream_t stream) {
  const MidCall c{{static_cast<const uint8_t*>(a.vals), a.nm_idx, a.vec_idx, a.pi_in, a.pi_out, nullptr},
                  a.s.M, a.s.K, a.s.V, a.s.Kv, a.N, static_cast<const uint16_t*>(a.X), a.ldx, a.Y, a.ldy, a.relu,
                  a.out_f32, a.plan};
  return a.s.dtype == HINM_F16 ? launch_planned<HINM_F16, kFromCanonical>(c, stream)
                               : launch_planned<HINM_BF16, kFromCanonical>(c, stream);
}

// The layer before its 2:4 step has twice the values per kept column.  Whole 64-column steps: as on the packed arrays.
// Otherwise the tile kernel is the register-staged one, which is ahead from about 1024 blocks on (2688 x 680, V = 64,
// Kv = 168, N = 1764, 1176 blocks: 15.8 against 16.6 us; 2752 x 1608, N = 3675, 2494 blocks: 43 and 58; 640 x 3872,
// V = 128, N = 1726, 270 blocks: 74 and 24) and ends at tiles of 128 rows.
bool spmm_mid_vectors_preferred(const VectorsArgs& a) {
  if (a.s.V % 32 != 0 || a.N == 1 || a.ldx % 8 != 0 || a.ldy % 8 != 0) return false;
  const int64_t blocks = plain_blocks(a.s.M, a.s.V, a.N);
  if (blocks >= (1 << 28)) return false;
  return a.N <= 64 || a.s.V > 128 || blocks <= (a.s.Kv % 64 != 0 ? 1024 : 640);
}

// Fitted to 210 random layers with 65 to 4000 columns (error 10 %).
double spmm_mid_vectors_us(const VectorsArgs& a) {
  const double steps = (a.s.Kv + 63) / 64;
  const double units = (double)plain_blocks(a.s.M, a.s.V, a.N) / 256;
  return a.s.V % 64 == 0 ? 3.9 + 0.068 * steps + units * (0.371 * steps + 0.73) : 4.0 + 0.045 * steps + units * 0.278 * steps;
}

hipError_t launch_spmm_mid_vectors(const VectorsArgs& a, hipStream_t stream) {
  const MidCall c{{static_cast<const uint8_t*>(a.vals_v), nullptr, a.vec_idx, a.pi_in, a.pi_out, nullptr},
                  a.s.M, a.s.K, a.s.V, a.s.Kv, a.N, static_cast<const uint16_t*>(a.X), a.ldx, a.Y, a.ldy, a.relu,
                  a.out_f32, a.plan};
  return a.s.dtype == HINM_F16 ? launch_planned<HINM_F16, kFromVectors>(c, stream)
                               : launch_planned<HINM_BF16, kFromVectors>(c, stream);
}

}  // namespace hinm
