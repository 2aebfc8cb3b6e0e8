// HiNM sparse GEMM with fused channel permutation, many columns, from the device-tuned layer form, waves with private rings
// of gathered input rows (arXiv 2407.20496, Section 3.2 and Section 5.3; layout in prepared_layout.h).
//
// One workgroup computes one tile of V = 32 * RB output channels for NB = 64 * NWC columns.  Its waves are NWC groups of
// 64 columns by NWK groups of steps (64 kept columns each, taken in turn).  A wave copies its own 64 columns of the rows its
// steps name, eight 128-byte row segments to a direct-to-LDS copy, into a ring of R slots of 32 rows that no other wave
// touches: what it multiplies needs no barrier and the copies behind it are never drained, one slot is refilled the moment
// its fragments are in registers.  Only the stored values and the row numbers are shared: 9 KB a step (128-row tiles), three
// slots, copied two stages ahead by all waves, one barrier a stage.
//
// Against whole stages behind a barrier (spmm_tile_prepared.hip: all copies of a 64-row stage requested at once, waited for
// in full): 16384 x 16384 at 50 %, N = 8192 1366 -> 1180 us, 4096 x 11008 at 50 %, N = 2048 83.3 -> 54.3, 11008 x 4096,
// N = 2048 81 -> 66, 4096 x 4096, V = 64, N = 1024 23.8 -> 18.5.  What bounds it: on large products the power limit.  With
// all units busy the clock falls from 2.4 GHz to 1.5 .. 1.9 GHz; a 64-row step of 512 columns then takes 1850 clocks, 1024 of
// them MFMA issue, 1170 the address unit (73 KB at 64 bytes a clock) and about 1000 LDS.  Rows that come from L1 instead
// of L2 and memory shorten the step by a fifth and the product by a tenth; four waves of 128 columns, which read half as
// many stored values from LDS, run at a 10 % higher clock and take as long.
#include "hinm_internal.h"
#include "mfma_types.h"
#include "prepared_layout.h"
#include "direct_lds.h"
#include "tile_epilogue.h"

#include <type_traits>

namespace hinm {
namespace {

// Where the stored values and row numbers come from: the device-tuned form, or the arrays of a layer before its 2:4 step.
enum RingSource { kRingPrepared = 0, kRingVectors = 1 };

constexpr int kUnitLds = 160 * 1024;

template <int SRC, int RB, int NWC, int NWK, int R>
struct RingCfg {
  static constexpr bool SPARSE = SRC == kRingPrepared;
  static constexpr int ROWS = RB, COLUMN_GROUPS = NWC, STEP_GROUPS = NWK, DEPTH = R;
  static constexpr int CBS = 2;                      // 32-column blocks of a wave
  static constexpr int WC = 32 * CBS;                // columns of a wave
  static constexpr int NB = NWC * WC;                // columns of a workgroup
  static constexpr int NW = NWC * NWK;               // waves
  static constexpr int THREADS = NW * 64;
  static constexpr int ROW_BYTES = WC * 2;
  static constexpr int COPIES = 32 * ROW_BYTES / 1024;  // wave-wide copies of a substep of 32 kept columns
  static constexpr int SLOT = 32 * ROW_BYTES;        // ring slot: one substep
  static constexpr int RING_BYTES = R * SLOT;
  static constexpr int A_STEP = SPARSE ? RB * kPrepBlockBytes : RB * 4096;  // before 2:4: 32 RB rows of 64 values
  static constexpr int A_STAGE = NWK * A_STEP;       // a stage: one step for every group, contiguous in the layer form
  static constexpr int A_GRANULES = A_STAGE / 16;
  static constexpr int A_INSTR = (A_GRANULES + 63) / 64;
  static constexpr int A_SLOT = A_INSTR * 1024;
  static constexpr int A_RING = 3;
  static constexpr int E_SLOT = NWK * 256;           // row numbers of a stage
  static constexpr int E_RING = 4;
  // wave-wide copies of a stage that all waves share (before 2:4 the row numbers are one wave's business)
  static constexpr int SHARED_INSTR = A_INSTR + (SPARSE ? NWK : 0);
  static constexpr int SHARED_ROUNDS = (SHARED_INSTR + NW - 1) / NW;
  static constexpr int SHARED_MIN = SHARED_INSTR / NW;  // every wave issues at least that many
  static constexpr int A_BASE = NW * RING_BYTES;
  static constexpr int E_BASE = A_BASE + A_RING * A_SLOT;
  static constexpr int V_BASE = E_BASE + E_RING * E_SLOT;  // before 2:4: vector indexes on their way to row numbers
  static constexpr int LOOP_BYTES = V_BASE + (SPARSE ? 0 : 4 * E_SLOT);
  static constexpr int EPI_BYTES = 32 * RB * kStageStride<NB>;
  // 32x32 blocks of the result that a wave leaves to the other groups: block b is finished by group b % NWK
  static constexpr int GIVEN = (NWK - 1) * ((RB * CBS + NWK - 1) / NWK);
  static constexpr int SUM_BYTES = NW * GIVEN * 4096;
  static constexpr int LOOP_OR_EPI = LOOP_BYTES > EPI_BYTES ? LOOP_BYTES : EPI_BYTES;
  static constexpr int LDS_BYTES = LOOP_OR_EPI > SUM_BYTES ? LOOP_OR_EPI : SUM_BYTES;
  // 256-column blocks run two side by side on the same tiles of a die: its 32 units then fetch 16 tiles and two column
  // panels, not 32 tiles and one (4096 x 4096, V = 128, N = 2048 28.6 -> 25.2 us with two groups of steps, 4096 x 11008
  // 57.0 -> 55.3; V = 64, 8192 x 4096, N = 2048 63.0 -> 60.3 with one).  The smaller the stored values of a tile are beside
  // the panel, the less there is to share.  Mean over 12 layers (M, K 2048..11008, N 1024..4096) of one block alone over two
  // together, two groups and one: V = 128 1.04 and 1.02, V = 96 1.01 and 1.00, V = 64 1.01 and 1.01, V = 32 0.99 and 0.97
  // (2048 x 8192, Kv = 2048, N = 4096 50.0 us alone, 56.4 together; 4096 x 4096, N = 1024 27.6 and 26.6); before 2:4, V = 128
  // to 32, one group 1.03, 1.01, 1.02, 1.01.  A panel of 512 columns is the larger part of what they fetch and stays alone
  // (16384 x 16384, N = 8192 1200 against 1260).
  static constexpr int BLOCKS_TOGETHER = NB == 256 ? 2 : 1;
  static_assert(NWK == 1 || NWK == 2 || NWK == 4, "groups of steps");
  static_assert(R == 3 || R == 4, "ring");
  static_assert(LDS_BYTES <= kUnitLds, "LDS of a compute unit");
  static constexpr int SLOTS = 256 * (kUnitLds / LDS_BYTES);  // workgroups that run at once
};

// The forms (variants 20 to 24): 512 columns; 256, two groups of steps; 256; 128, two groups; 128, four groups on halves of
// 128-row tiles.  Rings of four slots where the LDS has room for what runs at once.
constexpr int form_depth(int SRC, int RB, int form) {
  if (form == 4) return 3;
  if (SRC == kRingVectors) return form == 2 || RB == 1 || (RB == 2 && form != 1) ? 4 : 3;
  return form == 0 || form == 2 || RB <= 2 ? 4 : 3;
}
constexpr int kFormColumnGroups[5] = {8, 4, 4, 2, 2}, kFormStepGroups[5] = {1, 2, 1, 2, 4};
template <int SRC, int RB, int FORM>
using FormCfg = RingCfg<SRC, FORM == 4 ? 2 : RB, kFormColumnGroups[FORM], kFormStepGroups[FORM], form_depth(SRC, RB, FORM)>;

__device__ __forceinline__ void buffer_copy16_to_lds(__amdgpu_buffer_rsrc_t r, uint32_t offset, uint8_t* lds_wave_base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)lds_wave_base, 16, (int)offset, 0, 0, 0);
}
__device__ __forceinline__ void buffer_copy4_to_lds(__amdgpu_buffer_rsrc_t r, uint32_t offset, uint8_t* lds_wave_base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)lds_wave_base, 4, (int)offset, 0, 0, 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_buffer(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}

// LDS reads as raw instructions, not waited for here: the compiler would hold every one until all copies in flight had
// landed.  To it an output is written at once, so it has to stay in its register until `tie`: lds_reads.py looks at the built
// code and the build fails where anything touches such a register before the wait.
template <int OFFSET>
__device__ __forceinline__ void lds_read_b128(uint32_t addr, u32x4& r) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(r) : "v"(addr), "n"(OFFSET));
}
template <int OFFSET>
__device__ __forceinline__ void lds_read_tr16(uint32_t addr, uint64_t& r) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=&v"(r) : "v"(addr), "n"(OFFSET));
}
template <int OFFSET>
__device__ __forceinline__ void lds_read_b32(uint32_t addr, int& r) {
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=&v"(r) : "v"(addr), "n"(OFFSET));
}

__device__ __forceinline__ void lds_write_b32(uint32_t addr, int v) {
  asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v));
}

// No use of the register is moved before this point.
template <class T>
__device__ __forceinline__ void pin(T& r) {
  asm volatile("" : "+v"(r));
}

typedef uint64_t u64x4 __attribute__((ext_vector_type(4)));

template <int RB, int CBS, bool SPARSE>
struct Fragments {
  uint64_t part[CBS][4];  // of b, while the reads are in flight
  u32x8 b[CBS];
  u32x4 a[SPARSE ? RB : 2 * RB];  // before 2:4: both halves of 16 kept columns
  int idx[RB];
};

template <int I, int N, class F>
__device__ __forceinline__ void unroll(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll<I + 1, N>(f);
  }
}

struct RingParams {
  const uint8_t* values;    // prepared blocks, or the stored values before 2:4
  const int32_t* gather;    // row numbers, or the vector index
  const int32_t* pi_in;     // before 2:4 (or NULL)
  const int32_t* out_rows;  // before 2:4 possibly NULL
  const uint16_t* X;
  void* Y;
  int64_t ldy;
  uint32_t x_bytes;  // what of X may be read, from its first element on
  int row_bytes;     // of X
  int T, S, N, n_blocks, work_per_xcd;
  int K, Kv;
  int parts;         // four groups: workgroups that share a tile, 32 RB rows each
  bool relu, out_f32;
};

template <int SRC, int DT, int RB, int NWC, int NWK, int R>
__device__ __forceinline__ void ring_product(const RingParams& p) {
  using C = RingCfg<SRC, RB, NWC, NWK, R>;
  constexpr bool SPARSE = C::SPARSE;
  constexpr int CBS = C::CBS;
  constexpr int V = 32 * RB;
  constexpr int NW = C::NW;
  const int T = p.T, S = p.S, N = p.N, n_blocks = p.n_blocks, row_bytes = p.row_bytes;
  const int32_t* const gather = p.gather;
  const int32_t* const out_rows = p.out_rows;
  void* const Y = p.Y;
  const int64_t ldy = p.ldy;
  const bool relu = p.relu, out_f32 = p.out_f32;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

  // Consecutive workgroup ids go to different XCDs: every XCD has a contiguous run of the work list, in which the tiles of
  // BLOCKS_TOGETHER column blocks follow each other.
  const int xcd = blockIdx.x & 7;
  const int slot_in_xcd = blockIdx.x >> 3;
  const int work = xcd * p.work_per_xcd + slot_in_xcd;
  if (slot_in_xcd >= p.work_per_xcd || work >= n_blocks * T) return;
  const int group = work / (T * C::BLOCKS_TOGETHER), in_group = work % (T * C::BLOCKS_TOGETHER);
  const int width = min(C::BLOCKS_TOGETHER, n_blocks - group * C::BLOCKS_TOGETHER);
  const int t = in_group / width;
  const int nb = group * C::BLOCKS_TOGETHER + in_group % width;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % NWC, g = wave / NWC;
  const int n0 = nb * C::NB + wc * C::WC;  // first column of the wave
  const int stages = (S + NWK - 1) / NWK;

  const auto x_buf = make_buffer(p.X, p.x_bytes);
  const int entries = SPARSE ? S * 64 : p.Kv;  // of the tile in `gather`
  const uint32_t a_bytes = SPARSE ? (uint32_t)S * C::A_STEP : (uint32_t)V * p.Kv * 2;
  const int parts = NWK == 4 ? p.parts : 1, tile = t / parts;  // T and t count parts of tiles
  const uint32_t step_bytes = (uint32_t)parts * C::A_STEP, part_offset = (uint32_t)(t % parts) * C::A_STEP;
  const auto a_buf = make_buffer(p.values + (size_t)tile * parts * a_bytes + part_offset, parts * a_bytes - part_offset);
  const auto e_buf = make_buffer(gather + (size_t)tile * entries, (uint32_t)entries * 4);

  // ---- copies ----
  // Copy j of a substep: lane class c = lane / 8 takes row 8 j + c.  Its 32-byte units are stored at unit ^ (row & 3)
  // (applied to the source address, a direct copy writes LDS linearly): the four rows of a transposing read then fall on
  // different banks.  Row numbers of padded kept columns are -1, which lies beyond the buffer's end: such lanes write
  // zeros.  Lanes whose columns lie beyond N re-read the row's first ones; what they feed is never stored.
  const int c = lane >> 3;
  const int granule = (lane & 7) ^ ((c & 3) << 1);
  const int lane_off = (n0 + granule * 8 < N) ? (n0 + granule * 8) * 2 : 0;
  uint8_t* const ring = lds + wave * C::RING_BYTES;
  auto issue_row_copy = [&](int row, int slot_off, int j) {
    buffer_copy16_to_lds(x_buf, (uint32_t)(__mul24(row, row_bytes) + lane_off), ring + slot_off + j * 1024);
  };
  // Row numbers of a step in LDS: position e holds the row of lane class e / 8, substep (e / 4) % 2, copy e % 4, so that a
  // lane reads those of a substep's copies with one 16-byte read.
  const uint32_t e_src = (uint32_t)(((lane >> 2) & 1) * 32 + 8 * (lane & 3) + (lane >> 3)) * 4;
  uint32_t a_src[C::SHARED_ROUNDS];
  int a_first[C::SHARED_ROUNDS];  // before 2:4: kept column of the stage that a lane's 16 bytes begin at
#pragma unroll
  for (int m = 0; m < C::SHARED_ROUNDS; ++m) {
    const int i = wave + m * NW;
    if constexpr (SPARSE) {
      const int piece = min(i * 64 + lane, C::A_GRANULES - 1);  // of 16 bytes
      a_src[m] = parts == 1 ? (uint32_t)piece * 16
                            : piece / (C::A_STEP / 16) * step_bytes + (uint32_t)(piece % (C::A_STEP / 16)) * 16;
    } else {
      // eight rows of a step at a time, 128 bytes each, 16-byte piece x of row r at position x ^ (r / 2) % 8: the reads of
      // 32 consecutive rows fall on different banks
      const int row = i % (4 * RB) * 8 + (lane >> 3), piece = (lane & 7) ^ ((row >> 1) & 7);
      a_first[m] = i / (4 * RB) * 64 + piece * 8;
      a_src[m] = (uint32_t)(row * p.Kv + a_first[m]) * 2;
    }
  }
  // Before 2:4 the first wave of every group turns its vector indexes into row numbers: it copies those of the stage three
  // ahead of e_stage, has those of e_stage in a register by now (`index`) and gathers their input channels into LDS.
  const auto pi_buf = make_buffer(p.pi_in, (uint32_t)p.K * 4);
  const bool translates = !SPARSE && wc == 0;
  int index = 0;
  auto issue_shared = [&](int a_stage, int a_slot, int e_stage) {  // stored values of a_stage, row numbers of e_stage
#pragma unroll
    for (int m = 0; m < C::SHARED_ROUNDS; ++m) {
      const int i = wave + m * NW;
      if (i < C::A_INSTR) {
        uint32_t off = (uint32_t)a_stage * (SPARSE ? NWK * step_bytes : NWK * 128) + a_src[m];
        if (!SPARSE && a_first[m] + a_stage * NWK * 64 >= p.Kv) off = 0xFFFFFFF0u;  // beyond the row: zeros
        buffer_copy16_to_lds(a_buf, off, lds + C::A_BASE + a_slot + i * 1024);
      } else if (i < C::SHARED_INSTR) {
        buffer_copy4_to_lds(e_buf, (uint32_t)(e_stage * NWK + (i - C::A_INSTR)) * 256 + e_src,
                            lds + C::E_BASE + (e_stage & 3) * C::E_SLOT + (i - C::A_INSTR) * 256);
      }
    }
    if (translates) {
      buffer_copy4_to_lds(e_buf, (uint32_t)((e_stage + 3) * NWK + g) * 256 + e_src,
                          lds + C::V_BASE + ((e_stage + 3) & 3) * C::E_SLOT + g * 256);
      uint8_t* const at = lds + C::E_BASE + (e_stage & 3) * C::E_SLOT + g * 256;
      if (p.pi_in) buffer_copy4_to_lds(pi_buf, (uint32_t)index * 4, at);
      else lds_write_b32((uint32_t)(uintptr_t)(lds_void_t*)at + lane * 4, index);
    }
  };

  // ---- LDS reads ----
  const int i32 = lane & 31, qh = lane >> 5, i16 = lane & 15;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void_t*)lds;
  uint32_t b_lane[CBS];
#pragma unroll
  for (int cb = 0; cb < CBS; ++cb)
    b_lane[cb] = lds_base + wave * C::RING_BYTES + (8 * qh + (i16 >> 2)) * C::ROW_BYTES +
                 (((cb * 2 + (i32 >> 4)) ^ (i16 >> 2)) * 32) + (i16 & 3) * 8;
  uint32_t a_lane[SPARSE ? 1 : 4];  // before 2:4: by substep and half
  if constexpr (SPARSE) {
    a_lane[0] = lds_base + C::A_BASE + g * C::A_STEP + lane * 16;
  } else {
    unroll<0, 4>([&](auto q) {
      a_lane[decltype(q)::value] =
          lds_base + C::A_BASE + g * C::A_STEP + i32 * 128 + ((decltype(q)::value * 2 + qh) ^ ((i32 >> 1) & 7)) * 16;
    });
  }
  const uint32_t i_lane = lds_base + C::A_BASE + g * C::A_STEP + kPrepIdxOffset + lane * 4;
  const uint32_t e_lane = lds_base + C::E_BASE + g * 256 + c * 32;
  const uint32_t v_lane = lds_base + C::V_BASE + g * 256 + lane * 4;

  Fragments<RB, CBS, SPARSE> f[2];
  static_assert(C::COPIES == 4, "row numbers of a substep are one vector");
  u32x4 e0, e1;  // row numbers of the copies to come, by substep
  // LDS read U of the READS that make a substep's fragments: rows of X first, then the stored values, and at a step's first
  // substep the nibbles of both
  auto read_fragment = [&](Fragments<RB, CBS, SPARSE>& fr, int b_slot, int a_slot, auto u_tag, auto sub_tag) {
    constexpr int U = decltype(u_tag)::value, SUB = decltype(sub_tag)::value;
    if constexpr (U < 4 * CBS) {
      constexpr int CB = U / 4, Q = U % 4;
      lds_read_tr16<((Q >> 1) * 16 + (Q & 1) * 4) * C::ROW_BYTES>(b_lane[CB] + b_slot, fr.part[CB][Q]);
    } else if constexpr (!SPARSE) {
      constexpr int I = U - 4 * CBS;
      lds_read_b128<I % RB * 4096>(a_lane[SUB * 2 + I / RB] + a_slot, fr.a[I]);
    } else if constexpr (U < 4 * CBS + RB) {
      constexpr int I = U - 4 * CBS;
      lds_read_b128<I * kPrepBlockBytes + SUB * 1024>(a_lane[0] + a_slot, fr.a[I]);
    } else {
      constexpr int I = U - 4 * CBS - RB;
      lds_read_b32<I * kPrepBlockBytes>(i_lane + a_slot, fr.idx[I]);
    }
  };
  auto reads_of = [](int sub) constexpr { return 4 * CBS + (SPARSE ? RB + (sub == 0 ? RB : 0) : 2 * RB); };
  auto tie = [&](Fragments<RB, CBS, SPARSE>& fr, auto sub_tag) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::);
    unroll<0, CBS>([&](auto cbt) {
      constexpr int cb = decltype(cbt)::value;
      unroll<0, 4>([&](auto q) { pin(fr.part[cb][decltype(q)::value]); });
    });
    unroll<0, CBS>([&](auto cbt) {
      constexpr int cb = decltype(cbt)::value;
      fr.b[cb] = __builtin_bit_cast(u32x8, u64x4{fr.part[cb][0], fr.part[cb][1], fr.part[cb][2], fr.part[cb][3]});
      pin(fr.b[cb]);
    });
    unroll<0, SPARSE ? RB : 2 * RB>([&](auto i) { pin(fr.a[decltype(i)::value]); });
    if constexpr (SPARSE && decltype(sub_tag)::value == 0) unroll<0, RB>([&](auto rb) { pin(fr.idx[decltype(rb)::value]); });
  };

  f32x16 acc[RB][CBS];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < CBS; ++cb)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[rb][cb][e] = 0.f;

  auto mfma = [&](const Fragments<RB, CBS, SPARSE>& fr, auto m_tag, auto sub_tag) {
    constexpr int RBI = decltype(m_tag)::value / CBS % RB, CB = decltype(m_tag)::value % CBS;
    if constexpr (SPARSE) {
      acc[RBI][CB] = smfmac_32x32x32<DT, decltype(sub_tag)::value>(fr.a[RBI], fr.b[CB], acc[RBI][CB], fr.idx[RBI]);
    } else {
      constexpr int H = decltype(m_tag)::value / (RB * CBS);
      const u32x8 b = fr.b[CB];
      acc[RBI][CB] = mfma_32x32x16<DT>(fr.a[H * RB + RBI], H ? b.hi : b.lo, acc[RBI][CB]);
    }
  };

  // ---- pipeline ----
  constexpr int NM = RB * CBS * (SPARSE ? 1 : 2);  // MFMAs of a substep
  constexpr int W = NM >= 8 ? NM / 8 : 1;  // of these, before the wait for the next substep's rows
  constexpr int BEFORE = (W * C::COPIES + NM - 1) / NM;  // copies issued before that wait: copy j precedes MFMA j NM / COPIES
  // first two stages' row numbers straight into registers
  int first_rows[2][2][C::COPIES];
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int j = 0; j < C::COPIES; ++j) {
        const int entry = min(min(st * NWK + g, S - 1) * 64 + sub * 32 + 8 * j + c, entries - 1);
        first_rows[st][sub][j] = gather[(size_t)tile * entries + entry];
      }
  int first_index[3] = {0, 0, 0};  // before 2:4: the vector indexes of stages 2 to 4
  if constexpr (!SPARSE) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
      first_index[i] = gather[(size_t)tile * entries + min(((i + 2) * NWK + g) * 64 + (int)e_src / 4, entries - 1)];
    if (p.pi_in) {
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
          for (int j = 0; j < C::COPIES; ++j) first_rows[st][sub][j] = p.pi_in[first_rows[st][sub][j]];
    }
  }
  index = first_index[0];
  issue_shared(0, 0, 2);
#pragma unroll
  for (int j = 0; j < C::COPIES; ++j) issue_row_copy(first_rows[0][0][j], 0, j);
  index = first_index[1];
  issue_shared(1, C::A_SLOT, 3);
  index = first_index[2];
#pragma unroll
  for (int j = 0; j < C::COPIES; ++j) issue_row_copy(first_rows[0][1][j], C::SLOT, j);
#pragma unroll
  for (int j = 0; j < C::COPIES; ++j) issue_row_copy(first_rows[1][0][j], 2 * C::SLOT, j);
  if constexpr (R == 4) {
#pragma unroll
    for (int j = 0; j < C::COPIES; ++j) issue_row_copy(first_rows[1][1][j], 3 * C::SLOT, j);
  }
  if constexpr (R == 3) {
#pragma unroll
    for (int j = 0; j < C::COPIES; ++j) e1[j] = (uint32_t)first_rows[1][1][j];
  }
  wait_copies_outstanding<(R - 1) * C::COPIES + C::SHARED_MIN>();
  if constexpr (!SPARSE) asm volatile("s_waitcnt lgkmcnt(0)" ::);  // row numbers written to LDS
  __builtin_amdgcn_s_barrier();
  issue_shared(2, 2 * C::A_SLOT, 4);

  int b_slot = 0, a_slot = 0;  // of the substep and stage about to be multiplied
  auto next_b = [&](int s) { return s + C::SLOT == C::RING_BYTES ? 0 : s + C::SLOT; };
  auto next_a = [&](int s) { return s + C::A_SLOT == C::A_RING * C::A_SLOT ? 0 : s + C::A_SLOT; };

  u32x4 next_e0, next_e1;
  int next_index = 0;
  auto read_rows = [&](int stage) {  // and, before 2:4, the vector indexes of the stage three ahead of it
    const uint32_t at = e_lane + (stage & 3) * C::E_SLOT;
    lds_read_b128<0>(at, next_e0);
    lds_read_b128<16>(at, next_e1);
    if constexpr (!SPARSE) lds_read_b32<0>(v_lane + ((stage + 3) & 3) * C::E_SLOT, next_index);
  };
  auto tie_rows = [&]() {
    pin(next_e0);
    pin(next_e1);
    if constexpr (!SPARSE) pin(next_index);
  };

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  unroll<0, reads_of(0)>([&](auto u) { read_fragment(f[0], 0, 0, u, I0{}); });
  read_rows(2);
  tie(f[0], I0{});
  tie_rows();
  e0 = next_e0;
  if constexpr (R == 4) e1 = next_e1;
  index = next_index;

  // Substep SUB of stage s: the copies of the substep R ahead go into the slot just read, one by one between the MFMAs;
  // once the next substep's rows have landed, the reads of its fragments are spread over the rest of them.
  auto substep = [&](int s, auto sub_tag, auto issue_tag, auto shared_tag, auto wait_tag, auto read_tag, bool multiply) {
    constexpr int SUB = decltype(sub_tag)::value;
    constexpr bool ISSUE = decltype(issue_tag)::value;
    constexpr bool SHARED = decltype(shared_tag)::value;
    constexpr bool READ = decltype(read_tag)::value;
    // R = 4: rows of stage s + 2, substep SUB; R = 3: substep 0 -> stage s + 1 substep 1, substep 1 -> stage s + 2 substep 0
    const u32x4 rows = (R == 4) ? (SUB ? e1 : e0) : (SUB ? e0 : e1);
    const int write_slot = b_slot;
    b_slot = next_b(b_slot);
    constexpr int NR = reads_of(1 - SUB);
    constexpr int PER = (NR + (NM > W + 3 ? NM - W - 2 : 1) - 1) / (NM > W + 3 ? NM - W - 2 : 1);
    unroll<0, NM>([&](auto m) {
      constexpr int M = decltype(m)::value;
      if constexpr (READ && M == W) {
        wait_copies_outstanding<decltype(wait_tag)::value>();
        if constexpr (SUB == 1) {
          __builtin_amdgcn_s_barrier();
          if constexpr (SHARED) issue_shared(s + 3, a_slot, s + 5);
          a_slot = next_a(a_slot);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (ISSUE) {
        unroll<0, C::COPIES>([&](auto j) {
          if constexpr (decltype(j)::value * NM / C::COPIES == M)
            issue_row_copy((int)rows[decltype(j)::value], write_slot, decltype(j)::value);
        });
      }
      if constexpr (READ && M >= W) {
        unroll<0, PER>([&](auto p) {
          constexpr int U = (M - W) * PER + decltype(p)::value;
          if constexpr (U < NR)
            read_fragment(f[1 - SUB], b_slot, a_slot, std::integral_constant<int, U>{}, std::integral_constant<int, 1 - SUB>{});
        });
        if constexpr (SHARED && M == NM - 1) read_rows(s + 3);
      }
      if (multiply) mfma(f[SUB], m, sub_tag);
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (READ) {
      tie(f[1 - SUB], std::integral_constant<int, 1 - SUB>{});
      if constexpr (SPARSE && SUB == 0) unroll<0, RB>([&](auto rb) { f[1].idx[decltype(rb)::value] = f[0].idx[decltype(rb)::value]; });
      if constexpr (SHARED) tie_rows();
    }
  };
  using Yes = std::true_type;
  using No = std::false_type;
  // Copies that may be outstanding when the next substep's rows have to be there: those of the substeps behind it, those of
  // this substep issued so far, and what the wave issued of the shared copies since (at least SHARED_MIN).
  constexpr int BEHIND = (R - 2) * C::COPIES;
  using WaitEven = std::integral_constant<int, BEHIND + BEFORE + C::SHARED_MIN>;
  using WaitOdd = std::integral_constant<int, BEHIND + BEFORE + (R == 4 ? C::SHARED_MIN : 0)>;
  int s = 0;
  for (; s < stages - 2; ++s) {
    substep(s, I0{}, Yes{}, No{}, WaitEven{}, Yes{}, true);
    if constexpr (R == 3) e1 = next_e1;
    substep(s, I1{}, Yes{}, Yes{}, WaitOdd{}, Yes{}, true);
    e0 = next_e0;
    if constexpr (R == 4) e1 = next_e1;
    index = next_index;
  }
  using WaitTail0 = std::integral_constant<int, BEHIND + (R == 3 ? BEFORE : 0) + C::SHARED_MIN>;
  using WaitTail1 = std::integral_constant<int, C::COPIES + (R == 4 ? C::SHARED_MIN : 0)>;
  const int last_step = (stages - 1) * NWK + g;
  const bool whole = last_step < S;  // an odd number of steps: the last group has none in the last stage
  // Before 2:4 the rows of padded kept columns are some row of X: their values are zero, but a row may hold NaN.  Kept columns
  // come in eights, a lane's registers 4 h .. 4 h + 3 are eight of them.
  auto clear_padded = [&](Fragments<RB, CBS, SPARSE>& fr, int sub) {
    if (SPARSE || p.Kv - last_step * 64 >= 64) return;
    unroll<0, CBS>([&](auto cbt) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (last_step * 64 + 32 * sub + 16 * (i / 4) + 8 * qh >= p.Kv) fr.b[decltype(cbt)::value][i] = 0;
    });
  };
  substep(s, I0{}, std::integral_constant<bool, R == 3>{}, No{}, WaitTail0{}, Yes{}, true);
  substep(s, I1{}, No{}, No{}, WaitTail1{}, Yes{}, true);
  clear_padded(f[0], 0);
  substep(s + 1, I0{}, No{}, No{}, I0{}, Yes{}, whole);
  clear_padded(f[1], 1);
  substep(s + 1, I1{}, No{}, No{}, I0{}, No{}, whole);

  // ---- epilogue ----
  __builtin_amdgcn_s_barrier();  // every wave is done with the ring and the stored values
  auto out_row = [&](int row) -> int64_t { return SPARSE || out_rows ? out_rows[t * V + row] : t * V + row; };
  auto finish = [&](auto g_tag) {
    constexpr int G = decltype(g_tag)::value;
    if constexpr (NWK > 1) {
      // block b of group h, for group b % NWK: slot (b % NWK - h - 1) mod NWK of the wave's b / NWK-th set
      auto given = [&](int w, int h, int b) {
        return lds + (w * C::GIVEN + b / NWK * (NWK - 1) + (b % NWK - h - 1 + NWK) % NWK) * 4096 + lane * 16;
      };
      unroll<0, RB * CBS>([&](auto bt) {
        constexpr int b = decltype(bt)::value;
        if constexpr (b % NWK != G) {
          uint8_t* const dst = given(wave, G, b);
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4*>(dst + q * 1024) =
                f32x4{acc[b / CBS][b % CBS][4 * q], acc[b / CBS][b % CBS][4 * q + 1], acc[b / CBS][b % CBS][4 * q + 2],
                      acc[b / CBS][b % CBS][4 * q + 3]};
        }
      });
      __syncthreads();
      unroll<0, RB * CBS>([&](auto bt) {
        constexpr int b = decltype(bt)::value;
        if constexpr (b % NWK == G) {
          unroll<1, NWK>([&](auto dt) {
            constexpr int h = (G + decltype(dt)::value) % NWK;
            const uint8_t* const src = given(wc + h * NWC, h, b);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const f32x4 v = *reinterpret_cast<const f32x4*>(src + q * 1024);
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[b / CBS][b % CBS][4 * q + e] += v[e];
            }
          });
        }
      });
      __syncthreads();
    }
    unroll<0, RB * CBS>([&](auto bt) {
      constexpr int b = decltype(bt)::value, rb = b / CBS, cb = b % CBS;
      if constexpr (b % NWK == G) {
        if (out_f32) {
          const int n = n0 + cb * 32 + i32;
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            float* dst = static_cast<float*>(Y) + out_row(32 * rb + 8 * (e >> 2) + 4 * qh + (e & 3)) * ldy;
            float v = acc[rb][cb][e];
            if (relu) v = v > 0.f ? v : 0.f;
            if (n < N) dst[n] = v;
          }
        } else {
          stage_block<DT, kStageStride<C::NB>>(acc[rb][cb], lds + 32 * rb * kStageStride<C::NB> + (wc * C::WC + cb * 32) * 2, relu);
        }
      }
    });
  };
  unroll<0, NWK>([&](auto gt) {
    if (g == decltype(gt)::value) finish(gt);
  });
  if (out_f32) return;
  __syncthreads();
  store_staged_rows<V, C::NB, C::THREADS>(lds, Y, ldy, N, nb * C::NB, out_row);
}

// Two waves a SIMD are asked for where one would do, too: with more than 256 registers at hand the compiler parks fragments in
// accumulation registers before their LDS reads have landed.
template <int DT, int RB, int NWC, int NWK, int R>
__global__ __launch_bounds__(NWC * NWK * 64, 2) void spmm_rings_kernel(RingParams p) {
  ring_product<kRingPrepared, DT, RB, NWC, NWK, R>(p);
}
template <int DT, int RB, int NWC, int NWK, int R>
__global__ __launch_bounds__(NWC * NWK * 64, 2) void spmm_vectors_rings_kernel(RingParams p) {
  ring_product<kRingVectors, DT, RB, NWC, NWK, R>(p);
}

// The forms, by columns and groups of steps (variants 20 to 24), and what a launch of each takes by tile height (us):
//   start + (rounds of workgroups before the last) * (round + steps * full) + steps * (part + fill * more)
// where steps are those of a wave and `fill` is the share of the last round's slots that are taken: a step is slower the
// more units take part (clock, memory).  Fitted to 480 random layers (M, K 256..16384, N 65..8192, all tile heights, both
// types; error 5 to 15 %); the form chosen by it is 0.7 % off the best of the first four on average.  The last two of 32-row
// tiles are fitted to 804 layers of those (error 11 and 9 %, the choice 0.2 % off the best): two workgroups of 128 columns
// exceed the LDS of a unit by 2 KB, and two of 256 columns take as long side by side as one behind the other (2880 x 5888,
// Kv = 2944, N = 256 17.6 us on the kernel for a moderate number of columns, 12.2 on 128 columns; 9856 x 2864, Kv = 720,
// N = 288 19.4 on 128 columns, 14.6 on 256).  Examples, us in the order below: 4096 x 11008 at 50 %, N = 2048 67 / 53 / 57 /
// 75; 16384 x 16384 at 50 %, N = 8192 1178 / 1306 / 1375 / 1723; 4096 x 4096, V = 128, N = 1024 29 / 20 / 20 / 18; 1984 x
// 6376, V = 64, Kv = 3184, N = 6033 92 / 82 / 77 / 109.
struct RingForm {
  int columns, groups, slots;  // slots: workgroups of a round, as many as run at once or fewer (0: no such form)
  float start, full, part, more, round;
};
constexpr int kRingForms = 5;
constexpr RingForm kForms[4][kRingForms] = {  // [RB - 1]
    {{512, 1, 256, 3.2f, 0.76f, 0.55f, 0.21f, 1.4f}, {256, 2, 256, 3.3f, 0.91f, 0.58f, 0.32f, 1.5f},
     {256, 1, 256, 3.3f, 0.39f, 0.31f, 0.07f, 0.35f}, {128, 2, 256, 3.4f, 0.50f, 0.35f, 0.15f, 1.7f}},
    {{512, 1, 256, 4.4f, 0.93f, 0.55f, 0.18f, 3.7f}, {256, 2, 256, 4.5f, 0.99f, 0.57f, 0.34f, 2.8f},
     {256, 1, 512, 4.3f, 0.99f, 0.31f, 0.44f, 2.1f}, {128, 2, 256, 3.8f, 0.59f, 0.38f, 0.20f, 2.3f}},
    {{512, 1, 256, 5.8f, 0.99f, 0.56f, 0.25f, 6.3f}, {256, 2, 256, 5.2f, 1.15f, 0.63f, 0.38f, 3.9f},
     {256, 1, 256, 5.0f, 0.55f, 0.38f, 0.10f, 3.6f}, {128, 2, 256, 4.4f, 0.75f, 0.50f, 0.27f, 3.0f}},
    {{512, 1, 256, 6.4f, 1.04f, 0.66f, 0.43f, 10.8f}, {256, 2, 256, 5.8f, 1.24f, 0.74f, 0.42f, 6.3f},
     {256, 1, 256, 5.9f, 0.62f, 0.43f, 0.16f, 5.4f}, {128, 2, 256, 4.9f, 0.81f, 0.56f, 0.30f, 4.4f},
     {128, 4, 256, 4.0f, 1.51f, 0.69f, 0.64f, 1.0f}}};

// No more slots than the LDS of the form's configuration has room for.
template <int SRC, int RB, int FORM>
constexpr bool slots_hold(const RingForm& f) {
  using C = FormCfg<SRC, RB, FORM>;
  return f.columns == C::NB && f.groups == C::STEP_GROUPS && f.slots <= C::SLOTS;
}
template <int RB>
constexpr bool prepared_forms_hold() {
  const auto& f = kForms[RB - 1];
  return slots_hold<kRingPrepared, RB, 0>(f[0]) && slots_hold<kRingPrepared, RB, 1>(f[1]) &&
         slots_hold<kRingPrepared, RB, 2>(f[2]) && slots_hold<kRingPrepared, RB, 3>(f[3]) &&
         (RB == 4 ? slots_hold<kRingPrepared, RB, 4>(f[4]) : f[4].slots == 0);
}
static_assert(prepared_forms_hold<1>() && prepared_forms_hold<2>() && prepared_forms_hold<3>() && prepared_forms_hold<4>());

// Workgroups that share a tile: two of 64 rows each with four groups of steps (tiles of 128 rows only).
constexpr int form_parts(const RingForm& f) { return f.groups == 4 ? 2 : 1; }

double form_us(const RingForm& f, int S, int tiles, int N) {
  const int64_t work = (int64_t)tiles * form_parts(f) * ((N + f.columns - 1) / f.columns);
  const int64_t whole = (work - 1) / f.slots, last = work - whole * f.slots;
  const double steps = (S + f.groups - 1) / f.groups;
  return f.start + whole * (f.round + steps * f.full) + steps * (f.part + f.more * last / f.slots);
}

// `mid`: of the forms that split the steps, for fewer columns; against the kernel's own blocks they have to be 8 % ahead, 16 %
// with 32-row tiles, about what the estimates miss by (2720 x 8992, V = 32, Kv = 1120, N = 576: 12.7 us there, 13.9 here; 3200 x
// 10424, V = 128, Kv = 2608, N = 628: 21.6 us there, 22.4 here, estimated 24.8 and 23.3).
// Four groups are the form for the fewest columns, estimated on such products alone, and need no margin; up to 320 of the
// kernel's own blocks those are as good (11008 x 4096 at 50 %, N = 100, 344 blocks: 14.1 us there, 12.0 with four groups, 15.4
// with two; 4096 x 4096, N = 512, 512 blocks 17.6, 13.7 and 15.8; N = 256, 256 blocks 8.4 and 9.5).
// `far_rows`: by rows_are_far.
int best_form(const RingForm (&forms)[kRingForms], bool mid, int S, int tiles, int N, double* us, bool far_rows = false) {
  int best = -1;
  for (int i = 0; i < kRingForms; ++i) {
    const bool four = forms[i].groups == 4;
    if (forms[i].slots == 0 || (mid ? forms[i].groups == 1 : four)) continue;
    if (four && (S < 5 || (int64_t)tiles * 2 * ((N + 63) / 64) <= 320)) continue;
    const double t = form_us(forms[i], S, tiles, N) * (!mid || four ? 1.0 : &forms == &kForms[0] ? 1.16 : 1.08) *
                     (far_rows && i == 2 ? 1.1 : 1.0);
    if (best < 0 || t < *us) *us = t, best = i;
  }
  return best;
}

// Tiles of 32 rows that keep few of many rows of X find less of what they gather in L2 with 256 columns than with 512: beyond
// 32 MB of X with an eighth kept the former take 1.33 times their estimate, the latter 1.24 (16 drawn layers; 6336 x 12368,
// Kv = 1544, N = 4704 222 and 184 us).
bool rows_are_far(const PreparedArgs& a) {
  return a.s.V == 32 && a.s.K >= 6 * (int64_t)a.s.Kv && (double)a.s.K * a.N * 2 > 32e6;
}

// The tiles [first, first + count) of the layer.
template <int DT, class C>
hipError_t launch_form(const PreparedArgs& a, hipStream_t stream, int first, int count) {
  constexpr int RB = C::ROWS, NWK = C::STEP_GROUPS, R = C::DEPTH;
  const PreparedLayout L = prepared_layout(a.s);
  const int n_blocks = (a.N + C::NB - 1) / C::NB;
  const int parts = L.RB / RB;
  const int work_per_xcd = (int)(((int64_t)n_blocks * count * parts + 7) / 8);
  constexpr auto kernel = spmm_rings_kernel<DT, RB, C::COLUMN_GROUPS, NWK, R>;
  if (a.plan) {
    plan_record(a.plan, "spmm_rings_kernel<DT=%d,RB=%d,NB=%d,NWK=%d,R=%d> private rings, tiles=%d..%d grid=%d block=%d lds=%d", DT,
                RB, C::NB, NWK, R, first, first + count - 1, work_per_xcd * 8, C::THREADS, C::LDS_BYTES);
    return hipSuccess;
  }
  if (hipError_t e = raise_lds_limit<kernel>(C::LDS_BYTES); e != hipSuccess) return e;
  const uint8_t* base = static_cast<const uint8_t*>(a.prepared);
  const int64_t row_bytes = a.ldx * 2;
  RingParams p{};
  p.values = base + L.a_offset + (size_t)first * L.S * parts * C::A_STEP;
  p.gather = reinterpret_cast<const int32_t*>(base + L.gather_offset) + (size_t)first * L.S * 64;
  p.out_rows = reinterpret_cast<const int32_t*>(base + L.pi_out_offset) + (size_t)first * a.s.V;
  p.X = static_cast<const uint16_t*>(a.X);
  p.Y = a.Y;
  p.ldy = a.ldy;
  p.x_bytes = (uint32_t)((a.s.K - 1) * row_bytes + (int64_t)(a.N + 7) / 8 * 16);
  p.row_bytes = (int)row_bytes;  // checked by spmm_ring_prepared_supported
  p.T = count * parts;
  p.parts = parts;
  p.S = L.S;
  p.N = a.N;
  p.n_blocks = n_blocks;
  p.work_per_xcd = work_per_xcd;
  p.relu = a.relu;
  p.out_f32 = a.out_f32;
  kernel<<<dim3((unsigned)(work_per_xcd * 8)), C::THREADS, C::LDS_BYTES, stream>>>(p);
  return hipGetLastError();
}

template <int DT, int RB>
hipError_t launch_tiles(const PreparedArgs& a, hipStream_t stream, int form, int first, int count) {
  switch (form) {
    case 0: return launch_form<DT, FormCfg<kRingPrepared, RB, 0>>(a, stream, first, count);
    case 1: return launch_form<DT, FormCfg<kRingPrepared, RB, 1>>(a, stream, first, count);
    case 2: return launch_form<DT, FormCfg<kRingPrepared, RB, 2>>(a, stream, first, count);
    case 3: return launch_form<DT, FormCfg<kRingPrepared, RB, 3>>(a, stream, first, count);
    case 4:
      if constexpr (RB == 4) return launch_form<DT, FormCfg<kRingPrepared, RB, 4>>(a, stream, first, count);
      break;
    default: break;
  }
  return hipErrorInvalidValue;
}

template <int DT, int RB>
hipError_t launch_rb(const PreparedArgs& a, bool mid, hipStream_t stream) {
  const PreparedLayout L = prepared_layout(a.s);
  if (a.tile_variant) return launch_tiles<DT, RB>(a, stream, a.tile_variant - kRingFirstVariant, 0, L.T);
  double us = 0;
  const int form = best_form(kForms[RB - 1], mid, L.S, L.T, a.N, &us, rows_are_far(a));
  if (mid) return launch_tiles<DT, RB>(a, stream, form, 0, L.T);
  // Whole rounds of 512-column blocks, and the tiles that are left over in the form that suits them, behind them
  // (11008 x 4096 at 50 %, N = 2048, 344 blocks: 64.8 us, the best single launch 67.9).  With 32-row tiles, whose passes are the
  // shortest, by 1 us more than estimated (61 of 81 drawn splits are left, 0.93 times the best single launch's time on their
  // mean; without that some lose a tenth: 11584 x 2240, Kv = 1120, N = 352 1.09 times).
  const int wide = (a.N + 511) / 512;
  const int64_t rounds = (int64_t)L.T * wide / 256;
  const int whole = (int)(rounds * 256 / wide);
  if (rounds > 0 && whole < L.T) {
    double rest_us = 0;
    const int rest_form = best_form(kForms[RB - 1], false, L.S, L.T - whole, a.N, &rest_us, rows_are_far(a));
    if (form_us(kForms[RB - 1][0], L.S, whole, a.N) + rest_us + (RB == 1 ? 1.0 : 0.0) < us) {
      const hipError_t e = launch_tiles<DT, RB>(a, stream, 0, 0, whole);
      return e != hipSuccess ? e : launch_tiles<DT, RB>(a, stream, rest_form, whole, L.T - whole);
    }
  }
  return launch_tiles<DT, RB>(a, stream, form, 0, L.T);
}

}  // namespace

// Two stages at least, and what the copies' 32-bit byte offsets and 24-bit products can address.
bool spmm_ring_prepared_supported(const PreparedArgs& a) {
  if (a.N <= 1 || a.ldx % 8 != 0 || a.ldy % 8 != 0) return false;
  const PreparedLayout L = prepared_layout(a.s);
  const uint64_t row = (uint64_t)a.ldx * 2;
  if (a.tile_variant == kRingLastVariant && (L.S < 5 || L.RB != 4)) return false;  // two stages of four steps, two halves
  return L.S >= 3 && a.s.K < (1 << 23) && row < (1u << 23) && ((uint64_t)a.s.K + 1) * row <= (uint64_t{1} << 32) &&
         (int64_t)L.T * 2 * ((a.N + 127) / 128) < (1 << 30);
}

double spmm_ring_prepared_us(const PreparedArgs& a, bool mid) {
  double us = 0;
  best_form(kForms[a.s.V / 32 - 1], mid, (a.s.Kv + 63) / 64, a.s.M / a.s.V, a.N, &us, rows_are_far(a));
  return us;
}

hipError_t launch_spmm_ring_prepared(const PreparedArgs& a, bool mid, hipStream_t stream) {
  const int RB = a.s.V / 32;
#define HINM_RB(DT)                                    \
  switch (RB) {                                        \
    case 1: return launch_rb<DT, 1>(a, mid, stream);   \
    case 2: return launch_rb<DT, 2>(a, mid, stream);   \
    case 3: return launch_rb<DT, 3>(a, mid, stream);   \
    case 4: return launch_rb<DT, 4>(a, mid, stream);   \
  }
  if (a.s.dtype == HINM_F16) {
    HINM_RB(HINM_F16)
  } else {
    HINM_RB(HINM_BF16)
  }
#undef HINM_RB
  return hipErrorInvalidValue;
}

// ---- before the 2:4 step ------------------------------------------------------------------------------------------------

namespace {

// As kForms, fitted to 260 random layers (M, K up to 8192, N 65..4096; error 4 to 9 %, the form chosen 0.2 % off the best).  Two
// groups of steps on 256 columns leave no room in LDS for the dense values of 96 rows and more.  us, in the order of the
// forms: 4096 x 4096, V = 64, Kv = 2048, N = 1000 36 / 27 / 27 / 37 (tile kernel 37); 8192 x 8192, V = 128, Kv = 4096, N = 2048
// 120 / - / 137 / 179 (165); 4096 x 4096, V = 128, N = 1024 42 / - / 29 / 27 (42).
constexpr RingForm kVectorForms[4][kRingForms] = {  // [RB - 1]
    {{512, 1, 256, 4.0f, 1.13f, 0.52f, 0.25f, 1.5f}, {256, 2, 256, 4.2f, 1.13f, 0.54f, 0.41f, 1.8f},
     {256, 1, 512, 3.9f, 1.07f, 0.29f, 0.52f, 1.1f}, {128, 2, 256, 3.9f, 0.70f, 0.37f, 0.20f, 1.9f}},
    {{512, 1, 256, 5.4f, 1.59f, 0.58f, 0.52f, 3.7f}, {256, 2, 256, 4.9f, 1.64f, 0.70f, 0.56f, 2.8f},
     {256, 1, 256, 4.9f, 0.78f, 0.42f, 0.17f, 2.6f}, {128, 2, 256, 4.6f, 1.03f, 0.49f, 0.36f, 2.4f}},
    {{512, 1, 256, 6.2f, 2.05f, 0.84f, 0.62f, 0.0f}, {256, 2, 0, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f},
     {256, 1, 256, 5.8f, 0.78f, 0.54f, 0.21f, 6.8f}, {128, 2, 256, 5.4f, 1.32f, 0.73f, 0.30f, 3.1f}},
    {{512, 1, 256, 7.2f, 1.72f, 1.05f, 0.53f, 10.1f}, {256, 2, 0, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f},
     {256, 1, 256, 6.4f, 1.02f, 0.68f, 0.37f, 6.2f}, {128, 2, 256, 5.8f, 1.74f, 0.86f, 0.57f, 3.1f}}};

template <int RB>
constexpr bool vector_forms_hold() {
  const auto& f = kVectorForms[RB - 1];
  bool second = f[1].slots == 0;
  if constexpr (RB <= 2) second = slots_hold<kRingVectors, RB, 1>(f[1]);
  return slots_hold<kRingVectors, RB, 0>(f[0]) && second && slots_hold<kRingVectors, RB, 2>(f[2]) &&
         slots_hold<kRingVectors, RB, 3>(f[3]) && f[4].slots == 0;
}
static_assert(vector_forms_hold<1>() && vector_forms_hold<2>() && vector_forms_hold<3>() && vector_forms_hold<4>());

template <int DT, class C>
hipError_t launch_vectors_form(const VectorsArgs& a, hipStream_t stream) {
  const int T = a.s.M / a.s.V;
  const int n_blocks = (a.N + C::NB - 1) / C::NB;
  const int work_per_xcd = (int)(((int64_t)n_blocks * T + 7) / 8);
  constexpr auto kernel = spmm_vectors_rings_kernel<DT, C::ROWS, C::COLUMN_GROUPS, C::STEP_GROUPS, C::DEPTH>;
  if (hipError_t e = raise_lds_limit<kernel>(C::LDS_BYTES); e != hipSuccess) return e;
  const int64_t row_bytes = a.ldx * 2;
  RingParams p{};
  p.values = static_cast<const uint8_t*>(a.vals_v);
  p.gather = a.vec_idx;
  p.pi_in = a.pi_in;
  p.out_rows = a.pi_out;
  p.X = static_cast<const uint16_t*>(a.X);
  p.Y = a.Y;
  p.ldy = a.ldy;
  p.x_bytes = (uint32_t)((a.s.K - 1) * row_bytes + (int64_t)(a.N + 7) / 8 * 16);
  p.row_bytes = (int)row_bytes;  // checked by spmm_ring_vectors_supported
  p.T = T;
  p.S = (a.s.Kv + 63) / 64;
  p.N = a.N;
  p.n_blocks = n_blocks;
  p.work_per_xcd = work_per_xcd;
  p.K = a.s.K;
  p.Kv = a.s.Kv;
  p.relu = a.relu;
  p.out_f32 = a.out_f32;
  kernel<<<dim3((unsigned)(work_per_xcd * 8)), C::THREADS, C::LDS_BYTES, stream>>>(p);
  return hipGetLastError();
}

template <int DT, int RB>
hipError_t launch_vectors_rb(const VectorsArgs& a, hipStream_t stream) {
  double us = 0;
  switch (a.variant ? a.variant - kRingFirstVariant
                    : best_form(kVectorForms[RB - 1], false, (a.s.Kv + 63) / 64, a.s.M / a.s.V, a.N, &us)) {
    case 0: return launch_vectors_form<DT, FormCfg<kRingVectors, RB, 0>>(a, stream);
    case 1:
      if constexpr (RB <= 2) return launch_vectors_form<DT, FormCfg<kRingVectors, RB, 1>>(a, stream);
      break;
    case 2: return launch_vectors_form<DT, FormCfg<kRingVectors, RB, 2>>(a, stream);
    case 3: return launch_vectors_form<DT, FormCfg<kRingVectors, RB, 3>>(a, stream);
    default: break;
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool spmm_ring_vectors_supported(const VectorsArgs& a) {
  const int V = a.s.V;
  if (a.variant == kRingLastVariant || (a.variant == kRingFirstVariant + 1 && V > 64)) return false;
  if (!(V == 32 || V == 64 || V == 96 || V == 128) || a.N <= 1 || a.ldx % 8 != 0 || a.ldy % 8 != 0) return false;
  const uint64_t row = (uint64_t)a.ldx * 2;
  return (a.s.Kv + 63) / 64 >= 3 && a.s.K < (1 << 23) && row < (1u << 23) && ((uint64_t)a.s.K + 1) * row <= (uint64_t{1} << 32) &&
         (int64_t)(a.s.M / V) * ((a.N + 127) / 128) < (1 << 30);
}

// From 65 columns on.  Against the kernel for a moderate number of columns by estimate, 8 % ahead as for the prepared form, with
// more than five steps and more than 320 of its 64-column blocks (of 260 random layers two gained below); of
// what the tile kernel serves all but short passes of whole 64-column steps (2368 x 1536, V = 64, Kv = 384, N = 3856 19.0 us
// there, 21.4 here; Kv = 256, 3456 x 1040, N = 3943 20.0 and 20.5; but 1344 x 1616, Kv = 400, N = 3873 18.2 and 12.2).
bool spmm_ring_vectors_preferred(const VectorsArgs& a) {
  if (a.N <= 64 || !spmm_ring_vectors_supported(a)) return false;
  if (!spmm_mid_vectors_preferred(a)) return a.s.Kv % 64 != 0 || a.s.Kv > 6 * 64;
  const int64_t blocks = (int64_t)(a.s.M / (a.s.V % 64 == 0 ? 64 : 32)) * ((a.N + 63) / 64);
  if (blocks <= 320 || a.s.Kv <= 5 * 64) return false;
  double us = 0;
  best_form(kVectorForms[a.s.V / 32 - 1], false, (a.s.Kv + 63) / 64, a.s.M / a.s.V, a.N, &us);
  return us * 1.08 < spmm_mid_vectors_us(a);
}

hipError_t launch_spmm_ring_vectors(const VectorsArgs& a, hipStream_t stream) {
#define HINM_RB(DT)                                            \
  switch (a.s.V) {                                             \
    case 32: return launch_vectors_rb<DT, 1>(a, stream);       \
    case 64: return launch_vectors_rb<DT, 2>(a, stream);       \
    case 96: return launch_vectors_rb<DT, 3>(a, stream);       \
    case 128: return launch_vectors_rb<DT, 4>(a, stream);      \
  }
  if (a.s.dtype == HINM_F16) {
    HINM_RB(HINM_F16)
  } else {
    HINM_RB(HINM_BF16)
  }
#undef HINM_RB
  return hipErrorInvalidValue;
}

}  // namespace hinm
