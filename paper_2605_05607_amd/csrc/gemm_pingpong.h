// Main loops of the grouped GEMM tile: operands straight from memory into the LDS, slabs requested several k-steps ahead.
#pragma once
#include <type_traits>

#include "forward_types.h"

namespace moe355 {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x16 mfma_bf16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// FP8 operands (E4M3): a 16-byte fragment holds 16 reduction indices per lane; two fragments (32 bytes per lane)
// feed one 32x32x64 instruction.  Which reduction indices share an instruction, and where in the operand they sit,
// does not matter as long as A and B agree: both put the same two 16-byte chunks of the reduction range side by side.
__device__ __forceinline__ f32x16 mfma_fp8_pair(bf16x8 a_lo, bf16x8 a_hi, bf16x8 b_lo, bf16x8 b_hi, f32x16 c) {
  const i32x8 a = __builtin_shufflevector(__builtin_bit_cast(i32x4, a_lo), __builtin_bit_cast(i32x4, a_hi), 0, 1, 2, 3,
                                          4, 5, 6, 7);
  const i32x8 b = __builtin_shufflevector(__builtin_bit_cast(i32x4, b_lo), __builtin_bit_cast(i32x4, b_hi), 0, 1, 2, 3,
                                          4, 5, 6, 7);
  // both operands E4M3 (format selectors 0), no block scales (all scale operands 0)
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
}

// ---- loads into the LDS ----
// 16 bytes per lane from memory to LDS address lds + 16 lane.  Assembler, because the compiler would wait for every such
// load in front of any LDS read that it cannot tell apart from its target; the waits are placed by hand instead (the main
// loops have no other vector-memory operation: nothing is spilled).
__device__ __forceinline__ i32x4 lds_load_rsrc(const void *base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00027000;
  return r;
}
template <bool NT = false>  // NT: with the non-temporal hint
__device__ __forceinline__ void load_to_lds(i32x4 rsrc, uint32_t lds, uint32_t voff, uint32_t soff) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 :
                 : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
}
__device__ __forceinline__ void load_to_lds_far(const void *src, uint32_t lds) {  // a 64-bit address per lane
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds), "v"(src) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char *)p;
}
template <int N>
__device__ __forceinline__ void wait_loads() {  // at most N of this wave's vector-memory operations outstanding
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void slot_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// The lane's number, computed anew at every use: as a value that lives across a main loop (threadIdx is one) it takes a
// register that the full tiles do not have.
__device__ __forceinline__ int fresh_lane() {
  uint32_t zero = 0;
  asm volatile("" : "+s"(zero));
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// Where a lane reads its row of a 32-row block whose rows are 128 bytes with permuted chunks (see RowRequests): chunk
// 2 kk + lane / 32 of row `row` (row % 32 = lane % 32) is at this offset ^ 32 kk.
__device__ __forceinline__ int row_read_offset(int row, int lane) {
  return row * 128 + (((lane >> 5) ^ ((lane >> 1) & 7)) * 16);
}

// The rows of A as this wave requests them: instruction i of region h moves eight rows (128 bytes each, lane = row by
// chunk).  The stage image is [row][128 bytes] with the eight 16-byte chunks of a row permuted by (row >> 1) & 7 (gfx950's
// LDS has 64 banks and serves a 128-bit read 16 lanes at a time); the LDS side of the load is linear in the lane, so the
// permutation is applied to the memory side.  A chunk past K repeats a chunk of the same row in the last k-step (the
// packed tile holds zeros there).  FAR: matrices of 4 GiB and more, row numbers instead of byte offsets.
template <bool FP8, int H, int I, bool FAR>
struct RowRequests {
  static constexpr int EPC = FP8 ? 16 : 8, KS = FP8 ? 128 : kBK;
  i32x4 rsrc;
  const unsigned char *base;
  uint32_t at[H][I];
  uint32_t pitch;   // bytes of a row of A
  // FAR: this lane's chunk of instruction i, region h, 4 bits each.  Otherwise (no register to spare) scalar bits: whether
  // the instruction's first row is an odd multiple of eight, which with the lane gives the chunk.
  uint32_t chunks;
  // bytes: bound of the descriptor (0: every request is answered with zeros; FAR has no descriptor)
  __device__ __forceinline__ void init(const void *A, int lda, uint32_t bytes = 0xFFFFFFFFu) {
    base = static_cast<const unsigned char *>(A);
    pitch = (uint32_t)lda * (FP8 ? 1 : 2);
    rsrc = lds_load_rsrc(base, bytes);
    chunks = 0;
  }
  // row = row of the tile (image position: a multiple of eight plus lane / 8), a_row = row of the matrix
  __device__ __forceinline__ void set(int h, int i, int row, uint32_t a_row, int lane) {
    const uint32_t chunk = (lane & 7) ^ ((row >> 1) & 7);
    chunks |= FAR ? chunk << (4 * (h * I + i)) : (__builtin_amdgcn_readfirstlane(row >> 3) & 1) << (h * I + i);
    at[h][i] = FAR ? a_row : a_row * pitch + chunk * 16;
  }
  __device__ __forceinline__ uint32_t chunk_of(int h, int i) const {
    if (FAR) return (chunks >> (4 * (h * I + i))) & 7;
    const uint32_t lane = fresh_lane();
    return (lane & 7) ^ (lane >> 4) ^ ((chunks >> (h * I + i)) & 1) << 2;
  }
  // call before the first request of the last k-step
  __device__ __forceinline__ void clip(int K, int kt_last) {
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int i = 0; i < I; ++i) {
        const uint32_t c = chunk_of(h, i);
        if (kt_last * KS + (int)c * EPC >= K) {
          if (FAR) chunks &= ~(7u << (4 * (h * I + i))); else at[h][i] -= c * 16;
        }
      }
  }
  __device__ __forceinline__ void request(int h, int i, uint32_t lds, int kt) const {
    if constexpr (FAR)
      load_to_lds_far(base + (uint64_t)at[h][i] * pitch + chunk_of(h, i) * 16 + (uint32_t)kt * 128, lds);
    else
      load_to_lds(rsrc, lds, at[h][i], kt * 128);
  }
};

// ------------------------------------------------------------------------------------------------
// Full tiles (more than 128 rows): 256 x 256 outputs, two 64 KiB stages, 8 waves = 2 rows x 4 columns of RW x 64: RW = 128,
// or 96 for tiles of at most 192 rows.
// What bounds it: the matrix cores (2048 cycles per k-step and SIMD) and, as close, the LDS (192 KiB of fragment reads
// and 64 KiB of slab per k-step), so both have to run all the time.  The wave rows take turns: while one row's four waves
// (one per SIMD) issue the matrix instructions of a phase, the other row's read their next operands from the LDS and
// request slabs from memory; a barrier ends each such slot and the rows swap.  A k-step is four phases, the quadrants of
// the wave's block: rows 0-63 (A0) or the rest (A1) by columns 0-31 (B0) or 32-63 (B1), in the order A0 B0, A0 B1, A1 B1,
// A1 B0, so that every operand is read once per k-step and the memory slots are about equal:
//     M0: read B0(kt)            request A0(kt + 2)     then multiply A0 B0
//     M1: read B1(kt), half A1   request B0(kt + 2)                   A0 B1
//     M2: read the rest of A1    request B1(kt + 2)                   A1 B1
//     M3: read A0(kt + 1)        request A1(kt + 2)                   A1 B0
// A region of a stage is requested again right after both rows have read it, so a slab has 12 to 14 of the 16 slots of
// two k-steps to arrive.  Each wave requests two KiB of every region (A1 of RW = 96: one); it waits for its own requests (the counts below are
// the requests it has issued since) in a slot before the one in which either row reads the region, and the barrier at
// that slot's end tells the others.
// Measured: 16 384 rows x 4096 x 14336 (two GEMMs), dense rows: 1.22 PFLOP/s with slabs staged through registers, one
// barrier per k-step and all waves in step -> 1.38 PFLOP/s (the vendor library's dense product reaches 1.44 to 1.50 on
// the box); whole prefill step of that layer 9.64 -> 8.84 ms.
// ------------------------------------------------------------------------------------------------
// GRAD (weight gradients, wgrad_bf16.h), kGradSlabs: both operands are slabs of [column][128 bytes], `step` bytes from one
// k-step to the next, and both are requested and read as A is.
// kGradGatherA, kGradGatherB: the reduction index is the row of both operands and they are requested as they lie in memory,
// 64 rows per k-step; one operand's rows are gathered (byte offsets of the rows in the LDS table `tab`), the other's follow
// one another.  The stage holds blocks of [64 rows][64 columns] (B: [64 rows][32 columns] per region) and the reads
// transpose: a 16-lane group of ds_read_b64_tr_b16 turns four rows of sixteen columns into sixteen lanes of four reduction
// indices.  The halves of an A row swap where bit 1 of the row is set, so that four rows lie in different banks.  Rows past
// the last are offsets past the descriptor's end, i.e. zeros.
// ------------------------------------------------------------------------------------------------
constexpr int kGradSlabs = 1, kGradGatherA = 2, kGradGatherB = 3;
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ s16x4 lds_read_transposed(uint32_t at) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(uintptr_t)at);
}
// Eight reduction indices of a lane's column: two such reads, four rows (`four` bytes) apart.
__device__ __forceinline__ bf16x8 transposed_fragment(uint32_t at, int four) {
  const s16x4 lo = lds_read_transposed(at), hi = lds_read_transposed(at + four);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// Where a lane's address for such a read lies in a block of 64-column rows (sub-block i of 32 columns: ^ 64 i), from the
// first of eight rows: lane group of 16 = 16 columns and half of the eight rows' pairs, lane in it = row by 4 columns.
__device__ __forceinline__ uint32_t transposed_read_offset(int lane) {
  const uint32_t row = (lane >> 5) * 8 + ((lane & 15) >> 2);
  return row * 128 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8 + ((row >> 1) & 1) * 64;
}

template <bool FP8, int NB, int RW, bool LONE, bool FAR, int GRAD = 0>
struct PingPong {
  static constexpr int kStage = 65536, kB = 32768;
  static constexpr int NB0 = NB < 2 ? NB : 2, NB1 = NB > 2 ? NB - 2 : 0;  // row blocks with valid rows in A0, A1
  static constexpr int I1 = RW == 128 ? 2 : 1;  // requests of A1 per wave
  RowRequests<FP8, 2, 2, FAR> rows;
  i32x4 rb;
  uint32_t b_voff;
  uint32_t a_lds[2], b_soff;  // offsets of the first KiB this wave requests: of A0 and A1, of B0 (B1: 4 KiB further)
  uint32_t lds;            // LDS address of the stages
  const unsigned char *smem;
  int a_rd, b_rd;  // this lane's row / operand in a stage
  bf16x8 fa[2][2][4], fb[2][4];
  const unsigned char *slab_a, *slab_b;  // kGradSlabs: slab 0 of this workgroup's columns
  size_t step_a, step_b;
  uint32_t va[2][2], vb[2][2];           // this lane's offsets in them, by region and instruction
  // kGradGather*
  i32x4 gathered;              // the gathered matrix
  const unsigned char *next;   // the other operand: row 0, and the bytes from there to the end of its last row
  uint32_t next_bytes, pitch;
  uint32_t tab;                // LDS address of the table at this lane's row of instruction 0
  uint32_t col, col_next;      // gathered operand: this lane's byte in a row; the other: in a slab (region 0, instruction 0)
  uint32_t row[2];             // gathered operand: offsets of this lane's rows of the slab being requested

  __device__ __forceinline__ void find_rows(int kt) {  // instruction 1: 8 (B: 16) rows further
    const uint32_t at = tab + kt * 256;
    row[0] = *(const __attribute__((address_space(3))) uint32_t *)(uintptr_t)at;
    row[1] = *(const __attribute__((address_space(3))) uint32_t *)(uintptr_t)(at + (GRAD == kGradGatherA ? 32 : 64));
  }
  // region h of A or j of B, `wide` bytes of a row
  __device__ __forceinline__ void request_gathered(int region, int wide, uint32_t l) const {
    load_to_lds(gathered, l, row[0] + col + region * wide, 0);
    load_to_lds(gathered, l + 1024, row[1] + col + region * wide, 0);
  }
  __device__ __forceinline__ void request_next(int region, int wide, int rows_on, uint32_t l, int kt) const {
    const uint64_t skip = (uint64_t)kt * 64 * pitch;
    const i32x4 r = lds_load_rsrc(next + skip, skip < next_bytes ? next_bytes - (uint32_t)skip : 0u);
    load_to_lds(r, l, col_next + region * wide, 0);
    load_to_lds(r, l + 1024, col_next + region * wide + rows_on * pitch, 0);
  }

  __device__ __forceinline__ void request_slab(const unsigned char *slab, const uint32_t (&v)[2], uint32_t l) const {
    const i32x4 r = lds_load_rsrc(slab, 0xFFFFFFFFu);
    load_to_lds(r, l, v[0], 0);
    load_to_lds(r, l + 1024, v[1], 0);
  }
  __device__ __forceinline__ void request_a(int h, int kt) const {
    const uint32_t l = lds + (kt & 1) * kStage + a_lds[h];
    if constexpr (GRAD == kGradSlabs) {
      request_slab(slab_a + kt * step_a, va[h], l);
      return;
    }
    if constexpr (GRAD == kGradGatherA) {
      request_gathered(h, 128, l);
      return;
    }
    if constexpr (GRAD == kGradGatherB) {
      request_next(h, 128, 8, l, kt);
      return;
    }
    rows.request(h, 0, l, kt);
    if (h == 0 || I1 == 2) rows.request(h, 1, l + 1024, kt);
  }
  __device__ __forceinline__ void request_b(int j, int kt) const {
    const uint32_t l = lds + (kt & 1) * kStage + kB + b_soff + j * 4096, s = kt * kTileBytes + b_soff + j * 4096;
    if constexpr (GRAD == kGradSlabs) {
      request_slab(slab_b + kt * step_b, vb[j], l);
      return;
    }
    if constexpr (GRAD == kGradGatherA) {
      request_next(j, 64, 16, l, kt);
      return;
    }
    if constexpr (GRAD == kGradGatherB) {
      request_gathered(j, 64, l);
      return;
    }
    load_to_lds<LONE>(rb, l, b_voff, s);
    load_to_lds<LONE>(rb, l + 1024, b_voff, s + 1024);
  }
  __device__ __forceinline__ void read_a(int h, int i, int kt) {
    if constexpr (GRAD >= kGradGatherA) {
      const uint32_t s = lds + (kt & 1) * kStage + h * 8192 + (a_rd ^ i * 64);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) fa[h][i][kk] = transposed_fragment(s + kk * 2048, 512);
      return;
    }
    const unsigned char *s = smem + (kt & 1) * kStage + (h * 2 + i) * 4096;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) fa[h][i][kk] = *reinterpret_cast<const bf16x8 *>(s + (a_rd ^ kk * 32));
  }
  __device__ __forceinline__ void read_b(int j, int kt) {
    if constexpr (GRAD >= kGradGatherA) {
      const uint32_t s = lds + (kt & 1) * kStage + j * 4096 + b_rd;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) fb[j][kk] = transposed_fragment(s + kk * 1024, 256);
      return;
    }
    const unsigned char *s = smem + (kt & 1) * kStage + j * 4096;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      fb[j][kk] = *reinterpret_cast<const bf16x8 *>(s + (GRAD ? b_rd ^ kk * 32 : b_rd + kk * 1024));
  }
  template <int H, int J>
  __device__ __forceinline__ void multiply(f32x16 (&acc)[NB][2]) {
    constexpr int n = H == 0 ? NB0 : NB1;
    if constexpr (n > 0) {
      __builtin_amdgcn_s_setprio(1);
      if constexpr (FP8) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int i = 0; i < n; ++i)
            acc[H * 2 + i][J] = mfma_fp8_pair(fa[H][i][2 * p], fa[H][i][2 * p + 1], fb[J][2 * p], fb[J][2 * p + 1],
                                              acc[H * 2 + i][J]);
      } else {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int i = 0; i < n; ++i) acc[H * 2 + i][J] = mfma_bf16(fa[H][i][kk], fb[J][kk], acc[H * 2 + i][J]);
      }
      __builtin_amdgcn_s_setprio(0);
    }
    slot_barrier();
  }
  // LEFT: k-steps behind this one, 2 standing for two or more
  template <int LEFT>
  __device__ __forceinline__ void k_step(f32x16 (&acc)[NB][2], int kt) {
    read_b(0, kt);
    if (LEFT == 2 && GRAD == kGradGatherA) find_rows(kt + 2);
    if (LEFT == 2) request_a(0, kt + 2);
    wait_loads<LEFT == 2 ? 8 + I1 : LEFT == 1 ? 6 + I1 : 0>();
    wait_lds_reads();
    slot_barrier();
    multiply<0, 0>(acc);
    read_b(1, kt);
    if (NB > 2) read_a(1, 0, kt);
    if (LEFT == 2 && GRAD == kGradGatherB) find_rows(kt + 2);
    if (LEFT == 2) request_b(0, kt + 2);
    wait_lds_reads();
    slot_barrier();
    multiply<0, 1>(acc);
    if (NB > 3) read_a(1, 1, kt);
    if (LEFT == 2) request_b(1, kt + 2);
    if (LEFT >= 1) wait_loads<LEFT == 2 ? 10 + I1 : 4 + I1>();
    wait_lds_reads();
    slot_barrier();
    multiply<1, 1>(acc);
    if (LEFT >= 1) {
      read_a(0, 0, kt + 1);
      if (NB > 1) read_a(0, 1, kt + 1);
    }
    if (LEFT == 2) request_a(1, kt + 2);
    if (LEFT >= 1) wait_loads<LEFT == 2 ? 8 + 2 * I1 : 2 + I1>();
    wait_lds_reads();
    slot_barrier();
    multiply<1, 0>(acc);
  }
  // K: reduction length; wm: wave row (scalar)
  __device__ __forceinline__ void run(f32x16 (&acc)[NB][2], int KT, int K, int wm) {
    const bool tail = !GRAD && K % RowRequests<FP8, 2, 2, FAR>::KS != 0;
    auto slab = [&](int kt) {
      if (tail && kt == KT - 1) rows.clip(K, KT - 1);
      if (GRAD >= kGradGatherA) find_rows(kt);
      request_a(0, kt);
      request_b(0, kt);
      request_b(1, kt);
      request_a(1, kt);
    };
    slab(0);
    if (KT > 1) {
      slab(1);
      wait_loads<6 + I1>();
    } else {
      wait_loads<0>();
    }
    slot_barrier();
    read_a(0, 0, 0);
    if (NB > 1) read_a(0, 1, 0);
    wait_lds_reads();
    slot_barrier();
    if (wm == 1) slot_barrier();  // the second row starts one slot later ...
    int kt = 0;
    for (; kt + 2 < KT; ++kt) {
      if (tail && kt + 2 == KT - 1) rows.clip(K, KT - 1);
      k_step<2>(acc, kt);
    }
    if (KT > 1) k_step<1>(acc, kt++);
    k_step<0>(acc, kt);
    if (wm == 0) slot_barrier();  // ... and the first row waits for it at the end
  }
};

// ------------------------------------------------------------------------------------------------
// Tiles of at most 64 rows: bound by the weight stream, so what counts is the bytes a CU keeps in flight.  A ring of
// three stages (RW = 32: 8 KiB of rows and 32 KiB of weights); a k-step reads all its operands into registers first, so
// that the stage is free again and three slabs are on the way while it multiplies.  The wave rows share the rows, RW each,
// so that all four SIMDs have work.  RW = 64, two stages: tiles of 65 to 128 rows in kernels that leave LDS to others on
// their CU.
// ------------------------------------------------------------------------------------------------
template <bool FP8, int NB, int RW, bool LONE>
struct SlabRing {
  static constexpr int kA = RW * 2 * 128, kStage = kA + kTileBytes, kStages = RW == 64 ? 2 : 3;
  static constexpr int kRowLoads = RW / 32;                  // KiB of rows each wave requests per slab
  static constexpr int kLoads = kRowLoads + 4;
  RowRequests<FP8, 1, kRowLoads, false> rows;
  i32x4 rb;
  uint32_t b_voff, a_lds, b_soff, lds;
  const unsigned char *smem;
  int a_rd, b_rd;

  __device__ __forceinline__ void request(int stage, int kt) const {
    const uint32_t l = lds + stage * kStage;
#pragma unroll
    for (int i = 0; i < 4; ++i) load_to_lds<LONE>(rb, l + kA + b_soff + i * 1024, b_voff, kt * kTileBytes + b_soff + i * 1024);
#pragma unroll
    for (int i = 0; i < kRowLoads; ++i) rows.request(0, i, l + a_lds + i * 1024, kt);
  }
  __device__ __forceinline__ void run(f32x16 (&acc)[NB > 0 ? NB : 1][2], int KT, int K) {
    const bool tail = K % RowRequests<FP8, 1, kRowLoads, false>::KS != 0;
    auto ask = [&](int stage, int kt) {
      if (tail && kt == KT - 1) rows.clip(K, KT - 1);
      request(stage, kt);
    };
#pragma unroll
    for (int i = 0; i < kStages; ++i)
      if (i < KT) ask(i, i);
    int stage = 0;
    for (int kt = 0; kt < KT; ++kt) {
      // slab kt is here (this wave's part; the barrier: everybody's)
      if (kStages > 2 && kt + 2 < KT) wait_loads<2 * kLoads>();
      else if (kt + 1 < KT) wait_loads<kLoads>();
      else wait_loads<0>();
      slot_barrier();
      bf16x8 fa[NB > 0 ? NB : 1][4], fb[2][4];
      if constexpr (NB > 0) {
        const unsigned char *sa = smem + stage * kStage, *sb = smem + stage * kStage + kA + b_rd;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
          for (int j = 0; j < 2; ++j) fb[j][kk] = *reinterpret_cast<const bf16x8 *>(sb + j * 4096 + kk * 1024);
#pragma unroll
          for (int i = 0; i < NB; ++i)
            fa[i][kk] = *reinterpret_cast<const bf16x8 *>(sa + i * 4096 + (a_rd ^ kk * 32));
        }
      }
      // everybody has read it: its stage takes the slab kStages steps on
      wait_lds_reads();
      slot_barrier();
      if (kt + kStages < KT) ask(stage, kt + kStages);
      if constexpr (NB > 0) {
        if constexpr (FP8) {
#pragma unroll
          for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j)
                acc[i][j] = mfma_fp8_pair(fa[i][2 * p], fa[i][2 * p + 1], fb[j][2 * p], fb[j][2 * p + 1], acc[i][j]);
        } else {
#pragma unroll
          for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j) acc[i][j] = mfma_bf16(fa[i][kk], fb[j][kk], acc[i][j]);
        }
      }
      stage = stage == kStages - 1 ? 0 : stage + 1;
    }
  }
};

// ------------------------------------------------------------------------------------------------
// Tiles of 65 to 128 rows: a ring of three stages (16 KiB of rows and 32 KiB of weights), one barrier per k-step, in the
// middle of its matrix instructions.
// What bounds it: the weight stream, as long as a k-step's 1024 cycles of fragment reads (128 KiB) run under its 1024
// cycles of matrix instructions.  A wave reads slab kt, multiplies the first half as it arrives, and meets the others when
// everybody has read slab kt and its share of slab kt + 1 is here; slab kt + 3 then goes to the stage of slab kt, and the
// second half runs under the reads of slab kt + 1.
// Measured, about 100 rows per expert, against reading everything, a second barrier, then multiplying: 3200 tokens on 8 of
// 256 experts of 7168 x 2048 195 -> 180 us, 200 tokens on 8 of 16 experts of 2880 x 2880 149 -> 136 us, 100 tokens on 8
// experts of 4096 x 1536 130 -> 119 us, FP8 140 -> 136, 104 -> 101 and 91 -> 85 us (the barrier in front of the reads: 188,
// 137 and 122 us).  At 64 rows and less (SlabRing) the slabs on the way count for more.
// ------------------------------------------------------------------------------------------------
template <bool FP8, int NB, bool LONE>
struct FlowRing {
  static constexpr int kA = 128 * 128, kStage = kA + kTileBytes, kStages = 3, kRowLoads = 2, kLoads = kRowLoads + 4;
  RowRequests<FP8, 1, kRowLoads, false> rows;
  i32x4 rb;
  uint32_t b_voff, a_lds, b_soff, lds;
  const unsigned char *smem;
  int a_rd, b_rd;

  __device__ __forceinline__ void run(f32x16 (&acc)[NB][2], int KT, int K) {
    const bool tail = K % RowRequests<FP8, 1, kRowLoads, false>::KS != 0;
    auto ask = [&](int stage, int kt) {
      if (tail && kt == KT - 1) rows.clip(K, KT - 1);
      const uint32_t l = lds + stage * kStage;
#pragma unroll
      for (int i = 0; i < 4; ++i) load_to_lds<LONE>(rb, l + kA + b_soff + i * 1024, b_voff, kt * kTileBytes + b_soff + i * 1024);
#pragma unroll
      for (int i = 0; i < kRowLoads; ++i) rows.request(0, i, l + a_lds + i * 1024, kt);
    };
#pragma unroll
    for (int i = 0; i < kStages; ++i)
      if (i < KT) ask(i, i);
    if (KT > 2) wait_loads<2 * kLoads>(); else if (KT > 1) wait_loads<kLoads>(); else wait_loads<0>();
    slot_barrier();
    int stage = 0;
    for (int kt = 0; kt < KT; ++kt) {
      bf16x8 fa[NB][4], fb[2][4];
      const unsigned char *sa = smem + stage * kStage, *sb = smem + stage * kStage + kA + b_rd;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
        for (int j = 0; j < 2; ++j) fb[j][kk] = *reinterpret_cast<const bf16x8 *>(sb + j * 4096 + kk * 1024);
#pragma unroll
        for (int i = 0; i < NB; ++i) fa[i][kk] = *reinterpret_cast<const bf16x8 *>(sa + i * 4096 + (a_rd ^ kk * 32));
      }
      __builtin_amdgcn_sched_barrier(0);
      auto multiply = [&](int half) {
        if constexpr (FP8) {
#pragma unroll
          for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = mfma_fp8_pair(fa[i][2 * half], fa[i][2 * half + 1], fb[j][2 * half], fb[j][2 * half + 1], acc[i][j]);
        } else {
#pragma unroll
          for (int kk = 2 * half; kk < 2 * half + 2; ++kk)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j) acc[i][j] = mfma_bf16(fa[i][kk], fb[j][kk], acc[i][j]);
        }
      };
      multiply(0);
      __builtin_amdgcn_sched_barrier(0);
      wait_lds_reads();
      if (kt + 2 < KT) wait_loads<kLoads>(); else wait_loads<0>();
      slot_barrier();
      if (kt + kStages < KT) ask(stage, kt + kStages);
      multiply(1);
      stage = stage == kStages - 1 ? 0 : stage + 1;
    }
  }
};

}  // namespace moe355
