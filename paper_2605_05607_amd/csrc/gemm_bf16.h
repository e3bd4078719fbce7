// Grouped GEMMs on the matrix cores: tile, work item, the per-item kernels and the resident kernel, for bf16
// operands and (template flag FP8) for E4M3 operands.
#pragma once
#include <type_traits>

#include "combine_kernels.h"
#include "forward_types.h"
#include "gemm_pingpong.h"

namespace moe355 {

// ------------------------------------------------------------------------------------------------
// Grouped bf16 GEMM on the matrix cores.  C[rows of one expert tile, kBN/2 or kBN columns] = A * W_e.
//   A rows   : row_map == nullptr -> A[m0 + r, :]; else A[row_map[m0 + r], :] (token gather of Dispatch).
//   B tiles  : packed in operand order (pack_kernels.h), streamed linearly into the LDS and read linearly from it.
//   GATED    : epilogue h = silu(g) * u, written as bf16   (GEMM-1)
//   !GATED   : epilogue o = acc * row_w[row], written fp32 (GEMM-2, gate weight of Sec. III-C)
// Tile 256 x 256 x 64, one workgroup of 512 threads (8 waves = 2 rows x 4 columns) per CU.  Every operand byte enters the
// CU once (memory -> LDS) because the L2 -> CU path saturates soon on this chip.  RW = rows of a wave row (32 .. 128): the
// tile's 32-row blocks are split evenly over the two wave rows; NB = the blocks of this wave that hold valid rows (the
// others are skipped).  The main loops are in gemm_pingpong.h; this function sets up the operands and runs the epilogue.
// ------------------------------------------------------------------------------------------------

constexpr int kGemmThreads = 512;

// s_waitcnt immediate of the gfx9 encoding (gfx950 included) for "vmcnt(0)": the vector-memory counter at zero (bits
// 3:0 and 15:14), the export and LDS/scalar counters left at their maxima (bits 6:4 = 7, bits 11:8 = 15).  Used where
// a wait has to be spelled out around the device-scope hand-over of the resident kernel (see gemm_bf16_drain); any
// other instruction set encodes the counters differently, so the build is pinned to the target the waits were
// written for.
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "the explicit s_waitcnt encodings of the hand-over are written for gfx950"
#endif
constexpr int kWaitVmcnt0 = 0x0F70;
constexpr int kGemmLds = 3 * (kBM / 2 * kBK * 2 + kTileBytes);  // 144 KiB: the ring of the 128-row tiles (two 64 KiB stages
                                                                // and the epilogues take less)
constexpr int kGemmLdsBeside = 2 * 65536;  // the same with a ring of two stages there: the two stages of the full tiles
constexpr int kPatchBytes = 32 * 288;                     // per-wave epilogue patch (fits 8 x in the stages)

// Sixteen bytes past the L2 of this XCD, at a byte offset from `base` (a store of device scope, sc1): visible to the other
// XCDs as soon as it is acknowledged.  (Against two 8-byte stores the forward call is level: 328.6 and 329.8 us for 8192 tokens on
// 16 of 128 experts of 4096 x 1536, 685.5 and 686.0 for 4096 with a skewed load on 32 of 256 of 7168 x 2048.)
constexpr int kDeviceScope = 16;  // the sc1 bit in the cache policy of a buffer instruction
__device__ __forceinline__ void store_through(void *base, uint32_t at, const unsigned char *from) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0xFFFFFFFFu, 0x00027000);
  __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4 *>(from), r, at, 0, kDeviceScope);
}

__device__ __forceinline__ bool first_thread(int wave) { return wave == 0 && fresh_lane() == 0; }

// FP8: A and the packed B hold E4M3 codes; a k-step then covers 128 reduction indices in the same 128 bytes per row,
// so the slabs, the LDS image and the fragment reads are byte for byte those of the bf16 tile.  The scales
// (g.a_scale per token, g.b_scale per expert and output column, g.h_scale per expert) are applied in the epilogues
// and GEMM-1 writes h as codes.
// TRAIN selects the epilogues of the training path (bf16 only):
//   GATED  : as GEMM-1, and g and u are kept as well (g.aux = gu [rows, 2 N] bf16: g, then u) for the backward pass;
//   !GATED : the first GEMM of the backward pass, dh_raw = dy Wd^T (N = f).  With the kept g, u and the gate weight w:
//            dh = w dh_raw, dg = dh u silu'(g), du = dh silu(g)  ->  g.out = dgu [rows, 2 N] bf16 (dg, then du), and
//            g.aux2 = w silu(g) u [rows, N] bf16 (the h operand of the down-projection weight gradient, weight folded in).
template <bool GATED, bool RESIDENT, int NB, int RW, bool FP8, bool TRAIN, bool LONE, bool FAR, bool BESIDE>
__device__ __forceinline__ void gemm_bf16_tile(const GemmArgs &g, unsigned char *smem, int nt, int le, int m0,
                                               int rows, int wave, int poison = 0,
                                               int32_t *tickets = nullptr, int *pre = nullptr) {
  // wave: number of the wave (scalar).  RESIDENT (the kernel that loops over items): the lane is computed anew, so that
  // nothing derived from it counts as loop invariant; hoisting those values across items costs more registers than the
  // tile has to spare.
  const int lane = RESIDENT ? fresh_lane() : threadIdx.x & 63;
  const int w8 = wave, wm = wave >> 2, wn = wave & 3;

  f32x16 acc[NB > 0 ? NB : 1][2];
#pragma unroll
  for (int mi = 0; mi < NB; ++mi)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][j][r] = 0.f;

  const int l31 = lane & 31, khalf = lane >> 5;
  // Weight tiles of a streaming item (at most 64 rows), and of any item that is its expert's only M tile (LONE), are
  // read once by one workgroup: requested with the non-temporal hint so that they do not push the operands that other
  // tiles share out of the L2.
  typename std::conditional<
      (RW > 64), PingPong<FP8, (NB > 0 ? NB : 1), RW, LONE, FAR>,
      typename std::conditional<RW == 64 && !BESIDE, FlowRing<FP8, (NB > 0 ? NB : 1), LONE>,
                                SlabRing<FP8, NB, (RW > 64 ? 64 : RW), LONE || RW == 32>>::type>::type loop;
  loop.rows.init(g.A, g.lda, (uint32_t)poison - 1u);  // (a wait that gave up: nothing of an incomplete h is read)
  loop.rb = lds_load_rsrc(static_cast<const unsigned char *>(g.Bp) + ((size_t)(le * g.n_ntiles + nt) * g.n_ktiles) * kTileBytes,
                          (uint32_t)g.n_ktiles * kTileBytes);
  loop.lds = lds_address(smem);
  loop.smem = smem;
  // LDS -> operand addressing: lane l reads row l & 31 of a 32-row block, k half l >> 5
  loop.a_rd = row_read_offset(wm * RW + l31, lane);
  loop.b_rd = wn * 8192 + lane * 16;
  loop.b_voff = lane * 16;
  const auto a_row = [&](int row) {  // row of the matrix behind row `row` of the tile (padding: the last valid one)
    const int r = m0 + min(row, rows - 1);
    return (uint32_t)(g.row_map ? g.row_map[r] : r);
  };
  if constexpr (RW > 64) {
    typedef PingPong<FP8, 1, RW, false, FAR> PP;
    loop.b_rd += PP::kB;
    loop.b_soff = (wave >> 1) * 8192 + (wave & 1) * 2048;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = h == 0 ? 2 : PP::I1;  // requests of eight rows: wave's share of its wave row's A0 or A1
      const int row0 = (wave >> 2) * RW + h * 64 + (wave & 3) * 8 * n;
      loop.a_lds[h] = row0 * 128;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (i < n) {
          const int row = row0 + i * 8 + (lane >> 3);
          loop.rows.set(h, i, row, a_row(row), lane);
        }
    }
    loop.run(acc, g.n_ktiles, g.K, wave >> 2);
  } else {
    constexpr int n = RW / 32;
    loop.a_lds = wave * n * 1024;
    loop.b_soff = wave * 4096;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const int row = (wave * n + i) * 8 + (lane >> 3);
      loop.rows.set(0, i, row, a_row(row), lane);
    }
    loop.run(acc, g.n_ktiles, g.K);
  }

  // ---- epilogue ----
  // Accumulator register r of lane l holds C[8*(r/4) + 4*(l/32) + r%4][l%32] of its 32x32 block, i.e. a lane
  // owns one column.  Each wave turns its blocks around through a private LDS patch (the stages are dead now)
  // so that the global stores are 16 bytes per lane along a row instead of one element per lane.
  __syncthreads();  // every wave has finished reading the stages
  // RESIDENT: the ticket of this workgroup's next item is drawn now, by thread 0, so that the atomic's round trip
  // runs under the epilogue instead of in front of the next item; the value is parked in the LDS at the very end.
  int pre_v = -1;
  if (RESIDENT && first_thread(wave)) pre_v = atomicAdd(&tickets[((blockIdx.x + pre[1]) & 7) * kTicketStride], 1);
  unsigned char *patch = smem + w8 * kPatchBytes;
  // GEMM-2: the gate weights and the sole-slot marks of this wave's 128 rows come in once, coalesced, and wait in the
  // LDS behind the patches (1 KiB per wave), instead of 24 scattered loads in front of every 32-row block
  float *meta_w = reinterpret_cast<float *>(smem + 8 * kPatchBytes + w8 * 1024);
  int *meta_s = reinterpret_cast<int *>(meta_w + 128);
  if (!GATED && !TRAIN && NB > 0) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int row_l = wm * RW + hh * 64 + lane;
      meta_w[hh * 64 + lane] = row_l < rows ? (g.row_w ? g.row_w[m0 + row_l] : 1.f) : 0.f;
      meta_s[hh * 64 + lane] = (g.row_sole && row_l < rows) ? g.row_sole[m0 + row_l] : -1;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if (!GATED && TRAIN && NB > 0) {
    // first backward GEMM: the gate weights of this wave's rows, parked behind the wave's three blocks (which take
    // 13824 of its 16 KiB)
    meta_w = reinterpret_cast<float *>(smem + w8 * 16384 + 13824);
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int row_l = wm * RW + hh * 64 + lane;
      meta_w[hh * 64 + lane] = row_l < rows ? g.row_w[m0 + row_l] : 0.f;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if (GATED && FP8 && NB > 0) {
    // FP8 GEMM-1: the same for the scales of the tokens behind this wave's rows (rows past the end repeat the last)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int row_l = min(wm * RW + hh * 64 + lane, rows - 1);
      meta_w[hh * 64 + lane] = g.a_scale[g.row_map ? g.row_map[m0 + row_l] : m0 + row_l];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // FP8: the scales of this lane's columns, read once (inside the loop over the blocks the compiler would have to
  // read them again behind every global store).  GEMM-1: scale of the gate and of the up column of h column col_h
  // and the expert's scale of h; GEMM-2: the expert's scale of h times the scales of the lane's two output columns.
  float f8_s0 = 1.f, f8_s1 = 1.f, f8_sh = 1.f;
  if (FP8 && GATED && NB > 0) {
    const int col_h = nt * (kBN / 2) + wn * 32 + l31;
    const float *bs = g.b_scale + (size_t)le * 2 * g.N;
    f8_s0 = col_h < g.N ? bs[col_h] : 0.f;
    f8_s1 = col_h < g.N ? bs[g.N + col_h] : 0.f;
    f8_sh = g.h_scale[le];
  }
  if (FP8 && !GATED && NB > 0) {
    const int c0 = nt * kBN + wn * 64 + l31;
    const float sh = g.h_scale[le];
    f8_s0 = c0 < g.N ? sh * g.b_scale[(size_t)le * g.N + c0] : 0.f;
    f8_s1 = c0 + 32 < g.N ? sh * g.b_scale[(size_t)le * g.N + c0 + 32] : 0.f;
  }
#pragma unroll
  for (int mi = 0; mi < NB; ++mi) {
    const int blk_row0 = wm * RW + mi * 32;  // first tile row of this 32-row block
    if (!GATED && TRAIN) {
      // This wave's 32 x 64 block of g and of u comes in through the LDS in 16-byte pieces (row pitch 144 bytes, g
      // at 0, u at 4608 of a private 16 KiB region: the stages are dead), every lane replaces the elements it holds
      // accumulators for by dg and du in place and puts w silu(g) u into a third block at 9216, and the three
      // blocks leave in 16-byte pieces.
      unsigned char *blk = smem + w8 * 16384;
      const bf16_t *gu = static_cast<const bf16_t *>(g.aux);
      bf16_t *dgu = static_cast<bf16_t *>(g.out), *hw = static_cast<bf16_t *>(g.aux2);
      const int col0 = nt * kBN + wn * 64;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int c = it * 64 + lane;  // 16-byte chunk: 8 chunks per row
        const int rl = c >> 3, cc = c & 7;
        const int row_l = blk_row0 + rl, col = col0 + cc * 8;
        if (row_l < rows && col < g.N) {
          const bf16_t *src = gu + (size_t)(m0 + row_l) * 2 * g.N + col;
          *reinterpret_cast<u32x4 *>(blk + rl * 144 + cc * 16) = *reinterpret_cast<const u32x4 *>(src);
          *reinterpret_cast<u32x4 *>(blk + 4608 + rl * 144 + cc * 16) = *reinterpret_cast<const u32x4 *>(src + g.N);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // gate weights of the 16 rows this lane holds accumulators for (rows past the end: 0, the math stays finite
      // and nothing of them is stored)
      float wv[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 w4 = *reinterpret_cast<const f32x4 *>(meta_w + mi * 32 + q * 8 + khalf * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) wv[q * 4 + e] = w4[e];
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        // all reads of this half first, then the arithmetic, then all writes: the LDS operations of one kind go
        // out back to back instead of waiting on one another
        const int cb = (j * 32 + l31) * 2;
        float gv[16], uv[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
          gv[r] = (float)*reinterpret_cast<const bf16_t *>(blk + rl * 144 + cb);
          uv[r] = (float)*reinterpret_cast<const bf16_t *>(blk + 4608 + rl * 144 + cb);
        }
        bf16_t o_dg[16], o_du[16], o_hw[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-gv[r])), silu = gv[r] * sg;
          const float dh = wv[r] * acc[mi][j][r];
          o_dg[r] = (bf16_t)(dh * uv[r] * (sg * (1.0f + gv[r] * (1.0f - sg))));
          o_du[r] = (bf16_t)(dh * silu);
          o_hw[r] = (bf16_t)(wv[r] * silu * uv[r]);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
          *reinterpret_cast<bf16_t *>(blk + rl * 144 + cb) = o_dg[r];
          *reinterpret_cast<bf16_t *>(blk + 4608 + rl * 144 + cb) = o_du[r];
          *reinterpret_cast<bf16_t *>(blk + 9216 + rl * 144 + cb) = o_hw[r];
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int c = it * 64 + lane;
        const int rl = c >> 3, cc = c & 7;
        const int row_l = blk_row0 + rl, col = col0 + cc * 8;
        if (row_l < rows && col < g.N) {
          bf16_t *dst = dgu + (size_t)(m0 + row_l) * 2 * g.N + col;
          if (RESIDENT && !FAR) {  // other workgroups' second GEMM reads them in this launch
            const uint32_t at = ((uint32_t)(m0 + row_l) * 2 * g.N + col) * 2;
            store_through(dgu, at, blk + rl * 144 + cc * 16);
            store_through(dgu, at + g.N * 2, blk + 4608 + rl * 144 + cc * 16);
          } else {
            *reinterpret_cast<u32x4 *>(dst) = *reinterpret_cast<const u32x4 *>(blk + rl * 144 + cc * 16);
            *reinterpret_cast<u32x4 *>(dst + g.N) = *reinterpret_cast<const u32x4 *>(blk + 4608 + rl * 144 + cc * 16);
          }
          *reinterpret_cast<u32x4 *>(hw + (size_t)(m0 + row_l) * g.N + col) =
              *reinterpret_cast<const u32x4 *>(blk + 9216 + rl * 144 + cc * 16);
        }
      }
    } else if (GATED && FP8) {
      // h block: 32 rows x 32 columns of E4M3 codes, row pitch 48 bytes.  g and u get the scales of their token
      // and of their columns; h = silu(g) * u is divided by the expert's scale for h and converted.
      const float sg = f8_s0, su = f8_s1, rsh = __builtin_amdgcn_rcpf(f8_sh);
      f32x4 sx4[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) sx4[q] = *reinterpret_cast<const f32x4 *>(meta_w + mi * 32 + q * 8 + khalf * 4);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
        const float sx = sx4[r >> 2][r & 3];
        const float gv = acc[mi][0][r] * (sx * sg), uv = acc[mi][1][r] * (sx * su);
        patch[rl * 48 + l31] = to_e4m3((gv * __builtin_amdgcn_rcpf(1.0f + __expf(-gv))) * uv * rsh);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int ln = RESIDENT ? fresh_lane() : lane;
      const int rl = ln >> 1, cc = ln & 1;  // 16-byte chunk: 2 chunks per row
      const int row_l = blk_row0 + rl;
      const int col = nt * (kBN / 2) + wn * 32 + cc * 16;
      if (row_l < rows && col < g.N) {
        if (RESIDENT)
          store_through(g.out, (uint32_t)(m0 + row_l) * g.ldo + col, patch + rl * 48 + cc * 16);
        else
          *reinterpret_cast<u32x4 *>(static_cast<uint8_t *>(g.out) + (size_t)(m0 + row_l) * g.ldo + col) =
              *reinterpret_cast<const u32x4 *>(patch + rl * 48 + cc * 16);
      }
    } else if (GATED) {
      // h block: 32 rows x 32 columns bf16, row pitch 80 bytes (keeps the two half-waves on different banks);
      // TRAIN: two more such blocks for g and u, 2560 bytes apart
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
        const float gv = acc[mi][0][r], uv = acc[mi][1][r];
        // (the hardware reciprocal, 1 ulp, instead of the correctly rounded division: h is rounded to bf16 next)
        *reinterpret_cast<bf16_t *>(patch + rl * 80 + l31 * 2) =
            (bf16_t)((gv * __builtin_amdgcn_rcpf(1.0f + __expf(-gv))) * uv);
        if (TRAIN) {
          *reinterpret_cast<bf16_t *>(patch + 2560 + rl * 80 + l31 * 2) = (bf16_t)gv;
          *reinterpret_cast<bf16_t *>(patch + 5120 + rl * 80 + l31 * 2) = (bf16_t)uv;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const int c = it * 64 + (RESIDENT ? fresh_lane() : lane);  // 16-byte chunk: 4 chunks per row
        const int rl = c >> 2, cc = c & 3;
        const int row_l = blk_row0 + rl;
        const int col = nt * (kBN / 2) + wn * 32 + cc * 8;
        if (row_l < rows && col < g.N) {
          if (RESIDENT && !FAR)
            store_through(g.out, ((uint32_t)(m0 + row_l) * g.ldo + col) * 2, patch + rl * 80 + cc * 16);
          else
            *reinterpret_cast<u32x4 *>(static_cast<bf16_t *>(g.out) + (size_t)(m0 + row_l) * g.ldo + col) =
                *reinterpret_cast<const u32x4 *>(patch + rl * 80 + cc * 16);
          if (TRAIN) {
            bf16_t *gu = static_cast<bf16_t *>(g.aux) + (size_t)(m0 + row_l) * 2 * g.N + col;
            *reinterpret_cast<u32x4 *>(gu) = *reinterpret_cast<const u32x4 *>(patch + 2560 + rl * 80 + cc * 16);
            *reinterpret_cast<u32x4 *>(gu + g.N) = *reinterpret_cast<const u32x4 *>(patch + 5120 + rl * 80 + cc * 16);
          }
        }
      }
    } else {
      // o block: 32 rows x 64 columns fp32, row pitch 288 bytes.  A row whose token has no other local slot
      // is final already (the Combine sum would have one term): it goes to y in the output type, skipping o.
      // FP8: the scale of the expert's h times the scale of the lane's two output columns
      const float cs0 = f8_s0, cs1 = f8_s1;
      int sole[8];
#pragma unroll
      for (int it = 0; it < 8; ++it) sole[it] = meta_s[mi * 32 + it * 4 + (lane >> 4)];
      f32x4 w4[4];  // gate weights of the 16 rows this lane holds accumulators for (0 past the end)
#pragma unroll
      for (int q = 0; q < 4; ++q) w4[q] = *reinterpret_cast<const f32x4 *>(meta_w + mi * 32 + q * 8 + khalf * 4);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
        float wgt = w4[r >> 2][r & 3];
        if (poison) wgt = __builtin_nanf("");  // the wait for this item's h gave up: mark what it writes
        *reinterpret_cast<float *>(patch + rl * 288 + l31 * 4) = FP8 ? acc[mi][0][r] * cs0 * wgt : acc[mi][0][r] * wgt;
        *reinterpret_cast<float *>(patch + rl * 288 + 128 + l31 * 4) =
            FP8 ? acc[mi][1][r] * cs1 * wgt : acc[mi][1][r] * wgt;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int rl = it * 4 + (lane >> 4), cc = lane & 15;  // 16 chunks of 16 bytes per row
        const int row_l = blk_row0 + rl;
        const int col = nt * kBN + wn * 64 + cc * 4;
        const f32x4 v = *reinterpret_cast<const f32x4 *>(patch + rl * 288 + cc * 16);
        if (row_l < rows && col < g.N) {
          if (sole[it] >= 0) {
            bf16x4 b;
#pragma unroll
            for (int q = 0; q < 4; ++q) b[q] = (bf16_t)(v[q] + 0.0f);  // + 0 as in the sum that starts from zero
            // (y is not read again by this launch: streamed past the L2, which the operands need)
            __builtin_nontemporal_store(
                b, reinterpret_cast<bf16x4 *>(static_cast<bf16_t *>(g.y) + (size_t)sole[it] * g.ldo + col));
          }
          if (sole[it] < 0 || g.keep_rows) {
            *reinterpret_cast<f32x4 *>(static_cast<float *>(g.out) + (size_t)(m0 + row_l) * g.ldo + col) = v;
          }
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // the patch is reused by the next block
  }
  if (RESIDENT && first_thread(wave)) pre[0] = pre_v;
}

// One work item on the matrix cores.  Wave-uniform dispatch on the number of valid 32-row blocks: every variant
// executes the same sequence of barriers.  poison = 1 (GEMM-2 inside the resident kernel, after a wait that gave up):
// the rows are written as NaN.  FAR (an A matrix of 4 GiB or more): one tile shape with 64-bit addresses for every item,
// padding rows multiplied and not stored; kernels of its own, because beside the other variants it costs every kernel
// registers (the resident ones spilled up to 174).  RESIDENT: tickets = the queues' counters, pre = (ticket drawn ahead,
// queues tried so far).
template <bool GATED, bool RESIDENT, bool FP8, bool TRAIN, bool FAR, bool BESIDE>
__device__ __forceinline__ void gemm_bf16_item(const GemmArgs &g, unsigned char *smem, const int4 item, int wave,
                                               int poison = 0, int32_t *tickets = nullptr, int *pre = nullptr) {
  const int le = item.x, m0 = item.y, rows = item.z & kItemRowsMask, nt = item.w & ((1 << kTileShift) - 1);
  // the expert's only M tile (uniform).  Only the resident kernels, which run the layers made of such tiles, have
  // the variants with streaming weight loads: in the per-item kernels they cost six more registers, which the BESIDE ones
  // do not have.
  const bool lone = (item.z & kItemLone) != 0;
  const int nblk = (rows + 31) >> 5;                                     // 1..8 blocks of 32 rows
  const int wm = wave >> 2;                                              // wave row
  const int per_row = (nblk + 1) >> 1;                                   // blocks per wave row
  const int nb = max(0, min(per_row, nblk - per_row * wm));              // those of this wave that hold rows
#define MOE355_TILE_(NB_, RW_, LONE_)                                                                                 \
  gemm_bf16_tile<GATED, RESIDENT, NB_, RW_, FP8, TRAIN, LONE_, FAR, BESIDE>(g, smem, nt, le, m0, rows, wave, poison, \
                                                                            tickets, pre)
#define MOE355_TILE(NB_, RW_)                                                                                       \
  do {                                                                                                              \
    if (RESIDENT && RW_ > 32 && lone) MOE355_TILE_(NB_, RW_, (RESIDENT && RW_ > 32)); else MOE355_TILE_(NB_, RW_, false); \
  } while (0)
  if constexpr (FAR) {
    MOE355_TILE_(4, 128, false);
  } else if (nblk <= 2) {
    if (nb == 1) MOE355_TILE(1, 32); else MOE355_TILE(0, 32);
  } else if (nblk <= 4) {
    if (nb == 2) MOE355_TILE(2, 64); else MOE355_TILE(1, 64);  // (the second wave row holds at most one block less)
  } else if (nblk <= 6) {
    if (nb == 3) MOE355_TILE(3, 96); else MOE355_TILE(2, 96);
  } else {
    if (nb == 4) MOE355_TILE(4, 128); else MOE355_TILE(3, 128);
  }
#undef MOE355_TILE
#undef MOE355_TILE_
}

// One workgroup per work item; workgroup -> item by chunked_item.  BESIDE: the GEMMs of the backward pass, which share
// their CU with the operand transposes on the side stream: 248 registers (a SIMD has 512: 16 are left beside the two waves
// of the workgroup) and 128 KiB of LDS.
template <bool GATED, bool FP8 = false, bool TRAIN = false, bool FAR = false, bool BESIDE = false>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_bf16_kernel(const GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // kGemmLds, BESIDE: kGemmLdsBeside
  const int q = chunked_item(blockIdx.x, *g.n_items);
  if (q < 0) return;
  gemm_bf16_item<GATED, false, FP8, TRAIN, FAR, BESIDE>(g, smem, g.work[q], __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// ------------------------------------------------------------------------------------------------
// GEMM-1 and GEMM-2 of a layer in ONE launch of resident workgroups (one per CU), the one-GPU form of the
// tile-granular GEMM-1 => GEMM-2 hand-over of the fused kernel (Sec. IV-A, IV-B): a GEMM-2 tile starts as soon
// as the h rows of its M tile are complete, so the CUs that run out of GEMM-1 work (a launch of a few hundred
// tiles of ~100 us ends with many CUs idle) continue with GEMM-2 instead of waiting for a kernel boundary.
// moe_fused_forward uses it for bf16 layers whose experts get less than one full M tile of rows on average: the
// launches are then dominated by partial tiles and, under skewed routing, by the tail of the few large experts.  With fuller
// experts it depends on the time the launch takes (tile_gemm_launches).  Time of the forward call in one launch over two, by
// rows per expert:
//                                        even load:  50   100   200  |  300   600  2000   skewed:  50   100   200  |  300   600  2000
//   8 of 64 experts of 2048 x 512                   1.10  1.15  1.15 | 1.05  1.05  0.95           1.07  1.08  1.06 | 0.97  0.99  0.98
//   16 of 128 experts of 4096 x 1536                1.03  0.92  0.90 | 0.88  0.94  0.97           1.03  0.97  0.84 | 0.88  0.93  0.96
//   32 of 128 experts of 2880 x 2880                1.00  0.94  0.97 | 0.97  0.99  1.00           1.03  0.95  0.93 | 0.92  0.99  1.01
//   8 experts of 4096 x 14336                       0.98  0.93  0.99 | 0.99  1.01  1.00           0.93  0.90  0.95 | 0.95  0.98  0.99
//   32 of 256 experts of 7168 x 2048                1.00  0.91  0.95 | 0.93  0.99  0.99           0.89  0.91  0.93 | 0.94  0.97  0.98
// Where the rule takes one launch from 256 rows on, eight layers of 256 to 2000 rows, even and skewed: bf16 0.83 to 1.03 (median
// 0.97), FP8 0.88 to 1.03 (0.98), the training forward 0.84 to 1.04 (0.97); where it takes two, one launch would be 0.88 to 1.10
// (1.03).  What one launch owes to counters on lines of their own (kTicketStride, kReadyStride): 4096 FP8 tokens on 32 of 256 experts
// of 7168 x 2048 355 -> 331 us, 5003 tokens on 32 of 128 experts of 2880 x 2880 358 -> 339, 8192 on 16 of 128 of 4096 x 1536
// 334 -> 328.
//
// Work distribution: both lists are cut into 8 queues exactly as a plain launch would spread them over the XCDs
// (queue x = virtual blocks x, x + 8, ...; see chunked_item); a workgroup draws tickets from its home queue
// (blockIdx % 8, the XCD it runs on) and, when that is empty, from the others.  It moves on to GEMM-2 only after
// it has seen every GEMM-1 queue empty, i.e. when every GEMM-1 item is already in the hands of a running
// workgroup; GEMM-1 items never wait, so the counter a GEMM-2 item polls is always completed by workgroups that
// make progress: no deadlock for any number of resident workgroups and any placement.
// Hand-over: the producers of an M tile store h past their L2 (device-scope stores), wait for the acknowledgement and
// count themselves in tile_ready; the consumer polls the counter and loads.  The L2s of the XCDs are not coherent with each
// other, but neither a write-back nor an invalidate is needed: an XCD loads a line of h only after the line's M tile has been
// counted in full (rows start on a line of their own, see h_pitch, so no line belongs to two M tiles; a wait that gave up
// loads nothing), and lines of an earlier launch went at the start of this one.  Against one L2 write-back per GEMM-1 item and
// an invalidate per GEMM-2 item: about 5 us per item, forward of 4096 tokens on the skewed 7168 x 2048 layer 715 -> 683 us
// (two launches on the same boxes: 752, 738), 5003 tokens on 32 experts of 2880 x 2880 374 -> 352 us (364, 361).  FAR (h of
// 4 GiB and more) keeps both.
// ------------------------------------------------------------------------------------------------
struct PipelineArgs {
  GemmArgs g1, g2;
  int32_t *tickets;     // [16] x kTicketStride: queues of GEMM-1, then of GEMM-2
  int32_t *tile_ready;  // [M tiles] GEMM-1 items finished per M tile
  int32_t *error;       // set if a wait gave up (cannot happen unless the lists are corrupt)
  int nt1;              // GEMM-1 items per M tile a GEMM-2 item waits for
  int max_polls;        // bound on the polls of one wait (x ~1 us), so that no wave can wait forever
  // Combine stage (gemm_bf16_combine_kernel only)
  int32_t *tile_done;         // [M tiles] GEMM-2 items finished per M tile
  const int32_t *row_tile;    // [P] M tile of each local row
  const int32_t *topk_idx, *inv_perm, *offsets, *header;
  int T, k, e_lo, E_loc, P_cap, nt2, n_mtiles_cap;
};

constexpr int kMaxPolls = 1 << 22;  // default bound: several seconds

// All items of one GEMM that this workgroup can get hold of: home queue first, then the other queues.
// tile_done (GEMM-2 only, may be null): counter per M tile that every finished item of the tile is counted in, for
// the Combine stage that follows in the same launch; s_done: kDoneCap ints of LDS (tiles of the finished items).
constexpr int kDoneCap = 256;
// FIRST: the GEMM whose items are counted (else: the one that waits for them).
template <bool FIRST, bool GATED, bool FP8, bool TRAIN, bool FAR>
__device__ __forceinline__ void gemm_bf16_drain(const GemmArgs &g, unsigned char *smem, int *s_item, int wave,
                                                int32_t *__restrict__ tickets, int32_t *__restrict__ tile_ready,
                                                int32_t *__restrict__ error, int nt1, int max_polls,
                                                int32_t *__restrict__ tile_done = nullptr, int *s_done = nullptr) {
  const int home = blockIdx.x & 7;
  const int n_items = *g.n_items;
  const int n_virtual = (n_items + 8 * kChunk - 1) / (8 * kChunk) * (8 * kChunk);
  // s_item: [0] list position, [1] its wait gave up, [2] ticket drawn ahead (-1: none), [3] queues tried so far, in the
  // order home, home + 1, ...  Written by thread 0; in the LDS because the tile has no register to spare for them.
  // Next list position for this workgroup, or -1 when every queue is empty (thread 0 only).
  // pre >= 0: a ticket of the queue this workgroup is on, drawn ahead under the previous item's epilogue
  auto draw = [&]() {
    int q = -1, pre = s_item[2], qsel = s_item[3];
    while (qsel < 8) {
      const int queue = (home + qsel) & 7;
      const int v = queue + 8 * (pre >= 0 ? pre : atomicAdd(&tickets[queue * kTicketStride], 1));
      pre = -1;
      if (v < n_virtual) {
        if ((q = chunked_item(v, n_items)) >= 0) break;
        continue;  // a virtual block without an item
      }
      // this queue is empty: read all counters at once and go on with the next queue that still has positions
      // (an empty queue stays empty, so every queue is seen empty before the loop ends)
      unsigned open_queues = 0;  // bit i: queue i still has positions
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int t = __hip_atomic_load(&tickets[i * kTicketStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        open_queues |= (unsigned)(i + 8 * t < n_virtual) << i;
      }
      int next = 8;
#pragma unroll
      for (int i = 7; i >= 1; --i) {
        const int s2 = qsel + i;  // candidate position in the visiting order
        if (s2 < 8 && ((open_queues >> ((home + s2) & 7)) & 1u)) next = s2;
      }
      qsel = next;
    }
    s_item[2] = -1;
    s_item[3] = qsel;
    return q;
  };
  // GEMM-2 items that feed Combine in the same launch: the o rows (and the y rows of sole slots) of all items this
  // workgroup has finished become visible device-wide with ONE release, then every item is counted in its M tile's
  // counter.  (A release per item costs an L2 write-back of the fp32 rows each time: measured 4 % of the launch.)
  // Counting late is safe: the items are in the hands of a running workgroup until they are counted.
  int n_pending = 0;  // finished, not yet counted (the same in every thread)
  auto flush_done = [&]() {
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // this wave's stores have been acknowledged
    __syncthreads();
    if (first_thread(wave) && n_pending > 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // the write-back is complete before the counters move
      for (int i = 0; i < n_pending; ++i)
        __hip_atomic_fetch_add(&tile_done[s_done[i]], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    n_pending = 0;
    __syncthreads();  // the list may be overwritten
  };
  // (Drawing the next ticket a whole item ahead, to hide the latency of the atomic, was measured slower: a workgroup
  // that holds a long item while it finishes another one keeps that item from an idle workgroup.  What is drawn
  // ahead here is drawn under the epilogue of the item that is being finished, a few microseconds before it is used.)
  if (first_thread(wave)) {
    s_item[2] = -1;
    s_item[3] = 0;
  }
  for (;;) {
    __syncthreads();  // the previous item is done with the LDS (and with *s_item)
    if (first_thread(wave)) *s_item = draw();
    __syncthreads();
    const int q = __builtin_amdgcn_readfirstlane(*s_item);
    if (q < 0) break;  // nothing left in any queue
    int4 item = g.work[q];  // (the same in every lane: kept in scalar registers)
    item.x = __builtin_amdgcn_readfirstlane(item.x);
    item.y = __builtin_amdgcn_readfirstlane(item.y);
    item.z = __builtin_amdgcn_readfirstlane(item.z);
    item.w = __builtin_amdgcn_readfirstlane(item.w);
    const int tile = item.w >> kTileShift;
    if (FIRST) {
      gemm_bf16_item<GATED, true, FP8, TRAIN, FAR, false>(g, smem, item, wave, 0, tickets, s_item + 2);
      // Release side of the hand-over.  Every wave waits until its own h stores have been acknowledged (a workgroup
      // barrier alone does not wait for global stores); they went past the L2 (store_through), so there is nothing to write back.
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
      __syncthreads();  // every thread's h stores happen before thread 0's count
      if (first_thread(wave)) {
        if constexpr (FAR) {
          // h through the L2: written back with one release.  The write-back has to be complete before the counter moves.
          // The compiler places no wait between the two here (the wave has just waited for its stores, and the write-back
          // is not counted as outstanding), so the wait is spelled out.
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
          __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        }
        __hip_atomic_fetch_add(&tile_ready[(size_t)tile * kReadyStride], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ... then counted
      }
    } else {
      // Acquire side: thread 0 polls with relaxed device-scope loads; the barrier hands the result to the workgroup.  A wait
      // that gives up (corrupt lists; cannot happen otherwise) raises the error word and the
      // item runs with a NaN in place of the gate weight, so that nothing computed from incomplete h can pass as a
      // result.
      if (first_thread(wave)) {
        int polls = 0, gave_up = 0;
        while (__hip_atomic_load(&tile_ready[(size_t)tile * kReadyStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < nt1) {
          __builtin_amdgcn_s_sleep(32);
          if (++polls > max_polls) {
            __hip_atomic_store(error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            gave_up = 1;
            break;
          }
        }
        if constexpr (FAR) {
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // the invalidate is complete before the barrier lets the others load
        }
        s_item[1] = gave_up;
      }
      __syncthreads();
      gemm_bf16_item<false, true, FP8, false, FAR, false>(g, smem, item, wave, __builtin_amdgcn_readfirstlane(s_item[1]),
                                                          tickets, s_item + 2);
      if (tile_done) {
        // remembered, counted later (flush_done): one write-back for all the items of this workgroup
        if (first_thread(wave)) s_done[n_pending] = tile;
        // (every thread counts: a uniform decision.)  Counting every item at once towards the end of the launch, so
        // that idle workgroups can reduce tokens while the last items run, was measured: no gain, the rows of the
        // last items are what the reduction waits for.
        if (++n_pending == kDoneCap) flush_done();
      }
    }
  }
  if (!FIRST && tile_done) flush_done();
}

// ------------------------------------------------------------------------------------------------
// Combine as the last stage of the resident kernel (readiness-gated issue of Sec. IV-C on one GPU): a workgroup
// that has seen every GEMM-2 queue empty turns to the tokens.  One wave per token, tokens dealt round-robin over all
// resident waves.  The wave resolves the token's local slots (one lane per slot), waits until the GEMM-2 items of
// every M tile that holds one of those rows have been counted in tile_done (all of them are in the hands of running
// workgroups by then, so the wait ends), and sums the rows in slot order in fp32, exactly as combine_kernel does:
// bit-identical y.  Tokens with one local slot were written by GEMM-2 itself; tokens with none get zeros.
// Acquire side as in the GEMM-2 wait: relaxed device-scope polls, one acquire fence, then the loads.
// A wait that gives up raises the error word and the token's row is written as NaN.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void resident_combine(const PipelineArgs &p, int wave) {
  const int lane = fresh_lane();
  const int n_waves = gridDim.x * (kGemmThreads / 64);
  const int base = p.offsets[p.e_lo];
  const int P = min(p.header[1], p.P_cap);
  const int d = p.g2.N;
  const float *rows = static_cast<const float *>(p.g2.out);
  bf16_t *y = static_cast<bf16_t *>(p.g2.y);
  for (int t = blockIdx.x * (kGemmThreads / 64) + wave; t < p.T; t += n_waves) {  // t is wave-uniform
    const int row = combine_slot_row(p.topk_idx, p.inv_perm, t, p.k, lane, p.e_lo, p.E_loc, base, P);
    const int tile = row >= 0 ? min(max(p.row_tile[row], 0), p.n_mtiles_cap - 1) : 0;
    const uint64_t slots = __ballot(row >= 0);
    const int n = __popcll(slots);
    if (n == 1) continue;  // GEMM-2 has written this token's row
    bf16_t *yrow = y + (size_t)t * d;
    int poison = 0;
    if (n > 1) {
      int polls = 0;
      for (;;) {
        const bool ok = row < 0 || __hip_atomic_load(&p.tile_done[tile], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= p.nt2;
        if (__ballot(!ok) == 0) break;
        __builtin_amdgcn_s_sleep(32);
        if (++polls > p.max_polls) {
          if (lane == 0) __hip_atomic_store(p.error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          poison = 1;
          break;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    combine_token_rows<bf16_t, true>(rows, row, slots, d, yrow, lane, poison);
  }
}

template <bool FAR>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_bf16_pipeline_kernel(const PipelineArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // kGemmLds
  __shared__ int s_item[4];  // (see gemm_bf16_drain)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  gemm_bf16_drain<true, true, false, false, FAR>(p.g1, smem, s_item, wave, p.tickets, p.tile_ready, p.error, p.nt1, p.max_polls);
  gemm_bf16_drain<false, false, false, false, FAR>(p.g2, smem, s_item, wave, p.tickets + 8 * kTicketStride, p.tile_ready, p.error, p.nt1, p.max_polls);
}

// The resident kernel with Combine as its third stage: the whole layer after the tile table in one launch.
template <bool FAR>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_bf16_combine_kernel(const PipelineArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // kGemmLds
  __shared__ int s_item[4];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  gemm_bf16_drain<true, true, false, false, FAR>(p.g1, smem, s_item, wave, p.tickets, p.tile_ready, p.error, p.nt1, p.max_polls);
  __shared__ int s_done[kDoneCap];
  gemm_bf16_drain<false, false, false, false, FAR>(p.g2, smem, s_item, wave, p.tickets + 8 * kTicketStride, p.tile_ready, p.error, p.nt1, p.max_polls, p.tile_done,
                         s_done);
  resident_combine(p, wave);
}

// The same resident kernel for the training forward: GEMM-1 also keeps g and u.
template <bool FAR>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_train_pipeline_kernel(const PipelineArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // kGemmLds
  __shared__ int s_item[4];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  gemm_bf16_drain<true, true, false, true, FAR>(p.g1, smem, s_item, wave, p.tickets, p.tile_ready, p.error, p.nt1, p.max_polls);
  gemm_bf16_drain<false, false, false, false, FAR>(p.g2, smem, s_item, wave, p.tickets + 8 * kTicketStride, p.tile_ready, p.error, p.nt1, p.max_polls);
}

// The two GEMMs of the backward pass as one resident launch: the rows [dg | du] of the first (which also writes w h) are what
// the second one reads.  Where it is taken, with both forms' times: backward_one_launch.
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_backward_pipeline_kernel(const PipelineArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // kGemmLds
  __shared__ int s_item[4];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  gemm_bf16_drain<true, false, false, true, false>(p.g1, smem, s_item, wave, p.tickets, p.tile_ready, p.error, p.nt1, p.max_polls);
  gemm_bf16_drain<false, false, false, false, false>(p.g2, smem, s_item, wave, p.tickets + 8 * kTicketStride, p.tile_ready, p.error, p.nt1, p.max_polls);
}

// The same resident kernel on E4M3 operands (whose rows number less than 2^32 elements, i.e. bytes).
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_fp8_pipeline_kernel(const PipelineArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // kGemmLds
  __shared__ int s_item[4];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  gemm_bf16_drain<true, true, true, false, false>(p.g1, smem, s_item, wave, p.tickets, p.tile_ready, p.error, p.nt1, p.max_polls);
  gemm_bf16_drain<false, false, true, false, false>(p.g2, smem, s_item, wave, p.tickets + 8 * kTicketStride, p.tile_ready, p.error, p.nt1, p.max_polls);
}

}  // namespace moe355
