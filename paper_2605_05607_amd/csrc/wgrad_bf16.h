// Weight gradients of the expert FFN on the matrix cores: for every local expert, C = A^T B summed over the expert's
// rows (dW_gate = x^T dg, dW_up = x^T du, dW_down = (w h)^T dy).  The reduction index is the row, which is the slow
// index of both operands in memory, while a matrix-core operand wants 8 consecutive reduction indices per lane; so
// the operands are first transposed (and gathered: x and dy rows are fetched by token) into buffers of 64-row blocks,
// [block][column][64 rows], in which every expert's rows start at a block boundary and are zero-padded to one: what
// a workgroup stages per k-step is then one contiguous piece of memory per operand.  The GEMM is the forward tile's
// main loop with both operands staged like its A operand.
#pragma once
#include "gemm_bf16.h"

namespace moe355 {

// kb[le] = first 64-row block of local expert le in the padded row order, kb[E_loc] = number of blocks.
__global__ __launch_bounds__(256) void wgrad_blocks_kernel(const int32_t *__restrict__ offsets,
                                                           const int32_t *__restrict__ header, int e_lo, int E_loc,
                                                           int32_t *__restrict__ kb) {
  __shared__ int scratch[17];
  const int P = header[1], base = header[2];
  const int ipt = (E_loc + 255) / 256;
  const int lo = min(E_loc, (int)threadIdx.x * ipt), hi = min(E_loc, lo + ipt);
  int mine = 0;
  for (int le = lo; le < hi; ++le) {
    const int cnt = max(0, min(P, offsets[e_lo + le + 1] - base) - min(P, offsets[e_lo + le] - base));
    mine += (cnt + 63) >> 6;
  }
  int total;
  int run = block_exclusive_scan(mine, scratch, &total);
  for (int le = lo; le < hi; ++le) {
    const int cnt = max(0, min(P, offsets[e_lo + le + 1] - base) - min(P, offsets[e_lo + le] - base));
    kb[le] = run;
    run += (cnt + 63) >> 6;
  }
  if (threadIdx.x == 0) kb[E_loc] = total;
}

// dst[b][c][i] = src[row(r)][c0 + c] for the i-th row r of padded block b (zero where the block is padded), c < C,
// i < 64.  src rows have pitch ld; row(r) = row_map[r] or r.  grid (ceil(C / 64), block cap).
__global__ __launch_bounds__(256) void gather_transpose_kernel(const bf16_t *__restrict__ src,
                                                               const int32_t *__restrict__ row_map, int ld, int c0,
                                                               int C, const int32_t *__restrict__ offsets,
                                                               const int32_t *__restrict__ header,
                                                               const int32_t *__restrict__ kb, int e_lo, int E_loc,
                                                               bf16_t *__restrict__ dst) {
  __shared__ uint16_t tile[64][66];  // [row][column], 33 words per row: column reads hit distinct banks
  const int b = blockIdx.y;
  if (b >= kb[E_loc]) return;
  int lo = 0, hi = E_loc;  // expert that owns block b: largest le with kb[le] <= b (empty experts own no block)
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (kb[mid] <= b) lo = mid; else hi = mid;
  }
  const int le = lo;
  const int P = header[1], base = header[2];
  const int start = min(P, offsets[e_lo + le] - base);
  const int cnt = max(0, min(P, offsets[e_lo + le + 1] - base) - start);
  const int r_first = (b - kb[le]) * 64;  // first row of this block inside the expert
  const int cblk = blockIdx.x * 64;
  // load: thread t -> rows (t >> 3) and (t >> 3) + 32, 16-byte chunk t & 7
  for (int i = 0; i < 2; ++i) {
    const int rl = (threadIdx.x >> 3) + 32 * i, ch = threadIdx.x & 7;
    u32x4 v = {0u, 0u, 0u, 0u};
    const int c = cblk + ch * 8;
    if (r_first + rl < cnt && c < C) {
      const int r = start + r_first + rl;
      const size_t row = row_map ? (size_t)row_map[r] : (size_t)r;
      v = *reinterpret_cast<const u32x4 *>(src + row * ld + c0 + c);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      tile[rl][ch * 8 + 2 * q] = (uint16_t)(v[q] & 0xFFFFu);
      tile[rl][ch * 8 + 2 * q + 1] = (uint16_t)(v[q] >> 16);
    }
  }
  __syncthreads();
  // store: thread t -> columns (t >> 3) and (t >> 3) + 32, rows 8 (t & 7) .. + 8 as one 16-byte chunk
  for (int i = 0; i < 2; ++i) {
    const int cl = (threadIdx.x >> 3) + 32 * i, ch = threadIdx.x & 7;
    if (cblk + cl >= C) continue;
    u32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      v[q] = (uint32_t)tile[ch * 8 + 2 * q][cl] | ((uint32_t)tile[ch * 8 + 2 * q + 1][cl] << 16);
    *reinterpret_cast<u32x4 *>(dst + ((size_t)b * C + cblk + cl) * 64 + ch * 8) = v;
  }
}

struct WgradArgs {
  const bf16_t *AT;   // [block][lda][64]: rows a0 .. a0 + M of every block are the left operand's columns
  const bf16_t *BT;   // [block][ldb][64]: rows b0 .. b0 + N
  bf16_t *C;          // [E_loc][M][N]
  const int32_t *kb;  // [E_loc + 1]
  int lda, ldb, a0, b0;
  int M, N, n_mt, n_nt;
};

// Experts with at most kThinSteps blocks of 64 rows are left to wgrad_thin_bf16_kernel (those without rows to
// wgrad_zero_empty_kernel): their cost is writing the output, and that kernel's small workgroups overlap the stores of
// one tile with the loads of the next on the same CU.
constexpr int kStageBytes = 2 * kBM * kBK * 2;  // 64 KiB: A slab then B slab
constexpr int kThinSteps = 2;
constexpr int kThinTiles = 4;  // output tiles per workgroup of wgrad_thin_bf16_kernel

// Zero gradients of the local experts without rows: grid (shares, E_loc, 3 matrices), each workgroup clears one
// contiguous share of `units` 16-byte units.  Few registers and no LDS on purpose: its waves fit beside a GEMM
// workgroup on the same CU.
__global__ __launch_bounds__(256) void wgrad_zero_empty_kernel(const int32_t *__restrict__ kb, u32x4 *c0, u32x4 *c1,
                                                               u32x4 *c2, size_t units) {
  const int le = blockIdx.y;
  if (kb[le + 1] != kb[le]) return;
  u32x4 *C = (blockIdx.z == 0 ? c0 : blockIdx.z == 1 ? c1 : c2) + (size_t)le * units;
  const size_t share = (units + gridDim.x - 1) / gridDim.x;
  const size_t u0 = blockIdx.x * share, u1 = u0 + share < units ? u0 + share : units;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  for (size_t u = u0 + threadIdx.x; u < u1; u += 256) __builtin_nontemporal_store(zero, &C[u]);
}

// The gradients are written once and not read again by this library: all three kernels below store them with the
// non-temporal hint, so that 0.9 GB of output per product does not push the operands, which every tile of an expert
// shares, out of the L2s (measured: -9 % of the weight-gradient time on the GPT-OSS-shaped layer, -6.5 % on the
// Mixtral-shaped one, -9 % on the Qwen3-shaped one, -2 % on the DeepSeek-shaped one).
// One workgroup per (local expert, 256 x 256 output tile); 8 waves = 2 x 4, each 128 x 64 as 4 x 2 accumulators.
// LDS: two stages of (A 256 x 64, B 256 x 64), rows of 128 bytes with the forward tile's chunk swizzle; main loop of the
// forward's full tiles (slabs straight into the LDS, wave rows half a step apart) instead of slabs staged through registers
// with all waves in step.  What bounds it is the short reduction (8 k-steps for 512 rows) between a two-slab prologue and the
// store of 128 KiB: training step of 8192 tokens on 16 experts of 4096 x 1536 about 1277 -> 1267 us.
__global__ __launch_bounds__(kGemmThreads, 1) void wgrad_bf16_kernel(const WgradArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, w8 = tid >> 6;
  const int wm = w8 >> 2, wn = w8 & 3;
  const int le = blockIdx.y;
  const int mt = blockIdx.x / a.n_nt, nt = blockIdx.x % a.n_nt;
  const int m0 = mt * kBM, n0 = nt * kBN;
  const int kb0 = a.kb[le], KT = a.kb[le + 1] - kb0;
  if (KT <= kThinSteps) return;  // whole workgroup: the thin kernel owns this expert

  f32x16 acc[4][2];
#pragma unroll
  for (int mi = 0; mi < 4; ++mi)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][j][r] = 0.f;

  const int l31 = lane & 31, khalf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(w8);
  typedef PingPong<false, 4, 128, false, false, true> Loop;
  Loop loop;
  loop.lds = lds_address(smem);
  loop.smem = smem;
  loop.a_rd = row_read_offset(wm * 128 + l31, lane);
  loop.b_rd = Loop::kB + row_read_offset(wn * 64 + l31, lane);
  loop.b_soff = (wave >> 1) * 8192 + (wave & 1) * 2048;
  loop.step_a = (size_t)a.lda * 128;
  loop.step_b = (size_t)a.ldb * 128;
  loop.slab_a = reinterpret_cast<const unsigned char *>(a.AT) + ((size_t)kb0 * a.lda + a.a0 + m0) * 128;
  loop.slab_b = reinterpret_cast<const unsigned char *>(a.BT) + ((size_t)kb0 * a.ldb + a.b0 + n0) * 128;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    // sixteen columns of region h of either operand: eight per instruction, lane = column by 16-byte chunk; columns past
    // the end repeat the last one (not stored)
    const int row_a = (wave >> 2) * 128 + h * 64 + (wave & 3) * 16, row_b = (loop.b_soff >> 7) + h * 32;
    loop.a_lds[h] = row_a * 128;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int ra = row_a + i * 8 + (lane >> 3), rb = row_b + i * 8 + (lane >> 3);
      loop.va[h][i] = min(ra, a.M - 1 - m0) * 128 + ((lane & 7) ^ ((ra >> 1) & 7)) * 16;
      loop.vb[h][i] = min(rb, a.N - 1 - n0) * 128 + ((lane & 7) ^ ((rb >> 1) & 7)) * 16;
    }
  }
  loop.run(acc, KT, KT * kBK, wave >> 2);
  // epilogue: each wave turns its 32 x 64 blocks around through a private LDS patch (fp32, row pitch 288 bytes) so
  // that a row leaves as contiguous bf16
  __syncthreads();
  unsigned char *patch = smem + w8 * kPatchBytes;
  bf16_t *C = a.C + (size_t)le * a.M * a.N;
#pragma unroll
  for (int mi = 0; mi < 4; ++mi) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
      *reinterpret_cast<float *>(patch + rl * 288 + l31 * 4) = acc[mi][0][r];
      *reinterpret_cast<float *>(patch + rl * 288 + 128 + l31 * 4) = acc[mi][1][r];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int rl = it * 8 + (lane >> 3), cc = lane & 7;  // 8 groups of 8 columns per row: 16-byte stores
      const int m = m0 + wm * 128 + mi * 32 + rl, n = n0 + wn * 64 + cc * 8;
      const f32x4 v0 = *reinterpret_cast<const f32x4 *>(patch + rl * 288 + cc * 32);
      const f32x4 v1 = *reinterpret_cast<const f32x4 *>(patch + rl * 288 + cc * 32 + 16);
      if (m < a.M && n < a.N) {  // N % 8 == 0: the eight columns are inside together
        bf16x8 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          o[q] = (bf16_t)v0[q];
          o[4 + q] = (bf16_t)v1[q];
        }
        __builtin_nontemporal_store(o, reinterpret_cast<bf16x8 *>(C + (size_t)m * a.N + n));
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Experts with 0 .. kThinSteps blocks of rows: 128 x 128 output tiles, 4 waves = 2 x 2, each 64 x 64; one LDS stage of
// (A 128 x 64, B 128 x 64) = 32 KiB (the epilogue patches reuse it) and at most 128 registers, so that four workgroups
// share a CU.  (Measured on the DeepSeek-shaped layer: four workgroups per CU instead of three -2.5 %, four tiles per
// workgroup -1.5 % of the weight-gradient time; requesting the next tile's operands ahead of the epilogue needs 150
// registers, i.e. three workgroups per CU, and comes out the same.)
// grid (ceil(n_mt * n_nt / kThinTiles), E_loc); a.n_mt / a.n_nt count 128-tiles here.
__global__ __launch_bounds__(256, 4) void wgrad_thin_bf16_kernel(const WgradArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * kPatchBytes];  // 36 KiB >= one 32 KiB stage
  const int tid = threadIdx.x, lane = tid & 63, w4 = tid >> 6;
  const int wm = w4 >> 1, wn = w4 & 1;
  const int le = blockIdx.y;
  const int kb0 = a.kb[le], KT = a.kb[le + 1] - kb0;
  if (KT > kThinSteps || KT == 0) return;  // whole workgroup: wgrad_bf16_kernel / wgrad_zero_empty_kernel own this expert
  const int chunk = tid & 7, row0 = tid >> 3;  // rows row0 + 32 i
  const int l31 = lane & 31, khalf = lane >> 5, sw = (lane >> 1) & 7;
  // kThinTiles consecutive tiles per workgroup (a tile is a few microseconds of dependent latencies: load, LDS,
  // matrix instructions, LDS, store; what hides them is the number of workgroups a CU holds, four here, and not
  // having to start a new workgroup for every tile)
  for (int rep = 0; rep < kThinTiles; ++rep) {
  const int tile_id = blockIdx.x * kThinTiles + rep;
  if (tile_id >= a.n_mt * a.n_nt) break;  // (uniform)
  const int mt = tile_id / a.n_nt, nt = tile_id % a.n_nt;
  const int m0 = mt * 128, n0 = nt * 128;
  if (rep > 0) __syncthreads();  // the previous tile's patches are done with the LDS
  f32x16 acc[2][2];
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][j][r] = 0.f;
  for (int kt = 0; kt < KT; ++kt) {
    u32x4 ra[4], rb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const size_t blk = (size_t)(kb0 + kt);
      ra[i] = *reinterpret_cast<const u32x4 *>(
          a.AT + (blk * a.lda + a.a0 + min(m0 + row0 + 32 * i, a.M - 1)) * 64 + chunk * 8);
      rb[i] = *reinterpret_cast<const u32x4 *>(
          a.BT + (blk * a.ldb + a.b0 + min(n0 + row0 + 32 * i, a.N - 1)) * 64 + chunk * 8);
    }
    if (kt > 0) __syncthreads();  // the previous step's fragment reads are done
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = row0 + 32 * i;
      const int dst = (row * 8 + (chunk ^ ((row >> 1) & 7))) * 16;
      *reinterpret_cast<u32x4 *>(smem + dst) = ra[i];
      *reinterpret_cast<u32x4 *>(smem + 16384 + dst) = rb[i];
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int slot = ((kk * 2 + khalf) ^ sw) * 16;
      bf16x8 fa[2], fb[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        fa[q] = *reinterpret_cast<const bf16x8 *>(smem + (wm * 64 + q * 32 + l31) * 128 + slot);
        fb[q] = *reinterpret_cast<const bf16x8 *>(smem + 16384 + (wn * 64 + q * 32 + l31) * 128 + slot);
      }
#pragma unroll
      for (int mi = 0; mi < 2; ++mi) {
        acc[mi][0] = mfma_bf16(fa[mi], fb[0], acc[mi][0]);
        acc[mi][1] = mfma_bf16(fa[mi], fb[1], acc[mi][1]);
      }
    }
  }
  __syncthreads();  // the stage is dead: every wave takes a private patch
  unsigned char *patch = smem + w4 * kPatchBytes;
  bf16_t *C = a.C + (size_t)le * a.M * a.N;
#pragma unroll
  for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rl = (r >> 2) * 8 + khalf * 4 + (r & 3);
      *reinterpret_cast<float *>(patch + rl * 288 + l31 * 4) = acc[mi][0][r];
      *reinterpret_cast<float *>(patch + rl * 288 + 128 + l31 * 4) = acc[mi][1][r];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int rl = it * 8 + (lane >> 3), cc = lane & 7;  // 8 groups of 8 columns per row: 16-byte stores
      const int m = m0 + wm * 64 + mi * 32 + rl, n = n0 + wn * 64 + cc * 8;
      const f32x4 v0 = *reinterpret_cast<const f32x4 *>(patch + rl * 288 + cc * 32);
      const f32x4 v1 = *reinterpret_cast<const f32x4 *>(patch + rl * 288 + cc * 32 + 16);
      if (m < a.M && n < a.N) {  // N % 8 == 0: the eight columns are inside together
        bf16x8 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          o[q] = (bf16_t)v0[q];
          o[4 + q] = (bf16_t)v1[q];
        }
        __builtin_nontemporal_store(o, reinterpret_cast<bf16x8 *>(C + (size_t)m * a.N + n));
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  }  // tiles of this workgroup
}

}  // namespace moe355
