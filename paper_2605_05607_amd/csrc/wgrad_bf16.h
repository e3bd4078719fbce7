// Weight gradients of the expert FFN on the matrix cores: for every local expert, C = A^T B summed over the expert's
// rows (dW_gate = x^T dg, dW_up = x^T du, dW_down = (w h)^T dy).  The reduction index is the row, which is the slow
// index of both operands in memory, while a matrix-core operand wants 8 consecutive reduction indices per lane.  The kernels
// stage the rows as they lie in memory (x and dy rows by token) and transpose in the reads from the LDS.  All three products
// of the large experts are one launch, those of the small ones another.
// Operands of 4 GiB and more, which 32-bit offsets do not reach, are first transposed (and gathered) into buffers of 64-row
// blocks, [block][column][64 rows], in which every expert's rows start at a block boundary and are zero-padded to one: what a
// workgroup stages per k-step is then one contiguous piece of memory per operand (wgrad_slab_kernel, wgrad_thin_slab_kernel).
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

// Rows of local expert le (and its first one) in the local layout segment.
__device__ __forceinline__ int expert_rows(const int32_t *__restrict__ offsets, const int32_t *__restrict__ header, int e_lo,
                                           int le, int &start) {
  const int P = header[1], base = header[2];
  start = min(P, max(0, offsets[e_lo + le] - base));
  return max(0, min(P, offsets[e_lo + le + 1] - base) - start);
}

struct WgradArgs {
  const bf16_t *AT;   // [block][lda][64]: rows a0 .. a0 + M of every block are the left operand's columns
  const bf16_t *BT;   // [block][ldb][64]: rows b0 .. b0 + N
  bf16_t *C;          // [E_loc][M][N]
  const int32_t *kb;  // [E_loc + 1]
  int lda, ldb, a0, b0;
  int M, N, n_mt, n_nt;
};

// Experts with at most kThinSteps blocks of 64 rows are left to the thin kernels (those without rows to
// wgrad_zero_empty_kernel where the operands are transposed copies): their cost is writing the output, and that kernel's small workgroups overlap the stores of
// one tile with the loads of the next on the same CU.
constexpr int kStageBytes = 2 * kBM * kBK * 2;  // 64 KiB: A slab then B slab
constexpr int kThinSteps = 2;
constexpr int kThinTiles = 4;  // output tiles per workgroup of wgrad_thin_slab_kernel

// Zero gradients of the local experts without rows: grid (shares, E_loc, 3 matrices), each workgroup clears one
// contiguous share of `units` 16-byte units.  A launch of its own, ahead of the products: run beside them its writers cost the
// matrix-core workgroups more than they hide.
__global__ __launch_bounds__(256) void wgrad_zero_empty_kernel(const int32_t *__restrict__ offsets,
                                                               const int32_t *__restrict__ header, int e_lo, u32x4 *c0,
                                                               u32x4 *c1, u32x4 *c2, size_t units) {
  const int le = blockIdx.y;
  int start;
  if (expert_rows(offsets, header, e_lo, le, start) > 0) return;
  u32x4 *C = (blockIdx.z == 0 ? c0 : blockIdx.z == 1 ? c1 : c2) + (size_t)le * units;
  const size_t share = (units + gridDim.x - 1) / gridDim.x;
  const size_t u0 = blockIdx.x * share, u1 = u0 + share < units ? u0 + share : units;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  for (size_t u = u0 + threadIdx.x; u < u1; u += 256) __builtin_nontemporal_store(zero, &C[u]);
}

// The gradients are written once and not read again by this library: all kernels below store them with the
// non-temporal hint, so that 0.9 GB of output per product does not push the operands, which every tile of an expert
// shares, out of the L2s (measured: -9 % of the weight-gradient time on the GPT-OSS-shaped layer, -6.5 % on the
// Mixtral-shaped one, -9 % on the Qwen3-shaped one, -2 % on the DeepSeek-shaped one).
// One workgroup per (local expert, 256 x 256 output tile); 8 waves = 2 x 4, each 128 x 64 as 4 x 2 accumulators.
// LDS: two stages of (A 256 x 64, B 256 x 64), rows of 128 bytes with the forward tile's chunk swizzle; main loop of the
// forward's full tiles (slabs straight into the LDS, wave rows half a step apart) instead of slabs staged through registers
// with all waves in step.  What bounds it is the short reduction (8 k-steps for 512 rows) between a two-slab prologue and the
// store of 128 KiB: training step of 8192 tokens on 16 experts of 4096 x 1536, when every size took this form, 1277 -> 1267 us.
__global__ __launch_bounds__(kGemmThreads, 1) void wgrad_slab_kernel(const WgradArgs a) {
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
  typedef PingPong<false, 4, 128, false, false, kGradSlabs> Loop;
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
__global__ __launch_bounds__(256, 4) void wgrad_thin_slab_kernel(const WgradArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * kPatchBytes];  // 36 KiB >= one 32 KiB stage
  const int tid = threadIdx.x, lane = tid & 63, w4 = tid >> 6;
  const int wm = w4 >> 1, wn = w4 & 1;
  const int le = blockIdx.y;
  const int kb0 = a.kb[le], KT = a.kb[le + 1] - kb0;
  if (KT > kThinSteps || KT == 0) return;  // whole workgroup: wgrad_slab_kernel / wgrad_zero_empty_kernel own this expert
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

// ------------------------------------------------------------------------------------------------
// The weight gradients without transposed copies.  A row of an operand is read once per tile that needs its columns, by
// 128-byte (A) or 64-byte (B) pieces, where the copies cost a read and a write of every operand beside the GEMMs, which they
// slowed down.  What bounds them: a reduction of 8 k-steps (512 rows) between the start of a workgroup (row offsets, two
// slabs) and a 128 KiB epilogue, with one workgroup per CU.
// Measured, training step of 8192 tokens on 16 experts of 4096 x 1536: 1313 -> 1218 us (the two backward GEMMs 431 -> 380,
// products 414 -> about 400 in one launch, 11 launches less); backward pass of 100 rows on each of 8 experts of 2880 x 2880
// 409 -> 322 us, 400 rows 534 -> 484; of 7168 x 2048 518 -> 460 and 835 -> 782.  Same bits.
// ------------------------------------------------------------------------------------------------
struct WgradDirectArgs {
  const bf16_t *x, *dy;      // [T, d]
  const bf16_t *dgu, *hw;    // [P, 2 f]: dg, then du; [P, f]
  bf16_t *dW_gate, *dW_up, *dW_down;
  const int32_t *offsets, *header, *row_tok;
  int e_lo, E_loc, T, d, f;
  int n_items;               // E_loc * (tiles of [dW_gate | dW_up] and of dW_down)
};

constexpr int kWgradTable = 7680;  // rows whose offsets fit the LDS behind the stages; more are taken in several passes
constexpr int kWgradLds = 2 * kStageBytes + kWgradTable * 4;

// 32 x 64 block of C in a wave's patch (fp32, row pitch 288 bytes) -> bf16 rows m .., columns n ..; GU: n counts the columns
// of dW_gate and then those of dW_up (f % 64 == 0: eight columns never straddle the two).
template <bool GU>
__device__ __forceinline__ void wgrad_store_block(const WgradDirectArgs &a, const unsigned char *patch, int le, int m, int n) {
  const int lane = fresh_lane();
  const int M = GU ? a.d : a.f, N = GU ? 2 * a.f : a.d, ld = GU ? a.f : a.d;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int rl = it * 8 + (lane >> 3), cc = lane & 7;  // 8 groups of 8 columns per row: 16-byte stores
    const f32x4 v0 = *reinterpret_cast<const f32x4 *>(patch + rl * 288 + cc * 32);
    const f32x4 v1 = *reinterpret_cast<const f32x4 *>(patch + rl * 288 + cc * 32 + 16);
    int c = n + cc * 8;
    if (m + rl < M && c < N) {
      bf16x8 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        o[q] = (bf16_t)v0[q];
        o[4 + q] = (bf16_t)v1[q];
      }
      bf16_t *C = GU ? a.dW_gate : a.dW_down;
      if (GU && c >= a.f) {
        C = a.dW_up;
        c -= a.f;
      }
      __builtin_nontemporal_store(o, reinterpret_cast<bf16x8 *>(C + ((size_t)le * M + m + rl) * ld + c));
    }
  }
}

// One 256 x 256 tile.  GU: [dW_gate | dW_up] = x^T [dg | du], rows of x gathered; else dW_down = (w h)^T dy, rows of dy.
template <bool GU>
__device__ __forceinline__ void wgrad_direct_tile(const WgradDirectArgs &a, unsigned char *smem, int le, int mt, int nt,
                                                  int start, int cnt) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3, khalf = lane >> 5, l31 = lane & 31;
  f32x16 acc[4][2];
#pragma unroll
  for (int mi = 0; mi < 4; ++mi)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][j][r] = 0.f;
  typedef PingPong<false, 4, 128, false, false, GU ? kGradGatherA : kGradGatherB> Loop;
  Loop loop;
  loop.lds = lds_address(smem);
  loop.smem = smem;
  loop.a_rd = wm * 16384 + transposed_read_offset(lane);
  // B: rows of 64 bytes, no swap
  loop.b_rd = Loop::kB + wn * 8192 + ((lane >> 5) * 8 + ((lane & 15) >> 2)) * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
  loop.b_soff = (wave >> 1) * 8192 + (wave & 1) * 2048;
  loop.a_lds[0] = wm * 16384 + (wave & 3) * 2048;
  loop.a_lds[1] = loop.a_lds[0] + 8192;
  // A: an instruction is 8 rows of 128 bytes, lane = row by 16-byte chunk (the halves swapped where bit 1 of the row is
  // set); B: 16 rows of 64 bytes
  const int row_a = (wave & 3) * 16 + (lane >> 3), row_b = (wave & 1) * 32 + (lane >> 2);
  const uint32_t col_a = (mt * kBM + wm * 128) * 2 + (((lane & 7) * 16) ^ (((lane >> 4) & 1) * 64));
  const uint32_t col_b = (nt * kBN + (wave >> 1) * 64) * 2 + (lane & 3) * 16;
  loop.gathered = lds_load_rsrc(GU ? a.x : a.dy, (uint32_t)a.T * a.d * 2);
  loop.pitch = (GU ? 2 * a.f : a.f) * 2;
  loop.tab = loop.lds + 2 * kStageBytes + (GU ? row_a : row_b) * 4;
  loop.col = GU ? col_a : col_b;
  loop.col_next = GU ? row_b * loop.pitch + col_b : row_a * loop.pitch + col_a;
  uint32_t *tab = reinterpret_cast<uint32_t *>(smem + 2 * kStageBytes);
  for (int c0 = 0; c0 < cnt; c0 += kWgradTable) {
    const int n = min(cnt - c0, kWgradTable), KT = (n + 63) >> 6;
    if (c0 > 0) __syncthreads();  // every wave is done with the table and the stages
    for (int r = tid; r < KT * 64; r += kGemmThreads)
      tab[r] = (uint32_t)(r < n ? min(max(a.row_tok[start + c0 + r], 0), a.T - 1) : a.T) * (a.d * 2);
    __syncthreads();
    loop.next = reinterpret_cast<const unsigned char *>(GU ? a.dgu : a.hw) + (size_t)(start + c0) * loop.pitch;
    loop.next_bytes = (uint32_t)n * loop.pitch;
    loop.run(acc, KT, KT * kBK, wm);
  }
  // epilogue: each wave turns its 32 x 64 blocks around through a private LDS patch so that a row leaves as contiguous bf16
  __syncthreads();
  unsigned char *patch = smem + wave * kPatchBytes;
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
    wgrad_store_block<GU>(a, patch, le, mt * kBM + wm * 128 + mi * 32, nt * kBN + wn * 64);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// One workgroup per (expert, 256 x 256 tile) of all three matrices; experts of more than kThinSteps blocks of 64 rows.  The
// list of an expert goes through [dW_gate | dW_up], then dW_down, in blocks of up to 8 x 4 tiles, and is spread over the
// XCDs in runs of 32 (chunked_item), so that the workgroups of an XCD share operand slabs in its L2.
__global__ __launch_bounds__(kGemmThreads, 1) void wgrad_bf16_kernel(const WgradDirectArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // kWgradLds
  const int q = chunked_item(blockIdx.x, a.n_items);
  if (q < 0) return;
  const int td = (a.d + kBM - 1) / kBM, tf = (a.f + kBN - 1) / kBN, tg = (2 * a.f + kBN - 1) / kBN;
  const int per = td * tg + tf * td;
  const int le = q / per;
  int start;
  const int cnt = expert_rows(a.offsets, a.header, a.e_lo, le, start);
  if (cnt <= 64 * kThinSteps) return;  // whole workgroup: the thin kernel owns this expert
  int r = q - le * per;
  const bool gu = r < td * tg;
  if (!gu) r -= td * tg;
  const int Mt = gu ? td : tf, Nt = gu ? tg : td;
  const int Mg = min(Mt, kChunkM), mg = r / (Mg * Nt);
  r -= mg * Mg * Nt;
  const int Mcur = min(Mg, Mt - mg * Mg), G = kChunk / Mcur, ng = r / (Mcur * G);
  r -= ng * Mcur * G;
  const int mt = mg * Mg + r % Mcur, nt = ng * G + r / Mcur;
  if (gu) wgrad_direct_tile<true>(a, smem, le, mt, nt, start, cnt);
  else wgrad_direct_tile<false>(a, smem, le, mt, nt, start, cnt);
}

// Experts with 1 .. kThinSteps blocks of rows: 128 x 128 tiles, 4 waves = 2 x 2, each 64 x 64; one stage of 32 KiB through
// registers (what counts is the output; four workgroups per CU overlap one another's latencies, kThinTiles tiles each).
template <bool GU>
__device__ __forceinline__ void wgrad_thin_tile(const WgradDirectArgs &a, unsigned char *smem, int le, int mt, int nt,
                                                int start, int cnt) {
  // (the lane anew per tile: nothing derived from it is kept across the tiles of a workgroup, there is no register to spare)
  const int lane = fresh_lane(), w4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w4 >> 1, wn = w4 & 1;
  const int tid = w4 * 64 + lane, m0 = mt * 128, n0 = nt * 128;
  const int chunk = tid & 7, row0 = tid >> 3;
  const uint32_t lds = lds_address(smem), rd = transposed_read_offset(lane);
  f32x16 acc[2][2];
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][j][r] = 0.f;
  // rows past the last, and what lies behind the matrices, read as zeros; columns past the end are not stored
  const uint32_t gpitch = a.d * 2, npitch = (GU ? 2 * a.f : a.f) * 2;
  const __amdgpu_buffer_rsrc_t gathered =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(GU ? a.x : a.dy), 0, (uint32_t)a.T * gpitch, 0x00027000);
  const __amdgpu_buffer_rsrc_t next = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t *>(GU ? a.dgu : a.hw) + (size_t)start * (npitch / 2), 0, cnt * npitch, 0x00027000);
  const uint32_t col_g = (GU ? m0 : n0) * 2 + chunk * 16, col_n = (GU ? n0 : m0) * 2 + chunk * 16;
  for (int kt = 0; kt * 64 < cnt; ++kt) {
    u32x4 ra[4], rb[4];  // [row half][block of 64 columns]
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = kt * 64 + row0 + 32 * i;
      const uint32_t og = (uint32_t)(r < cnt ? min(max(a.row_tok[start + r], 0), a.T - 1) : a.T) * gpitch + col_g;
      const uint32_t on = r * npitch + col_n;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        ra[i * 2 + b] = __builtin_amdgcn_raw_buffer_load_b128(GU ? gathered : next, (GU ? og : on) + b * 128, 0, 0);
        rb[i * 2 + b] = __builtin_amdgcn_raw_buffer_load_b128(GU ? next : gathered, (GU ? on : og) + b * 128, 0, 0);
      }
    }
    if (kt > 0) __syncthreads();  // the previous step's fragment reads are done
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int row = row0 + 32 * i, dst = b * 8192 + row * 128 + ((chunk * 16) ^ (((row >> 1) & 1) * 64));
        *reinterpret_cast<u32x4 *>(smem + dst) = ra[i * 2 + b];
        *reinterpret_cast<u32x4 *>(smem + 16384 + dst) = rb[i * 2 + b];
      }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8 fa[2], fb[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint32_t at = lds + (rd ^ q * 64) + kk * 2048;
        fa[q] = transposed_fragment(at + wm * 8192, 512);
        fb[q] = transposed_fragment(at + 16384 + wn * 8192, 512);
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
  const int l31 = lane & 31, khalf = lane >> 5;
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
    wgrad_store_block<GU>(a, patch, le, m0 + wm * 64 + mi * 32, n0 + wn * 64);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Zero gradients of an expert without rows: workgroup `share` of `shares` clears a contiguous share of its three matrices.
__device__ __forceinline__ void wgrad_zero_share(const WgradDirectArgs &a, int le, uint32_t share, uint32_t shares) {
  const uint64_t units = (uint64_t)a.d * a.f / 8, all = 3 * units, per = (all + shares - 1) / shares;  // of 16 bytes
  const uint64_t end = per * (share + 1) < all ? per * (share + 1) : all;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  for (uint64_t u = per * share + threadIdx.x; u < end; u += 256) {
    const uint32_t m = (u >= units) + (u >= 2 * units);
    bf16_t *C = m == 0 ? a.dW_gate : m == 1 ? a.dW_up : a.dW_down;
    __builtin_nontemporal_store(zero, reinterpret_cast<u32x4 *>(C) + (size_t)le * units + (u - m * units));
  }
}

// grid (ceil(tiles of 128 x 128 of all three matrices / kThinTiles), E_loc).  Experts without rows as well: what either takes
// is the time of its stores, and a launch that finds no such expert still costs 5 us.
__global__ __launch_bounds__(256, 4) void wgrad_thin_bf16_kernel(const WgradDirectArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * kPatchBytes];  // 36 KiB >= one 32 KiB stage
  const int le = blockIdx.y;
  int start;
  const int cnt = expert_rows(a.offsets, a.header, a.e_lo, le, start);
  if (cnt > 64 * kThinSteps) return;  // whole workgroup: wgrad_bf16_kernel owns it
  if (cnt == 0) {
    wgrad_zero_share(a, le, blockIdx.x, gridDim.x);
    return;
  }
  const int td = (a.d + 127) / 128, tf = (a.f + 127) / 128, tg = (2 * a.f + 127) / 128, gu = td * tg;
  for (int rep = 0; rep < kThinTiles; ++rep) {
    int id = blockIdx.x * kThinTiles + rep;
    if (id >= gu + tf * td) break;  // (uniform)
    if (rep > 0) __syncthreads();  // the previous tile's patches are done with the LDS
    if (id < gu) {
      wgrad_thin_tile<true>(a, smem, le, id / tg, id % tg, start, cnt);
    } else {
      id -= gu;
      wgrad_thin_tile<false>(a, smem, le, id / td, id % td, start, cnt);
    }
  }
}

}  // namespace moe355
