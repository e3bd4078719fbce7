// Tile table: work lists of the two GEMMs and per-row metadata of the local layout segment.
#pragma once
#include "combine_kernels.h"
#include "forward_types.h"
#include "fp8_kernels.h"

namespace moe355 {

// ------------------------------------------------------------------------------------------------
// Work lists and per-row metadata of the local layout segment.
// header[0] = work items of GEMM-1, header[1] = P (local rows), header[2] = first layout row of the segment,
// header[3] = work items of GEMM-2, header[4] = M tiles; header[24] = error flag of the resident GEMM kernel
// and tickets[0 .. 7] / [8 .. 15] x kTicketStride = ticket counters of its GEMM-1 / GEMM-2 queues (all cleared here).  row_tile / tile_done
// (both may be null): M tile of every local row and the per-tile counter of finished GEMM-2 items, for the resident
// kernel that also runs Combine.
//
// A work item is one output tile (expert, M tile, N tile): int4 (local expert, first local row, valid rows,
// N tile | M-tile id << 12).  An expert's partial tile (its last rows) walks with the expert's full tiles when it has
// more than 64 rows: it needs the same weight panels, and running it in the same chunks fetches them once instead of
// twice (measured on layers whose experts hold one or two full tiles and a partial one: the L2 fills of GEMM-1 were
// twice the weights).  Partial tiles of at most 64 rows (pure weight streaming) are mixed into those chunks or
// trail them (see the list order below).
// The order of the list is also what keeps the L2 useful:
// the chip has 8 XCDs with a private 4 MiB L2 each and workgroup i runs on XCD i % 8, so every GEMM workgroup
// maps its index to a list position such that XCD x works through the 32-item chunks x, x + 8, x + 16, ...;
// and a chunk is a block of (up to 8 M tiles) x (32 / that many N tiles) of ONE expert, so the 32 workgroups
// that are resident on an XCD at the same time share a few A slabs and a few weight panels instead of
// streaming 32 different ones through the L2.
// ------------------------------------------------------------------------------------------------

// Rows up to which a partial tile counts as "streaming": its cost is reading the expert's weights from HBM, not
// the matrix cores.
constexpr int kStreamRows = 64;

// The FP8 form's codes of x, made by the same launch: the tile table is a chain of latencies on a few hundred workgroups, the
// codes are bound by HBM, and a row that no local slot names is not read (4096 tokens, k = 8, 32 of 256 experts of 7168: a
// third of the rows; 17.1 + 5.2 us as two launches, step 372 -> 359).
struct TokenCodes {
  const uint4 *x;
  int cols;
  uint8_t *codes;
  float *scales;
  const int32_t *inv_perm;
};

// Two kinds of blocks run side by side, since each is a short chain of dependent reads and together they made one twice as
// long: the first list_blocks blocks write the work lists (each rebuilds the small per-expert tables in its LDS), the others
// the per-row metadata.  (8192 tokens, k = 8, 128 experts: 9.6 us with every block doing both, one after the other, and
// looking each item's expert up in `offsets`; 6.3 us.)  QUANT: behind them a block per token.
template <bool QUANT>
__global__ __launch_bounds__(256) void fwd_prep_kernel(const int32_t *__restrict__ offsets,
                                                       const int32_t *__restrict__ perm,
                                                       const float *__restrict__ topk_w, int T, int k, int e_lo,
                                                       int E_loc, int bm, int P_cap, int max_mtiles, int nt1, int nt2,
                                                       int list_blocks, int32_t *__restrict__ header,
                                                       int32_t *__restrict__ tickets,
                                                       int4 *__restrict__ work1, int4 *__restrict__ work2,
                                                       int32_t *__restrict__ row_tok, float *__restrict__ row_w,
                                                       const int32_t *__restrict__ topk_idx,
                                                       int32_t *__restrict__ row_sole,
                                                       int32_t *__restrict__ tile_ready,
                                                       int32_t *__restrict__ row_tile,
                                                       int32_t *__restrict__ tile_done, const TokenCodes tokens) {
  const int base = offsets[e_lo], end = offsets[e_lo + E_loc];
  const int P = max(0, min(P_cap, end - base));
  if (QUANT && (int)blockIdx.x >= 2 * list_blocks) {
    const int t = blockIdx.x - 2 * list_blocks;
    const int row = combine_slot_row(topk_idx, tokens.inv_perm, t, k, threadIdx.x & 63, e_lo, E_loc, base, P_cap);
    if (__ballot(row >= 0) == 0) return;  // (the same in all four waves)
    fp8_quantize_row(tokens.x, t, tokens.cols, tokens.codes, tokens.scales);
    return;
  }
  if ((int)blockIdx.x >= list_blocks) {
    const long long npairs = (long long)T * k;
    const int stride = list_blocks * blockDim.x;
    for (int r = (blockIdx.x - list_blocks) * blockDim.x + threadIdx.x; r < P; r += stride) {
      int p = perm[base + r];
      p = p < 0 ? 0 : (p >= npairs ? (int)(npairs - 1) : p);
      const int t = p / k;
      row_tok[r] = t;
      row_w[r] = topk_w[p];
      if (row_sole) {
        // a row that is its token's only local slot needs no reduction: GEMM-2 writes it straight to y
        int n_local = 0;
#pragma unroll 8
        for (int j = 0; j < k; ++j) {
          const int e = topk_idx[(size_t)t * k + j];
          n_local += e >= e_lo && e < e_lo + E_loc;
        }
        row_sole[r] = n_local == 1 ? t : -1;
      }
    }
    return;
  }
  // LDS: part[E_loc] per expert: rows of its partial tile (0 = none) << 16 | E_loc - expert, i.e. ordered by rows, then by
  //      lower expert | start[E_loc + 1] first row | full0[E_loc + 1] first tile of class F | order[E_loc] experts with a
  //      streaming partial tile, largest first | only with row_tile: pos[E_loc] place of each expert's partial tile in
  //      `order` | number of streaming tiles | 17 ints of scan scratch
  extern __shared__ int lds[];
  int *part = lds;
  int *start = part + E_loc;
  int *full0 = start + E_loc + 1;
  int *order = full0 + E_loc + 1;
  int *pos = order + E_loc;
  int *s_small = row_tile ? pos + E_loc : pos;
  int *scratch = s_small + 1;
  const int nthr = list_blocks * blockDim.x, me = blockIdx.x * blockDim.x + threadIdx.x;
  for (int le = threadIdx.x; le <= E_loc; le += blockDim.x) start[le] = min(P, offsets[e_lo + le] - base);
  if (threadIdx.x == 0) *s_small = 0;
  __syncthreads();
  // An expert with cnt rows has cnt / bm full tiles and, if cnt % bm != 0, one partial tile.
  const int ipt = (E_loc + blockDim.x - 1) / blockDim.x;
  const int lo = min(E_loc, (int)threadIdx.x * ipt);
  const int hi = min(E_loc, lo + ipt);
  const auto tiles_of = [&](int le) {  // tiles of class F: a large partial tile walks with the expert's full tiles
    const int cnt = max(0, start[le + 1] - start[le]);
    return cnt / bm + ((cnt % bm) > kStreamRows);
  };
  int local_full = 0, local_small = 0;
  for (int le = lo; le < hi; ++le) {
    const int rest = max(0, start[le + 1] - start[le]) % bm;
    part[le] = rest << 16 | (E_loc - le);
    local_full += tiles_of(le);
    local_small += rest != 0 && rest <= kStreamRows;
  }
  if (local_small) atomicAdd(s_small, local_small);
  int n_full;
  int run = block_exclusive_scan(local_full, scratch, &n_full);  // (its barriers publish part[] and the count as well)
  for (int le = lo; le < hi; ++le) {
    full0[le] = run;
    run += tiles_of(le);
  }
  if (threadIdx.x == 0) full0[E_loc] = n_full;
  // rank sort of the streaming partial tiles: how many of them compare larger
  for (int le = lo; le < hi; ++le) {
    const int mine = part[le];
    if ((mine >> 16) == 0 || (mine >> 16) > kStreamRows) continue;
    const unsigned above = ((kStreamRows + 1) << 16) - mine - 1;  // keys of streaming tiles lie below (kStreamRows + 1) << 16
    int rank = 0, o = 0;
#pragma unroll 4
    for (; o + 4 <= E_loc; o += 4) {
      const int4 v = *reinterpret_cast<const int4 *>(part + o);
      rank += ((unsigned)(v.x - mine - 1) < above) + ((unsigned)(v.y - mine - 1) < above) +
              ((unsigned)(v.z - mine - 1) < above) + ((unsigned)(v.w - mine - 1) < above);
    }
    for (; o < E_loc; ++o) rank += (unsigned)(part[o] - mine - 1) < above;
    order[rank] = le;
    if (row_tile) pos[le] = rank;
  }
  __syncthreads();
  n_full = min(n_full, max_mtiles);
  const int n_small = min(*s_small, max_mtiles - n_full);
  const int n_tiles = n_full + n_small;
  const int n1 = n_tiles * nt1, n2 = n_tiles * nt2;
  if (me == 0) {
    header[0] = n1;
    header[1] = P;
    header[2] = base;
    header[3] = n2;
    header[4] = n_tiles;
    header[24] = 0;
  }
  if (me < 16) tickets[me * kTicketStride] = 0;
  for (int i = me; i < n_tiles; i += nthr) {
    tile_ready[(size_t)i * kReadyStride] = 0;
    if (tile_done) tile_done[i] = 0;
  }
  // M tile of every local row (the resident kernel's Combine stage looks up the tile whose GEMM-2 items it waits for)
  if (row_tile) {
    for (int r = me; r < P; r += nthr) {
      // expert of row r: largest le whose first row is <= r
      int a = 0, b = E_loc;
      while (b - a > 1) {
        const int mid = (a + b) >> 1;
        if (start[mid] <= r) a = mid; else b = mid;
      }
      const int cnt = start[a + 1] - start[a];
      const int mt = (r - start[a]) / bm;
      const int tile = (mt < cnt / bm || (part[a] >> 16) > kStreamRows) ? full0[a] + mt : n_full + pos[a];
      row_tile[r] = min(tile, max(n_tiles - 1, 0));
    }
  }
  for (int q = me; q < n1 + n2; q += nthr) {
    const bool second = q >= n1;
    const int Nt = second ? nt2 : nt1;
    const int qq = second ? q - n1 : q;
    // List order.  Classes: F = full tiles and partial tiles of more than kStreamRows rows, S = streaming partial tiles.
    //   [ mixed chunks: each 32-item chunk holds 8 items of S, then 24 items of F, so that some CUs of every XCD
    //     stream weights from HBM while the others multiply; only when S is at least half as large as F,
    //     otherwise the few S items would just push full tiles into an extra round ]
    //   [ rest of F ] [ rest of S, largest first ]  -- the launch ends with its shortest items
    const int nF = n_full * Nt, nS = n_small * Nt;
    constexpr int nsc = 8, nfc = kChunk - nsc;
    const int n_mix = (nF > 0 && 2 * nS >= nF) ? min(nF / nfc, nS / nsc) : 0;
    // F items that share operands form groups of gsz consecutive list positions; gsz follows the F share of a chunk
    const int gsz = n_mix > 0 ? nfc : kChunk;
    bool streams;  // class S
    int idx;       // position inside the class list
    if (qq < n_mix * kChunk) {
      const int c = qq / kChunk, sl = qq % kChunk;
      streams = sl < nsc;
      idx = streams ? c * nsc + sl : c * nfc + (sl - nsc);
    } else {
      const int r = qq - n_mix * kChunk, f_rem = nF - n_mix * nfc;
      streams = r >= f_rem;
      idx = streams ? n_mix * nsc + (r - f_rem) : n_mix * nfc + r;
    }
    int le, mt, nt, tile;
    if (!streams) {
      // expert that owns F position idx: largest le with full0[le] * Nt <= idx
      int a = 0, b = E_loc;
      while (b - a > 1) {
        const int mid = (a + b) >> 1;
        if (full0[mid] * Nt <= idx) a = mid; else b = mid;
      }
      le = a;
      const int Mt = full0[le + 1] - full0[le];
      int r = idx - full0[le] * Nt;
      // inside the expert: M groups of up to 8 tiles; inside an M group: N groups of gsz / (M tiles) tiles.
      // (A slab and B panel of a tile are equally large, so the bytes a chunk pulls into its L2 are smallest
      // when the chunk is close to square: 8 x 4 rather than 32 x 1.)
      const int Mg = min(Mt, kChunkM);
      const int mg = r / (Mg * Nt);
      r -= mg * Mg * Nt;
      const int Mcur = min(Mg, Mt - mg * Mg);
      const int G = max(1, gsz / Mcur);
      const int ng = r / (Mcur * G);
      r -= ng * Mcur * G;
      const int Gcur = min(G, Nt - ng * G);
      // Inside the group the shorter side runs fastest.  The workgroups of an XCD start a few microseconds apart
      // (one whenever a CU becomes free), and the L2 keeps only the last few k-steps of what they stream; two items
      // share a panel through it only if they sit within a few list positions of each other, and with the shorter
      // side innermost both the A sharers and the B sharers do.
      if (Gcur <= Mcur) {
        mt = mg * Mg + r / Gcur;
        nt = ng * G + r % Gcur;
      } else {
        mt = mg * Mg + r % Mcur;
        nt = ng * G + r / Mcur;
      }
      tile = full0[le] + mt;
    } else {
      le = order[idx / Nt];
      tile = n_full + idx / Nt;
      nt = idx % Nt;
      mt = (start[le + 1] - start[le]) / bm;
    }
    const int first = start[le], cnt = start[le + 1] - first;
    const int rows = mt < cnt / bm ? bm : part[le] >> 16;  // the last tile of class F may be the expert's large partial tile
    const int4 item = make_int4(le, first + mt * bm, rows | (cnt <= bm ? kItemLone : 0), nt | (tile << kTileShift));
    if (second) work2[qq] = item; else work1[qq] = item;
  }
}

}  // namespace moe355
