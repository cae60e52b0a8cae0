// Stable grouping of a step's (token, expert) pairs by key (layer, expert slot).
//
// On an EP group this is the dispatch all-to-all (Section 2.2); with several
// micro-batches at different layers in one step (Section 4.1) the key carries
// the layer, so one grouped GEMM launch covers every (layer, expert) group.
//
//   perm_count_kernel    per 256-token chunk: routed pairs per expert (LDS atomics)
//   perm_scan_kernel     one workgroup: per-key totals, offsets, per-chunk bases,
//                        the GEMM tile list (each BM-row block's group record:
//                        key, first row, rows, index of its first row block);
//                        it also clears the work counters of the step's
//                        grouped GEMM launches
//                        (the three above and perm_scatter_kernel: one launch,
//                        perm_small_kernel, for steps of up to 1000 to 2000 tokens,
//                        with the gather's copies for those of a few)
//   perm_scatter_kernel  per chunk: stable rank of each pair inside its key from
//                        per-wavefront 64-bit expert masks (popcount of the lanes
//                        below), then inv, and perm where a caller asks for it
//   gather_tokens_kernel one wavefront per (token, 1 KB piece of its row):
//                        the piece, read once, to a_perm[inv[q]] for each of
//                        the token's k+S pairs q
//
// Pair q = (tok_base[rho] + t) * (k+S) + r; key = layer*(E+S) + slot expert.
// All results are integers fixed by the inputs (no order-dependent atomics).
#include "eb_internal.h"
#include "eb_numeric.h"

namespace eb {
namespace {

constexpr int kScanThreads = 1024;

__device__ __forceinline__ int clamp_expert(int e, int E) { return e < 0 ? 0 : (e >= E ? E - 1 : e); }

template <class RTA>
__global__ __launch_bounds__(kPermChunk) void perm_count_kernel(RTA rta, int32_t* __restrict__ hist) {
  const RunTable& rt = rta.get();
  __shared__ int cnt[1024];
  const int b = blockIdx.x;
  if (b >= rt.chunk_base[rt.n]) return;  // past the live chunks (grid sized for the largest step)
  for (int e = threadIdx.x; e < rt.E; e += blockDim.x) cnt[e] = 0;
  __syncthreads();
  const int rho = find_entry(rt.chunk_base, rt.n, b);
  const int T = rt.tok_base[rho + 1] - rt.tok_base[rho];
  const int t = (b - rt.chunk_base[rho]) * kPermChunk + threadIdx.x;
  if (t < T) {
    const int32_t* ix = in_global(rt.idx[rho]) + (size_t)t * rt.k;
    for (int r = 0; r < rt.k; ++r) atomicAdd(&cnt[clamp_expert(ix[r], rt.E)], 1);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < rt.E; e += blockDim.x) hist[(size_t)b * rt.E + e] = cnt[e];
}

constexpr int kScanWaves = kScanThreads / kWave;
constexpr int kMaxKeys = 15360;      // L * (E + S) limit of the descriptor check
constexpr int kHistWindow = 16384;   // histogram cells held in LDS at once

// Block-wide exclusive scan of one value per thread (1024 threads): a
// shuffle scan inside each wavefront, then over the 16 wavefront totals;
// returns the exclusive prefix and writes the total to *total.
__device__ int block_exclusive_scan(int v, int* wtot, int* total) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int x = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int y = __shfl_up(x, off, kWave);
    if (lane >= off) x += y;
  }
  if (lane == kWave - 1) wtot[wave] = x;
  __syncthreads();
  if (wave == 0) {
    int t = lane < kScanWaves ? wtot[lane] : 0;
#pragma unroll
    for (int off = 1; off < kScanWaves; off <<= 1) {
      const int y = __shfl_up(t, off, kWave);
      if (lane >= off) t += y;
    }
    if (lane < kScanWaves) wtot[lane] = t;
  }
  __syncthreads();
  const int before = wave > 0 ? wtot[wave - 1] : 0;
  *total = wtot[kScanWaves - 1];
  __syncthreads();  // wtot is reused by the next scan
  return before + x - v;
}

// Offsets and GEMM tile list from the per-key totals in running[] (1024
// threads, running[] complete); leaves each key's offset in running[].
__device__ void offsets_and_tiles(int* running, int n_keys, int* wtot, int32_t* __restrict__ offsets,
                                  int4* __restrict__ tiles, int bm, TailRule tail, int max_tiles,
                                  int32_t* __restrict__ work_ctr) {
  const int tid = threadIdx.x;
  // exclusive scan over keys -> offsets; thread tid owns a contiguous span
  const int span = (n_keys + kScanThreads - 1) / kScanThreads;
  const int k0 = min(tid * span, n_keys), k1 = min(k0 + span, n_keys);
  int local = 0;
  for (int i = k0; i < k1; ++i) local += running[i];
  int total = 0;
  int base = block_exclusive_scan(local, wtot, &total);
  for (int i = k0; i < k1; ++i) {
    const int v = running[i];
    offsets[i] = base;
    running[i] = base;  // becomes the running cursor of key i
    base += v;
  }
  if (tid == 0) offsets[n_keys] = total;
  __syncthreads();

  // tile list: ceil(M/bm) row blocks per non-empty key, keys ascending,
  //    the first tail.tiles groups of at most tail.rows rows (one block each,
  //    tail.rows <= bm) after all the others
  auto rows_of = [&](int i) { return (i + 1 < n_keys ? running[i + 1] : total) - running[i]; };
  int local_tiles = 0, local_small = 0;
  for (int i = k0; i < k1; ++i) {
    const int M = rows_of(i);
    local_tiles += (M + bm - 1) / bm;
    local_small += M > 0 && M <= tail.rows;
  }
  int tiles_total = 0, small_total = 0;
  int tb = block_exclusive_scan(local_tiles, wtot, &tiles_total);
  int sb = block_exclusive_scan(local_small, wtot, &small_total);
  const int main_total = tiles_total - min(small_total, tail.tiles);
  for (int i = k0; i < k1; ++i) {
    const int r0 = running[i], M = rows_of(i);
    if (M == 0) continue;
    const bool small = M <= tail.rows;
    const int at = small && sb < tail.tiles ? main_total + sb : tb - min(sb, tail.tiles);
    const int4 g = make_int4(i, r0, M, at);
    const int n = (M + bm - 1) / bm;
    for (int m = 0; m < n; ++m)
      if (at + m < max_tiles) tiles[at + m] = g;
    tb += n;
    sb += small;
  }
  if (tid == 0) {
    work_ctr[kWorkTiles] = min(tiles_total, max_tiles);
    work_ctr[kWorkTiles + 1] = min(main_total, max_tiles);
  }
  __syncthreads();  // running[] may change from here on
}

// offsets: [L*(E+S)+1]; chunk_base: [n_chunks][E+S]; tiles: [max_tiles].
// The histogram cells (chunk b, column c) go through LDS in windows of
// kHistWindow / (E+S) chunks (one window unless the step is very large);
// every global load of a phase is independent of the others.
template <class RTA>
__global__ __launch_bounds__(kScanThreads) void perm_scan_kernel(
    RTA rta, const int32_t* __restrict__ hist, int32_t* __restrict__ chunk_base,
    int32_t* __restrict__ offsets, int4* __restrict__ tiles, int bm, TailRule tail,
    int max_tiles, int32_t* __restrict__ work_ctr) {
  __shared__ int running[kMaxKeys];              // per-key totals, then offsets / cursors
  __shared__ int hl[kHistWindow];                // one window of histogram cells
  __shared__ int wtot[kScanWaves];
  __shared__ int s_cb[EB_MAX_RUN + 1], s_tb[EB_MAX_RUN + 1], s_ly[EB_MAX_RUN];
  const RunTable& rt = rta.get();
  const int tid = threadIdx.x;
  if (tid < kWorkWords && tid != kWorkTiles && tid != kWorkTiles + 1) work_ctr[tid] = 0;
  const int E = rt.E, ES = rt.E + rt.S, n = rt.n;
  const int n_chunks = rt.chunk_base[n];
  const int n_keys = rt.L * ES;
  for (int i = tid; i < n_keys; i += kScanThreads) running[i] = 0;
  if (tid <= n) {
    s_cb[tid] = rt.chunk_base[tid];
    s_tb[tid] = rt.tok_base[tid];
  }
  if (tid < n) s_ly[tid] = rt.layer[tid];
  __syncthreads();

  // cell (b, c): routed pairs of chunk b on expert c, or (shared slot c >= E)
  // the chunk's tokens; *key = (layer of b's entry, c)
  auto cell = [&](int b, int c, int* key) {
    const int rho = find_entry(s_cb, n, b);
    *key = s_ly[rho] * ES + c;
    if (c < E) return (int)hist[(size_t)b * E + c];
    return min(kPermChunk, s_tb[rho + 1] - s_tb[rho] - (b - s_cb[rho]) * kPermChunk);
  };
  const int win = kHistWindow / ES;  // >= 16 chunks (ES <= 1024)
  const int n_win = (n_chunks + win - 1) / win;

  // 1) per-key totals (integer LDS atomics: order-free); the last window
  //    stays in hl
  for (int w0 = 0; w0 < n_chunks; w0 += win) {
    const int cells = min(win, n_chunks - w0) * ES;
    for (int i = tid; i < cells; i += kScanThreads) {
      int key;
      const int v = cell(w0 + i / ES, i % ES, &key);
      hl[i] = v;
      atomicAdd(&running[key], v);
    }
  }
  __syncthreads();

  // 2), 3)
  offsets_and_tiles(running, n_keys, wtot, offsets, tiles, bm, tail, max_tiles, work_ctr);

  // 4) per-chunk bases: for every column, the entries' chunks in order; a
  //    key's cursor lives in LDS across entries, in a register within one
  for (int w = 0; w < n_win; ++w) {
    const int w0 = w * win, nw = min(win, n_chunks - w0);
    if (n_win > 1) {
      for (int i = tid; i < nw * ES; i += kScanThreads) {
        int key;
        hl[i] = cell(w0 + i / ES, i % ES, &key);
      }
      __syncthreads();
    }
    for (int c = tid; c < ES; c += kScanThreads) {
      for (int rho = 0; rho < n; ++rho) {
        const int b_lo = max(s_cb[rho], w0), b_hi = min(s_cb[rho + 1], w0 + nw);
        if (b_lo >= b_hi) continue;
        const int key = s_ly[rho] * ES + c;
        int cur = running[key];
        for (int b = b_lo; b < b_hi; ++b) {
          chunk_base[(size_t)b * ES + c] = cur;
          cur += hl[(b - w0) * ES + c];
        }
        running[key] = cur;
      }
    }
    __syncthreads();  // hl is refilled by the next window
  }
}

// One block per chunk, one token per thread.  `elem_bytes` is 2 (bf16) or 4.
template <class RTA>
__global__ __launch_bounds__(kPermChunk) void perm_scatter_kernel(
    RTA rta, const int32_t* __restrict__ chunk_base, int32_t* __restrict__ perm,
    int32_t* __restrict__ inv) {
  __shared__ unsigned long long mask[kPermChunk / kWave][1024];
  const RunTable& rt = rta.get();
  const int E = rt.E, S = rt.S, k = rt.k, ES = E + S, slots = k + S;
  const int b = blockIdx.x;
  if (b >= rt.chunk_base[rt.n]) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int i = threadIdx.x; i < (kPermChunk / kWave) * E; i += blockDim.x)
    mask[i / E][i % E] = 0ull;
  __syncthreads();
  const int rho = find_entry(rt.chunk_base, rt.n, b);
  const int T = rt.tok_base[rho + 1] - rt.tok_base[rho];
  const int t0 = (b - rt.chunk_base[rho]) * kPermChunk;
  const int t = t0 + threadIdx.x;
  const bool valid = t < T;
  const int32_t* ix = in_global(rt.idx[rho]) + (size_t)t * k;
  if (valid)
    for (int r = 0; r < k; ++r) atomicOr(&mask[wave][clamp_expert(ix[r], E)], 1ull << lane);
  __syncthreads();
  if (valid) {
    const unsigned long long below = (1ull << lane) - 1ull;
    const int32_t* cb = chunk_base + (size_t)b * ES;
    const size_t q0 = (size_t)(rt.tok_base[rho] + t) * slots;
    for (int r = 0; r < slots; ++r) {
      int pos;
      if (r < k) {
        const int e = clamp_expert(ix[r], E);
        int rank = __popcll(mask[wave][e] & below);
        for (int w2 = 0; w2 < wave; ++w2) rank += __popcll(mask[w2][e]);
        pos = cb[e] + rank;
      } else {
        pos = cb[E + (r - k)] + threadIdx.x;  // every token of the chunk has it
      }
      inv[q0 + r] = pos;
      if (perm) perm[pos] = (int32_t)(q0 + r);
    }
  }
}

// ---------------------------------------------------------------------------
// Count, scan and scatter of a small step in one workgroup.  The three
// launches above each take about 5 us for a step of a few hundred tokens
// whatever they do, one after the other; here the pairs of 64 tokens at a time
// (a piece, one token per lane) are counted in LDS, scanned and placed without
// leaving the CU.  The same integers as the three kernels give, also for a
// token that picks an expert more than once (a caller's picks may): such pairs
// share the token's row, one for each token of a kPermChunk-token chunk, and
// the next chunk starts after all the pairs counted.
// Bound by the latency of its phases, then by one CU's LDS atomics and
// scattered stores; a wavefront takes a second piece from the 17th on.
// Kernel times: 8 to 10 us up to 4 pieces, 11 at 8 pieces of 8 slots (over 64
// experts) and 16 of 2, 16 at 16 of 8, 15 at 32 of 2; 20 at 16 of 8 over 256
// experts.  What the three launches take depends on their chunks; per step of
// a pass, one workgroup less three launches, in us:
//   entries of 64 tokens (a chunk each): 20 pieces of 2 slots over 8 experts
//     -3.0, of 4 over 256 -4.1, of 6 over 64 -1.4; 16 of 8 over 64 +0.9, over
//     128 -0.6;
//   entries of 128 tokens (two pieces a chunk): 16 pieces of 8 over 60 -2.3, over
//     256 +2.3; 32 of 2 over 8 +0.2;
//   entries of 256 tokens (four pieces a chunk): 16 pieces of 2 slots over 8
//     experts -1.6, of 6 over 64 -1.4, of 4 over 256 -0.7, of 8 over 64 +1.0,
//     of 8 over 256 +3.1; 12 of 8 over 256 -1.2; 28 of 2 over 8 +1.1, of 4
//     over 256 +4.5.
// Hence the limits (perm_small): with a chunk for every two pieces up to 32
// pieces and 128 pieces x slots, fewer with many experts; else one piece per
// wavefront and 128 pieces x (slots + experts / 96).
constexpr int kSmallPieces = 32;      // pieces of a small step
constexpr int kSmallSlots = 128;      // pieces x slots of a small step
constexpr int kSmallWords = 23040;    // LDS words for the pieces' expert masks and counts (90 KB)
static_assert(EB_MAX_RUN <= kWave, "one lane per entry");
// Grouped rows of up to kSmallCopy bytes are written here too (row_bytes > 0):
// a launch less.  One token of 8 slots at H = 2048: step + combine 41.5 ->
// 39.8 us; two tokens 57.0 -> 55.2; from eight tokens on one CU's stores take
// as long as the launch saved.
constexpr int kSmallCopy = 128 * 1024;
constexpr int kSmallRows = kSmallCopy / 512;  // a row has at least 512 bytes (H is a multiple of 256)
constexpr int kSmallRowPiece = kWave * 16;    // bytes of a row one wavefront copies

template <class RTA>
__global__ __launch_bounds__(kScanThreads) void perm_small_kernel(
    RTA rta, int32_t* __restrict__ offsets, int4* __restrict__ tiles, int bm, TailRule tail, int max_tiles,
    int32_t* __restrict__ work_ctr, int32_t* __restrict__ perm, int32_t* __restrict__ inv, int row_bytes,
    uint8_t* __restrict__ a_perm) {
  __shared__ int running[kMaxKeys];                        // per-key totals, then offsets / cursors
  __shared__ unsigned long long masks[kSmallWords / 2];    // [pieces][E] lanes per expert, then the counts
  __shared__ int wtot[kScanWaves], s_layer[kSmallPieces];
  __shared__ int s_pos[kSmallRows];                        // inv of a step whose rows are copied here
  const RunTable& rt = rta.get();
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int E = rt.E, S = rt.S, k = rt.k, n = rt.n, ES = E + S, slots = k + S, n_keys = rt.L * ES;

  // value of a uniform lane, in a scalar register (a shuffle goes through LDS)
  auto lane_of = [](int v, int from) { return __builtin_amdgcn_readlane(v, from); };
  // lane i: entry i's first piece (pieces of an entry in token order, entries in order)
  const int tok0 = lane < n ? rt.tok_base[lane] : 0, len = lane < n ? rt.tok_base[lane + 1] - tok0 : 0;
  int upto = (len + kWave - 1) / kWave;
  const int own = upto;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int y = __shfl_up(upto, off, kWave);
    if (lane >= off) upto += y;
  }
  const int np = min(lane_of(upto, kWave - 1), kSmallPieces);
  int* cnt = reinterpret_cast<int*>(masks + np * E);       // [pieces][ES] counts, then first positions

  // this lane's token of piece p and its picks
  struct Token {
    int rho, q0, rows;     // entry, first pair, tokens of the piece
    int last;              // last piece of its chunk
    int e[kMaxSlots];
  } tk;
  auto load = [&](int p) {
    tk.rho = __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < n && upto <= p)));
    const int last = lane_of(upto, tk.rho), first = last - lane_of(own, tk.rho), t0 = (p - first) * kWave;
    tk.rows = min(kWave, lane_of(len, tk.rho) - t0);
    tk.last = min(first + ((p - first) | (kPermChunk / kWave - 1)), last - 1);
    tk.q0 = (lane_of(tok0, tk.rho) + t0 + lane) * slots;
    const int32_t* ix = in_global(rt.idx[tk.rho]) + (size_t)(t0 + lane) * k;
#pragma unroll
    for (int r = 0; r < kMaxSlots; ++r)
      if (r < k && lane < tk.rows) tk.e[r] = clamp_expert(ix[r], E);
  };
  int p_last = -1;         // the piece in tk
  if (wave < np) load(p_last = wave);

  // copy unit u: 1 KB piece u % row_pieces of token u / row_pieces; a
  // wavefront's first one is read now
  const int row_pieces = (row_bytes + kSmallRowPiece - 1) / kSmallRowPiece;
  const int units = rt.tok_base[n] * row_pieces;
  uint4 row = make_uint4(0, 0, 0, 0);
  auto read_row = [&](int u) {
    const int g = u / row_pieces, at = (u - g * row_pieces) * kSmallRowPiece + lane * 16;
    const int rho = __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < n && tok0 + len <= g)));
    const int t = g - lane_of(tok0, rho);
    const uint8_t* src = in_global(static_cast<const uint8_t*>(rt.a[rho])) + (size_t)t * row_bytes;
    if (at < row_bytes) row = *reinterpret_cast<const uint4*>(src + at);
  };
  if (wave < units) read_row(wave);

  if (tid < kWorkWords && tid != kWorkTiles && tid != kWorkTiles + 1) work_ctr[tid] = 0;
  for (int i = tid; i < n_keys; i += kScanThreads) running[i] = 0;
  for (int i = tid; i < np * E; i += kScanThreads) masks[i] = 0ull;
  for (int i = tid; i < np * ES; i += kScanThreads) cnt[i] = 0;
  __syncthreads();
  for (int p = wave; p < np; p += kScanWaves) {
    if (p != p_last) load(p_last = p);
    if (lane == 0) s_layer[p] = rt.layer[tk.rho];
    if (lane < S) cnt[p * ES + E + lane] = tk.rows;
#pragma unroll
    for (int r = 0; r < kMaxSlots; ++r)
      if (r < k && lane < tk.rows) {
        atomicOr(&masks[p * E + tk.e[r]], 1ull << lane);
        // a repeated pick has no row of its own: it counts at the chunk's end
        bool again = false;
#pragma unroll
        for (int i = 0; i < r; ++i) again |= tk.e[i] == tk.e[r];
        atomicAdd(&cnt[(again ? tk.last : p) * ES + tk.e[r]], 1);
      }
  }
  __syncthreads();
  for (int i = tid; i < np * ES; i += kScanThreads) {
    const int p = i / ES;
    const int v = cnt[i];
    if (v) atomicAdd(&running[s_layer[p] * ES + i - p * ES], v);
  }
  __syncthreads();
  offsets_and_tiles(running, n_keys, wtot, offsets, tiles, bm, tail, max_tiles, work_ctr);
  // first position of every (piece, column): the pieces in order
  for (int c = tid; c < ES; c += kScanThreads) {
    int layer = -1, cur = 0;
    for (int p0 = 0; p0 < np; p0 += 8) {
      int v[8], l[8];  // read ahead of the stores
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (p0 + j < np) {
          v[j] = cnt[(p0 + j) * ES + c];
          l[j] = s_layer[p0 + j];
        }
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (p0 + j < np) {
          if (l[j] != layer) {
            if (layer >= 0) running[layer * ES + c] = cur;
            cur = running[l[j] * ES + c];
            layer = l[j];
          }
          cnt[(p0 + j) * ES + c] = cur;
          cur += v[j];
        }
    }
  }
  __syncthreads();
  for (int p = p_last; p >= 0; p -= kScanWaves) {
    if (p != p_last) load(p);
    if (lane >= tk.rows) continue;
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < kMaxSlots; ++r)
      if (r < slots) {
        const int pos = r < k ? cnt[p * ES + tk.e[r]] + __popcll(masks[p * E + tk.e[r]] & below)
                              : cnt[p * ES + E + (r - k)] + lane;
        inv[tk.q0 + r] = pos;
        if (perm) perm[pos] = tk.q0 + r;
        if (row_bytes > 0) s_pos[tk.q0 + r] = pos;
      }
  }
  if (units == 0) return;
  __syncthreads();
  for (int u = wave; u < units; u += kScanWaves) {
    if (u != wave) read_row(u);
    const int g = u / row_pieces, at = (u - g * row_pieces) * kSmallRowPiece + lane * 16;
    for (int r = 0; r < slots; ++r)
      if (at < row_bytes) *reinterpret_cast<uint4*>(a_perm + (size_t)s_pos[g * slots + r] * row_bytes + at) = row;
  }
}

// One wavefront per (token, 1 KB piece of its row): the piece is read once
// (one 16-byte load per lane) and written to the grouped positions inv[q]
// of all the token's k+S pairs.  Reading each row once per pair instead (one
// wavefront per grouped row) moves up to k+S times the read bytes; pieces of
// 2 KB keep fewer wavefronts in flight.
constexpr int kGatherU = 1;                  // 16-byte loads per lane per piece
constexpr int kGatherPiece = 64 * kGatherU;  // 16-byte chunks per piece

template <class RTA>
__global__ __launch_bounds__(256) void gather_tokens_kernel(RTA rta, int pieces, int elem_bytes,
                                                          const int32_t* __restrict__ inv,
                                                          uint8_t* __restrict__ a_perm) {
  const RunTable& rt = rta.get();
  const int total = rt.tok_base[rt.n];
  const int lane = threadIdx.x & 63;
  const long long wv = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (wv >= (long long)total * pieces) return;
  const int g = (int)(wv / pieces);  // global token of the step
  const int c0 = (int)(wv - (long long)g * pieces) * kGatherPiece;
  const int slots = rt.k + rt.S;
  const int P = total * slots;
  const int rho = find_entry(rt.tok_base, rt.n, g);
  const int t = g - rt.tok_base[rho];
  const size_t row_bytes = (size_t)rt.H * elem_bytes;
  const uint4* src = reinterpret_cast<const uint4*>(in_global(static_cast<const uint8_t*>(rt.a[rho])) + (size_t)t * row_bytes);
  // lane r < slots holds the grouped position of slot r (clamped into range)
  const int pos = lane < slots ? min(max(inv[(size_t)g * slots + lane], 0), P - 1) : 0;
  const int n16 = (int)(row_bytes / 16);
  uint4 v[kGatherU];
#pragma unroll
  for (int j = 0; j < kGatherU; ++j) {
    const int c = c0 + 64 * j + lane;
    if (c < n16) v[j] = src[c];
  }
  for (int r = 0; r < slots; ++r) {
    uint4* dst = reinterpret_cast<uint4*>(a_perm + (size_t)__shfl(pos, r, 64) * row_bytes);
#pragma unroll
    for (int j = 0; j < kGatherU; ++j) {
      const int c = c0 + 64 * j + lane;
      if (c < n16) dst[c] = v[j];
    }
  }
}

}  // namespace

// Launch helpers shared by the host-built (ByValue) and device-written
// (InMemory) tables; grids are the live sizes or the largest step's.
namespace {

template <class RTA>
void perm_count_impl(RTA a, int grid, int32_t* hist, hipStream_t s) {
  prof_start(EB_K_PERM_COUNT, s);
  if (grid > 0) hipLaunchKernelGGL(perm_count_kernel<RTA>, dim3(grid), dim3(kPermChunk), 0, s, a, hist);
  prof_stop(EB_K_PERM_COUNT, s);
}

template <class RTA>
void perm_scan_impl(RTA a, const int32_t* hist, int32_t* chunk_base, int32_t* offsets, int4* tiles,
                    int bm, TailRule tail, int max_tiles, int32_t* work_ctr, hipStream_t s) {
  prof_start(EB_K_PERM_SCAN, s);
  hipLaunchKernelGGL(perm_scan_kernel<RTA>, dim3(1), dim3(kScanThreads), 0, s, a, hist, chunk_base,
                     offsets, tiles, bm, tail, max_tiles, work_ctr);
  prof_stop(EB_K_PERM_SCAN, s);
}

template <class RTA>
void perm_scatter_impl(RTA a, int grid_chunks, const int32_t* chunk_base, int32_t* perm, int32_t* inv, hipStream_t s) {
  prof_start(EB_K_PERM_SCATTER, s);
  if (grid_chunks > 0)
    hipLaunchKernelGGL(perm_scatter_kernel<RTA>, dim3(grid_chunks), dim3(kPermChunk), 0, s, a,
                       chunk_base, perm, inv);
  prof_stop(EB_K_PERM_SCATTER, s);
}

// Whether a step of `pieces` 64-token pieces and `chunks` chunks runs in
// perm_small_kernel: the pieces' masks and counts fit its LDS, and there are
// few enough of them that one workgroup is faster than three launches
// (measured there).
bool perm_small(const eb_model_desc& d, int pieces, int chunks) {
  if (pieces > kSmallPieces || pieces * (3 * d.E + d.S) > kSmallWords) return false;
  const int slots = d.k + d.S;
  const int cost = pieces * (96 * slots + d.E);  // 96 experts count as a slot
  if (2 * chunks >= pieces) return pieces * slots <= kSmallSlots && cost <= 96 * kSmallSlots + 2048;
  return pieces <= kScanWaves && cost <= 96 * kSmallSlots;
}

template <class RTA>
void perm_small_impl(RTA a, const StepBuffers& b, int bm, TailRule tail, int row_bytes, hipStream_t s) {
  prof_start(EB_K_PERM_SCAN, s);
  hipLaunchKernelGGL(perm_small_kernel<RTA>, dim3(1), dim3(kScanThreads), 0, s, a, b.offsets, b.tiles, bm, tail,
                     b.max_tiles, b.work_ctr, b.perm, b.inv, row_bytes, static_cast<uint8_t*>(b.a_perm));
  prof_stop(EB_K_PERM_SCAN, s);
}

template <class RTA>
void gather_impl(RTA a, int H, int grid_tokens, int elem_bytes, const int32_t* inv, void* a_perm, hipStream_t s) {
  const size_t row_bytes = (size_t)H * elem_bytes;
  prof_start(EB_K_PERM_GATHER, s);
  if (grid_tokens > 0) {
    const int n16 = (int)(row_bytes / 16);
    const int pieces = (n16 + kGatherPiece - 1) / kGatherPiece;
    const long long waves = (long long)grid_tokens * pieces;
    hipLaunchKernelGGL(gather_tokens_kernel<RTA>, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, a,
                       pieces, elem_bytes, inv, static_cast<uint8_t*>(a_perm));
  }
  prof_stop(EB_K_PERM_GATHER, s);
}

// The whole grouping: grid_chunks / grid_tokens are the chunks and tokens the
// grids cover, pieces the most 64-token pieces the entries can have.
template <class RTA>
void permute_impl(RTA a, const eb_model_desc& d, int grid_chunks, int grid_tokens, int pieces, const StepBuffers& b,
                  hipStream_t s) {
  const int bm = gemm_bm(d.dtype);
  const TailRule tail = gemm_tail(d.dtype, d.F);
  const int elem_bytes = d.dtype == EB_DTYPE_BF16 ? 2 : 4;
  if (perm_small(d, pieces, grid_chunks)) {
    const bool copy = (long long)grid_tokens * (d.k + d.S) * d.H * elem_bytes <= kSmallCopy;
    perm_small_impl(a, b, bm, tail, copy ? d.H * elem_bytes : 0, s);
    if (copy) return;
  } else {
    perm_count_impl(a, grid_chunks, b.hist, s);
    perm_scan_impl(a, b.hist, b.chunk_base, b.offsets, b.tiles, bm, tail, b.max_tiles, b.work_ctr, s);
    perm_scatter_impl(a, grid_chunks, b.chunk_base, b.perm, b.inv, s);
  }
  gather_impl(a, d.H, grid_tokens, elem_bytes, b.inv, b.a_perm, s);
}

bool scan_fits(int L, int E, int S, int n) {
  return (long)L * (E + S) <= kMaxKeys && E + S <= kScanThreads && n <= EB_MAX_RUN;
}

}  // namespace

hipError_t launch_permute(const eb_model_desc& d, const RunTable& rt, const StepBuffers& b, hipStream_t s) {
  if (!scan_fits(d.L, d.E, d.S, rt.n)) return hipErrorInvalidValue;
  int pieces = 0;
  for (int i = 0; i < rt.n; ++i) pieces += (rt.tok_base[i + 1] - rt.tok_base[i] + kWave - 1) / kWave;
  permute_impl(ByValue<RunTable>{rt}, d, rt.chunk_base[rt.n], rt.tok_base[rt.n], pieces, b, s);
  return hipGetLastError();
}

hipError_t launch_permute_dev(const eb_model_desc& d, const RunTable* rt, int N, int T, const StepBuffers& b,
                              hipStream_t s) {
  if (!scan_fits(d.L, d.E, d.S, 0)) return hipErrorInvalidValue;
  permute_impl(InMemory<RunTable>{rt}, d, N * ((T + kPermChunk - 1) / kPermChunk), N * T,
               N * ((T + kWave - 1) / kWave), b, s);
  return hipGetLastError();
}

}  // namespace eb
