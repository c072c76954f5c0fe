// Small data-movement kernels around the attention kernels:
//  - transpose: V -> V^T (so the PV product reads 16-byte MFMA operands);
//  - gather_strips: K rows and V^T columns gathered by selected column index into
//    compact per-head arrays (Algorithm 1, merge_index: column strips);
//  - strip_prep: the selected columns and offsets (plus the local window) as
//    bitmaps, and the list of 64-key tile diagonals that hold at least one kept
//    offset (Algorithm 1, merge_index: slash strips extended over the matrix);
//  - block granularity (Algorithm 1, block_reduction with blk > 1): token scores
//    summed over blocks, and the block lists turned into the same metadata.
#include "sa_device.h"
#include "sa_kernels.h"

namespace sa {

namespace {

constexpr int GT_ROW_B = 260;   // bytes per gathered row in LDS (256 + 4 pad)

// 64 rows staged in LDS -> 128 transposed rows of 64 entries (128 bytes each)
__device__ __forceinline__ void store_transposed(const char* tile, uint16_t* out, size_t out_stride, int tid) {
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    int c = tid + 256 * n;
    int drow = c >> 3, kc = c & 7;
    uint16_t e[8];
#pragma unroll
    for (int x = 0; x < 8; ++x)
      e[x] = *reinterpret_cast<const uint16_t*>(tile + (8 * kc + x) * GT_ROW_B + drow * 2);
    uint4 v;
    v.x = e[0] | ((uint32_t)e[1] << 16);
    v.y = e[2] | ((uint32_t)e[3] << 16);
    v.z = e[4] | ((uint32_t)e[5] << 16);
    v.w = e[6] | ((uint32_t)e[7] << 16);
    *reinterpret_cast<uint4*>(out + (size_t)drow * out_stride + 8 * kc) = v;
  }
}

__device__ __forceinline__ void stage_chunk(char* tile, int row, int col, uint4 v) {
  uint32_t* dst = reinterpret_cast<uint32_t*>(tile + row * GT_ROW_B + col * 16);
  dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
}

// V -> V^T, zero padded to S_pad keys
__global__ __launch_bounds__(256) void transpose_kernel(const uint16_t* v, uint16_t* vt, int S, int S_pad) {
  __shared__ __attribute__((aligned(16))) char tile[64 * GT_ROW_B];
  const int g = blockIdx.y, c0 = blockIdx.x * 64, tid = threadIdx.x;
  if (c0 >= ((S + 63) & ~63)) return;   // nothing reads beyond the last partial tile
  const uint16_t* src = v + (size_t)g * S * kHeadDim;
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const int c = tid + 256 * n, row = c >> 4, col = c & 15;
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (c0 + row < S) x = *reinterpret_cast<const uint4*>(src + (size_t)(c0 + row) * kHeadDim + col * 8);
    stage_chunk(tile, row, col, x);
  }
  __syncthreads();
  store_transposed(tile, vt + (size_t)g * kHeadDim * S_pad + c0, S_pad, tid);
}

// The column side of the strip mask: a workgroup takes 64 entries of one head's list, writes
// the padded copy of them (INT_MAX marks "no column"), their K rows and, transposed through
// LDS, their V rows.  K and V go in one launch: both read the list, and a launch of its own
// costs 5 us, as much as the whole gather of a short sequence.
__global__ __launch_bounds__(256) void gather_strips_kernel(GatherParams P) {
  __shared__ __attribute__((aligned(16))) char tile[64 * GT_ROW_B];
  const int g = blockIdx.y;
  const int c0 = blockIdx.x * 64;
  const int cnt = min(max(P.cnt[g], 0), P.S);
  const int tid = threadIdx.x;
  if (P.dlist[(size_t)g * P.dlist_stride] & kSweepBit) return;
  const int32_t* list = P.idx + (size_t)g * P.S;
  if (tid < 64) P.idx_pad[(size_t)g * P.S_pad + c0 + tid] = (c0 + tid < cnt) ? list[c0 + tid] : 0x7FFFFFFF;
  if (c0 >= ((cnt + 63) & ~63)) return;   // nothing reads beyond the last partial tile
  // rows of an earlier segment see no key at or after their end: a tile of the ascending
  // list that starts there is left alone
  const int key_limit = P.key_limit[g / P.heads_per_seg];
  if (key_limit > 0 && list[c0] >= key_limit) return;
  const size_t kv = (size_t)((P.head0 + g % P.heads_per_seg) / P.group) * P.S * kHeadDim;
  uint4 kr[4], vr[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const int c = tid + 256 * n, cc = c0 + (c >> 4), col = c & 15;
    kr[n] = vr[n] = make_uint4(0u, 0u, 0u, 0u);
    if (cc < cnt) {
      const int j = min(max(list[cc], 0), P.S - 1);   // a malformed list must not read out of bounds
      const size_t at = kv + (size_t)j * kHeadDim + col * 8;
      kr[n] = *reinterpret_cast<const uint4*>(P.k + at);
      vr[n] = *reinterpret_cast<const uint4*>(P.v + at);
    }
  }
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const int c = tid + 256 * n, row = c >> 4, col = c & 15;
    *reinterpret_cast<uint4*>(P.kc + ((size_t)g * P.S_pad + c0 + row) * kHeadDim + col * 8) = kr[n];
    stage_chunk(tile, row, col, vr[n]);
  }
  __syncthreads();
  store_transposed(tile, P.vct + (size_t)g * kHeadDim * P.S_pad + c0, P.S_pad, tid);
}

constexpr int PT = 1024;               // threads of the metadata kernels
constexpr int kBitSegWords = 32768;    // bitmap words a workgroup holds in LDS: 1M keys or offsets

// word w of a bitmap whose set bits are the run [lo, hi]
__device__ __forceinline__ uint32_t run_word(int w, int lo, int hi) {
  const int x0 = w << 5;
  if (x0 > hi || x0 + 31 < lo) return 0u;
  uint32_t m = 0xFFFFFFFFu;
  if (lo > x0) m &= 0xFFFFFFFFu << (lo - x0);
  if (hi < x0 + 31) m &= 0xFFFFFFFFu >> (x0 + 31 - hi);
  return m;
}

// any kept offset in [lo, hi] (0 <= lo <= hi)?  offset o sits at bit off_max - o
__device__ bool any_offset(const uint32_t* ob, int off_max, int lo, int hi) {
  int x_lo = off_max - hi, x_hi = off_max - lo;
  for (int w = x_lo >> 5; w <= (x_hi >> 5); ++w) {
    uint32_t m = 0xFFFFFFFFu;
    if (w == (x_lo >> 5)) m &= 0xFFFFFFFFu << (x_lo & 31);
    if (w == (x_hi >> 5)) m &= 0xFFFFFFFFu >> (31 - (x_hi & 31));
    if (ob[w] & m) return true;
  }
  return false;
}

// Tile diagonal d pairs the 256-row query tile starting at row i0 with the
// 64-key tile starting at key i0 + 192 - 64 d: it spans offsets
// [64 d - 255, 64 d + 63], the 32 rows of wave w (of 8) the 95 offsets from
// 64 d - 255 + 32 w on.  dlist = ascending d with at least one kept offset; an
// entry is d | (mask << 24), bit w of mask set when wave w sees a kept offset.
//
// Sum of x over the workgroup, known to every thread.
__device__ __forceinline__ long long block_sum(long long x, long long* scratch) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = x;
  __syncthreads();
  long long t = 0;
  for (int w = 0; w < PT / 64; ++w) t += scratch[w];
  return t;
}

// Whether a head is swept: every causal key tile visited once, columns and offsets kept in
// one mask, instead of the gathered columns first and then every tile diagonal with a kept
// offset, columns masked out.  Where the lists are full the two passes visit nearly every
// key twice (8K tokens of a diffuse head at alpha = 0.95: 1.9 x the tiles of a sweep).
//
// The rule compares tile costs in 1/128 of a tile of the dense kernel, fitted at 2K, 16K and
// 64K tokens (32 heads, 5-90 % of the columns, 0.4-20 runs of four offsets per 2000):
// a gathered tile 132, a range tile 76 + 7 per wave that works on it (idle waves are cheaper,
// but the tile's loads and barrier are paid), a swept tile 134 to 144.  At 64K, 60 % columns:
// 32 runs 19.2 ms in two passes / 30.9 swept, 218 runs 29.7 / 30.9, 436 runs 35.7 / 30.9,
// 1638 runs 45.2 / 31.1.
constexpr int kColTileCost = 132, kRangeTileCost = 76, kRangeWaveCost = 7, kSweepTileCost = 140;
// Which core a head in two passes is for (kSparseBit: core 1): what core 0 gains on a gathered tile and on
// every wave that works on a range tile, against what it loses on a range tile whose other waves wait, in the unit of
// the costs above.  Core 0 / core 1, 32 heads of 64K: 20 % of the columns 5.9 / 6.2 ms (5 a tile), runs of one offset every
// 1000 6.6 / 5.1 (-18 a range tile, 2.4 waves at work), four every 300 20.8 / 16.5 (-15), 128 every 1000 10.0 / 9.0 (-9, 4 waves), 700
// every 4000 6.8 / 7.2 (+6, 6.2 waves), head patterns 34.1 / 35.2 (7.7 waves).  The line lies where heads of one layer seldom
// fall on both sides, because a launch with both cores is slower than either alone (8 heads of 128K, alpha = 0.95, 4.9 waves:
// 29.3 / 29.3 ms, half and half 30.6): planted slashes at alpha of 0.8 to 0.98 leave 3.4 to 6.1 waves and run up to 5 %
// faster on core 1 (at 0.98 up to 5 % slower), smeared ones 6.4 to 7.8.
constexpr int kCoreColTile = 2, kCoreWave = 5, kCoreRangeTile = 33;

// Written by one workgroup: `active(d, w)` says whether wave w has work on diagonal d.  A
// thread takes one (d, w) pair, a wave eight diagonals at a time (one ballot is eight
// masks), and every wave owns a contiguous run of diagonals: it counts its entries, the
// counts are exchanged once, and it forms the masks again to write them in order.  The
// list of a head that is swept holds every diagonal, with the bits of `swept(d, w)`.
// `col_tiles`: the gathered tiles this thread counted.  `cores`: the launch asks for the core of heads in two
// passes (the sum for it costs 1 us: metadata of 32 heads of 16K with it / without, strips 25.7 / 24.5, blocks 11.1 / 10.2).
template <typename F, typename G>
__device__ __forceinline__ void write_dlist(int nd, int q_lo, int q_hi, long long col_tiles, bool cores, int32_t* dl, int32_t* dcnt,
                                            F&& active, G&& swept) {
  __shared__ int wave_cnt[PT / 64];
  __shared__ long long sums[PT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_groups = (nd + 7) / 8;
  const int g_lo = n_groups * wave / (PT / 64), g_hi = n_groups * (wave + 1) / (PT / 64);
  auto mask_of = [&](int g) {                      // mask of diagonal 8 g + lane / 8
    const int d = 8 * g + (lane >> 3);
    const unsigned long long b = __ballot(d < nd && active(d, lane & 7));
    return (uint32_t)(b >> (lane & ~7)) & 0xFFu;
  };
  // diagonal d is met by the query tiles a with 4 a + 3 >= d
  auto met = [&](int d) { return (long long)max(q_hi - max(q_lo, d / 4), 0); };
  int n = 0;
  long long two_pass = kColTileCost * col_tiles, sweep = 0, core = kCoreColTile * col_tiles;
  for (int g = g_lo; g < g_hi; ++g) {
    const uint32_t mask = mask_of(g);
    const int d = 8 * g + (lane >> 3);
    const bool first = (lane & 7) == 0 && d < nd;
    n += __popcll(__ballot(first && mask != 0u));
    if (first) {
      sweep += kSweepTileCost * met(d);
      if (mask != 0u) two_pass += (kRangeTileCost + kRangeWaveCost * __popc(mask)) * met(d);
      if (mask != 0u) core += (kCoreWave * (int)__popc(mask) - kCoreRangeTile) * met(d);
    }
  }
  if (lane == 0) wave_cnt[wave] = n;
  if (block_sum(two_pass - sweep, sums) > 0) {
    for (int g = g_lo; g < g_hi; ++g) {
      const int d = 8 * g + (lane >> 3);
      const unsigned long long b = __ballot(d < nd && swept(d, lane & 7));
      const uint32_t mask = (uint32_t)(b >> (lane & ~7)) & 0xFFu;
      if ((lane & 7) == 0 && d < nd) dl[d] = (int32_t)((uint32_t)(d | kSweepBit) | (mask << 24));
    }
    if (tid == 0) *dcnt = nd;
    return;
  }
  const uint32_t flag = cores && block_sum(core, sums) < 0 ? (uint32_t)kSparseBit : 0u;
  int at = 0, total = 0;
  for (int w = 0; w < PT / 64; ++w) {
    at += w < wave ? wave_cnt[w] : 0;
    total += wave_cnt[w];
  }
  for (int g = g_lo; g < g_hi; ++g) {
    const uint32_t mask = mask_of(g);
    const bool mine = (lane & 7) == 0 && mask != 0u;
    const unsigned long long b = __ballot(mine);
    if (mine) dl[at + __popcll(b & ((1ull << lane) - 1ull))] = (int32_t)((uint32_t)(8 * g + (lane >> 3)) | flag | (mask << 24));
    at += __popcll(b);
  }
  if (tid == 0) *dcnt = total;
}

// gathered tiles of the query tiles this thread takes: 64 listed columns each, up to the last row
__device__ __forceinline__ long long count_col_tiles(const int32_t* list, int n, int q_lo, int q_hi, int row_hi) {
  long long tiles = 0;
  for (int a = q_lo + (int)threadIdx.x; a < q_hi; a += PT) {
    const int last = min(a * kFlashBQ + kFlashBQ, row_hi) - 1;
    int lo = 0, hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (list[mid] <= last) lo = mid + 1; else hi = mid;
    }
    tiles += (lo + kFlashBK - 1) / kFlashBK;
  }
  return tiles;
}

// Strip masks: wave w meets the offsets [64 d - 255 + 32 w, 64 d - 161 + 32 w] on diagonal d.
__device__ __forceinline__ void write_strip_dlist(const MaskPrepParams& P, int h, const uint32_t* ob) {
  const SegmentJob& J = P.seg[h / P.heads_per_seg];
  const int q_lo = J.qtile0, q_hi = J.qtile0 + J.n_qtiles;
  const long long col = count_col_tiles(P.col_idx + (size_t)h * P.S, min(max(P.col_cnt[h], 0), P.S), q_lo, q_hi, J.row_hi);
  write_dlist((P.S + 63) / 64 + 3, q_lo, q_hi, col, P.cores != 0, P.dlist + (size_t)h * P.dlist_stride, P.dcnt + h,
              [&](int d, int w) {
                const int lo = max(0, 64 * d - 255 + 32 * w), hi = min(P.S - 1, 64 * d - 255 + 32 * w + 94);
                return lo <= hi && any_offset(ob, P.off_max, lo, hi);
              },
              [&](int d, int w) { return 64 * d - 255 + 32 * w + 94 >= 0 && 64 * d - 255 + 32 * w <= P.S - 1; });
}

// The metadata of a strip mask in one launch.  One workgroup builds a head's offset bitmap in
// LDS (the window first, then the listed offsets), stores it and lists the tile diagonals it
// touches; another builds the head's column bitmap.  Two fills, a bit-setting launch over
// global atomics (12 us for one head of 1K tokens, 41 us for 32 heads of 8K: neighbouring
// list entries hit the same word) and a list launch became this one.  A bitmap longer than
// kBitSegWords (1M tokens) is cut into segments, each of which goes through the whole list;
// the tile diagonals are then listed by dlist_kernel.
__global__ __launch_bounds__(PT) void strip_prep_kernel(MaskPrepParams P, int n_seg) {
  extern __shared__ __attribute__((aligned(16))) uint32_t bits[];
  const int h = blockIdx.y, tid = threadIdx.x;
  const bool cols = (int)blockIdx.x >= n_seg;
  const int w0 = ((int)blockIdx.x - (cols ? n_seg : 0)) * kBitSegWords;
  const int words = cols ? P.cb_words : P.rb_words;
  const int nw = min(kBitSegWords, words - w0);
  if (nw <= 0) return;
  if (blockIdx.x == 0 && tid == 0 && P.tiles != nullptr && h < P.heads_per_seg) P.tiles[h] = 0ull;
  const int32_t* list = (cols ? P.col_idx : P.slash_idx) + (size_t)h * P.S;
  const int n = min(max((cols ? P.col_cnt : P.slash_cnt)[h], 0), P.S);
  // bit x of the offset bitmap is offset off_max - x: the window is the run of bits up to off_max
  const int win_lo = cols ? 0x7FFFFFFF : P.off_max - (min(P.window, P.S) - 1);
  for (int x = tid; x < nw; x += PT) bits[x] = run_word(w0 + x, win_lo, P.off_max);
  __syncthreads();
  constexpr int B = 8;                      // entries a thread requests before it uses the first
  for (int c0 = 0; c0 < n; c0 += B * PT) {
    int v[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int c = c0 + u * PT + tid;
      v[u] = c < n ? list[c] : -1;
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      if (v[u] < 0 || v[u] >= P.S) continue;          // (also entries a malformed list may hold)
      const int x = cols ? v[u] : P.off_max - v[u];
      const int at = (x >> 5) - w0;
      if (at >= 0 && at < nw) atomicOr(bits + at, 1u << (x & 31));
    }
  }
  __syncthreads();
  uint32_t* out = cols ? P.col_bits + (size_t)h * P.cb_words : P.off_bits + (size_t)h * P.rb_words;
  for (int x = tid; x < nw; x += PT) out[w0 + x] = bits[x];
  if (cols || n_seg != 1) return;
  write_strip_dlist(P, h, bits);
}

// the tile diagonals of a head whose offset bitmap was written in several segments
__global__ __launch_bounds__(PT) void dlist_kernel(MaskPrepParams P) {
  write_strip_dlist(P, blockIdx.x, P.off_bits + (size_t)blockIdx.x * P.rb_words);
}

// ---- block granularity ----------------------------------------------------------
// out[g][b] = sum of in[g][b*blk .. (b+1)*blk) (the last block may be short): one
// wave per block, lanes stride the block, fp64 partial sums combined in a fixed
// butterfly order, so the result does not depend on the launch.
__global__ __launch_bounds__(256) void block_reduce_kernel(const float* in, float* out, int S, int blk, int nb) {
  const int g = blockIdx.y;
  const int b = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (b >= nb) return;
  const float* src = in + (size_t)g * S;
  const int lo = b * blk, hi = min(lo + blk, S);
  double acc = 0.0;
  for (int e = lo + lane; e < hi; e += 64) acc += (double)src[e];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
  if (lane == 0) out[(size_t)g * nb + b] = (float)acc;
}

__device__ __forceinline__ int floor_div(int x, int y) { return x >= 0 ? x / y : -((-x + y - 1) / y); }

// The metadata of a block mask in one launch, in the format of the strip path.
//
// Job 0 of a head lists the tile diagonals.  Kept block diagonals (block row minus block
// column): a full block on diagonal delta spans the offsets blk*delta - (blk-1) ..
// blk*delta + (blk-1), so a selected block b of offsets [blk*b, blk*b + blk) lies on
// diagonals b and b + 1, and the window [0, w) on every diagonal with blk*delta - (blk-1)
// <= w - 1.  With 256-row query tiles, 64-key tiles and blk in {64, 128, 256}, the 32 rows
// of wave w lie in one row block and the key tile of tile diagonal d in one column block,
// floor(32 w / blk) - floor((192 - 64 d) / blk) block diagonals apart whatever the query
// tile: the per-wave bit of a list entry says "this wave's block is kept".
//
// The other jobs take kBlockSpan keys each and write, for the selected key blocks seen as
// the token columns they hold, their part of the padded index list (only the last block of
// the sequence can be short, and an ascending list has it last, so slot c belongs to list
// entry c / blk) and of the column bitmap, and their part of the offset bitmap, in which
// every offset 0 .. S-1 is kept (kept blocks are kept whole).
constexpr int kBlockSpan = 8192;
__global__ __launch_bounds__(PT) void block_prep_kernel(BlockPrepParams P) {
  extern __shared__ __attribute__((aligned(16))) uint32_t bits[];   // block diagonals / key blocks
  const int h = blockIdx.y, tid = threadIdx.x;
  const bool diag = blockIdx.x == 0;
  if (diag && tid == 0 && P.tiles != nullptr && h < P.heads_per_seg) P.tiles[h] = 0ull;
  const int32_t* list = (diag ? P.slash_blk : P.col_blk) + (size_t)h * P.nb;
  const int n = min(max((diag ? P.slash_bcnt : P.col_bcnt)[h], 0), P.nb);
  const int n_words = (P.nb + 1) / 32 + 1;
  // the window's diagonals are the run [0, (w + blk - 2) / blk]
  const int win_hi = diag ? (int)min(((long long)P.window + P.blk - 2) / P.blk, (long long)P.nb) : -1;
  for (int x = tid; x < n_words; x += PT) bits[x] = run_word(x, 0, win_hi);
  __syncthreads();
  for (int c = tid; c < n; c += PT) {
    const int b = list[c];
    if (b < 0 || b >= P.nb) continue;
    atomicOr(bits + (b >> 5), 1u << (b & 31));
    if (diag) atomicOr(bits + ((b + 1) >> 5), 1u << ((b + 1) & 31));
  }
  __syncthreads();
  auto has = [&](int b) { return ((bits[b >> 5] >> (b & 31)) & 1u) != 0u; };
  if (diag) {
    // column tiles: the selected key blocks as runs of blk columns
    const SegmentJob& J = P.seg[h / P.heads_per_seg];
    const int q_lo = J.qtile0, q_hi = J.qtile0 + J.n_qtiles;
    long long col = 0;
    const int32_t* cb = P.col_blk + (size_t)h * P.nb;
    const int nc = min(max(P.col_bcnt[h], 0), P.nb);
    for (int c = tid; c < nc; c += PT)
      col += (long long)(P.blk / kFlashBK) * max(q_hi - max(q_lo, (int)((long long)cb[c] * P.blk / kFlashBQ)), 0);
    auto meets = [&](int d, int w) {       // the offsets of the wave on this tile reach into [0, S)
      const int o_lo = 64 * d - 255 + 32 * w;
      return o_lo + 94 >= 0 && o_lo <= P.S - 1;
    };
    auto kept = [&](int d, int w) {
      const int delta = (32 * w) / P.blk - floor_div(192 - 64 * d, P.blk);
      return delta >= 0 && delta <= P.nb && meets(d, w) && has(delta);
    };
    write_dlist((P.S + 63) / 64 + 3, q_lo, q_hi, col, false, P.dlist + (size_t)h * P.dlist_stride, P.dcnt + h, kept, kept);
    return;
  }
  const int span = (int)blockIdx.x - 1, n_span = (int)gridDim.x - 1;
  int n_tok = 0;
  if (n > 0) n_tok = min((n - 1) * P.blk + min(P.blk, P.S - min(max(list[n - 1], 0), P.nb - 1) * P.blk), P.S);
  if (span == 0 && tid == 0) P.tok_cnt[h] = n_tok;
  const int c_lo = span * kBlockSpan, c_hi = min(c_lo + kBlockSpan, P.idx_pad_stride);
  for (int c = c_lo + tid; c < c_hi; c += PT) {
    const int r = c / P.blk;
    int j = 0x7FFFFFFF;
    if (c < n_tok) j = min(min(max(list[r], 0), P.nb - 1) * P.blk + c % P.blk, P.S - 1);   // (a malformed list must not lead out of bounds)
    P.idx_pad[(size_t)h * P.idx_pad_stride + c] = j;
  }
  // words of the two bitmaps: kBlockSpan / 32 a job, the last job takes the few beyond
  const int w_lo = span * (kBlockSpan / 32);
  const int cw_hi = span + 1 < n_span ? w_lo + kBlockSpan / 32 : P.cb_words;
  for (int x = w_lo + tid; x < cw_hi; x += PT) {
    const int b = x * 32 / P.blk;
    P.col_bits[(size_t)h * P.cb_words + x] = (b < P.nb && has(b)) ? run_word(x, 0, P.S - 1) : 0u;
  }
  const int ow_hi = span + 1 < n_span ? w_lo + kBlockSpan / 32 : P.rb_words;
  for (int x = w_lo + tid; x < ow_hi; x += PT)
    P.off_bits[(size_t)h * P.rb_words + x] = run_word(x, P.off_max - (P.S - 1), P.off_max);
}

}  // namespace

hipError_t launch_block_reduce(const float* in, float* out, int n_rows, int S, int blk, hipStream_t st) {
  const int nb = (S + blk - 1) / blk;
  if (n_rows == 0 || nb == 0) return hipSuccess;
  hipLaunchKernelGGL(block_reduce_kernel, dim3((nb + 3) / 4, n_rows), dim3(256), 0, st, in, out, S, blk, nb);
  return hipGetLastError();
}

// Kernels with a sequence-sized LDS array.  The limit belongs to the kernel, for all threads of
// the process, so it is the most that any launch asks for, never what this launch asks for.
constexpr size_t kStripPrepLds = (size_t)kBitSegWords * 4;
constexpr size_t kBlockPrepLds = (size_t)((kMaxSeqLen / kFlashBK + 1) / 32 + 1) * 4;   // (blocks of 64 keys are the shortest)
template <typename K>
static hipError_t allow_lds(K kernel, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_block_prep(const BlockPrepParams& P, hipStream_t st) {
  const size_t lds = (size_t)((P.nb + 1) / 32 + 1) * 4;
  hipError_t e = allow_lds(&block_prep_kernel, kBlockPrepLds);
  if (e != hipSuccess) return e;
  dim3 grid(1 + (P.idx_pad_stride + kBlockSpan - 1) / kBlockSpan, P.n_bh);
  hipLaunchKernelGGL(block_prep_kernel, grid, dim3(PT), lds, st, P);
  return hipGetLastError();
}

hipError_t launch_transpose(const uint16_t* v, uint16_t* vt, int n, int S, int S_pad, hipStream_t st) {
  dim3 grid(S_pad / 64, n);
  if (grid.x == 0 || grid.y == 0) return hipSuccess;
  hipLaunchKernelGGL(transpose_kernel, grid, dim3(256), 0, st, v, vt, S, S_pad);
  return hipGetLastError();
}

hipError_t launch_gather_strips(const GatherParams& P, hipStream_t st) {
  dim3 grid(P.S_pad / 64, P.n_heads);
  if (grid.x == 0 || grid.y == 0) return hipSuccess;
  hipLaunchKernelGGL(gather_strips_kernel, grid, dim3(256), 0, st, P);
  return hipGetLastError();
}

hipError_t launch_mask_prep(const MaskPrepParams& P, hipStream_t st) {
  const int n_seg = (P.rb_words + kBitSegWords - 1) / kBitSegWords;   // (the column bitmap is the shorter one)
  const size_t lds = (size_t)(n_seg == 1 ? P.rb_words : kBitSegWords) * 4;
  hipError_t e = allow_lds(&strip_prep_kernel, kStripPrepLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(strip_prep_kernel, dim3(2 * n_seg, P.n_bh), dim3(PT), lds, st, P, n_seg);
  if (n_seg > 1) {
    hipLaunchKernelGGL(dlist_kernel, dim3(P.n_bh), dim3(PT), 0, st, P);
  }
  return hipGetLastError();
}

}  // namespace sa
