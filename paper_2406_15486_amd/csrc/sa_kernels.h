// Host-visible declarations of the kernel launchers (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sa {

constexpr int kHeadDim = 128;  // the only supported head dimension
constexpr int kFlashBQ = 256;  // query rows per workgroup of the flash kernels
constexpr int kFlashBK = 64;   // keys per tile
constexpr int kMaxSeqLen = 1 << 24;   // kernels keep 32-bit byte offsets into V^T
constexpr int kSweepBit = 1 << 23;   // in every entry of a tile-diagonal list: the head is swept
constexpr int kSparseBit = 1 << 22;  // ... or (strips, see two_cores) its tiles leave many waves without work

// One launch may take up to kMaxSegs query segments (Algorithm 1's chunks), each with lists of its own;
// tile0, part0: tiles and parts of the segments before.
constexpr int kMaxSegs = 8;
struct SegmentJob {
  int qtile0, n_qtiles, tile0;   // modes 0 and 2: its query tiles of the launch
  int row_lo, row_hi;            // its rows of the launch: others are neither computed nor written (mode 1: the sampled rows)
  int part0;                     // (set by the launch)
  int lse_parts;                 // mode 1: parts the keys of a query tile are cut into (a power of two); lse is
                                 // [lse_parts, n_slots, n_qrows] partial values, combined by launch_lse_combine
  int k_splits;                  // ... and the workgroups they are given to (a power of two, <= lse_parts)
};

struct FlashParams {
  const uint16_t* q;        // [n_bh, S, 128] bf16
  const uint16_t* k;        // [n_bkv, S, 128] bf16
  const uint16_t* vt;       // [n_bkv, 128, S_pad] bf16 (V transposed, zero padded)
  void* out;                // [n_bh, S, 128] bf16 or fp32
  float* lse;               // nullable
  int S, S_pad;
  int n_bh, n_bkv, group;   // batch*q-heads, batch*kv-heads, q heads per kv head
  int head0;                // strip-masked mode: q, out, lse, tiles and the per-head metadata start at this
                            // (batch*q-)head, n_bh counts the heads of this pass; KV head = (head0 + h) / group
  float scale_log2;         // softmax scale * log2(e)
  int n_seg;                // segments of the launch; per-head metadata and row log-sum-exps are [n_seg, n_bh]
  SegmentJob seg[kMaxSegs];
  int n_slots;              // n_seg * n_bh
  int n_qtiles;             // 256-row query tiles of all segments; mode 1: of each
  int n_qrows;              // mode 1: sampled rows of a segment
  int cols_in_place;        // strip-masked mode, block lists: column tiles are read from k / vt themselves
                            // (kc, vct unused); col_idx_pad then holds runs of 64 consecutive keys per tile
  int all_tiles;            // modes 0 and 2: query tiles of all heads of the call (of its shortest segment here), whatever this launch takes
  int short_lists;          // mode 2 (set by the launch): heads in two passes take core 1
  int part_m;               // modes 0 and 2: > 0: tile a's schedule is cut into ceil((a + 1) / part_m) workgroups
  float* part_o;            // ... whose sums [part, 256, 128] and then [part, 256, 2] lie here (flash_parts_bytes)
  float* part_ml;           // (set by the launch)
  int parts_per_head;       // (set by the launch)
  // strip-masked mode only
  const uint16_t* kc;           // [n_slots, S_pad, 128] K rows gathered by column index
  const uint16_t* vct;          // [n_slots, 128, S_pad] V rows gathered and transposed
  const int32_t* col_idx_pad;   // [n_slots, cidx_stride] ascending, padded with INT_MAX
  const int32_t* col_cnt;       // [n_slots]
  const uint32_t* col_bits;     // [n_slots, cb_words]  bit j: key j is a selected column
  const uint32_t* off_bits;     // [n_slots, rb_words]  bit x: offset off_max - x is kept
  const int32_t* dlist;         // [n_slots, dlist_stride] ascending touched tile-diagonals
  const int32_t* dcnt;          // [n_slots]
  unsigned long long* tiles;    // nullable [n_bh]: over all segments
  int cidx_stride, cb_words, rb_words, dlist_stride, off_max;
};

// mode 0: dense causal; 1: row log-sum-exp of the n_qrows rows from seg[].row_lo on of every segment; 2: strip mask
hipError_t launch_flash(int mode, bool out_f32, const FlashParams& P, hipStream_t st);
// parts of the keys of a query tile (from the sequence alone, at most max_parts) and the workgroups
// that share them (from the heads of the launch too)
void lse_splits(int row_first, int n_s, int n_bh, int max_parts, int* parts, int* workgroups);
// whether heads in two passes may run on either core in a call of S tokens and all_tiles query tiles (core 1 otherwise)
bool two_cores(bool blocks, int S, int all_tiles);
// part_m of a launch over segments of n_bh heads (0: not cut), and the bytes of the partial sums of
// n_heads of them
constexpr int kMaxParts = 256;
constexpr size_t kMaxPartsBytes = (size_t)kMaxParts * kFlashBQ * (kHeadDim + 2) * 4;
int flash_parts(int n_bh, int n_seg, const SegmentJob* seg);
int parts_of(int m, int n_seg, const SegmentJob* seg);
size_t flash_parts_bytes(int m, int n_heads, int n_seg, const SegmentJob* seg);
hipError_t launch_lse_combine(const FlashParams& P, float* out, hipStream_t st);

// vt[g][d][c] = v[g][c][d], zero up to the 64-key tile that ends the sequence
hipError_t launch_transpose(const uint16_t* v, uint16_t* vt, int n, int S, int S_pad, hipStream_t st);

// per head g of the pass, c < cnt[g] (zero up to the end of the 64-entry tile):
//   kc[g][c][:] = k[kv(g)][idx[g][c]][:],  vct[g][:][c] = v[kv(g)][idx[g][c]][:]
struct GatherParams {
  const uint16_t* k; const uint16_t* v;   // [n_kv, S, 128]
  const int32_t* idx;       // [n_heads, S] ascending
  const int32_t* cnt;       // [n_heads]
  uint16_t* kc;             // [n_heads, S_pad, 128]
  uint16_t* vct;            // [n_heads, 128, S_pad]
  int32_t* idx_pad;         // [n_heads, S_pad]: copy of idx padded with INT_MAX
  int n_heads, group;       // source head of head g is (head0 + g) / group
  int head0;
  int S, S_pad;
  const int32_t* dlist;     // [n_heads, dlist_stride]: nothing is gathered for a head that is swept
  int dlist_stride;
  int heads_per_seg;        // n_heads counts the heads of every segment
  int key_limit[kMaxSegs];  // of a segment, > 0: no reader looks at a key >= key_limit; tiles of 64 list entries
                            // that start there are not gathered (their idx_pad entries still are written)
};
hipError_t launch_gather_strips(const GatherParams& P, hipStream_t st);

struct MaskPrepParams {
  const int32_t* col_idx; const int32_t* col_cnt;      // [n_bh, S], [n_bh]
  const int32_t* slash_idx; const int32_t* slash_cnt;
  uint32_t* col_bits; uint32_t* off_bits;
  int32_t* dlist; int32_t* dcnt;
  unsigned long long* tiles;                           // nullable [heads_per_seg]: cleared
  int n_bh, S, window, cb_words, rb_words, dlist_stride, off_max;
  int cores;                                           // the attention launch reads kSparseBit
  int heads_per_seg;                                   // n_bh counts the heads of every segment
  SegmentJob seg[kMaxSegs];                            // the query tiles a segment's masks are for, and the end of their rows
};
hipError_t launch_mask_prep(const MaskPrepParams& P, hipStream_t st);

// block granularity: lists of selected key blocks / offset blocks of blk tokens
struct BlockPrepParams {
  const int32_t* col_blk; const int32_t* col_bcnt;     // [n_bh, nb], [n_bh]
  const int32_t* slash_blk; const int32_t* slash_bcnt;
  int32_t* idx_pad; int32_t* tok_cnt;                  // [n_bh, idx_pad_stride], [n_bh]: the key blocks as token
                                                       // columns, padded with INT_MAX
  uint32_t* col_bits; uint32_t* off_bits;
  int32_t* dlist; int32_t* dcnt;
  unsigned long long* tiles;                           // nullable [heads_per_seg]: cleared
  int n_bh, S, window, cb_words, rb_words, dlist_stride, off_max;
  int heads_per_seg;                                   // n_bh counts the heads of every segment
  SegmentJob seg[kMaxSegs];                            // the query tiles a segment's masks are for, and the end of their rows
  int blk, nb, idx_pad_stride;
};
hipError_t launch_block_prep(const BlockPrepParams& P, hipStream_t st);
// out[r][b] = sum of in[r][b*blk .. (b+1)*blk), r < n_rows, rows of S floats
hipError_t launch_block_reduce(const float* in, float* out, int n_rows, int S, int blk, hipStream_t st);

struct ScoreParams {
  const uint16_t* q; const uint16_t* k;
  const float* lse;         // [n_bh, n_s] natural log
  float* col;               // [n_bh, S]
  float* slash;             // [n_bh, S]
  float* partial;           // workspace for slash partial sums
  int S, n_s, n_bh, n_bkv, group;   // n_bh: heads of every segment
  int heads_per_seg;
  int row_first[kMaxSegs];  // the sampled rows of a segment are [row_first, row_first + n_s)
  float scale_log2;
  int n_kblocks, n_chunks, chunk_rows, win;   // win = floats per (key block, chunk) partial
};
hipError_t launch_score_accumulate(const ScoreParams& P, hipStream_t st);
hipError_t launch_score_finalize(const ScoreParams& P, hipStream_t st);
size_t score_partial_floats(int S, int n_s, int n_bh);
void score_geometry(int S, int n_s, int* n_kblocks, int* n_chunks, int* chunk_rows, int* win);

// measurement aids: back-to-back MFMA loop and plain copy
hipError_t launch_probe_mfma(int iters, int waves_per_simd, float* sink, hipStream_t st);
hipError_t launch_probe_copy(const void* src, void* dst, size_t bytes, hipStream_t st);

struct SelectParams {
  const float* scores;      // [n_prob, S]
  int32_t* idx;             // [n_prob, S]
  int32_t* cnt;             // [n_prob]
  int n_prob, S;
  float alpha;
  // optional second set of n_prob problems of the same size, solved by the same launch
  const float* scores2; int32_t* idx2; int32_t* cnt2; float alpha2;
};
hipError_t launch_select(const SelectParams& P, hipStream_t st);

}  // namespace sa
