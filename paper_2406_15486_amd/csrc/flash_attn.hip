// Flash-style attention kernels for gfx950: dense causal attention (Eq. 1-2),
// row log-sum-exp of the sampled queries (stage 1, pass 1) and attention under
// the merged column / slash / window mask (Eq. 3, Algorithm 1 last step).
//
// A workgroup owns 256 query rows of one head; each of its 8 waves owns 32 of
// them.  Keys are visited in tiles of 64, one K/V stream per workgroup.  For every
// tile a wave forms S^T = K Q^T (keys x queries) with bf16 MFMAs, so that one lane
// holds scores of one or two queries: the row-wise online softmax is then in-lane
// arithmetic plus a rare exchange between lanes.  The probabilities, rounded to bf16, are
// directly the B operand of O^T += V^T P^T, so the accumulators (O^T, head_dim x
// queries) again keep their queries per lane and the rescale is a per-lane scalar.
// K tiles live in LDS as [key][d]; V is read from a pre-transposed copy
// (V^T, [d][key]) so both MFMA A operands are 16-byte LDS reads.  Four stages of each are
// resident in LDS, filled by direct global->LDS loads two and three tiles ahead.
//
// What bounds it.  Long launches run at the card's power limit: the clock falls to 1.5 to 2 GHz (dense
// 1.5 with 32x32x16 MFMAs, 1.9 with 16x16x32), and taking instructions or waits out of the loop returns
// little unless it saves energy.
// Launches whose waves often have no work run at 2.3 GHz and are bound by one wave's chain of
// instructions from barrier to barrier.  Hence two cores, one of them in two shapes (parameter CORE of
// flash_body):
//
// Core 0, 16x16x32 MFMAs (two groups of 16 queries per wave, one LDS operand for both): the same
// products as 32x32x16 at some 12 % less energy (at the power limit an MFMA loop reaches 2003 against 1755
// TFLOP/s, with an LDS operand each 1790 against 1645, with an exponential beside it 1511 against 1442), but a
// vector port that is blocked by twice as many MFMAs (four fma in the stream of each 32 MFMA cycles: 46
// against 33 cycles).  Core 2, the same schedule with 32x32x16 MFMAs (32 queries per wave), for launches that
// do not reach the power limit; its results are those of core 0 bit for bit.
// The waves form two groups of four (rows 0..127 and 128..255); waves
// w and w+4 share a SIMD.  Left alone, two waves that alternate an MFMA section
// and a vector-ALU (softmax) section fall into step - both on the matrix pipe,
// then both on the vector pipe - and each pipe idles half the time.  Here the
// groups run the two phases of a tile in opposite order - group 0 the MFMAs of
// P V(t-1) and K Q^T(t) and then the softmax of tile t, group 1 the softmax of
// tile t-1 and then the same MFMAs - and one workgroup barrier per tile re-aligns
// them, so every SIMD always has one wave feeding the matrix pipe and one feeding
// the vector pipe.
//
// Core 1, 32x32x16 MFMAs (32 queries per wave), heads in two passes: every wave issues the softmax of one
// 32-key half between the MFMAs of the next, so that a tile is one chain of about half the length.
//
// Core 2 / core 0 / core 1, whole path or kernel: dense 16K 1948 / 1860 / 1961 us, 8 heads of 8300 174 / 187 / 177;
// 8K swept 672 / 620 / 652; blocks of 128 at 32K 3261 / 3040 / 3146, swept, 16 heads of 4500 165 / 176 / 170; 64K head
// patterns 35.2 / 34.1 / 35.2 ms; 50001 tokens at alpha = 0.8 5383 / 5430 / 5230 us; runs of four offsets
// every 300 of 64K 20.6 / 20.4 / 16.2 ms, every 1000 6.97 / 6.85 / 5.47 ms.
// The log-sum-exp sweep (core 2) stages no V and needs half the registers: two of its
// workgroups share a CU, and it is bound by their vector instructions.  On core 0 16 heads of 4000 tokens and 256
// rows 19.7 / 22.8 us, 32 of 16384 and 832 132 / 143, but of 65536 and 3328 1628 / 1582.
#include <type_traits>

#include "sa_device.h"
#include "sa_kernels.h"

namespace sa {

namespace {

constexpr int BQ = kFlashBQ;          // 256 query rows per workgroup
constexpr int BK = kFlashBK;          // 64 keys per tile
constexpr int NT = 512;               // two groups of four waves
constexpr int NSTAGE = 4;             // K and V^T tiles resident in LDS
constexpr int NAUX = 8;               // ring of aux-word slots
constexpr int kDiagMask = 0x003FFFFF;  // a tile-diagonal list entry: diagonal in bits 0..21, kSparseBit, kSweepBit, one bit per wave above
// LDS tiles are unpadded (the direct global->LDS loads write 1 KB runs); bank
// conflicts are avoided by XOR-swizzling the 16-byte chunk index with the row.
constexpr int KROW_B = 256;           // bytes per K row in LDS: 16 chunks, chunk c of row p stored at c ^ (p & 15)
constexpr int VROW_B = 128;           // bytes per V^T row in LDS: 8 chunks, chunk c of row d stored at c ^ ((d >> 1) & 7)
constexpr int KTILE_B = BK * KROW_B;
constexpr int VTILE_B = kHeadDim * VROW_B;
constexpr int AUX_B = 256;            // 64 dwords per tile: key indices or mask words
constexpr int OFF_K = 0;
constexpr int OFF_V = OFF_K + NSTAGE * KTILE_B;
constexpr int OFF_A = OFF_V + NSTAGE * VTILE_B;
constexpr int OFF_DUMP = OFF_A + NAUX * AUX_B;      // 1 KB per wave: where loads of tiles past the end go
constexpr int LDS_B = OFF_DUMP + 8 * 1024;          // 141312 bytes
// The log-sum-exp sweep stages K only: its dump area follows the K stages, and with
// 72 KB of LDS and at most 128 registers per lane two of its workgroups share a CU.
constexpr int OFF_DUMP_LSE = OFF_V;
constexpr int LDS_B_LSE = OFF_DUMP_LSE + 8 * 1024;  // 73728 bytes
constexpr float kSumBound = 256.0f;    // a tile's exponentials may sum to 2^8 per lane before the reference maximum moves

// Query tiles per head up to which a strip-masked launch goes by tile, not by head.  By head / by
// tile, 32 heads, whole path: 4K tokens 273 / 233 us, 8K 707 / 708, blocks of 128 at 8K 596 / 579,
// 12K 1422 / 1431.
constexpr int kByTileMax = 32;

enum TileKind : int { TK_PLAIN = 0, TK_CAUSAL = 1, TK_COLIDX = 2, TK_RANGE = 3 };
// What a stretch of the tile loop knows at compile time about the tiles it touches
// (the tile of an iteration, the one before and the four ahead).  KIND: nothing (0),
// all of them gathered-column tiles (1), or none of them (2); REAL: all of them lie
// inside the schedule; INTERIOR: the tiles up to the next one hold only keys before the
// workgroup's first row, so every wave works on them and nothing is masked.  The loop
// runs in stretches, so that the long ones carry no per-tile choice between the two kinds
// of addressing, aux words and activity tests, and no stand-ins for tiles past the end.
template <int KIND_, bool REAL_, bool INTERIOR_ = false, bool FIRST_ = false>
struct Stretch {
  static constexpr int KIND = KIND_;
  static constexpr bool REAL = REAL_;
  static constexpr bool INTERIOR = INTERIOR_;
  static constexpr bool FIRST = FIRST_;      // iteration 0: there is no tile before this one
  using AtFirst = Stretch<KIND_, REAL_, INTERIOR_, true>;
};
// The MFMA operands of one iteration (see flash_body): V^T operands if V, K operands if K, in two
// halves; where there are both they take turns.
template <bool V, bool K>
struct Steps {
  static constexpr int HALF = 8 * (V + K);
  static constexpr bool is_v(int i) { return V && (!K || (i & 1)); }
  static constexpr int index(int i) { return V && K ? (i % HALF) / 2 : i & 7; }   // of the eight of its kind in a half
};
using AnyTiles = Stretch<0, false>;
using PlainTiles = Stretch<0, true, true>;       // dense / log-sum-exp sweep below the diagonal
using ColTiles = Stretch<1, true, true>;
using RngTiles = Stretch<2, false>;
using RngRealTiles = Stretch<2, true>;

// a wave-uniform 64-bit value / pointer, forced into scalar registers (the inline
// assembly below takes its base address in a scalar register pair; left alone, the
// compiler may do wave-uniform address arithmetic in vector registers)
__device__ __forceinline__ uint64_t scalar_u64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t scalar_ptr(const void* p) { return scalar_u64(reinterpret_cast<uint64_t>(p)); }
// Direct global -> LDS load: lane l of the wave moves N bytes from global address
// `base` + `off` (base wave-uniform, in scalar registers; off per lane) to LDS
// address `lds` + N * l (`lds` wave-uniform, passed in M0).  It is written as inline
// assembly so that the waits on it are the explicit vm_wait calls below: the
// compiler, when it issues this instruction itself, makes every later LDS read wait
// for all of them (it cannot tell the buffers apart), which serialises the prefetch
// with the arithmetic.  The loads of a wave complete in order.
// The wave-uniform operands are forced into scalar registers here, whatever the
// compiler made of the address arithmetic (free when they already are scalar).
__device__ __forceinline__ void dma16(uint64_t base, uint32_t off, uint32_t lds) {
  const uint64_t sbase = scalar_u64(base);
  const uint32_t slds = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(sbase), "s"(slds)
               : "memory", "m0");
}
__device__ __forceinline__ void dma4(uint64_t base, uint32_t off, uint32_t lds) {
  const uint64_t sbase = scalar_u64(base);
  const uint32_t slds = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(sbase), "s"(slds)
               : "memory", "m0");
}
// wait until at most N of this wave's vector-memory loads are still in flight
template <int N>
__device__ __forceinline__ void vm_wait() {
  static_assert(N >= 0 && N < 16, "vmcnt immediate");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// workgroup barrier
__device__ __forceinline__ void wg_meet() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// ... LDS reads issued before it have returned
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0), as the builtin: the compiler's own counters see it too
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Parts of the query tiles [q0, q1) of a head, ceil((a + 1) / m) for tile a.
__host__ __device__ inline int parts_upto(int m, int n) { return m * (n / m) * (n / m + 1) / 2 + (n % m) * (n / m + 1); }
// What a workgroup does: part `split` of n_parts of query tile a of head bh, rows [row_lo, row_hi) of
// segment seg.  Log-sum-exp: the sampled rows of the segment (a counts from the first of them), and
// how its keys are cut.  part0: the tile's first part among those of its head.
struct TileJob {
  int bh, a, seg, row_lo, row_hi, split, n_parts, part0, lse_parts, k_splits;
};
// tile f of the launch (segments one after the other): its segment, and the tile
__host__ __device__ inline int segment_of(const FlashParams& P, int f) {
  int m = 0;
  while (m + 1 < P.n_seg && f >= P.seg[m + 1].tile0) ++m;
  return m;
}
__host__ __device__ inline int parts_before(int m, int q0, int q1) { return parts_upto(m, q1) - parts_upto(m, q0); }

}  // namespace

// MODE: 0 dense causal, 1 row log-sum-exp only (no V), 2 strip-masked sparse.
// IN_PLACE (strip-masked mode, block lists): the gathered-column tiles are runs of 64
// consecutive keys (blocks of 64, 128 or 256 keys), so they are read from K and V^T
// themselves instead of from gathered copies; the padded index list still travels with
// every tile (causal edge, short last block).
// SWEEP (strip-masked mode, heads whose lists are nearly full): one causal sweep over every
// key tile in order, as in the dense mode, with columns and offsets joined in one mask; no
// gathered tiles.  The kernel below picks the body by head.  As a run-time flag inside one
// body the choice cost the long unswept launches 2.5 % (128K tokens, alpha = 0.95); as a
// body of its own it knows at compile time that interior tiles are active.
// PARTS (dense and strip-masked modes): the workgroup takes part `split` of the `n_parts` equal
// parts of its query tile's schedule and leaves unnormalised sums for parts_combine_kernel.
template <int MODE, bool OUT_F32, bool IN_PLACE, bool SWEEP, bool PARTS, int CORE>
__device__ __forceinline__ void flash_body(const FlashParams& P, const TileJob& J) {
  const int bh = J.bh, a = J.a, split = J.split, n_parts = J.n_parts;
  const int hs = MODE == 2 ? J.seg * P.n_bh + bh : bh;   // the head's metadata: one set for every segment
  static_assert(!SWEEP || MODE == 2, "only the strip mask is swept");
  static_assert(!IN_PLACE || MODE == 2, "in-place column tiles belong to the strip-masked mode");
  static_assert(CORE == 2 || MODE != 1, "the log-sum-exp sweep runs on core 2");
  static_assert(CORE != 0 || !PARTS, "cut tiles run on cores 1 and 2");
  static_assert(CORE != 1 || (MODE == 2 && !SWEEP), "core 1 takes heads in two passes");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr bool WITH_V = (MODE != 1);
  // Where a wave issues its share of the tile loads.  Each direct load stalls the wave
  // 40-100 cycles; the two MFMA phases of a SIMD hardly overlap, so a stall there costs
  // the iteration, while the softmax phase is the shorter one and has room.  The
  // log-sum-exp sweep is the other way round (short MFMA phase, no P V).
  constexpr bool kLoadsInSoftmax = WITH_V;
  constexpr int kOffDump = WITH_V ? OFF_DUMP : OFF_DUMP_LSE;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // 0..7, wave-uniform, kept in an SGPR
  const int grp = wave >> 2;           // phase group
  const int lane = tid & 63;
  const uint32_t smem_lds = __builtin_amdgcn_readfirstlane((int)(uintptr_t)(__attribute__((address_space(3))) char*)smem);

  const int bkv = ((MODE == 2 ? P.head0 : 0) + bh) / P.group;
  const int S = P.S;
  const int i0 = (MODE == 1 ? J.row_lo : 0) + a * BQ;                     // first query row of the workgroup
  const int i_last_wg = min(i0 + BQ, J.row_hi) - 1;      // last valid row
  const int iw0 = i0 + 32 * wave;                        // first query row of the wave
  const int a64 = i0 / BK;   // index of the 64-key tile that holds row i0 (i0 % 256 == 0 in MODE 2)
  const uint16_t* kbase = P.k + (size_t)bkv * S * kHeadDim;
  const uint16_t* vtbase = WITH_V ? P.vt + (size_t)bkv * kHeadDim * P.S_pad : nullptr;

  // ---- tile schedule: gathered-column tiles, then range tiles (sparse), or the
  //      causal sweep (dense / log-sum-exp) ------------------------------------------
  const int32_t* cidx = nullptr;
  const int32_t* dl = nullptr;
  const uint32_t* cbits = nullptr;
  const uint32_t* obits = nullptr;
  const uint16_t* kc = nullptr;
  const uint16_t* vct = nullptr;
  int n_col_tiles = 0, n_rng = 0;
  if (SWEEP) {
    dl = P.dlist + (size_t)hs * P.dlist_stride;
    cbits = P.col_bits + (size_t)hs * P.cb_words;
    obits = P.off_bits + (size_t)hs * P.rb_words;
  } else if (MODE == 2) {
    cidx = P.col_idx_pad + (size_t)hs * P.cidx_stride;
    int cnt = min(max(P.col_cnt[hs], 0), S);
    int lo = 0, hi = cnt;          // selected columns j <= last row of the tile (ascending list)
    while (lo < hi) {
      int mid = (lo + hi) >> 1;
      if (cidx[mid] <= i_last_wg) lo = mid + 1; else hi = mid;
    }
    n_col_tiles = (lo + BK - 1) / BK;
    dl = P.dlist + (size_t)hs * P.dlist_stride;
    int dc = min(max(P.dcnt[hs], 0), P.dlist_stride);
    lo = 0; hi = dc;               // tile diagonals d whose key tile a64 + 3 - d is >= 0
    while (lo < hi) {
      int mid = (lo + hi) >> 1;
      if ((dl[mid] & kDiagMask) <= a64 + 3) lo = mid + 1; else hi = mid;
    }
    n_rng = lo;
    cbits = P.col_bits + (size_t)hs * P.cb_words;
    obits = P.off_bits + (size_t)hs * P.rb_words;
    kc = P.kc + (size_t)hs * P.S_pad * kHeadDim;
    vct = P.vct + (size_t)hs * kHeadDim * P.S_pad;
  }
  int t_base = 0;                        // first key tile of this workgroup's share of the causal sweep
  const int n_sweep = min(i_last_wg, S - 1) / BK + 1;
  int n_sched = (MODE == 2 && !SWEEP) ? (n_col_tiles + n_rng) : n_sweep;
  // Log-sum-exp sweep: the keys of the query tile are cut into lse_parts equal parts, each summed
  // from nothing, and this workgroup takes the parts [part, part_stop) one after the other.
  int part = 0, part_stop = 1;
  if (MODE == 1) {
    part = J.lse_parts / J.k_splits * split;
    part_stop = part + J.lse_parts / J.k_splits;
    t_base = n_sweep * part / J.lse_parts;
    n_sched = n_sweep * part_stop / J.lse_parts - t_base;
  }
  // tile that ends part `part` (counted from t_base); the workgroup's last part ends with the schedule
  auto end_of_part = [&]() { return part + 1 < part_stop ? n_sweep * (part + 1) / J.lse_parts - t_base - 1 : -1; };
  int part_last = MODE == 1 ? __builtin_amdgcn_readfirstlane(end_of_part()) : -1;
  if (PARTS) {
    t_base = n_sched * split / n_parts;
    n_sched = n_sched * (split + 1) / n_parts - t_base;
    if (MODE == 2 && !SWEEP) {           // tile t of this part is tile t + t_base of the schedule
      const int col_before = min(t_base, n_col_tiles);
      n_rng -= t_base - col_before;
      n_col_tiles = min(n_col_tiles - col_before, n_sched);
      cidx += BK * col_before;
      kc += (size_t)col_before * BK * kHeadDim;
      vct += (size_t)col_before * BK;
    }
  }
  t_base = __builtin_amdgcn_readfirstlane(t_base);
  n_col_tiles = __builtin_amdgcn_readfirstlane(n_col_tiles);
  n_rng = __builtin_amdgcn_readfirstlane(n_rng);
  const int n_tiles = __builtin_amdgcn_readfirstlane(n_sched);
  constexpr bool SHIFTED = MODE == 1 || (PARTS && (MODE == 0 || SWEEP));   // a causal sweep that starts at tile t_base

  // Kind of tile t (wave-uniform; no memory access), and whether t lies inside the schedule.
  // `kc` is the Stretch the calling iteration belongs to: what it knows at compile time.
  auto is_col = [&](auto kc, int t) __attribute__((always_inline)) -> bool {
    constexpr int KIND = decltype(kc)::KIND;
    return MODE == 2 && !SWEEP && (KIND == 1 || (KIND == 0 && t < n_col_tiles));
  };
  auto is_real = [&](auto kc, int t) __attribute__((always_inline)) -> bool { return decltype(kc)::REAL || t < n_tiles; };
  // Descriptor of tile t.  A range tile is named by its tile diagonal d: key tile
  // a64 + 3 - d, which the 256 rows meet at offsets [64 d - 255, 64 d + 63].  The d
  // values come from a list in global memory; they are fetched (fetch_d) four tiles
  // ahead of their first use and handed on in scalar registers, so that no phase
  // waits on a scalar load.
  auto fetch_d = [&](auto kc, int t) __attribute__((always_inline)) -> int {
    // read through the constant address space: the list is not written while the kernel
    // runs, and only so does the load stay a scalar one (tracked apart from the vector
    // loads in flight) behind the barriers and inline assembly of the loop
    typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
    if (IN_PLACE && is_col(kc, t))
      return ((const_i32_ptr)(uintptr_t)cidx)[BK * t];                       // first key of the tile's block
    if (SWEEP) {
      // the list holds every diagonal; only block masks need its entry (which waves keep the tile)
      if (IN_PLACE && is_real(kc, t)) return ((const_i32_ptr)(uintptr_t)dl)[a64 + 3 - t - (SHIFTED ? t_base : 0)];
      return 0;
    }
    if (MODE == 2 && !is_col(kc, t) && is_real(kc, t))
      return ((const_i32_ptr)(uintptr_t)dl)[n_rng - 1 - (t - n_col_tiles)];   // far to near
    return 0;
  };
  // first key of tile t
  auto first_key = [&](auto kc, int t, int d) __attribute__((always_inline)) -> int {  // contiguous tiles only; d = list entry
    if (IN_PLACE && is_col(kc, t)) return d;         // the entry of an in-place column tile is its first key
    return (MODE == 2 && !SWEEP) ? (a64 + 3 - (d & kDiagMask)) * BK : (t + (SHIFTED ? t_base : 0)) * BK;
  };
  // array bases as scalars, once
  const uint64_t s_kbase = scalar_ptr(kbase), s_vtbase = scalar_ptr(vtbase);
  const uint64_t s_kc = scalar_ptr(kc), s_vct = scalar_ptr(vct), s_cidx = scalar_ptr(cidx);
  const uint64_t s_cbits = scalar_ptr(cbits), s_obits = scalar_ptr(obits);

  // ---- staging ---------------------------------------------------------------------
  // One wave instruction writes a 1 KB run of LDS, lane l its bytes [16 l, 16 l + 16):
  // for K that is 4 physical rows, for V^T 8 rows.  Each lane therefore fetches the
  // global chunk that belongs at its LDS position: the K row whose slot it is (see krow_slot16)
  // and the chunk that the XOR
  // swizzle maps there.  A tile is 16 runs of K and 16 of V^T; wave w issues runs w
  // and w + 8 of each.  The lane's byte offset inside a run is fixed for the whole
  // kernel, and run w + 8 lies a constant 32 K rows / 64 V^T rows after run w
  // (neither the swizzle nor the slot permutation sees that step): per tile and per
  // load only the scalar base address changes, so issuing costs no vector arithmetic.
  uint32_t koff0, voff0;
  {
    int p = 4 * wave + (lane >> 4);                // physical K row of run `wave`
    int c = (lane & 15) ^ (p & 15);                // logical 16-byte chunk stored there
    koff0 = (CORE == 0 ? krow_slot16(p) : krow_slot32(p)) * KROW_B + c * 16;   // key row within the tile, byte in the row
    int d = 8 * wave + (lane >> 3);                // V^T row
    int cv = (lane & 7) ^ ((d >> 1) & 7);
    voff0 = (uint32_t)d * (uint32_t)P.S_pad * 2u + cv * 16;
  }
  // The loads are issued one at a time (load_v_one / load_k_one, n = 0, 1), so the
  // caller can spread them between its exponentials (or its MFMAs): a wave that issues
  // them back to back stalls on each.  Loads of a tile past the end of the schedule still go out (to a
  // stand-in address and the wave's dump area), which keeps the number of loads per
  // phase, and with it the vmcnt arithmetic, constant.
  uint64_t ld_vbase = 0, ld_vbase1 = 0, ld_kbase = 0;
  uint32_t ld_vdst = 0, ld_kdst = 0, ld_vstep = 0, ld_kstep = 0, ld_klim = 0;   // step: LDS distance of run w + 8
  // A tile past the end of the schedule is replaced by a stand-in: the first tile of
  // K / V^T, always readable, loaded into the wave's dump kilobyte.
  auto load_v_begin = [&](auto kc, int t, int d) __attribute__((always_inline)) {
    if (!WITH_V) return;
    const bool real = is_real(kc, t), col = !IN_PLACE && real && is_col(kc, t);   // col: from the gathered copy
    const uint32_t off = !real ? 0u : (col ? (uint32_t)t : (uint32_t)first_key(kc, t, d)) * 2u;   // bytes into a V^T row; t * 64 keys for a gathered tile
    ld_vbase = col ? s_vct + (uint64_t)((uint32_t)t * (BK * 2u)) : s_vtbase + off;
    ld_vbase1 = ld_vbase + 128ull * (uint32_t)P.S_pad;            // run w + 8: 64 rows of V^T further on
    ld_vdst = smem_lds + 1024 * wave + (real ? OFF_V + (t & (NSTAGE - 1)) * VTILE_B : kOffDump);
    ld_vstep = real ? 8192 : 0;                    // a stand-in tile writes both runs to the same dump kilobyte
  };
  auto load_k_begin = [&](auto kc, int t, int d) __attribute__((always_inline)) {
    const bool real = is_real(kc, t), col = !IN_PLACE && real && is_col(kc, t);
    const int kmax = col ? P.S_pad - 1 : S - 1;    // last row of the array that may be read
    // a range tile may start past the last key (all of it masked): the base row is
    // clamped, and so is each lane's byte offset, to the last row that exists
    const int row0 = min(!real ? 0 : (col ? t * BK : first_key(kc, t, d)), kmax);
    ld_kbase = (col ? s_kc : s_kbase) + ((uint64_t)(uint32_t)row0 << 8);
    ld_klim = (uint32_t)(kmax - row0) * KROW_B + (koff0 & (KROW_B - 1));
    ld_kdst = smem_lds + 1024 * wave + (real ? OFF_K + (t & (NSTAGE - 1)) * KTILE_B : kOffDump);
    ld_kstep = real ? 8192 : 0;
  };
  auto load_v_one = [&](int n) {
    if (!WITH_V) return;
    dma16(n == 0 ? ld_vbase : ld_vbase1, voff0, ld_vdst + ld_vstep * n);
  };
  auto load_k_one = [&](int n) {
    dma16(ld_kbase, min(koff0 + 32 * KROW_B * n, ld_klim), ld_kdst + ld_kstep * n);
  };
  // the 64 dwords that go with a tile: the key indices of a gathered tile, or for a
  // range tile 16 words of the offset bitmap (covering every offset of the 256 x 64
  // tile) followed by the 2 words of the column bitmap.  One load, by wave t % 8.
  const uint32_t aux_lane = lane < 16 ? 4u * lane : 4u * (lane & 1);
  auto dma_aux = [&](auto kc, int t, int d) __attribute__((always_inline)) {
    if (MODE != 2 || wave != (t & 7)) return;
    const bool real = is_real(kc, t);
    const uint32_t dst = smem_lds + (real ? OFF_A + (t & (NAUX - 1)) * AUX_B : kOffDump);
    if (real && is_col(kc, t)) {
      dma4(s_cidx + (uint64_t)((uint32_t)t * (BK * 4u)), 4u * lane, dst);
    } else {
      const int j0 = real ? first_key(kc, t, d) : 0;
      const int wb = (P.off_max - (i0 - j0 + BQ - 1)) >> 5;          // first offset-bitmap word needed
      // lanes 0..15: offset words wb ..; lanes 16..63: the two column words, alternating.
      // The column bitmaps lie below the offset bitmaps in the workspace (and within
      // 4 GB of them), so offsets from the column word are non-negative 32-bit values.
      const uint64_t cw = s_cbits + (uint64_t)((uint32_t)(j0 >> 5) * 4u);
      const uint32_t gap = (uint32_t)(s_obits + (uint64_t)((uint32_t)wb * 4u) - cw);
      dma4(cw, aux_lane + (lane < 16 ? gap : 0u), dst);
    }
  };

  // Whether this wave has anything to do on tile t.
  //  - gathered tile: its first key index (an aux word) must not lie after the wave's rows.
  //    The word is read early (act_word) and looked at later (tile_active), so that the wait
  //    for it hides behind MFMAs;
  //  - range tile: one of the 95 offsets between the wave's 32 rows and the tile's 64
  //    keys must be kept.  That depends on the tile diagonal and the wave only, not on
  //    the query tile, so the list entry carries it as a bit per wave (bits 24..31; a
  //    key after a row gives a negative offset, never kept).  Also not all 64 keys may
  //    be selected columns (the column pass covered those), and the tile must start
  //    before the sequence end: settle() clears the bits of such an entry.  (A sweep that needs
  //    the entries keeps tiles of selected columns instead: there it sets them.)  The two words
  //    of the column bitmap are fetched like the entries, as scalars and a tile later, so that
  //    activity is scalar arithmetic: read from the aux words it cost a wait for every LDS read
  //    in flight in the middle of the P V sweep.
  constexpr bool kBits = MODE == 2 && (!SWEEP || IN_PLACE);      // range tiles have list entries
  auto fetch_cols = [&](auto kc, int t, int d) __attribute__((always_inline)) -> uint64_t {
    typedef const __attribute__((address_space(4))) uint64_t* const_u64_ptr;
    if (!kBits || is_col(kc, t) || !is_real(kc, t)) return 0;
    return *(const_u64_ptr)(uintptr_t)(s_cbits + (uint64_t)((uint32_t)(first_key(kc, t, d) >> 5) * 4u));
  };
  auto settle = [&](auto kc, int t, int d, uint64_t cols) __attribute__((always_inline)) -> int {
    if (!kBits || is_col(kc, t)) return d;
    if (SWEEP) return cols == ~0ull ? (int)((uint32_t)d | 0xFF000000u) : d;
    return (cols == ~0ull || first_key(kc, t, d) >= S) ? (int)((uint32_t)d & 0x00FFFFFFu) : d;
  };
  auto act_word = [&](auto kc, int t, int& w0) __attribute__((always_inline)) {
    if (MODE != 2 || SWEEP || decltype(kc)::INTERIOR || !is_col(kc, t)) return;
    w0 = *reinterpret_cast<const int*>(smem + OFF_A + (t & (NAUX - 1)) * AUX_B);
  };
  auto tile_active = [&](auto kc, int t, int d, int w0) __attribute__((always_inline)) -> bool {
    if (decltype(kc)::INTERIOR) return true;
    bool act;
    const int j0 = first_key(kc, t, d);
    if (is_col(kc, t)) {
      act = w0 <= iw0 + 31;
    } else if (kBits) {
      act = (((uint32_t)d >> (24 + wave)) & 1u) && (!SWEEP || j0 <= iw0 + 31);
    } else {
      act = j0 <= iw0 + 31;                        // else every key of the tile lies after the wave's rows
      // ... or the wave has no row.  (Half of the waves for 128 sampled rows: left to work on copies
      // of the last row they took half the vector pipe; 32 heads, 128K keys 276 / 155 us, 32K
      // 73 / 48 us; 32K with 1664 rows, whose last tile is half full, 478 / 458 us.)
      if (MODE == 1) act = act && iw0 <= i_last_wg;
    }
    return __builtin_amdgcn_readfirstlane((int)act) != 0;
  };

#define SA_PIN() __builtin_amdgcn_sched_barrier(0)
  if constexpr (CORE != 1) {
    // Two shapes of the MFMAs, the same results bit for bit: both form a score and an element of O by the same
    // additions in the same order (eight products after eight), and the sums and references below are kept
    // for the same groups of keys.
    // CORE 0, 16x16x32: a lane has two queries, 16 apart, and eight keys of each 32.
    // CORE 2, 32x32x16: a lane has one query, and two groups of eight keys of each 32, 16 apart.
    // `n` is the query of a lane or the group of its keys.
    constexpr bool WIDE = CORE == 2;
    constexpr int NQ = WIDE ? 1 : 2;                       // queries of a lane
    using Acc = std::conditional_t<WIDE, f32x16, f32x4>;
    constexpr int NR = WIDE ? 16 : 4, NO = WIDE ? 4 : 16, NS = WIDE ? 2 : 8;   // elements of an accumulator, accumulators of O and of S
    const int ql = WIDE ? lane & 31 : lane & 15;   // query within a group / row within an operand
    const int kg = WIDE ? lane >> 5 : lane >> 4;   // which part of the contraction block this lane feeds
    const int i_me = iw0 + ql;                             // this lane's first query row; the second is 16 on
    auto row_ok = [&](int n) { const int i = i_me + 16 * n; return i <= i_last_wg && (MODE != 2 || i >= J.row_lo); };
    // ---- Q^T operand: two groups of 16 queries and 4 contraction steps of 32 (or 32 queries and 8 of 16), resident in registers
    constexpr int KS = 8 / NQ;
    bf16x8 qf[8];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      int qr = row_ok(n) ? i_me + 16 * n : max(min(i_last_wg, S - 1), 0);
      const uint16_t* qrow = P.q + ((size_t)bh * S + qr) * kHeadDim;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        qf[KS * n + ks] = as_bf16x8(*reinterpret_cast<const uint4*>(qrow + ks * (kHeadDim / KS) + kg * 8));
    }

    Acc o[NO];                             // query n: o[8 n ..]
#pragma unroll
    for (int x = 0; x < NO; ++x)
#pragma unroll
      for (int r = 0; r < NR; ++r) o[x][r] = 0.f;
    float m_run[NQ];                       // reference maximum, in log2 units (score * scale * log2 e)
#pragma unroll
    for (int n = 0; n < NQ; ++n) m_run[n] = kNegBig;
    constexpr int NL = MODE == 1 ? 1 : 2;  // (the log-sum-exp sweep, bound by vector instructions, has one shape and one sum)
    float l_run[2] = {0.f, 0.f};           // running sums of exp2 for this lane's keys
    const float c2 = P.scale_log2;

    // ---- operand ring and the MFMA phase -------------------------------------------
    // A phase takes up to 32 operands from LDS: 16 of P V(t-1) (16 rows: head-dim blocks 0..7 for each of
    // two 32-key halves; 32 rows: blocks 0..3 for each of four 16-key groups) and 16 of
    // K Q^T(t) (16-key blocks 0..3 for each of 4 contraction steps; 32-key halves for each of 8).  They
    // come through a ring of 8 registers x 16 bytes: after the MFMAs of operand i (one per group of 16
    // queries, or one) have consumed slot i % 8, operand i + 8 is read into it, so every read has the MFMAs of seven
    // operands (~250 cycles) to return and the matrix pipe does not wait on LDS round trips.  sched_barrier pins the order: the
    // compiler would otherwise sink each read down to its use.
    Acc s[NS];
    uint4 pk[2][2];
    uint4 R[8];
    // score e of 32-key half sb and query / key group n: see mm_qk
    auto score_at = [](int sb, int n, int e) { return WIDE ? sb : 4 * n + 2 * sb + (e >> 2); };
    auto score_el = [](int n, int e) { return WIDE ? 8 * n + e : e & 3; };
    // K operand i = 4 ks + b: contraction step ks, 16-key block b (2 ks + b: step ks, half b)
    auto ld_k = [&](int slot, int i, int buf) {
      // row p = 16 b + ql (32 b + ql); logical chunk 4 ks + kg (2 ks + kg) lives at physical chunk (..) ^ (p & 15)
      const int b = WIDE ? i & 1 : i & 3, ks = WIDE ? i >> 1 : i >> 2;
      const char* kp = smem + OFF_K + buf * KTILE_B + ((WIDE ? 32 : 16) * b + ql) * KROW_B;
      R[slot] = *reinterpret_cast<const uint4*>(kp + ((((WIDE ? 2 : 4) * ks + kg) ^ (WIDE ? ql & 15 : ql)) << 4));
    };
    // V^T operand i = 8 sb + mb: keys 32 sb .., head-dim block mb (8 sb + 4 n + mb: keys 32 sb + 16 n ..)
    auto ld_v = [&](int slot, int i, int buf) {
      // row d = 16 mb + ql (32 mb + ql); logical chunk 4 sb + kg (4 sb + 2 n + kg) lives at physical chunk (..) ^ ((d >> 1) & 7)
      const int sb = i >> 3, mb = WIDE ? i & 3 : i & 7, n = WIDE ? (i >> 2) & 1 : 0;
      const char* vp = smem + OFF_V + buf * VTILE_B + ((WIDE ? 32 : 16) * mb + ql) * VROW_B;
      R[slot] = *reinterpret_cast<const uint4*>(vp + (((4 * sb + 2 * n + kg) ^ (WIDE ? (ql >> 1) & 7 : ql >> 1)) << 4));
    };
    // P V: on entry the ring holds V operands 0..7 (read during the softmax phase);
    // the second half of the sweep re-fills it with the first 8 K operands of the next
    // tile (read even when that tile turns out to need no work from this wave).
    auto mm_pv = [&](int bufp, int bufq, auto&& look, auto&& decide) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (i == 3) look();                          // read the words that say whether the next tile needs this wave
        if (i == 9) decide();                        // ... and decide, under the MFMAs
        const int sb = i >> 3;
        if constexpr (WIDE) {                                                // O^T += V^T P^T
          o[i & 3] = mfma_32x32x16(as_bf16x8(R[i & 7]), as_bf16x8(pk[(i >> 2) & 1][sb]), o[i & 3]);
        } else {
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            const int n = (i & 1) ? 1 - m : m, x = 8 * n + (i & 7);
            o[x] = mfma_16x16x32(as_bf16x8(R[i & 7]), as_bf16x8(pk[n][sb]), o[x]);
          }
        }
        SA_PIN();
        if (i + 8 < 16) ld_v(i & 7, i + 8, bufp); else ld_k(i & 7, i - 8, bufq);
        SA_PIN();
      }
    };
    // first 8 K operands of a tile into the ring (when no P V sweep did it)
    auto warm_k = [&](int bufq) {
#pragma unroll
      for (int i = 0; i < 8; ++i) ld_k(i, i, bufq);
      SA_PIN();
    };
    // K Q^T: the ring holds K operands 0..7.  Without P V this sweep issues the loads of the tiles
    // further ahead, one every three operands.
    // Element r of s[4 n + b] is key j0 + 32 (b / 2) + 8 kg + 4 (b % 2) + r against query i_me + 16 n.
    // (WIDE: of s[b] key j0 + 32 b + 16 (r / 8) + 8 kg + r % 8 against query i_me.)
    auto mm_qk = [&](int bufq) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (!kLoadsInSoftmax) {
          if (i == 8) load_k_one(0);
          if (i == 11) load_k_one(1);
        }
        const int b = WIDE ? i & 1 : i & 3, ks = WIDE ? i >> 1 : i >> 2;
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
          const int n = (!WIDE && (i & 1)) ? 1 - m : m, x = 4 * n + b;
          if (ks == 0) {
#pragma unroll
            for (int r = 0; r < NR; ++r) s[x][r] = 0.f;
          }
          if constexpr (WIDE) s[x] = mfma_32x32x16(as_bf16x8(R[i & 7]), qf[ks], s[x]);
          else s[x] = mfma_16x16x32(as_bf16x8(R[i & 7]), qf[KS * n + ks], s[x]);
        }
        SA_PIN();
        if (i + 8 < 16) ld_k(i & 7, i + 8, bufq);
        SA_PIN();
      }
    };

    // log-sum-exp of part `part` of this lane's row (mode 1).  The store joins the loads in flight and
    // so only makes the vmcnt waits of the loop wait for more than they must.
    // (one order of the four groups of keys in both shapes)
    auto row_sum = [&](int n) __attribute__((always_inline)) -> float {
      if constexpr (NL == 1) return half_sum(l_run[0]);
      else if constexpr (WIDE) return half_sum(l_run[0]) + half_sum(l_run[1]);
      else return quad_sum(l_run[n]);
    };
    auto store_part_lse = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        const float l_tot = row_sum(n);
        if (row_ok(n) && kg == 0)
          P.lse[((size_t)part * P.n_slots + J.seg * P.n_bh + bh) * P.n_qrows + (i_me + 16 * n - J.row_lo)] = m_run[n] * kLn2 + __logf(l_tot);
      }
    };

    // ---- the softmax phase: mask, online softmax (two queries per lane), bf16 --------
    auto step_softmax = [&](auto kc, int t, int d, auto&& fetch) __attribute__((always_inline)) {
      const int j0 = first_key(kc, t, d);
      constexpr bool INTERIOR = decltype(kc)::INTERIOR;
      const int kind = is_col(kc, t) ? TK_COLIDX : (MODE == 2 && !(SWEEP && IN_PLACE)) ? TK_RANGE : (!INTERIOR && j0 + BK - 1 > i0) ? TK_CAUSAL : TK_PLAIN;
      const int buf = t & (NSTAGE - 1);
      // Mask: one 32-bit pattern per lane and 32-key half, set = keep: bit e (e = 0..7) <-> key
      // j0 + 32 sb + 8 kg + e against the lane's SECOND query, bit 16 + e against its first.  (The
      // offset of the second query is the larger one by 16, so a window of the reversed offset
      // bitmap has its bits 16 places lower.)  WIDE: bit 16 n + e <-> key j0 + 32 sb + 16 n + 8 kg + e.
      // Either way bit b is offset first_off - 32 sb - b.  The pattern is built per tile kind; one loop
      // applies it (a 1-bit signed extract and a bitwise select between the score and -inf per element).
      bool masked = false;                   // wave-uniform
      uint32_t km[2] = {0xFFFFFFFFu, 0xFFFFFFFFu};
      const int first_off = i_me - (j0 + 8 * kg) + (WIDE ? 0 : 16);
      // keep key <= query, i.e. e <= tl for the first query, e <= tl + 16 for the second
      auto causal = [](int tl) -> uint32_t {
        if (WIDE) return tl < 0 ? 0u : (tl >= 31 ? 0xFFFFFFFFu : (2u << tl) - 1u);
        auto low = [](int n) { return (1u << min(max(n, 0), 8)) - 1u; };   // the lowest n of 8 bits
        return (low(tl + 1) << 16) | low(tl + 17);
      };
      if (kind == TK_CAUSAL) {
        if (j0 + BK - 1 > iw0) {
          masked = true;
#pragma unroll
          for (int sb = 0; sb < 2; ++sb) km[sb] = causal(i_me - (j0 + 32 * sb + 8 * kg));
        }
      } else if (MODE == 2 && kind == TK_COLIDX) {
        const int32_t* il = reinterpret_cast<const int32_t*>(smem + OFF_A + (t & (NAUX - 1)) * AUX_B);
        if (!INTERIOR && il[BK - 1] > iw0) {   // only the last gathered tiles reach past a row: keep index <= query
          masked = true;
#pragma unroll
          for (int sb = 0; sb < 2; ++sb) {
            uint32_t m = 0;
#pragma unroll
            for (int g = 0; g < (WIDE ? 2 : 1); ++g) {
              const int4* ip = reinterpret_cast<const int4*>(il + 32 * sb + 16 * g + 8 * kg);
              int4 x0 = ip[0], x1 = ip[1];
              int jj[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                if (WIDE) m |= (jj[e] <= i_me ? 1u : 0u) << (16 * g + e);
                else m |= ((jj[e] <= i_me ? 1u : 0u) << (16 + e)) | ((jj[e] <= i_me + 16 ? 1u : 0u) << e);
              }
            }
            km[sb] = m;
          }
        }
      } else if (MODE == 2 && kind == TK_RANGE) {
        masked = true;
        const uint32_t* mw = reinterpret_cast<const uint32_t*>(smem + OFF_A + (t & (NAUX - 1)) * AUX_B);
        const int wb = (P.off_max - (i0 - j0 + BQ - 1)) >> 5;
        const int x0 = P.off_max - first_off;                // >= 0 by construction of the bitmap
        const int k = (x0 >> 5) - wb;                        // 0 .. 9: word of the staged window
        const uint32_t w0 = mw[k], w1 = mw[k + 1], w2 = mw[k + 2];
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
          const uint32_t ow = __builtin_amdgcn_alignbit(sb == 0 ? w1 : w2, sb == 0 ? w0 : w1, x0 & 31);
          const uint32_t cb = __builtin_amdgcn_ubfe(mw[16 + sb], 8 * kg, 8);   // bit e <-> key is a selected column
          const uint32_t cw = WIDE ? mw[16 + sb] >> (8 * kg) : cb | (cb << 16);
          // columns were taken by the gathered tiles - or, in a sweep, are kept here as well (a
          // column bit, unlike an offset bit, says nothing about j <= i)
          km[sb] = SWEEP ? (ow | cw) : (ow & ~cw);
          if (SWEEP && !INTERIOR) km[sb] &= causal(first_off - (WIDE ? 0 : 16) - 32 * sb);
        }
        // a tile that keeps every pair (a whole block of the block mask, the inside of a
        // band of offsets) needs no masking at all
        masked = __builtin_amdgcn_ballot_w64((km[0] & km[1] & 0x00FF00FFu) != 0x00FF00FFu) != 0ull;
      }
      if (masked) {
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe(km[sb], ((WIDE ? n == 1 : n == 0) ? 16 : 0) + e, 1);   // all-ones where kept
              const int x = score_at(sb, n, e), r = score_el(n, e);
              s[x][r] = __uint_as_float((__float_as_uint(s[x][r]) & keep) | (0xFF800000u & ~keep));
            }
      }

      // the operand ring is idle: fetch the first 8 V operands of this tile's P V now,
      // so that the reads return under the exponentials
      // (the log-sum-exp sweep fetches nothing: a pin alone costs it 4 %)
      if (WITH_V) {
        SA_PIN();
        fetch();
        SA_PIN();
#pragma unroll
        for (int i = 0; i < 8; ++i) ld_v(i, i, buf);
        SA_PIN();
      } else {
        fetch();
      }
      // Online softmax, optimistic: the exponentials are taken against the reference
      // maximum the row already has, and only their sum is looked at.  A sum within
      // 2^8 means that no probability exceeds 2^8, which is all the reference is
      // for (exact in fp32 and bf16 alike); then the tile costs no maximum at all.
      // Otherwise (first tiles of a row, or a score far above what the row has seen: the
      // sum is large, inf or NaN) the row maximum of the tile is formed, the reference
      // moved up to it, the accumulators rescaled and the exponentials taken again.
      float rs[2];
      auto exponentials = [&](auto first_tag) {
        constexpr bool FIRST = decltype(first_tag)::value;
        rs[0] = rs[1] = 0.f;
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
          for (int n = 0; n < 2; ++n) {
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              if (kLoadsInSoftmax && FIRST && e == 4) {   // the loads of the tiles ahead, spread over the exponentials
                if (sb == 0) load_v_one(n); else load_k_one(n);
              }
              p[e] = fast_exp2(fmaf(s[score_at(sb, n, e)][score_el(n, e)], c2, -m_run[n % NQ]));
              rs[n % NL] += p[e];
            }
            pk[n][sb] = make_uint4(pack_bf16x2(p[0], p[1]), pack_bf16x2(p[2], p[3]), pack_bf16x2(p[4], p[5]), pack_bf16x2(p[6], p[7]));
          }
      };
      exponentials(std::true_type{});
      if (__any(!(rs[0] <= kSumBound && (NL == 1 || rs[1] <= kSumBound)))) {
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
          // (the maximum starts from a value the compiler cannot see through: otherwise it
          // forms the whole maximum ahead of the branch, on every tile)
          float mx = s[4 * n][0];
          asm volatile("" : "+v"(mx));
#pragma unroll
          for (int x = 0; x < NS / NQ; ++x)
#pragma unroll
            for (int r = 0; r < NR; ++r) mx = fmaxf(mx, s[4 * n + x][r]);
          if constexpr (WIDE) mx = half_max(mx); else mx = quad_max(mx);   // the lanes of a row agree on its reference
          const float m_cand = mx * c2;
          const float m_new = (m_cand > m_run[n]) ? m_cand : m_run[n];
          const float alpha = fast_exp2(m_run[n] - m_new);
          m_run[n] = m_new;
          l_run[n] *= alpha;
          if (WIDE && NL > 1) l_run[1] *= alpha;
          if (WITH_V) {
#pragma unroll
            for (int x = 0; x < NO / NQ; ++x)
#pragma unroll
              for (int r = 0; r < NR; ++r) o[8 * n + x][r] *= alpha;
          }
        }
        exponentials(std::false_type{});
      }
      l_run[0] += rs[0];
      if (NL > 1) l_run[1] += rs[1];
      // (a part ends well before the diagonal: every wave that has rows works on its last tile)
      if (MODE == 1 && t == part_last) {
        store_part_lse();
        ++part;
        part_last = __builtin_amdgcn_readfirstlane(end_of_part());
        m_run[0] = kNegBig;
        l_run[0] = 0.f;
      }
    };

    // ---- the two-phase pipeline --------------------------------------------------------
    // MFMA phase(u):    P V(u-1), K Q^T(u)
    // softmax phase(u): softmax(u)
    // Iteration u also issues the loads of aux(u+3), V(u+2), K(u+3): from its softmax phase
    // (dense and strip-masked kernels) or from its MFMA phase (log-sum-exp sweep).
    // Group 0 runs MFMA phase u in the first half of iteration u, group 1 in the second.
    // Slot t % 4 of the K (V^T) ring is re-filled with tile t + 4 only after the barrier
    // that follows its last reader - K Q^T(t) (P V(t)) of group 1; a load is waited for
    // by the wave that issued it before the barrier that precedes its first reader.  Loads complete
    // in order, so "at most n in flight" means everything but the last n has landed: at
    // the end of iteration u the loads of iteration u - 1 that feed the next softmax and
    // K Q^T (V(u+1), and K(u+1) from iteration u - 2) must be in, the rest may still fly.
    unsigned long long tiles_done = 0;
    bool act_t = false;                        // this wave has work on the tile whose softmax comes next
    // list entries of tiles u .. u+3, settled up to u+2
    int dq0 = fetch_d(AnyTiles{}, 0), dq1 = fetch_d(AnyTiles{}, 1), dq2 = fetch_d(AnyTiles{}, 2), dq3 = fetch_d(AnyTiles{}, 3);
    int dq4 = 0;                               // fetched by the iteration: the entry of tile u+4
    uint64_t cols3 = 0;                        // ... and the column words of tile u+3
    // The scores, the probabilities and the operand ring are written on some paths only
    // (a wave may have no work on a tile).  An empty asm that "defines" them where their
    // old contents are dead tells the compiler so; without it every path that skips a
    // write carries the old value along, and the register allocator copies whole arrays
    // between two homes inside the loop.
    auto forget_ring = [&]() {
#pragma unroll
      for (int i = 0; i < 8; ++i) asm volatile("" : "=v"(R[i]));
    };
    auto forget_ring_and_p = [&]() {
      forget_ring();
#pragma unroll
      for (int i = 0; i < 4; ++i) asm volatile("" : "=v"(pk[i >> 1][i & 1]));
    };
    auto forget_scores = [&]() {
#pragma unroll
      for (int i = 0; i < NS; ++i) asm volatile("" : "=v"(s[i]));
    };
    // (An interior stretch knows that the wave works on every tile: as a run-time flag the answer
    // left a join in front of the K Q^T sweep, at which the compiler waited for the whole ring.)
    auto softmax_phase = [&](auto kc, int u, int d_u, int it) __attribute__((always_inline)) {   // list entry of tile u; iteration
      const bool act = decltype(kc)::INTERIOR ? !(decltype(kc)::FIRST && u < it) : act_t;   // (u < it: group 1)
      forget_ring_and_p();                     // consumed by the MFMA phase before
      if (kLoadsInSoftmax) {
        // the loads of iteration `it`: aux(it + 3), V(it + 2), K(it + 3)
        dma_aux(kc, it + 3, dq3);
        load_v_begin(kc, it + 2, dq2);
        load_k_begin(kc, it + 3, dq3);
        if (!act) { load_v_one(0); load_v_one(1); load_k_one(0); load_k_one(1); }
      }
      // The scalar loads are collected by the barrier's lgkmcnt(0).  While one is in flight every wait for
      // an LDS read waits for everything, so they go out where the next such wait is far away.
      auto fetch = [&]() {
        dq4 = fetch_d(kc, it + 4);
        cols3 = fetch_cols(kc, it + 3, dq3);
      };
      if (act) step_softmax(kc, u, d_u, fetch); else fetch();
    };
    auto mfma_phase = [&](auto kc, int u) __attribute__((always_inline)) {
      forget_scores();                         // consumed by the softmax phase before
      const bool have = is_real(kc, u);
      // (nothing is in flight: the V operands were requested a softmax ago.  Told so, the compiler does not
      // wait for the whole ring where the paths below meet in front of the K Q^T sweep.)
      if (WITH_V && !decltype(kc)::INTERIOR) __builtin_amdgcn_s_waitcnt(0xc07f);
      __builtin_amdgcn_s_setprio(1);
      const bool pv = WITH_V && (decltype(kc)::INTERIOR ? !decltype(kc)::FIRST : act_t);
      const bool late = MODE == 2 && !SWEEP && !decltype(kc)::INTERIOR && is_col(kc, u);   // activity from an aux word
      int aw0 = 0;
      bool act_n = !late && have && tile_active(kc, u, dq0, 0);
      if (pv) {
        auto look = [&]() { if (late && have) act_word(kc, u, aw0); };
        auto decide = [&]() { if (late) act_n = have && tile_active(kc, u, dq0, aw0); };
        mm_pv((u - 1) & (NSTAGE - 1), u & (NSTAGE - 1), look, decide);
      } else {
        if (!kLoadsInSoftmax) load_k_begin(kc, u + 3, dq3);
        if (late && have) {
          act_word(kc, u, aw0);
          act_n = tile_active(kc, u, dq0, aw0);
        }
        if (act_n) warm_k(u & (NSTAGE - 1)); else forget_ring();
      }
      if (act_n) mm_qk(u & (NSTAGE - 1));
      __builtin_amdgcn_s_setprio(0);
      if (!kLoadsInSoftmax && !act_n) { load_k_one(0); load_k_one(1); }
      tiles_done += act_n ? 1 : 0;
      act_t = act_n;
      // everything but this phase's loads and the K loads of the one before has landed
      if (!kLoadsInSoftmax) vm_wait<4>();
    };
    // before the barrier that ends an iteration everything has landed but that iteration's
    // loads and the K loads of the one before
    // (the wave that also fetched aux words waits for one load more than it must)
    auto end_of_iteration_wait = [&]() {
      if (kLoadsInSoftmax) vm_wait<6>();
    };

    // prologue: K(0..2), V(0..1) and the aux words of tiles 0..2
    {
      const AnyTiles any{};
      dma_aux(any, 0, dq0); dma_aux(any, 1, dq1); dma_aux(any, 2, dq2);
      load_k_begin(any, 0, dq0); load_k_one(0); load_k_one(1);
      load_k_begin(any, 1, dq1); load_k_one(0); load_k_one(1);
      load_k_begin(any, 2, dq2); load_k_one(0); load_k_one(1);
      load_v_begin(any, 0, dq0); load_v_one(0); load_v_one(1);
      load_v_begin(any, 1, dq1); load_v_one(0); load_v_one(1);
      const uint64_t c0 = fetch_cols(any, 0, dq0), c1 = fetch_cols(any, 1, dq1), c2w = fetch_cols(any, 2, dq2);
      dq0 = settle(any, 0, dq0, c0); dq1 = settle(any, 1, dq1, c1); dq2 = settle(any, 2, dq2, c2w);
    }
    // vmcnt(0), as the builtin: the compiler then also knows that the Q loads above have
    // landed and places no waits of its own for them inside the loop, where they would
    // wait for the loads in flight there as well
    __builtin_amdgcn_s_waitcnt(0x0f70);
    wg_barrier();
    // Iteration n: group 0 runs MFMA phase n, then softmax phase n; group 1 runs softmax
    // phase n - 1, then MFMA phase n; one workgroup barrier ends the iteration.  The
    // barrier is all the LDS traffic needs (a stage is re-filled, and a landed tile is
    // first read, at least one iteration after the other side touched it - see above);
    // starting the two groups on opposite phases after each barrier is what keeps one
    // wave of every SIMD on the matrix pipe while the other is on the vector pipe.
    // (The loop is written out once per group: one loop that picks the phase at run
    // time keeps the registers of both phases alive everywhere and spills.)
    // Iteration n touches tiles n - 1 .. n + 4 and decides on the work of tiles n and n + 1.
    // Strip-masked kernel: the selected keys that are not before the workgroup's first row
    // (at most 256) lie in the last five gathered tiles, so the iterations n + 1 <
    // n_col_tiles - 5 see gathered tiles only, with work for every wave and nothing to mask;
    // the iterations n > n_col_tiles see range tiles only; the few in between take the
    // general form.  Dense and log-sum-exp sweeps: the tiles below key tile a64 (the one
    // that holds the first row) are interior.  The iterations n + 4 < n_tiles see no tile
    // past the end of the schedule.
    const int n_gen0 = (MODE == 2 && !SWEEP) ? max(n_col_tiles - 6, 0)                 // first iteration of the general form
                                   : (MODE == 1 && i_last_wg - i0 < BQ - 32) ? 0      // (waves without rows look at every tile)
                                   : max(min(a64 - t_base - 1, n_tiles - 4), 0);
    const int n_gen1 = (MODE == 2 && !SWEEP) ? min(n_col_tiles, n_tiles) : n_tiles;    // its last
    const int n_real = n_tiles - 4;                                          // first iteration that may see a tile past the end
    if (grp == 0) {
      auto iteration = [&](auto kc, int n) __attribute__((always_inline)) {
        mfma_phase(kc, n);                     // n = 0: K Q^T(0) only; n = n_tiles: the last P V
        softmax_phase(kc, n, dq0, n);
        end_of_iteration_wait();
        wg_barrier();
        SA_PIN();
        dq0 = dq1; dq1 = dq2; dq2 = settle(kc, n + 3, dq3, cols3); dq3 = dq4;
      };
      int n = 0;
      auto interior = [&](auto kc) __attribute__((always_inline)) {
        if (n_gen0 > 0) iteration(typename decltype(kc)::AtFirst{}, n++);
        for (; n < n_gen0; ++n) iteration(kc, n);
      };
      if (SWEEP && IN_PLACE) {
        for (; n < n_real; ++n) iteration(RngRealTiles{}, n);
        for (; n <= n_tiles; ++n) iteration(RngTiles{}, n);
      } else if (MODE == 2 && !SWEEP) {
        interior(ColTiles{});
        for (; n <= n_gen1; ++n) iteration(AnyTiles{}, n);
        for (; n < n_real; ++n) iteration(RngRealTiles{}, n);
        for (; n <= n_tiles; ++n) iteration(RngTiles{}, n);
      } else {
        interior(PlainTiles{});
        for (; n <= n_gen1; ++n) iteration(AnyTiles{}, n);
      }
    } else {
      int dprev = 0;                           // tile diagonal of tile n - 1
      auto iteration = [&](auto kc, int n) __attribute__((always_inline)) {
        softmax_phase(kc, n - 1, dprev, n);
        mfma_phase(kc, n);
        end_of_iteration_wait();
        wg_barrier();
        SA_PIN();
        dprev = dq0; dq0 = dq1; dq1 = dq2; dq2 = settle(kc, n + 3, dq3, cols3); dq3 = dq4;
      };
      int n = 0;
      auto interior = [&](auto kc) __attribute__((always_inline)) {
        if (n_gen0 > 0) iteration(typename decltype(kc)::AtFirst{}, n++);
        for (; n < n_gen0; ++n) iteration(kc, n);
      };
      if (SWEEP && IN_PLACE) {
        for (; n < n_real; ++n) iteration(RngRealTiles{}, n);
        for (; n <= n_tiles; ++n) iteration(RngTiles{}, n);
      } else if (MODE == 2 && !SWEEP) {
        interior(ColTiles{});
        for (; n <= n_gen1; ++n) iteration(AnyTiles{}, n);
        for (; n < n_real; ++n) iteration(RngRealTiles{}, n);
        for (; n <= n_tiles; ++n) iteration(RngTiles{}, n);
      } else {
        interior(PlainTiles{});
        for (; n <= n_gen1; ++n) iteration(AnyTiles{}, n);
      }
    }
    vm_wait<0>();                              // nothing may still be writing LDS when the workgroup ends

    // ---- epilogue -------------------------------------------------------------
    if (MODE == 1) {
      store_part_lse();
      return;
    }
    if (MODE == 2 && P.tiles != nullptr && lane == 0 && tiles_done > 0) atomicAdd(P.tiles + bh, tiles_done);
    // four d in a run: 16 mb + 4 kg .. + 3 of both rows of a lane (WIDE: 32 mb + 8 g + 4 kg .. + 3 of its row)
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      const float l_tot = row_sum(n);
      if (!row_ok(n)) continue;
      const int i = i_me + 16 * n;
      if (PARTS) {
        const size_t slot = (size_t)bh * P.parts_per_head + J.part0 + split;
        const int r = 32 * wave + 16 * n + ql;
        if (kg == 0) reinterpret_cast<float2*>(P.part_ml)[slot * BQ + r] = make_float2(m_run[n], l_tot);
        float* po = P.part_o + (slot * BQ + r) * kHeadDim + 4 * kg;
#pragma unroll
        for (int x = 0; x < NO / NQ; ++x)
#pragma unroll
          for (int g = 0; g < NR / 4; ++g) {
            const Acc& a = o[8 * n + x];
            *reinterpret_cast<float4*>(po + (WIDE ? 32 * x + 8 * g : 16 * x)) = make_float4(a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]);
          }
        continue;
      }
      if (P.lse != nullptr && kg == 0) P.lse[(size_t)bh * S + i] = m_run[n] * kLn2 + __logf(l_tot);
      const float inv = 1.0f / l_tot;
      const size_t at = ((size_t)bh * S + i) * kHeadDim + 4 * kg;
#pragma unroll
      for (int x = 0; x < NO / NQ; ++x)
#pragma unroll
        for (int g = 0; g < NR / 4; ++g) {
          const Acc& a = o[8 * n + x];
          const float x0 = a[4 * g] * inv, x1 = a[4 * g + 1] * inv, x2 = a[4 * g + 2] * inv, x3 = a[4 * g + 3] * inv;
          const size_t d = at + (WIDE ? 32 * x + 8 * g : 16 * x);
          if (OUT_F32)
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(P.out) + d) = make_float4(x0, x1, x2, x3);
          else
            *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(P.out) + d) = make_uint2(pack_bf16x2(x0, x1), pack_bf16x2(x2, x3));
        }
    }
  } else {
    const int ql = lane & 31;   // query within the wave / row within a 32-row operand
    const int hf = lane >> 5;   // which half of the contraction block this lane feeds
    const int i_me = iw0 + ql;                             // this lane's query row
    const bool row_ok = i_me <= i_last_wg && i_me >= J.row_lo;
    // ---- Q^T operand: 8 contraction steps of 16, resident in registers -------
    bf16x8 qf[8];
    {
      int qr = row_ok ? i_me : max(min(i_last_wg, S - 1), 0);
      const uint16_t* qrow = P.q + ((size_t)bh * S + qr) * kHeadDim;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
        qf[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(qrow + ks * 16 + hf * 8));
    }

    f32x16 o[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[mb][r] = 0.f;
    float m_run = kNegBig;   // reference maximum, in log2 units (score * scale * log2 e)
    float l_run = 0.f;       // running sum of exp2 for this lane's keys
    const float c2 = P.scale_log2;

    // list entries of tiles u .. u+3 of iteration u, settled up to u+2
    int dq0 = fetch_d(AnyTiles{}, 0), dq1 = fetch_d(AnyTiles{}, 1), dq2 = fetch_d(AnyTiles{}, 2), dq3 = fetch_d(AnyTiles{}, 3);
    int dq4 = 0;                               // fetched by the iteration: the entry of tile u+4
    uint64_t cols3 = 0;                        // ... and the column words of tile u+3

    // ---- operands ----------------------------------------------------------------------
    // The MFMAs of an iteration take up to 32 operands of 32 rows from LDS: 16 of P V(u-1) (head-dim
    // blocks 0..3 for each of four 16-key groups) and 16 of K Q^T(u) (8 contraction steps for each of
    // two 32-key halves).  They come through a ring of 8 registers x 16 bytes: after the MFMA of operand
    // i has consumed slot i % 8, operand i + 8 is read into it, so every read has 7 MFMAs (~250 cycles)
    // to return and the matrix pipe does not wait on LDS round trips.  sched_barrier pins the order: the
    // compiler would otherwise sink each read down to its use.
    // Element r of s[sb] is key j0 + 32 sb + 16 (r / 8) + 8 hf + r % 8 against query i_me.
    f32x16 s[2];
    uint32_t pk[2][8];                         // probabilities of half sb as bf16
    // What the sum of a tile's second half starts from: infinity on the wave's first tile, so that the reference is looked for
    // there too and covers a whole tile, as in the other cores.  A row's largest probabilities are then close to 1, where
    // bf16 is exact; with the first 32 keys alone the error against fp64 was up to 2.5 % larger (8 heads of 3001, 10 %
    // of the columns, core 2 / first half / whole tile: 1.346e-3 / 1.369e-3 / 1.336e-3).
    float rs_first = __builtin_huge_valf();
    uint4 R[8];
    // operand i of iteration u; `st` (Steps) says which operands there are
    auto load_operand = [&](auto st, int i, int u) __attribute__((always_inline)) {
      using St = decltype(st);
      const int h = i / St::HALF, j = St::index(i);
      if (St::is_v(i)) {
        // row d = 32 mb + ql of V^T; logical chunk 4 h + 2 g + hf lives at physical chunk (..) ^ ((d >> 1) & 7)
        const int g = j >> 2, mb = j & 3;
        const char* vp = smem + OFF_V + ((u - 1) & (NSTAGE - 1)) * VTILE_B + (32 * mb + ql) * VROW_B;
        R[i & 7] = *reinterpret_cast<const uint4*>(vp + (((4 * h + 2 * g + hf) ^ ((ql >> 1) & 7)) << 4));
      } else {
        // row p = 32 h + ql of K; logical chunk 2 j + hf lives at physical chunk (..) ^ (p & 15)
        const char* kp = smem + OFF_K + (u & (NSTAGE - 1)) * KTILE_B + (32 * h + ql) * KROW_B;
        R[i & 7] = *reinterpret_cast<const uint4*>(kp + (((2 * j + hf) ^ (ql & 15)) << 4));
      }
    };
    auto multiply = [&](auto st, int i) __attribute__((always_inline)) {
      using St = decltype(st);
      const int h = i / St::HALF, j = St::index(i);
      if (St::is_v(i)) {                         // O^T += V^T P^T
        const int g = j >> 2, mb = j & 3;
        const uint4 pw = {pk[h][4 * g], pk[h][4 * g + 1], pk[h][4 * g + 2], pk[h][4 * g + 3]};
        o[mb] = mfma_32x32x16(as_bf16x8(R[i & 7]), as_bf16x8(pw), o[mb]);
      } else {                                   // S^T = K Q^T
        if (j == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) s[h][r] = 0.f;
        }
        s[h] = mfma_32x32x16(as_bf16x8(R[i & 7]), qf[j], s[h]);
      }
    };

    // ---- masks ---------------------------------------------------------------------------
    // One 32-bit pattern per lane and 32-key half, bit b <-> key j0 + 32 sb + 8 hf + b of the lane's 16
    // (b = 0..7, 16..23), set = keep.  The pattern is built per tile kind when the tile's
    // scores are under way; that of half 1 is used an iteration later.  A score is masked by a 1-bit
    // signed extract and a bitwise select between it and -inf: with its exponential (where every
    // tile is masked), or in a pass of its own that is left out where the half keeps every pair (a
    // whole block of the block mask, the inside of a band, tiles away from the causal edge).
    uint32_t km[2] = {0xFFFFFFFFu, 0xFFFFFFFFu};
    auto masked_score = [&](int sb, int r) __attribute__((always_inline)) -> float {
      const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe(km[sb], 16 * (r >> 3) + (r & 7), 1);   // all-ones where kept
      return __uint_as_float((__float_as_uint(s[sb][r]) & keep) | (0xFF800000u & ~keep));
    };
    auto mask_half = [&](int sb) __attribute__((always_inline)) {
      if (__builtin_amdgcn_ballot_w64((km[sb] & 0x00FF00FFu) != 0x00FF00FFu) == 0ull) return;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[sb][r] = masked_score(sb, r);
    };
    // words of a range tile's pattern, read a half iteration before they are used
    uint32_t rw[5] = {0, 0, 0, 0, 0};
    auto read_range_words = [&](auto kc, int t, int d) __attribute__((always_inline)) {
      if (is_col(kc, t)) return;
      const uint32_t* mw = reinterpret_cast<const uint32_t*>(smem + OFF_A + (t & (NAUX - 1)) * AUX_B);
      const int j0 = first_key(kc, t, d);
      const int wb = (P.off_max - (i0 - j0 + BQ - 1)) >> 5;
      const int x0 = P.off_max - (i_me - (j0 + 8 * hf));        // >= 0 by construction of the bitmap
      const int k = (x0 >> 5) - wb;                             // 0 .. 9: word of the staged window
      rw[0] = mw[k]; rw[1] = mw[k + 1]; rw[2] = mw[k + 2];
      rw[3] = mw[16]; rw[4] = mw[17];                           // the column words
    };
    auto build_masks = [&](auto kc, int t, int d) __attribute__((always_inline)) {
      constexpr bool INTERIOR = decltype(kc)::INTERIOR;
      if (!is_col(kc, t)) {
        const int tl = i_me - (first_key(kc, t, d) + 8 * hf);     // offset of the lane's first key
        const int x0 = P.off_max - tl;
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
          const uint32_t ow = __builtin_amdgcn_alignbit(rw[sb + 1], rw[sb], x0 & 31);  // bit b <-> offset tl - 32 sb - b
          const uint32_t cw = rw[3 + sb] >> (8 * hf);                                  // bit 16u+e <-> key is a selected column
          km[sb] = ow & ~cw;                       // columns were taken by the gathered tiles
        }
        return;
      }
      km[0] = km[1] = 0xFFFFFFFFu;
      const int32_t* il = reinterpret_cast<const int32_t*>(smem + OFF_A + (t & (NAUX - 1)) * AUX_B);
      if (!INTERIOR && il[BK - 1] > iw0) {         // only the last gathered tiles reach past a row: keep index <= query
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
          uint32_t m = 0;
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const int4* ip = reinterpret_cast<const int4*>(il + 32 * sb + 16 * g + 8 * hf);
            int4 x0 = ip[0], x1 = ip[1];
            int jj[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) m |= (jj[e] <= i_me ? 1u : 0u) << (16 * g + e);
          }
          km[sb] = m;
        }
      }
    };

    // ---- one iteration of a wave ------------------------------------------------------------
    // Iteration u issues the MFMAs of P V(u-1) and of K Q^T(u), and with them, in the same
    // instruction stream, the softmax of the scores that are there: half 1 (keys 32..63) of tile u-1
    // beside the first half of the MFMAs (P V of half 0, K Q^T of half 0), half 0 of tile u beside the
    // second (P V of half 1, K Q^T of half 1).  So a wave feeds the matrix and the vector pipe
    // at once, whatever the other wave of its SIMD does.
    //
    // Online softmax, optimistic: the exponentials are taken against the reference
    // maximum the row already has, and only their sum is looked at.  A sum within
    // 2^8 means that no probability exceeds 2^8, which is all the reference is
    // for (exact in fp32 and bf16 alike); then the tile costs no maximum at all.
    // Otherwise (first tiles of a row, or a score far above what the row has seen: the
    // sum is large, inf or NaN) the row maximum of the half is formed, the reference
    // moved up to it, the accumulators rescaled and the exponentials taken again.
    //
    // PREV, CUR: tile u-1 / u has work for this wave.  MM: masks are applied not at all (0), with
    // the exponentials (1), in a pass (2).  AHEAD: the ring holds the first eight operands already and
    // is left with those of the next iteration (which has work on both tiles too).
    auto run = [&](auto kc, auto prev_tag, auto cur_tag, auto ahead_tag, int u, auto&& fetch) __attribute__((always_inline)) {
      constexpr bool PREV = decltype(prev_tag)::value, CUR = decltype(cur_tag)::value, AHEAD = decltype(ahead_tag)::value;
      constexpr int KIND = decltype(kc)::KIND;
      constexpr int MM = (!IN_PLACE && KIND == 2) ? 1 : decltype(kc)::INTERIOR ? 0 : 2;
      using St = Steps<PREV, CUR>;
      constexpr int H = St::HALF;
      if (!AHEAD) {
#pragma unroll
        for (int i = 0; i < (H > 0 ? 8 : 0); ++i) load_operand(St{}, i, u);
        SA_PIN();
      }
      if (CUR && MM != 0) read_range_words(kc, u, dq0);
      auto half = [&](auto h_tag) __attribute__((always_inline)) {
        constexpr int h = decltype(h_tag)::value, sb = 1 - h;
        constexpr bool SM = h == 0 ? PREV : CUR;
        if (SM && MM == 2) mask_half(sb);
        auto score = [&](int r) __attribute__((always_inline)) -> float { return MM == 1 ? masked_score(sb, r) : s[sb][r]; };
        float rs = h == 0 ? rs_first : 0.f, p[16];
        if (SM && h == 0) rs_first = 0.f;
        auto element = [&](int r) __attribute__((always_inline)) {
          p[r] = fast_exp2(fmaf(score(r), c2, -m_run));
          rs += p[r];
          if (r & 1) pk[sb][r >> 1] = pack_bf16x2(p[r - 1], p[r]);
        };
        // the loads of the tiles ahead, one at a time: V in the first half, K in the second
        if (h == 0) load_v_begin(kc, u + 2, dq2); else load_k_begin(kc, u + 3, dq3);
        auto load_one = [&](int n) __attribute__((always_inline)) { if (h == 0) load_v_one(n); else load_k_one(n); };
        if (H == 0) { load_one(0); load_one(1); }
        if (h == 1) fetch();
#pragma unroll
        for (int i = 0; i < H; ++i) {
          const int x = h * H + i;
          multiply(St{}, x);
          SA_PIN();
          if (x + 8 < 2 * H) load_operand(St{}, x + 8, u);
          else if (AHEAD) load_operand(St{}, x + 8 - 2 * H, u + 1);
          if (i == H / 4) load_one(0);
          if (i == H / 4 + H / 2) load_one(1);
          SA_PIN();
          if (SM) {
#pragma unroll
            for (int e = 16 * i / H; e < 16 * (i + 1) / H; ++e) element(e);
            SA_PIN();
          }
        }
        if (SM && H == 0) {
#pragma unroll
          for (int e = 0; e < 16; ++e) element(e);
        }
        if (SM) {
          if (__builtin_expect(__any(!(rs <= kSumBound)), 0)) {
            // (the maximum starts from a value the compiler cannot see through: otherwise it
            // forms the whole maximum ahead of the branch, on every tile)
            float mx = score(0);
            asm volatile("" : "+v"(mx));
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, score(r));
            mx = half_max(mx);                     // the two lanes of a row agree on its reference
            const float m_cand = mx * c2;
            const float m_new = (m_cand > m_run) ? m_cand : m_run;
            const float alpha = fast_exp2(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int mb = 0; mb < 4; ++mb)
#pragma unroll
              for (int r = 0; r < 16; ++r) o[mb][r] *= alpha;
            rs = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) element(r);
          }
          l_run += rs;
        }
      };
      half(std::integral_constant<int, 0>{});
      if (CUR && MM != 0) build_masks(kc, u, dq0);
      half(std::integral_constant<int, 1>{});
    };

    // ---- the tile loop -------------------------------------------------------------------
    // Iteration u reads V(u-1) and K(u) and issues the loads of aux(u+3), V(u+2), K(u+3); one
    // workgroup barrier ends it.  Slot t % 4 of the K (V^T) ring is re-filled with tile t + 4 from
    // iteration t + 1 (t + 2) on, after the barrier that follows its last reader.  A load is waited for
    // by the wave that issued it before a barrier: loads complete in order, and before the barrier that
    // ends iteration u everything has landed but that iteration's four loads, so that V(u+1)
    // and K(u+2) are there: what iteration u+1 reads, and the first operands of the next that it
    // reads ahead.
    unsigned long long tiles_done = 0;
    bool act_prev = false;                     // this wave has work on the tile before
    // prologue: K(0..2), V(0..1) and the aux words of tiles 0..2
    {
      const AnyTiles any{};
      dma_aux(any, 0, dq0); dma_aux(any, 1, dq1); dma_aux(any, 2, dq2);
      load_k_begin(any, 0, dq0); load_k_one(0); load_k_one(1);
      load_k_begin(any, 1, dq1); load_k_one(0); load_k_one(1);
      load_k_begin(any, 2, dq2); load_k_one(0); load_k_one(1);
      load_v_begin(any, 0, dq0); load_v_one(0); load_v_one(1);
      load_v_begin(any, 1, dq1); load_v_one(0); load_v_one(1);
      const uint64_t c0 = fetch_cols(any, 0, dq0), c1 = fetch_cols(any, 1, dq1), c2w = fetch_cols(any, 2, dq2);
      dq0 = settle(any, 0, dq0, c0); dq1 = settle(any, 1, dq1, c1); dq2 = settle(any, 2, dq2, c2w);
    }
    // vmcnt(0), as the builtin: the compiler then also knows that the Q loads above have
    // landed and places no waits of its own for them inside the loop, where they would
    // wait for the loads in flight there as well
    __builtin_amdgcn_s_waitcnt(0x0f70);
    wg_barrier();
    constexpr std::true_type YES{};
    constexpr std::false_type NO{};
    // The arrays are written on some paths only (a wave may have no work on a tile).  An empty asm
    // that "defines" what an iteration hands on, where its contents are dead, tells the compiler so;
    // without it every path that skips a write carries the old values along, and the register
    // allocator copies whole arrays between two homes inside the loop.
    auto hand_on_nothing = [&]() __attribute__((always_inline)) {
      asm volatile("" : "=v"(s[1]));
#pragma unroll
      for (int i = 0; i < 8; ++i) asm volatile("" : "=v"(pk[0][i]));
    };
    auto iteration = [&](auto kc, auto ahead, int u) __attribute__((always_inline)) {
      using Kc = decltype(kc);
      // The scalar loads are collected at the barrier.  While one is in flight every wait for
      // an LDS read waits for everything.
      auto fetch = [&]() __attribute__((always_inline)) {
        dq4 = fetch_d(kc, u + 4);
        cols3 = fetch_cols(kc, u + 3, dq3);
      };
      dma_aux(kc, u + 3, dq3);
      bool act = true;
      if constexpr (Kc::INTERIOR) {
        if constexpr (Kc::FIRST) run(kc, NO, YES, NO, u, fetch); else run(kc, YES, YES, ahead, u, fetch);
      } else {
        int w0 = 0;
        if (is_real(kc, u)) act_word(kc, u, w0);
        act = is_real(kc, u) && tile_active(kc, u, dq0, w0);
        if (act_prev && act) {
          run(kc, YES, YES, NO, u, fetch);
        } else if (act) {
          run(kc, NO, YES, NO, u, fetch);
        } else {
          if (act_prev) {
            run(kc, YES, NO, NO, u, fetch);
          } else {
            load_v_begin(kc, u + 2, dq2); load_v_one(0); load_v_one(1);
            load_k_begin(kc, u + 3, dq3); load_k_one(0); load_k_one(1);
            fetch();
          }
          hand_on_nothing();
        }
      }
      tiles_done += act ? 1 : 0;
      act_prev = act;
      vm_wait<4>();
      // (the operands read ahead stay in flight: their stages are not re-filled in the next iteration)
      if constexpr (decltype(ahead)::value) wg_meet(); else wg_barrier();
      SA_PIN();
      dq0 = dq1; dq1 = dq2; dq2 = settle(kc, u + 3, dq3, cols3); dq3 = dq4;
    };
    // Iteration n touches tiles n - 1 .. n + 4 and decides on the work of tile n.
    // Strip-masked kernel: the selected keys that are not before the workgroup's first row
    // (at most 256) lie in the last five gathered tiles, so the iterations n + 1 <
    // n_col_tiles - 5 see gathered tiles only, with work for every wave and nothing to mask;
    // the iterations n > n_col_tiles see range tiles only; the few in between take the
    // general form.  The iterations n + 4 < n_tiles see no tile past the end of the schedule.
    const int n_gen0 = max(n_col_tiles - 6, 0);                              // first iteration of the general form
    const int n_gen1 = min(n_col_tiles, n_tiles);                            // its last
    const int n_real = n_tiles - 4;                                          // first iteration that may see a tile past the end
    int n = 0;
    if (n_gen0 > 0) {
      iteration(ColTiles::AtFirst{}, NO, n++);
#pragma unroll
      for (int i = 0; i < 8; ++i) load_operand(Steps<true, true>{}, i, n);
      for (; n < n_gen0; ++n) iteration(ColTiles{}, YES, n);
      act_prev = true;
    }
    for (; n <= n_gen1; ++n) iteration(AnyTiles{}, NO, n);
    for (; n < n_real; ++n) iteration(RngRealTiles{}, NO, n);
    for (; n <= n_tiles; ++n) iteration(RngTiles{}, NO, n);
    vm_wait<0>();                              // nothing may still be writing LDS when the workgroup ends

    // ---- epilogue -------------------------------------------------------------
    float l_tot = half_sum(l_run);
    if (P.tiles != nullptr && lane == 0 && tiles_done > 0) atomicAdd(P.tiles + bh, tiles_done);
    if (!row_ok) return;
    if (PARTS) {
      const size_t slot = (size_t)bh * P.parts_per_head + J.part0 + split;
      const int r = 32 * wave + ql;
      if (hf == 0) reinterpret_cast<float2*>(P.part_ml)[slot * BQ + r] = make_float2(m_run, l_tot);
      float* po = P.part_o + (slot * BQ + r) * kHeadDim;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<float4*>(po + 32 * mb + 8 * g + 4 * hf) =
              make_float4(o[mb][4 * g], o[mb][4 * g + 1], o[mb][4 * g + 2], o[mb][4 * g + 3]);
      return;
    }
    if (P.lse != nullptr && hf == 0) P.lse[(size_t)bh * S + i_me] = m_run * kLn2 + __logf(l_tot);
    float inv = 1.0f / l_tot;
    size_t rowoff = ((size_t)bh * S + i_me) * kHeadDim;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        int d = 32 * mb + 8 * g + 4 * hf;
        float x0 = o[mb][4 * g] * inv, x1 = o[mb][4 * g + 1] * inv;
        float x2 = o[mb][4 * g + 2] * inv, x3 = o[mb][4 * g + 3] * inv;
        if (OUT_F32) {
          float4 v4 = {x0, x1, x2, x3};
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(P.out) + rowoff + d) = v4;
        } else {
          uint2 v2 = {pack_bf16x2(x0, x1), pack_bf16x2(x2, x3)};
          *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(P.out) + rowoff + d) = v2;
        }
      }
  }
#undef SA_PIN
}

// CORE: the core (see the top of the file) of dense and swept tiles.  Heads in two passes take core 1, or
// core 0 where the call is large and long (short_lists) and the head's list does not leave too many waves without
// work (kSparseBit; strips only).
template <int MODE, bool OUT_F32, bool IN_PLACE, bool PARTS, int CORE>
__global__ __launch_bounds__(NT, (MODE == 1) ? 4 : 1) void flash_kernel(FlashParams P) {
  // ---- which (head, query tile) this workgroup owns ------------------------
  // (the log-sum-exp sweep may also give the keys of a query tile to k_splits workgroups)
  TileJob J;
  J.split = 0; J.n_parts = 1; J.part0 = 0; J.lse_parts = J.k_splits = 1;
  {
    const int bid = blockIdx.x;
    int f = 0;                           // tile, counted over the segments
    SegmentJob seg = P.seg[0];
    J.seg = 0;
    if (PARTS) {
      // heavy (late) query tiles first, the heads of a part side by side
      // (a segment's values are read once: a load for every tile passed over is 1 us of a small call)
      J.bh = bid % P.n_bh;
      J.split = bid / P.n_bh;
      const int pm = P.part_m;
      for (int m = P.n_seg - 1; m > 0; --m) {   // (both loops end: the grid has exactly the parts of these tiles)
        const int n = parts_before(pm, P.seg[m].qtile0, P.seg[m].qtile0 + P.seg[m].n_qtiles);
        if (J.split < n) {
          seg = P.seg[m];
          J.seg = m;
          break;
        }
        J.split -= n;
      }
      const int q0 = seg.qtile0, q1 = q0 + seg.n_qtiles;
      int a = q1 - 1, before = parts_before(pm, q0, q1), rem;
      J.n_parts = a / pm + 1;
      rem = a % pm;
      while (J.split >= J.n_parts && a > q0) {
        J.split -= J.n_parts;
        before -= J.n_parts;
        --a;
        if (--rem < 0) {
          rem = pm - 1;
          --J.n_parts;
        }
      }
      J.a = a;
      J.part0 = seg.part0 + before - J.n_parts;
    } else if (MODE == 2) {
      // heads are sliced over the 8 XCDs (workgroups go round-robin to XCDs) and an
      // XCD works through one head at a time, heavy (late) query tiles first: the
      // workgroups resident on it then stream the gathered columns of the same head,
      // a working set (tens of MB per XCD) that the memory-side cache can hold.
      if (P.n_bh >= 8) {
        // Where an XCD's heads have few query tiles each, that leaves the last head's heavy
        // tiles for the end, with no light ones left to even them out (8K tokens: 32 CUs go
        // through 4 x 32 tiles): there the heavy tiles of all its heads come first.
        const int xcd = bid & 7, slot = bid >> 3, heads = (P.n_bh + 7) >> 3;
        const bool by_tile = P.n_qtiles <= kByTileMax;
        f = P.n_qtiles - 1 - (by_tile ? slot / heads : slot % P.n_qtiles);
        J.bh = xcd + 8 * (by_tile ? slot % heads : slot / P.n_qtiles);
        if (J.bh >= P.n_bh) return;
      } else {
        f = P.n_qtiles - 1 - bid / P.n_bh;
        J.bh = bid % P.n_bh;
        if (f < 0) return;
      }
    } else {
      // a bundle = the query heads sharing one KV head at one query tile; the
      // bundle's workgroups land on one XCD so the K/V stream is shared in L2.
      // (Log-sum-exp: n_qtiles of every segment, cut by each into its own k_splits.)
      int xcd = bid & 7, slot = bid >> 3;
      int bl = slot / P.group, hg = slot % P.group;
      int bundle = bl * 8 + xcd;
      if (MODE == 1) {
        // (late segments first, as everywhere: their rows see the most keys.  Sweep, early first / late first: 16 heads
        // of 20000 in four segments 48.7 / 46.0 us, 32 in eight of 512 rows 443 / 425)
        for (int m = P.n_seg - 1; m > 0; --m) {
          const int n = P.n_qtiles * P.seg[m].k_splits * P.n_bkv;
          if (bundle < n) {
            seg = P.seg[m];
            J.seg = m;
            break;
          }
          bundle -= n;
        }
        J.lse_parts = seg.lse_parts;
        J.k_splits = seg.k_splits;
      }
      const int ks = J.k_splits;
      if (bundle >= P.n_qtiles * ks * P.n_bkv) return;
      const int av = P.n_qtiles * ks - 1 - bundle / P.n_bkv;
      J.split = av % ks;
      J.bh = bundle % P.n_bkv * P.group + hg;
      J.a = av / ks;
    }
    if (!PARTS && MODE == 2) {
      if (P.n_seg > 1) {
        J.seg = segment_of(P, f);
        seg = P.seg[J.seg];
      }
      J.a = seg.qtile0 + f - seg.tile0;
    }
    J.row_lo = seg.row_lo;
    J.row_hi = seg.row_hi;
  }
  if constexpr (MODE == 2) {
    // (diagonal 0 is in every list, and its entry is the first)
    const int first = __builtin_amdgcn_readfirstlane(P.dlist[(size_t)(J.seg * P.n_bh + J.bh) * P.dlist_stride]);
    if (first & kSweepBit) {
      flash_body<MODE, OUT_F32, IN_PLACE, MODE == 2, PARTS, CORE>(P, J);
    } else if (PARTS || P.short_lists || (!IN_PLACE && (first & kSparseBit))) {
      flash_body<MODE, OUT_F32, IN_PLACE, false, PARTS, 1>(P, J);
    } else if constexpr (!PARTS) {
      flash_body<MODE, OUT_F32, IN_PLACE, false, false, 0>(P, J);
    }
  } else {
    flash_body<MODE, OUT_F32, IN_PLACE, false, PARTS, CORE>(P, J);
  }
}

// The parts of a query tile brought to one reference maximum, added in fixed order and
// normalised.  Eight rows per workgroup, 32 lanes of four columns each.
// (SEGMENTS: there are several.  Found in a loop over the arguments, the one of most launches cost 1.1 us of
// the 7.7 that 8 heads of 3001 tokens take.)
template <bool OUT_F32, bool SEGMENTS>
__global__ __launch_bounds__(256) void parts_combine_kernel(FlashParams P) {
  const int bh = blockIdx.y, tid = threadIdx.x;
  const int r_launch = blockIdx.x * 8 + (tid >> 5);
  const int seg = SEGMENTS ? segment_of(P, r_launch / BQ) : 0;
  const int a = P.seg[seg].qtile0 + r_launch / BQ - P.seg[seg].tile0, r = r_launch % BQ;
  const int i = a * BQ + r, c4 = tid & 31;
  if (i < P.seg[seg].row_lo || i >= P.seg[seg].row_hi) return;
  const size_t slot = (size_t)bh * P.parts_per_head + P.seg[seg].part0 + parts_before(P.part_m, P.seg[seg].qtile0, a);
  const int n_parts = a / P.part_m + 1;
  const float2* ml = reinterpret_cast<const float2*>(P.part_ml) + slot * BQ + r;
  const float4* po = reinterpret_cast<const float4*>(P.part_o + (slot * BQ + r) * kHeadDim) + c4;
  float m = ml[0].x;
  for (int s = 1; s < n_parts; ++s) m = fmaxf(m, ml[s * BQ].x);
  float l = 0.f;
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s = 0; s < n_parts; ++s) {
    const float2 e = ml[s * BQ];
    const float w = fast_exp2(e.x - m);
    const float4 y = po[(size_t)s * BQ * (kHeadDim / 4)];
    l = fmaf(e.y, w, l);
    x.x = fmaf(y.x, w, x.x); x.y = fmaf(y.y, w, x.y); x.z = fmaf(y.z, w, x.z); x.w = fmaf(y.w, w, x.w);
  }
  const float inv = 1.0f / l;
  const size_t at = ((size_t)bh * P.S + i) * kHeadDim + 4 * c4;
  if (OUT_F32)
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(P.out) + at) = make_float4(x.x * inv, x.y * inv, x.z * inv, x.w * inv);
  else
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(P.out) + at) =
        make_uint2(pack_bf16x2(x.x * inv, x.y * inv), pack_bf16x2(x.z * inv, x.w * inv));
  if (P.lse != nullptr && c4 == 0) P.lse[(size_t)bh * P.S + i] = m * kLn2 + __logf(l);
}

// out[i] = log sum_s exp(part[s][i]): the key parts of the log-sum-exp sweep, in fixed order.  A few
// blocks with up to 64 loads a thread: bound by their latency unless several are in flight (32 parts
// of 4096 rows one by one / eight at a time: sweep and combination 58.5 / 49.7 us).
// (A segment's values [heads, rows] lie behind each other, its parts n apart; k of them each.)
struct LseParts { int per_seg, k[kMaxSegs]; };
__global__ void lse_combine_kernel(const float* part, float* out, size_t n, LseParts L) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int k = L.k[i / L.per_seg];
  float m = part[i];
#pragma unroll 8
  for (int s = 1; s < k; ++s) m = fmaxf(m, part[(size_t)s * n + i]);
  float z = 0.f;
#pragma unroll 8
  for (int s = 0; s < k; ++s) z += __expf(part[(size_t)s * n + i] - m);
  out[i] = m + __logf(z);
}

hipError_t launch_lse_combine(const FlashParams& P, float* out, hipStream_t st) {
  const size_t n = (size_t)P.n_slots * P.n_qrows;
  if (n == 0) return hipSuccess;
  LseParts L;
  L.per_seg = P.n_bh * P.n_qrows;
  for (int m = 0; m < kMaxSegs; ++m) L.k[m] = m < P.n_seg ? P.seg[m].lse_parts : 1;
  hipLaunchKernelGGL(lse_combine_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, P.lse, out, n, L);
  return hipGetLastError();
}

// The log-sum-exp launch cuts the keys of a query tile into equal parts, which are summed apart
// and combined in fixed order, and gives them to workgroups, some neighbouring ones to each.
// How many workgroups: W of them fill the 512 slots (256 CUs x 2) unevenly, and 128 sampled rows
// are one query tile per head, a serial chain over every key on a chip that is nearly idle.  A
// workgroup costs its tiles and kStartTiles tiles' worth of start and end; one that has a CU to
// itself runs its tiles in 0.6 of the time.
// How many parts: what a call of kFewHeads heads would take as workgroups, whatever the heads of
// this call or pass, so that a row's bits follow from its sequence alone.  (With the parts left
// to the workgroups a row's last bits, and with them strips at the selection's cut, followed the
// batch and the room in the workspace.)  A part keeps kMinPartTiles tiles, more than the five that
// a query tile can span, so that every row sees a key in every part.
// Parts of at least 64 tiles / of at least eight, whole path: three segments of two sequences of
// 5003 tokens 523 / 422 us, blocks at 32K 2535 / 2450 us, 8K 770 / 690 us.  The sweep alone, parts
// left to the workgroups / from the sequence: 32 heads of 128K and 6592 rows 6235 / 6233 us, of
// 50001 and 2560 rows 949 / 952, of 32K and 1664 rows 486 / 476, of 32K and 128 rows 50 / 50, of 128K
// and 128 rows 150 / 155.
constexpr int kStartTiles = 6, kMinPartTiles = 8, kFewHeads = 4;
static int lse_workgroups(int n_qtiles, int n_bh, int min_tiles, int k_max) {
  const long long W = (long long)n_qtiles * n_bh;
  auto cost = [&](int k) {
    const long long n = W * k;
    return (n <= 256 ? 0.6 : (double)((n + 511) / 512)) * ((double)min_tiles / k + kStartTiles);
  };
  int best = 1;
  for (int k = 2; k <= k_max && min_tiles / k >= kMinPartTiles; k *= 2)
    if (cost(k) < cost(best)) best = k;
  return best;
}

void lse_splits(int row_first, int n_s, int n_bh, int max_parts, int* parts, int* workgroups) {
  const int n_qtiles = (n_s + kFlashBQ - 1) / kFlashBQ;
  const int min_tiles = row_first / kFlashBK;       // key tiles the first sampled row sees, at least
  *parts = lse_workgroups(n_qtiles, kFewHeads, min_tiles, max_parts);
  *workgroups = lse_workgroups(n_qtiles, n_bh, min_tiles, *parts);
}

// Parts of the schedules of a dense or strip-masked launch over the query tiles [q0, q1).  A
// workgroup has a CU to itself, so fewer workgroups than the 256 CUs leave part of the chip
// idle while the last query tile goes through all its key tiles alone.  Tile a, of 4 (a + 1)
// key tiles in a causal sweep, is then cut into ceil((a + 1) / m) equal parts of at most 4 m.
// Short parts fill the chip, but each leaves 132 KB of sums to be written and read: m follows
// the length (the last tile in six parts) and grows only in coarse steps, until there are no
// more parts than CUs; then the cut is made if the estimate says that it pays (a key tile takes
// kTileUs, the combination kCombineUs and kPartUs a part).  All this depends on the shape of the
// call alone, so that a tile's result does not depend on how the call divides heads and queries over
// its launches.  It does depend on the number of heads, batch included: of the 300 shapes of 1, 2, 4 .. 32
// heads and up to 128 tiles at which a sequence or two of them are cut, 237 are cut differently
// for one and two, and their results agree to rounding only.  One cut for every batch would have to
// be made where the chip is full as well, and there the sums would cost more than the work (32
// sequences of 8 heads and 3001 tokens, computed: 1 GB of them written and read at the rate of a
// copy 0.45 ms, the key tiles at kTileUs on 256 CUs 0.35 ms).
// Dense kernel, uncut / cut (parts): 1 head of 1024 tokens 29.5 / 20.9 us (10), of 4096
// 81 / 33 (51), 4 of 2048 47 / 31 (80), of 8192 156 / 88 (240), 8 of 1500 37 / 31 (168), of 3001
// 64 / 41 (240); left uncut: 16 of 3000 66.6 / 66.0 (256), 32 of 600 21.7 / 29.8 (192).
// Up to two query tiles there are eight key tiles at most to share, and a second launch costs as much.
// Uncut / cut, whole call: dense 1 head of 257 tokens 20.6 / 25.5 us, 4 of 384 20.8 / 23.8, 1 of
// 512 25.0 / 24.0; strips 4 of 384 29.6 / 32.9; blocks of 128 4 of 384 28.4 / 29.6, of 512 31.0 / 30.0.
// Three tiles: dense 8 of 640 25.2 / 26.2, 8 of 768 29.6 / 27.1, strips 4 of 640 35.5 / 34.6, blocks 1 of
// 640 31.0 / 30.2, 8 of 768 36.0 / 33.5; blocks 4 of 1024 40.2 / 32.9, of 2047 59.2 / 40.6.
constexpr int kMinCutTiles = 3;
constexpr double kTileUs = 1.1, kCombineUs = 3.0, kPartUs = 0.065;
// Several segments in one launch are one set of tiles, cut by one m.
int flash_parts(int n_bh, int n_seg, const SegmentJob* seg) {
  int q1 = 0, tiles = 0;
  double spread = 0;
  for (int k = 0; k < n_seg; ++k) {
    const int lo = seg[k].qtile0, hi = lo + seg[k].n_qtiles;
    q1 = q1 > hi ? q1 : hi;
    tiles += hi - lo;
    spread += n_bh * 2.0 * ((double)hi * (hi + 1) - (double)lo * (lo + 1)) / 256;
  }
  if (q1 < kMinCutTiles || (long long)n_bh * tiles > kMaxParts) return 0;
  const double longest = 4.0 * q1;
  const int base = (q1 + 5) / 6;
  for (int step : {2, 3, 4, 6, 8}) {
    const int m = (base * step + 1) / 2;
    const long long n = (long long)n_bh * parts_of(m, n_seg, seg);
    if (n > kMaxParts) continue;
    const double part = 4.0 * m;
    const double t = (part > spread ? part : spread) * kTileUs + kCombineUs + kPartUs * n;
    return m < q1 && t < longest * kTileUs ? m : 0;
  }
  return 0;
}

int parts_of(int m, int n_seg, const SegmentJob* seg) {
  int n = 0;
  for (int k = 0; k < n_seg; ++k) n += parts_before(m, seg[k].qtile0, seg[k].qtile0 + seg[k].n_qtiles);
  return n;
}

size_t flash_parts_bytes(int m, int n_heads, int n_seg, const SegmentJob* seg) {
  return m == 0 ? 0 : (size_t)n_heads * parts_of(m, n_seg, seg) * BQ * (kHeadDim + 2) * sizeof(float);
}

template <int MODE, bool OUT_F32, bool IN_PLACE, bool PARTS, int CORE>
static hipError_t launch_one(const FlashParams& P, int grid, hipStream_t st) {
  size_t shmem = (MODE == 1) ? LDS_B_LSE : LDS_B;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&flash_kernel<MODE, OUT_F32, IN_PLACE, PARTS, CORE>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((flash_kernel<MODE, OUT_F32, IN_PLACE, PARTS, CORE>), dim3(grid), dim3(NT), shmem, st, P);
  return hipGetLastError();
}
template <int MODE, bool IN_PLACE>
static hipError_t launch_whole(bool out_f32, int core, const FlashParams& P, int grid, hipStream_t st) {
  if (core == 0) return out_f32 ? launch_one<MODE, true, IN_PLACE, false, 0>(P, grid, st) : launch_one<MODE, false, IN_PLACE, false, 0>(P, grid, st);
  return out_f32 ? launch_one<MODE, true, IN_PLACE, false, 2>(P, grid, st) : launch_one<MODE, false, IN_PLACE, false, 2>(P, grid, st);
}

// The core of a launch's dense and swept tiles.  Core 0 and core 2 give the same bits, so this choice may
// follow the launch.  Up to some 1.5 rounds of the 256 CUs the chain of the heaviest tile decides and core 2
// is faster, above them the power.  Core 0 / core 2 against the faster one, whole path: dense, 8 heads of 8300 (264 tiles) 186 /
// 174 us, of 10800 (344) 255 / 249, of 12000 (376) 293 / 290, of 14000 (440) 348 / 355, 32 of 2100 (288) 58.6 / 57.6, 64 of 2100
// (576) 100 / 98.6, 32 of 3500 (448) 118.6 / 120; swept strips, 4 of 15000 (236) 431 / 416, 16 of 4500 (288) 184 / 181, of 5003 (320) 199 /
// 199, of 6000 (384) 233 / 236; swept blocks of 128, whose sweep has no interior stretch, 16 of 4500 176 / 165, 8 of 12000
// 364 / 355, of 14000 420 / 421, 32 of 5000 (640) 277 / 276, of 7000 (896) 435 / 439.
// Not core 1, though its chain is the shortest (dense, 32 heads of 500 21.5 / 22.2 us, 4 of 2000 in parts 30.6 / 31.1): its
// references begin with 32 keys where the others take 64, so a row's largest probabilities are less often close to 1, where
// bf16 is exact.  Error against fp64, cores 2 / 1: 2 heads of 600 1.177e-3 / 1.214e-3, 8 of 3001 1.200e-3 / 1.219e-3.
constexpr int kWideDense = 384, kWideStrips = 320, kWideBlocks = 640, kWideLength = 3072;
static int sweep_core(int mode, const FlashParams& P) {
  const long long tiles = (long long)P.n_bh * P.n_qtiles;
  if (mode == 0) return P.S < kWideLength || tiles <= kWideDense ? 2 : 0;
  return tiles <= (P.cols_in_place ? kWideBlocks : kWideStrips) ? 2 : 0;
}

// Which calls have heads in two passes on core 0 (if their lists are not sparse): of more tiles than CUs, of
// sequences long enough.  By the length alone, so that a head's bits above 256 query tiles do not follow the
// batch.  Gain over core 2, core 0 / core 1: strips 32 heads of 3000 0.95 / 1.02, of 6001 0.93 / 1.05, 16 of 20000
// 0.97 / 1.05, 8 of 40000 0.99 / 1.02, but 32 of 65536 1.04 / 1.00.  Block lists 32 of 16384 1.02 / 1.06, of 32768 1.06 / 1.04.
constexpr int kLongStrips = 49152, kLongBlocks = 24576;
bool two_cores(bool blocks, int S, int all_tiles) { return all_tiles > kMaxParts && S >= (blocks ? kLongBlocks : kLongStrips); }

// a launch whose schedules are cut into parts, and the combination
static hipError_t launch_parts(int mode, bool out_f32, const FlashParams& P0, hipStream_t st) {
  FlashParams P = P0;
  P.parts_per_head = parts_of(P.part_m, P.n_seg, P.seg);
  for (int k = 1; k < P.n_seg; ++k) P.seg[k].part0 = parts_of(P.part_m, k, P.seg);
  const int n = P.n_bh * P.parts_per_head;
  P.part_ml = P.part_o + (size_t)n * BQ * kHeadDim;
  hipError_t e = mode == 0 ? launch_one<0, false, false, true, 2>(P, n, st)
               : P.cols_in_place ? launch_one<2, false, true, true, 2>(P, n, st) : launch_one<2, false, false, true, 2>(P, n, st);
  if (e != hipSuccess) return e;
  const dim3 grid(P.n_qtiles * (BQ / 8), P.n_bh);
  if (P.n_seg > 1) {
    if (out_f32) hipLaunchKernelGGL((parts_combine_kernel<true, true>), grid, dim3(256), 0, st, P);
    else hipLaunchKernelGGL((parts_combine_kernel<false, true>), grid, dim3(256), 0, st, P);
  } else {
    if (out_f32) hipLaunchKernelGGL((parts_combine_kernel<true, false>), grid, dim3(256), 0, st, P);
    else hipLaunchKernelGGL((parts_combine_kernel<false, false>), grid, dim3(256), 0, st, P);
  }
  return hipGetLastError();
}

hipError_t launch_flash(int mode, bool out_f32, const FlashParams& P, hipStream_t st) {
  int grid;
  if (mode != 1 && P.part_m > 0) return launch_parts(mode, out_f32, P, st);
  if (mode == 2) {
    grid = (P.n_bh >= 8) ? 8 * P.n_qtiles * ((P.n_bh + 7) / 8) : P.n_qtiles * P.n_bh;
  } else {
    int bundles = 0;
    for (int k = 0; k < P.n_seg; ++k) bundles += P.n_qtiles * (mode == 1 ? P.seg[k].k_splits : 1) * P.n_bkv;
    grid = ((bundles + 7) / 8) * 8 * P.group;
  }
  if (grid <= 0) return hipSuccess;
  FlashParams L = P;
  if (mode == 2) L.short_lists = !two_cores(P.cols_in_place != 0, P.S, P.all_tiles);
  const int core = sweep_core(mode, P);
  switch (mode) {
    case 0: return launch_whole<0, false>(out_f32, core, P, grid, st);
    case 1: return launch_one<1, false, false, false, 2>(P, grid, st);
    default: return P.cols_in_place ? launch_whole<2, true>(out_f32, core, L, grid, st) : launch_whole<2, false>(out_f32, core, L, grid, st);
  }
}

}  // namespace sa
