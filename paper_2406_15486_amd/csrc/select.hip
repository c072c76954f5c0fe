// Stage 2 (Algorithm 1 stage 2; Sec. 4.3): per head and direction, the fewest
// strips whose score mass reaches alpha * total, ties to the lower index.
//
// Sorting is not needed to find the cut.  With candidates ordered by (score
// descending, index ascending) the kept set is {score > v} plus the first m
// candidates with score == v, for the cut value v.  v is found by a most-
// significant-digit radix descent over the fp32 bit patterns (non-negative
// floats order like their bits): the exponent first, then the mantissa in
// digits of 8, 8 and 7 bits.  Each pass builds a histogram, over the candidates
// that match the digits fixed so far, of (count, sum of the 23-bit mantissas);
// all candidates of a bin share their exponent, so the bin's score mass is
// (count * 2^23 + mantissa sum) * 2^(e - 150) EXACTLY, from integer sums whose
// order cannot matter.  One wave then walks the bins from the top: a lane holds
// four bins, the running sums come from an fp64 scan over the lanes in a fixed
// order, and the first bin whose running sum reaches the target is the digit.
// Nothing in the kernel adds floating-point numbers atomically: repeated runs
// give identical lists.  (One thread walking the 256 bins pays an LDS round trip
// per bin and was 17 us in each of the four passes.)
//
// Measured, both directions of a layer in one launch: 1 head of 1024 candidates
// 76 -> 13 us, 32 heads of 8192 88 -> 19 us, of 32768 112 -> 45 us, of 131072
// 211 -> 145 us.  The small ones are four passes of three barriers; the large ones
// are bound by the LDS atomics (about one per clock and CU, 64 CUs at work).
//
// The histogram lives in LDS and is updated with one 64-bit integer atomic per
// candidate (count in the upper bits, mantissa sum below).  Scores of one head
// crowd into a few exponents, and atomics of one wave to one address are served
// one after the other; so every bin has kCopies copies, indexed by lane % kCopies
// (then a wave's atomics land on distinct addresses and banks), which are added
// up before the walk.
//
// A last double sweep writes the kept indices in ascending order: every wave owns
// a contiguous segment of the candidates, counts what it will keep, and after one
// exchange of the counts writes its part of the list.  One workgroup per problem.
#include "sa_device.h"
#include "sa_kernels.h"

namespace sa {

namespace {

constexpr int NT = 1024;
constexpr int NW = NT / 64;
constexpr int kCopies = 32;                 // copies of every histogram bin
constexpr int kCntShift = 43;               // packed bin: count << 43 | mantissa sum (2^24 candidates at most:
                                            // a copy sees 2^19 of them, mantissa sum < 2^42, count < 2^20)
constexpr unsigned int kNoKey = 0xFFFFFFFFu;
constexpr int kBatch = 16;                  // scores a lane requests before it uses the first
constexpr size_t kSelectLds = 256 * kCopies * sizeof(unsigned long long);

// the bit pattern a score is ranked by: negative, infinite and NaN scores carry no
// mass and rank with the zeros
__device__ __forceinline__ unsigned int score_key(float v) {
  const unsigned int u = __float_as_uint(v);
  return (v > 0.0f && u < 0x7F800000u) ? u : 0u;
}

__global__ __launch_bounds__(NT) void select_kernel(SelectParams P) {
  extern __shared__ __attribute__((aligned(16))) unsigned long long hist[];   // [256 bins][kCopies]
  __shared__ unsigned int hcnt[256];
  __shared__ double bsum[256];                // mass per bin
  __shared__ double sh_above, sh_target;
  __shared__ unsigned int sh_prefix, sh_m, sh_done;
  __shared__ unsigned int w_gt[NW], w_tie[NW];

  // workgroups [0, n_prob) take the first set of problems, [n_prob, 2 n_prob) the
  // second one (the two directions of a layer in one launch)
  const bool second = (int)blockIdx.x >= P.n_prob;
  const int prob = second ? (int)blockIdx.x - P.n_prob : (int)blockIdx.x;
  const int S = P.S;
  const float* sc = (second ? P.scores2 : P.scores) + (size_t)prob * S;
  int32_t* idx = (second ? P.idx2 : P.idx) + (size_t)prob * S;
  int32_t* cnt_out = (second ? P.cnt2 : P.cnt) + prob;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double alpha = (double)(second ? P.alpha2 : P.alpha);

  if (alpha >= 1.0) {                       // keep everything
    for (int i = tid; i < S; i += NT) idx[i] = i;
    if (tid == 0) *cnt_out = S;
    return;
  }

  // every wave owns a contiguous run of whole 64-candidate groups
  const int n_groups = (S + 63) / 64;
  const int g_lo = (int)((long long)n_groups * wave / NW), g_hi = (int)((long long)n_groups * (wave + 1) / NW);

  // kBatch loads in flight per lane: a wave that waits for every score before it asks for
  // the next spends the pass waiting.  Up to 16384 candidates a wave's run is one batch: it
  // is read once and stays in registers for all six sweeps.
  unsigned int key[kBatch];                  // kNoKey past the end: matches no digit, exceeds no cut (as a signed number)
  auto load_batch = [&](int g0) {
    float v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = (g0 + u) * 64 + lane;
      v[u] = (g0 + u < g_hi && i < S) ? sc[i] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = (g0 + u) * 64 + lane;
      key[u] = (g0 + u < g_hi && i < S) ? score_key(v[u]) : kNoKey;
    }
  };
  const bool resident = n_groups <= NW * kBatch;
  if (resident) load_batch(g_lo);

  if (tid == 0) { sh_above = 0.0; sh_prefix = 0u; sh_done = 0u; sh_m = 0u; }
  for (int x = tid; x < 256 * kCopies; x += NT) hist[x] = 0ull;
  __syncthreads();
  // digit p: bits [shift, shift + width) of the 31-bit key
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = (pass == 3) ? 0 : 23 - 8 * pass;
    const int above_shift = (pass == 0) ? 31 : 31 - 8 * pass;    // bits from here up are fixed
    const unsigned int dmask = (pass == 3) ? 127u : 255u;
    const unsigned int prefix = sh_prefix;
    const unsigned int fixed = prefix >> above_shift;
    unsigned long long* my_hist = hist + (lane & (kCopies - 1));
    for (int g0 = g_lo; g0 < g_hi; g0 += kBatch) {
      if (!resident) load_batch(g0);
      auto credit = [&](unsigned int x) {
        if ((x >> above_shift) == fixed) {
          const unsigned int b = (x >> shift) & dmask;
          atomicAdd(my_hist + b * kCopies, (1ull << kCntShift) | (unsigned long long)(x & 0x7FFFFFu));
        }
      };
      if (g0 + kBatch <= g_hi) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) credit(key[u]);
      } else {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          if (g0 + u >= g_hi) break;                           // (wave-uniform: short problems skip the empty steps)
          credit(key[u]);
        }
      }
    }
    __syncthreads();
    {
      // four threads per bin, eight copies each (started at different copies, to spread the
      // LDS banks), left cleared for the next pass
      const int bin = tid >> 2;
      unsigned long long* part = hist + bin * kCopies + (tid & 3) * (kCopies / 4);
      unsigned long long c = 0ull, ms = 0ull;
#pragma unroll
      for (int x = 0; x < kCopies / 4; ++x) {
        const int at = (x + bin) & (kCopies / 4 - 1);
        const unsigned long long v = part[at];
        part[at] = 0ull;
        c += v >> kCntShift;
        ms += v & ((1ull << kCntShift) - 1ull);
      }
      unsigned int c32 = (unsigned int)c;
      c32 += __shfl_xor(c32, 1, 64); c32 += __shfl_xor(c32, 2, 64);
      ms += __shfl_xor(ms, 1, 64); ms += __shfl_xor(ms, 2, 64);
      if ((tid & 3) == 0) {
        // exponent of the bin's candidates: the bin itself in the first pass
        const unsigned int e = (pass == 0) ? (unsigned int)bin : (prefix >> 23);
        const unsigned long long units = (e > 0u ? ((unsigned long long)c32 << 23) : 0ull) + ms;
        hcnt[bin] = c32;
        bsum[bin] = ldexp((double)units, e > 0u ? (int)e - 150 : -149);   // exact: units < 2^53
      }
    }
    __syncthreads();
    if (wave == 0) {
      // The walk from the top bin down, by one wave: lane l holds the bins 255 - 4 l .. 252 - 4 l.
      // The running sums are formed in one fixed order (four bins in a row, a scan over the
      // lanes), so repeated runs agree bit for bit.
      double b4[4];
      unsigned int c4[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        b4[x] = bsum[255 - 4 * lane - x];
        c4[x] = hcnt[255 - 4 * lane - x];
      }
      double incl = ((b4[0] + b4[1]) + b4[2]) + b4[3];
      for (int step = 1; step < 64; step <<= 1) {
        const double o = __shfl_up(incl, step, 64);
        if (lane >= step) incl += o;
      }
      double target = sh_target;
      if (pass == 0) {
        target = alpha * __shfl(incl, 63, 64);
        if (lane == 0) {
          sh_target = target;
          if (!(target > 0.0)) sh_done = 1u;       // alpha == 0 or no mass: keep nothing
        }
      }
      double run = __shfl_up(incl, 1, 64);
      run = sh_above + (lane == 0 ? 0.0 : run);    // mass above this lane's bins
      int cut = -1, low = -1;                      // first bin that reaches the target; lowest non-empty bin
      double cut_above = 0.0, low_above = 0.0;
      unsigned int cut_n = 0u, low_n = 0u;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        if (c4[x] != 0u) {
          const int b = 255 - 4 * lane - x;
          if (cut < 0 && run + b4[x] >= target) { cut = b; cut_above = run; cut_n = c4[x]; }
          low = b; low_above = run; low_n = c4[x];
          run += b4[x];
        }
      }
      const unsigned long long has_cut = __ballot(cut >= 0), has_low = __ballot(low >= 0);
      // without a cut (only by fp64 rounding of the running sum): inside the lowest non-empty bin
      const bool mine = has_cut != 0ull ? lane == __ffsll((unsigned long long)has_cut) - 1
                                        : (has_low != 0ull && lane == 63 - __clzll((long long)has_low));
      if (mine && target > 0.0) {
        const int chosen = has_cut != 0ull ? cut : low;
        const double above = has_cut != 0ull ? cut_above : low_above;
        const unsigned int new_prefix = prefix | ((unsigned int)chosen << shift);
        sh_above = above;
        sh_prefix = new_prefix;
        if (pass == 3) {
          // all candidates left share the exact value v: how many are needed
          const double v = (double)__uint_as_float(new_prefix);
          const unsigned int c = has_cut != 0ull ? cut_n : low_n;
          unsigned int m = 1u;
          if (v > 0.0) {
            const double need = (target - above) / v;
            m = (need <= 1.0) ? 1u : (need >= (double)c ? c : (unsigned int)need);
            while (m > 1u && above + (double)(m - 1u) * v >= target) --m;
            while (m < c && above + (double)m * v < target) ++m;
          }
          sh_m = m;
        }
      }
    }
    __syncthreads();
    if (sh_done) {
      if (tid == 0) *cnt_out = 0;
      return;
    }
  }

  // ---- ordered compaction: count per wave segment, exchange, write -------------
  const unsigned int vkey = sh_prefix;
  const unsigned int m = sh_m;
  const unsigned long long lt = (1ull << lane) - 1ull;
  unsigned int n_gt = 0u, n_tie = 0u;
  for (int g0 = g_lo; g0 < g_hi; g0 += kBatch) {
    if (!resident) load_batch(g0);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (g0 + u >= g_hi) break;
      n_gt += (unsigned int)__popcll(__ballot((int)key[u] > (int)vkey));
      n_tie += (unsigned int)__popcll(__ballot(key[u] == vkey));
    }
  }
  if (lane == 0) { w_gt[wave] = n_gt; w_tie[wave] = n_tie; }
  __syncthreads();
  unsigned int tie_run = 0u, pos_run = 0u;   // ties before this wave's segment; list position of its first kept index
  for (int w = 0; w < wave; ++w) {
    const unsigned int t = w_tie[w];
    const unsigned int kept_ties = (tie_run >= m) ? 0u : ((m - tie_run < t) ? m - tie_run : t);
    pos_run += w_gt[w] + kept_ties;
    tie_run += t;
  }
  for (int g0 = g_lo; g0 < g_hi; g0 += kBatch) {
    if (!resident) load_batch(g0);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (g0 + u >= g_hi) break;
      const int i = (g0 + u) * 64 + lane;
      const bool gt = (int)key[u] > (int)vkey;
      const bool tie = key[u] == vkey;
      const unsigned long long bt = __ballot(tie);
      const unsigned int trank = tie_run + (unsigned int)__popcll(bt & lt);
      const bool sel = gt || (tie && trank < m);
      const unsigned long long bs = __ballot(sel);
      if (sel) idx[pos_run + (unsigned int)__popcll(bs & lt)] = i;
      tie_run += (unsigned int)__popcll(bt);
      pos_run += (unsigned int)__popcll(bs);
    }
  }
  if (wave == NW - 1 && lane == 0) *cnt_out = (int)pos_run;
}

}  // namespace

hipError_t launch_select(const SelectParams& P, hipStream_t st) {
  if (P.n_prob <= 0) return hipSuccess;
  const int sets = (P.scores2 != nullptr) ? 2 : 1;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&select_kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSelectLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(select_kernel, dim3(sets * P.n_prob), dim3(NT), kSelectLds, st, P);
  return hipGetLastError();
}

}  // namespace sa
