// Budget-to-threshold mapping (App. C.1) on the device: from the contribution
// scores c [n_rows, k] of one score pass (one or more layers), the threshold
// tau_q for each requested skip ratio q.
//
//  * N_all = n_rows * k routed slots.  Candidates exclude slot 0 (the top-1
//    expert) and, with m_min > 1, the m_min - 1 highest-c other slots of each
//    row (ties to the lower slot): Alg. 4's restore step never skips them.
//  * m_q = clip(round-half-even(q N_all), 0, N_cand); tau_q lies between the
//    m_q-th and (m_q+1)-th smallest candidate scores: their midpoint when they
//    differ; at a tie on value v, tau = v (realising #{c < v}) or the midpoint
//    of v and the next larger score (realising #{c <= v}), whichever count is
//    closer to m_q, the lower one on a draw; m_q = 0 gives 0, m_q = N_cand +inf.
//  * The order statistics come from a radix select on 32-bit order-preserving
//    keys, all budgets at once: a top digit (top_bin), then the keys' bits 10-19
//    and 0-9.  Two order statistics per budget are jobs; jobs with the same prefix share a histogram
//    (the slot of the lowest of them), and a key finds its slot through a table
//    of the digits chosen so far, so the work per key does not grow with the
//    budgets.  The ranks left over give #{c < v} and #{c <= v} of a boundary tie,
//    and the last pass keeps the smallest key above each prefix, so a tie needs
//    no further pass.  All counting is integer, so the result is exact and
//    deterministic; the midpoint is formed in fp64 from the two fp32 scores and
//    rounded once.
// What bounds it: launches and dependent steps, hardly the bytes (12.6 MB for 48
// layers x 8192 tokens).  Up to kSmallRows rows one workgroup does all of it with
// its keys in registers; more rows take five launches over at most 256 workgroups
// (clear, then a pass per digit, each starting with the pick of the digit before
// it in every workgroup, then the finish).  Four 8-bit digits, a tie count and a
// second select in 23 launches took 131 us for 4096 rows and one budget, now
// 18 us, and 318 us for 393216 rows and four budgets, now 45 us (128 or 512
// workgroups: 46 and 64).
// Every step runs on the caller's stream with no host synchronisation; ranks
// that depend on earlier results are read from device memory.
#include "ace_internal.h"

namespace ace {

namespace {

constexpr int kJobs = 2 * kTauMaxQ;  // two order statistics per budget
constexpr int kLowBits = 10, kBins = 1 << kLowBits;  // of the second and third digit
constexpr int kTopBins = 8192;                       // of the top digit (top_bin)
constexpr int kThreads = 1024;  // of every workgroup: 16 waves, one per job in the picks
static_assert(kThreads / 64 == kJobs, "a wave per job");

// one selection: the job's rank among all candidates (0-based), the candidates
// below its prefix, the digits fixed so far, and its histogram slot (the lowest
// job with the same prefix; -1: not active)
struct Select {
  unsigned long long n_cand;
  unsigned long long target[kJobs], below[kJobs], count[kJobs];  // count: candidates with the prefix
  uint32_t prefix[kJobs], next[kJobs];  // top bin, then key >> 10, then the key; next: smallest larger key known
  int slot[kJobs];
  long long m_q[kTauMaxQ];
};

struct TauArgs {
  const float *scores;
  long long n_rows;
  int k, m_min, n_q;
  bool vec;                  // rows of 4 or 8 scores, 16-byte aligned
  double q[kTauMaxQ];
  Select *sel;               // [2]: after the first and after the second pick
  unsigned long long *top;   // [kTopBins]
  unsigned long long *mid;   // [kJobs][kBins]
  unsigned long long *low;   // [kJobs][kBins]
  uint32_t *next;            // [kTauMaxQ]
  float *tau;
  long long *m_q_out;        // optional
  long long *n_cand_out;     // optional
};

// order-preserving key of a non-NaN float (-0 taken as +0)
__device__ __forceinline__ uint32_t key_of(float c) {
  const uint32_t u = __float_as_uint(c + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float value_of(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

// Top digit: the key's upper 12 bits, but 512 bins per octave for values in
// [2^-8, 1), where the scores of a token (k shares of one) lie.  With 8 bins per
// octave there (the upper 12 bits alone) the lanes of a wave met in few LDS bins
// and each selection carried 5% of all keys into the next digit (the digit passes
// of 393216 rows and four budgets took 56 us instead of 37).
constexpr uint32_t kFineLo = 0xBB800000u, kFineHi = 0xBF800000u;  // keys of 2^-8 and 1
constexpr uint32_t kFineBin0 = kFineLo >> 20, kAboveBin0 = kFineBin0 + ((kFineHi - kFineLo) >> 14);
static_assert(kAboveBin0 + ((0xFFFFFFFFu - kFineHi) >> 20) < kTopBins, "bins of the top digit");
__device__ __forceinline__ uint32_t top_bin(uint32_t key) {
  return key < kFineLo   ? key >> 20
         : key < kFineHi ? kFineBin0 + ((key - kFineLo) >> 14)
                         : kAboveBin0 + ((key - kFineHi) >> 20);
}
// smallest key of a top bin
__device__ __forceinline__ uint32_t bin_key(uint32_t bin) {
  return bin < kFineBin0    ? bin << 20
         : bin < kAboveBin0 ? kFineLo + ((bin - kFineBin0) << 14)
                            : kFineHi + ((bin - kAboveBin0) << 20);
}

// candidate slots of one row: bit i set if slot i may be skipped
__device__ __forceinline__ unsigned row_candidates(const float (&c)[kMaxK], int k, int m_min) {
  if (m_min == 1) return (1u << k) - 2u;
  unsigned cand = 0;
#pragma unroll
  for (int i = 1; i < kMaxK; ++i) {
    int rank = 0;  // higher-c other slots (ties: lower slot first)
#pragma unroll
    for (int j = 1; j < kMaxK; ++j)
      if (j < k && j != i && (c[j] > c[i] || (c[j] == c[i] && j < i))) ++rank;
    if (i < k && rank >= m_min - 1) cand |= 1u << i;
  }
  return cand;
}

__device__ __forceinline__ void load_row(const TauArgs &a, long long r, float (&c)[kMaxK]) {
  if (a.vec) {
    const float4 *p = reinterpret_cast<const float4 *>(a.scores + r * a.k);
    const float4 lo = p[0];
    const float4 hi = a.k == 8 ? p[1] : make_float4(0.f, 0.f, 0.f, 0.f);
    c[0] = lo.x; c[1] = lo.y; c[2] = lo.z; c[3] = lo.w;
    c[4] = hi.x; c[5] = hi.y; c[6] = hi.z; c[7] = hi.w;
  } else {
#pragma unroll
    for (int i = 0; i < kMaxK; ++i) c[i] = i < a.k ? a.scores[r * a.k + i] : 0.f;
  }
}

// f(key) for every candidate of this workgroup's rows
template <typename F> __device__ __forceinline__ void each_candidate(const TauArgs &a, F f) {
  const long long step = static_cast<long long>(kThreads) * gridDim.x;
  for (long long r = static_cast<long long>(blockIdx.x) * kThreads + threadIdx.x; r < a.n_rows; r += step) {
    float c[kMaxK];
    load_row(a, r, c);
    const unsigned cand = row_candidates(c, a.k, a.m_min);
#pragma unroll
    for (int i = 1; i < kMaxK; ++i)
      if ((cand >> i) & 1u) f(key_of(c[i]));
  }
}

__device__ __forceinline__ unsigned long long wave_scan(unsigned long long v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long n = __shfl_up(v, o);
    if (lane >= o) v += n;
  }
  return v;
}

// minimum over the wave, in every lane
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  v = min(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x128, 0xF, 0xF, true)));  // row_ror 8
  v = min(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x124, 0xF, 0xF, true)));
  v = min(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x122, 0xF, 0xF, true)));
  v = min(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x121, 0xF, 0xF, true)));
  v = min(v, static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), 16)));
  return min(v, static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), 32)));
}

// jobs with the same prefix share the slot of the lowest of them
__device__ __forceinline__ void share_slots(Select &s) {
  __syncthreads();
  const int j = threadIdx.x;
  if (j < 64) {
    int slot[kJobs];
    uint32_t prefix[kJobs];
#pragma unroll
    for (int i = 0; i < kJobs; ++i) {
      slot[i] = s.slot[i];
      prefix[i] = s.prefix[i];
    }
    if (j < kJobs && s.slot[j] >= 0) {
      const uint32_t p = s.prefix[j];
      int first = j;
#pragma unroll
      for (int i = kJobs - 1; i >= 0; --i)
        if (i < j && slot[i] >= 0 && prefix[i] == p) first = i;
      s.slot[j] = first;  // one wave: every lane has read before one writes
    }
  }
  __syncthreads();
}

// N_cand, the jobs of every budget, and their top digit from its histogram
template <typename C> __device__ __forceinline__ void pick_top(const TauArgs &a, const C *hist, Select &s) {
  __shared__ unsigned long long part[kThreads / 64];
  constexpr int kPer = kTopBins / kThreads;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  unsigned long long c[kPer], sum = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    c[i] = hist[kPer * tid + i];
    sum += c[i];
  }
  const unsigned long long incl = wave_scan(sum);
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  unsigned long long before = incl - sum, n_cand = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    if (w < wave) before += part[w];
    n_cand += part[w];
  }
  if (tid < kJobs) {
    const int i = tid >> 1;
    long long m = 0;
    const long long nc = static_cast<long long>(n_cand);
    if (i < a.n_q) {
      m = static_cast<long long>(rint(a.q[i] * (static_cast<double>(a.n_rows) * a.k)));
      m = m < 0 ? 0 : (m > nc ? nc : m);
    }
    const bool inner = m > 0 && m < nc;
    s.target[tid] = inner ? static_cast<unsigned long long>(m - 1 + (tid & 1)) : ~0ull;  // ~0: in no bin
    s.slot[tid] = inner ? tid : -1;
    s.below[tid] = s.count[tid] = 0ull;
    s.prefix[tid] = 0u;
    s.next[tid] = 0xFFFFFFFFu;
    if ((tid & 1) == 0) s.m_q[i] = m;
    if (tid == 0) s.n_cand = n_cand;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kJobs; ++j) {
    const unsigned long long t = s.target[j];
    if (t < before || t >= before + sum) continue;
    unsigned long long b = before;  // exactly one bin holds the rank
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (t >= b && t < b + c[i]) {
        s.prefix[j] = static_cast<uint32_t>(kPer * tid + i);
        s.below[j] = b;
        s.count[j] = c[i];
      }
      b += c[i];
    }
  }
  share_slots(s);
}

// the next digit of every job (wave w: job w) from its slot's histogram; LAST:
// also the next larger key if this histogram has one
template <bool LAST, typename C> __device__ __forceinline__ void pick_next(const C *hist, Select &s) {
  constexpr int kPer = kBins / 64;
  const int lane = threadIdx.x & 63, j = threadIdx.x >> 6;
  if (s.slot[j] >= 0) {
    const C *h = hist + static_cast<size_t>(s.slot[j]) * kBins + kPer * lane;
    C c[kPer];
    unsigned long long sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      c[i] = h[i];
      sum += c[i];
    }
    unsigned long long before = s.below[j] + wave_scan(sum) - sum;
    const unsigned long long t = s.target[j];
    int bin = -1;
    unsigned long long b = 0, n = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (t >= before && t < before + c[i]) {  // exactly one bin of the wave's 1024
        bin = kPer * lane + i;
        b = before;
        n = c[i];
      }
      before += c[i];
    }
    const int owner = __ffsll(static_cast<long long>(__ballot(bin >= 0))) - 1;
    bin = __shfl(bin, owner);
    const uint32_t prefix = (LAST ? s.prefix[j] : bin_key(s.prefix[j]) >> 20) << kLowBits;
    uint32_t next = 0xFFFFFFFFu;
    if (LAST) {
#pragma unroll
      for (int i = kPer - 1; i >= 0; --i)
        if (c[i] && kPer * lane + i > bin) next = prefix | static_cast<uint32_t>(kPer * lane + i);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) next = min(next, static_cast<uint32_t>(__shfl_xor(static_cast<int>(next), o)));
    }
    if (lane == owner) {
      s.prefix[j] = prefix | static_cast<uint32_t>(bin);
      s.below[j] = b;
      s.count[j] = n;
      if (LAST) s.next[j] = min(s.next[j], next);
    }
  }
}

// word copy of a selection by the first wave
__device__ __forceinline__ void copy_select(Select *dst, const Select *src) {
  static_assert(sizeof(Select) % 8 == 0, "whole words");
  constexpr int n = sizeof(Select) / 8;
  if (threadIdx.x < 64)
    for (int i = threadIdx.x; i < n; i += 64)
      reinterpret_cast<unsigned long long *>(dst)[i] = reinterpret_cast<const unsigned long long *>(src)[i];
}

// key -> slot of its digits: table[digit] of the top digit, then of (slot, digit)
__device__ __forceinline__ void clear_slots(uint8_t *table, int n) {
  for (int i = threadIdx.x; i < n / 4; i += kThreads) reinterpret_cast<uint32_t *>(table)[i] = 0xFFFFFFFFu;
}

// thresholds from the whole keys; at a tie on v (the two keys are equal) the count
// on v's side that is closer to m_q, the lower one on a draw
__device__ __forceinline__ void finish(const TauArgs &a, const Select &s) {
  const int i = threadIdx.x;
  if (i < a.n_q) {
    const long long m = s.m_q[i], nc = static_cast<long long>(s.n_cand);
    const uint32_t lo = s.prefix[2 * i], hi = s.prefix[2 * i + 1];
    float t;
    if (m == 0) {
      t = 0.f;
    } else if (m == nc) {
      t = INFINITY;
    } else {
      uint32_t other = hi;
      bool inf = false;
      if (lo == hi) {
        const long long below = static_cast<long long>(s.below[2 * i]);
        const long long above = below + static_cast<long long>(s.count[2 * i]);
        const long long db = below > m ? below - m : m - below;
        const long long da = above > m ? above - m : m - above;
        if (db > da) {  // else tau = v, the midpoint of v and v
          inf = above == nc;  // every candidate skipped
          other = s.next[2 * i];
        }
      }
      t = inf ? INFINITY
              : lo == other ? value_of(lo)
                            : static_cast<float>(0.5 * (static_cast<double>(value_of(lo)) +
                                                        static_cast<double>(value_of(other))));
    }
    a.tau[i] = t;
    if (a.m_q_out) a.m_q_out[i] = m;
  }
  if (i == 0 && a.n_cand_out) a.n_cand_out[0] = static_cast<long long>(s.n_cand);
}

// add a workgroup's LDS counts of N bins into the global ones
template <int N> __device__ __forceinline__ void merge(unsigned long long *out, const uint32_t *h) {
  static_assert(N % kThreads == 0, "whole rounds");
  uint32_t v[N / kThreads];
#pragma unroll
  for (int i = 0; i < N / kThreads; ++i) v[i] = h[i * kThreads + threadIdx.x];
#pragma unroll
  for (int i = 0; i < N / kThreads; ++i)
    if (v[i]) atomicAdd(&out[i * kThreads + threadIdx.x], static_cast<unsigned long long>(v[i]));
}

__device__ __forceinline__ void clear_bins(uint32_t *h, int n) {
  for (int i = threadIdx.x; i < n / 4; i += kThreads) reinterpret_cast<uint4 *>(h)[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ __launch_bounds__(kThreads) void tau_clear_kernel(TauArgs a) {
  const int n = kTopBins + 2 * kJobs * kBins;  // top, mid and low are adjacent
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) a.top[i] = 0ull;
  if (blockIdx.x == 0 && threadIdx.x < kTauMaxQ) a.next[threadIdx.x] = 0xFFFFFFFFu;
}

__global__ __launch_bounds__(kThreads) void tau_top_kernel(TauArgs a) {
  __shared__ __align__(16) uint32_t h[kTopBins];
  clear_bins(h, kTopBins);
  __syncthreads();
  each_candidate(a, [&](uint32_t key) { atomicAdd(&h[top_bin(key)], 1u); });
  __syncthreads();
  merge<kTopBins>(a.top, h);
}

__global__ __launch_bounds__(kThreads) void tau_mid_kernel(TauArgs a) {
  __shared__ Select s;
  __shared__ __align__(16) uint32_t h[kJobs][kBins];
  __shared__ uint8_t slot1[kTopBins];
  clear_slots(slot1, kTopBins);
  clear_bins(&h[0][0], kJobs * kBins);
  pick_top(a, a.top, s);
  const int tid = threadIdx.x;
  if (tid < kJobs && s.slot[tid] == tid) slot1[s.prefix[tid]] = static_cast<uint8_t>(tid);
  if (blockIdx.x == 0) copy_select(&a.sel[0], &s);
  __syncthreads();
  each_candidate(a, [&](uint32_t key) {
    const int v = slot1[top_bin(key)];
    if (v < kJobs) atomicAdd(&h[v][(key >> kLowBits) & (kBins - 1)], 1u);
  });
  __syncthreads();
  merge<kJobs * kBins>(a.mid, &h[0][0]);
}

__global__ __launch_bounds__(kThreads) void tau_low_kernel(TauArgs a) {
  __shared__ Select s;
  __shared__ __align__(16) uint32_t h[kJobs][kBins];
  __shared__ uint8_t slot1[kTopBins], slot2[kJobs][kBins];
  __shared__ uint32_t next[kTauMaxQ];
  const int tid = threadIdx.x;
  clear_slots(slot1, kTopBins);
  clear_slots(&slot2[0][0], kJobs * kBins);
  clear_bins(&h[0][0], kJobs * kBins);
  if (tid < kTauMaxQ) next[tid] = 0xFFFFFFFFu;
  copy_select(&s, &a.sel[0]);
  __syncthreads();
  const int up = tid < kJobs ? s.slot[tid] : -1;  // this job's slot of the digit before
  if (up == tid) slot1[s.prefix[tid]] = static_cast<uint8_t>(tid);
  __syncthreads();  // the prefixes are read before the waves extend them
  pick_next<false>(a.mid, s);
  share_slots(s);
  if (up >= 0 && s.slot[tid] == tid) slot2[up][s.prefix[tid] & (kBins - 1)] = static_cast<uint8_t>(tid);
  if (blockIdx.x == 0) copy_select(&a.sel[1], &s);
  // where a budget's two keys may tie, the smallest key above their prefix
  uint32_t above[kTauMaxQ], mn[kTauMaxQ];
#pragma unroll
  for (int q = 0; q < kTauMaxQ; ++q) {
    above[q] = s.slot[2 * q] >= 0 && s.prefix[2 * q] == s.prefix[2 * q + 1] ? s.prefix[2 * q] : 0xFFFFFFFFu;
    mn[q] = 0xFFFFFFFFu;
  }
  __syncthreads();
  each_candidate(a, [&](uint32_t key) {
    const int u = slot1[top_bin(key)];
    if (u < kJobs) {
      const int v = slot2[u][(key >> kLowBits) & (kBins - 1)];
      if (v < kJobs) atomicAdd(&h[v][key & (kBins - 1)], 1u);
    }
#pragma unroll
    for (int q = 0; q < kTauMaxQ; ++q)
      if (q < a.n_q && (key >> kLowBits) > above[q]) mn[q] = min(mn[q], key);
  });
#pragma unroll
  for (int q = 0; q < kTauMaxQ; ++q) {
    const uint32_t v = wave_min(mn[q]);
    if ((tid & 63) == q && v != 0xFFFFFFFFu) atomicMin(&next[q], v);
  }
  __syncthreads();
  merge<kJobs * kBins>(a.low, &h[0][0]);
  if (tid < a.n_q && next[tid] != 0xFFFFFFFFu) atomicMin(&a.next[tid], next[tid]);
}

__global__ __launch_bounds__(kThreads) void tau_finish_kernel(TauArgs a) {
  __shared__ Select s;
  copy_select(&s, &a.sel[1]);
  __syncthreads();
  if (threadIdx.x < a.n_q) s.next[2 * threadIdx.x] = a.next[threadIdx.x];
  __syncthreads();
  pick_next<true>(a.low, s);
  __syncthreads();
  finish(a, s);
}

// Keys of all selections a small mapping ranks directly (each against its slot's)
constexpr int kListMax = 512;

// The whole mapping by one workgroup, RPT rows per thread, keys in registers
// through the top digit (what follows rarely needs them again and reads them again).
// After the top digit a selection holds a few dozen keys of a score pass: up to
// kListMax of them are gathered and ranked directly, else the digits go on.
template <int RPT> __global__ __launch_bounds__(kThreads) void tau_small_kernel(TauArgs a) {
  __shared__ Select s;
  __shared__ __align__(16) uint32_t h[kJobs * kBins];  // the top digit's histogram first
  static_assert(kTopBins <= kJobs * kBins, "histograms share their place");
  __shared__ uint8_t slot1[kTopBins], slot2[kJobs][kBins];
  __shared__ uint32_t next[kTauMaxQ];
  __shared__ uint32_t list[kListMax];                 // gathered keys, each slot's together
  __shared__ uint8_t list_slot[kListMax];
  __shared__ int from[kJobs], fill[kJobs];            // a slot's first and next place in the list
  __shared__ int rank[kJobs];                         // rank of each job's key in its slot
  __shared__ int2 tie[kJobs];                         // ... among its equals, and how many they are
  const int tid = threadIdx.x;
  uint32_t key[RPT][kMaxK];
  unsigned cand[RPT];
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const long long row = tid + static_cast<long long>(r) * kThreads;
    float c[kMaxK];
    load_row(a, row < a.n_rows ? row : 0, c);
    cand[r] = row < a.n_rows ? row_candidates(c, a.k, a.m_min) : 0u;
#pragma unroll
    for (int i = 1; i < kMaxK; ++i) key[r][i] = key_of(c[i]);
  }
  auto each = [&](auto f) {
#pragma unroll
    for (int r = 0; r < RPT; ++r)
#pragma unroll
      for (int i = 1; i < kMaxK; ++i)
        if ((cand[r] >> i) & 1u) f(key[r][i]);
  };
  clear_bins(h, kTopBins);
  clear_slots(slot1, kTopBins);
  if (tid < kTauMaxQ) next[tid] = 0xFFFFFFFFu;
  __syncthreads();
  each([&](uint32_t u) { atomicAdd(&h[top_bin(u)], 1u); });
  __syncthreads();
  pick_top(a, h, s);
  const int up = tid < kJobs ? s.slot[tid] : -1;
  unsigned long long total = 0, lower = 0;  // keys of all slots, of the slots below this thread's job's
#pragma unroll
  for (int j = 0; j < kJobs; ++j) {
    const unsigned long long c = s.slot[j] == j ? s.count[j] : 0ull;
    total += c;
    if (j < up) lower += c;
  }
  if (total <= kListMax) {  // uniform over the workgroup
    if (tid < kJobs) {
      rank[tid] = up >= 0 ? static_cast<int>(s.target[tid] - s.below[tid]) : -1;
      from[tid] = fill[tid] = up >= 0 ? static_cast<int>(lower) : 0;
    }
    if (up == tid) slot1[s.prefix[tid]] = static_cast<uint8_t>(tid);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      int v[kMaxK];
#pragma unroll
      for (int i = 1; i < kMaxK; ++i) {
        asm("" : "+v"(key[r][i]));  // its bin is computed again, not kept since the histogram
        v[i] = slot1[top_bin(key[r][i])];
      }
#pragma unroll
      for (int i = 1; i < kMaxK; ++i)
        if (((cand[r] >> i) & 1u) && v[i] < kJobs) {
          const int p = atomicAdd(&fill[v[i]], 1);
          list[p] = key[r][i];
          list_slot[p] = static_cast<uint8_t>(v[i]);
        }
    }
    __syncthreads();
    if (tid < static_cast<int>(total)) {
      const int slot = list_slot[tid];
      const int i0 = from[slot], i1 = fill[slot];
      const uint32_t x = list[tid];
      int less = 0, le = 0;
      uint32_t up_key = 0xFFFFFFFFu;  // smallest larger key of the slot
      for (int i = i0; i < i1; ++i) {
        const uint32_t v = list[i];
        less += v < x ? 1 : 0;
        le += v <= x ? 1 : 0;
        if (v > x) up_key = min(up_key, v);
      }
      for (int j = slot; j < 2 * a.n_q; ++j) {
        const int r = rank[j];
        if (s.slot[j] != slot || r < less || r >= le) continue;  // equal keys write the same values
        s.prefix[j] = x;
        s.next[j] = up_key;
        tie[j] = make_int2(r - less, le - less);
      }
    }
    __syncthreads();
    if (up >= 0) {
      s.below[tid] = s.target[tid] - static_cast<unsigned long long>(tie[tid].x);
      s.count[tid] = static_cast<unsigned long long>(tie[tid].y);
    }
    // a tie whose next larger key lies in another bin
    for (int q = 0; q < a.n_q; ++q) {
      if (s.slot[2 * q] < 0 || s.prefix[2 * q] != s.prefix[2 * q + 1] || s.next[2 * q] != 0xFFFFFFFFu) continue;
      const uint32_t v = s.prefix[2 * q];
      uint32_t mn = 0xFFFFFFFFu;
      each_candidate(a, [&](uint32_t u) {
        if (u > v) mn = min(mn, u);
      });
      mn = wave_min(mn);
      if ((tid & 63) == 0 && mn != 0xFFFFFFFFu) atomicMin(&next[q], mn);
    }
    __syncthreads();
    if (tid < a.n_q) s.next[2 * tid] = min(s.next[2 * tid], next[tid]);
    __syncthreads();
    finish(a, s);
    return;
  }
  clear_slots(&slot2[0][0], kJobs * kBins);
  clear_bins(h, kJobs * kBins);
  if (up == tid) slot1[s.prefix[tid]] = static_cast<uint8_t>(tid);
  __syncthreads();
  each_candidate(a, [&](uint32_t u) {
    const int v = slot1[top_bin(u)];
    if (v < kJobs) atomicAdd(&h[v * kBins + ((u >> kLowBits) & (kBins - 1))], 1u);
  });
  __syncthreads();
  pick_next<false>(h, s);
  share_slots(s);
  if (up >= 0 && s.slot[tid] == tid) slot2[up][s.prefix[tid] & (kBins - 1)] = static_cast<uint8_t>(tid);
  clear_bins(h, kJobs * kBins);
  __syncthreads();
  each_candidate(a, [&](uint32_t u) {
    const int w = slot1[top_bin(u)];
    if (w < kJobs) {
      const int v = slot2[w][(u >> kLowBits) & (kBins - 1)];
      if (v < kJobs) atomicAdd(&h[v * kBins + (u & (kBins - 1))], 1u);
    }
  });
  for (int q = 0; q < a.n_q; ++q) {
    if (s.slot[2 * q] < 0 || s.prefix[2 * q] != s.prefix[2 * q + 1]) continue;  // uniform
    const uint32_t above = s.prefix[2 * q];
    uint32_t mn = 0xFFFFFFFFu;
    each_candidate(a, [&](uint32_t u) {
      if ((u >> kLowBits) > above) mn = min(mn, u);
    });
    mn = wave_min(mn);
    if ((tid & 63) == 0 && mn != 0xFFFFFFFFu) atomicMin(&next[q], mn);
  }
  __syncthreads();
  if (tid < a.n_q) s.next[2 * tid] = next[tid];
  __syncthreads();
  pick_next<true>(h, s);
  __syncthreads();
  finish(a, s);
}

// Rows up to which one workgroup maps them: 4096 rows take 18-23 us (one to eight
// budgets) against 27-35 us by five launches; with 8 rows a thread its registers
// spill and 8192 rows take 55-88 us against 27-35.
constexpr long long kSmallRows = 4 * kThreads;

constexpr size_t align256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

size_t tau_workspace_bytes() {
  return align256(2 * sizeof(Select) + kTauMaxQ * sizeof(uint32_t)) +
         (kTopBins + 2 * kJobs * kBins) * sizeof(unsigned long long);
}

hipError_t launch_tau_map(const float *scores, long long n_rows, int k, int m_min, const double *q, int n_q,
                          float *tau, long long *m_q_out, long long *n_cand_out, void *workspace,
                          hipStream_t stream) {
  TauArgs a{};
  a.scores = scores;
  a.n_rows = n_rows;
  a.k = k;
  a.m_min = m_min;
  a.n_q = n_q;
  a.vec = k % 4 == 0 && (reinterpret_cast<uintptr_t>(scores) & 15u) == 0;
  for (int i = 0; i < kTauMaxQ; ++i) a.q[i] = i < n_q ? q[i] : 0.0;
  char *ws = static_cast<char *>(workspace);
  a.sel = reinterpret_cast<Select *>(ws);
  a.next = reinterpret_cast<uint32_t *>(ws + 2 * sizeof(Select));
  a.top = reinterpret_cast<unsigned long long *>(ws + align256(2 * sizeof(Select) + kTauMaxQ * sizeof(uint32_t)));
  a.mid = a.top + kTopBins;
  a.low = a.mid + kJobs * kBins;
  a.tau = tau;
  a.m_q_out = m_q_out;
  a.n_cand_out = n_cand_out;
  if (n_rows > 0 && n_rows <= kSmallRows) {
    if (n_rows <= kThreads)
      tau_small_kernel<1><<<1, kThreads, 0, stream>>>(a);
    else if (n_rows <= 2 * kThreads)
      tau_small_kernel<2><<<1, kThreads, 0, stream>>>(a);
    else
      tau_small_kernel<4><<<1, kThreads, 0, stream>>>(a);
    return hipGetLastError();
  }
  const long long blocks = (n_rows + kThreads - 1) / kThreads;
  const unsigned grid = static_cast<unsigned>(blocks < 1 ? 1 : blocks > 256 ? 256 : blocks);
  tau_clear_kernel<<<32, kThreads, 0, stream>>>(a);
  tau_top_kernel<<<grid, kThreads, 0, stream>>>(a);
  tau_mid_kernel<<<grid, kThreads, 0, stream>>>(a);
  tau_low_kernel<<<grid, kThreads, 0, stream>>>(a);
  tau_finish_kernel<<<1, kThreads, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace ace
