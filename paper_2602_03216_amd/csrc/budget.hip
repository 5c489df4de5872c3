// Dynamic Token Coverage budget: the budget steps of Algorithm 1 of the paper (Section 2.3): cross-head
// sum of the token scores, normalisation, ascending order, cumulative-mass threshold.
// s_l[t] = sum_h s_h[t] (normalised by its total); k_sparse = the smallest k whose k
// least important tokens carry a cumulative mass >= tau; k_keep = L - k_sparse.
//
// No sort is needed: the answer only depends on the value at which the ascending cumulative mass
// crosses tau * total.  A radix descent over the order-preserving uint32 image of s_l finds it
// in 4 passes of 8 bits, least important bin first: every pass builds, for the keys that match
// the prefix found so far, a 256-bin histogram of (count, mass); the next kernel walks the bins
// upwards until count/mass below plus the bin's mass reaches the target.  After the last pass
// the bin is a single fp32 value v, and the number of tied tokens to take is
// ceil((target - mass_below) / v).
// Masses are EXACT and do not depend on the order of the additions: the keys of one bin differ by at
// most one step of the binary exponent (first pass) or share it (later passes), so a bin's mass is kept
// as the integer sum of the 24-bit significands (shifted by the lowest exponent bit), accumulated with
// integer atomics, and becomes a double only when the bins are walked, in a fixed order.  Two runs on
// the same scores give the same count bit for bit.
// Rows of up to kRowTokens take all of that in one launch (bud_row_kernel, below); longer ones the chain of small kernels.
#include "tsa_internal.h"

#include <climits>

namespace tsa {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kSlice = 2048;      // tokens per workgroup: few rows (one per batch entry), so short slices fill the chip

struct BudState {
  uint32_t prefix;       // digits found so far
  uint32_t count_below;  // tokens strictly below the prefix range
  double mass_below;     // their mass
};

struct BudRow {
  double total;                        // written by the first slice of pass 1, read by the later launches
  unsigned long long isum[4][256];     // per bin: sum of significands, in units of 2^(E - 150), E = bin_exponent()
  uint32_t count[4][256];
  BudState state[5];     // state[p]: before pass p; state[4]: final
};

struct BudArgs {
  const float* scores;   // [B,Hq,L]
  float* sl;             // [B,L]
  BudRow* rows;          // [B]; NULL: the row kernel follows, no histograms to clear
  int32_t* k_keep;       // [B]
  int Hq, L;
  double tau;
  int k_max;             // upper bound of the result (capacity of the caller's buffers)
  int k_min;             // lower bound of the result (at least 1)
};

__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u << 1) == 0u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// A float as significand x 2^(exponent - 150): finite v, sig < 2^24 (subnormals: exponent field 1).
__device__ __forceinline__ void split_float(float v, uint32_t& sig, int& e) {
  const uint32_t u = __float_as_uint(v);
  e = (int)((u >> 23) & 255u);
  sig = u & 0x7fffffu;
  if (e) sig |= 0x800000u; else e = 1;
}
// Exponent unit of a bin's integer sum: the exponent field of the bin's smallest magnitude.  The first
// pass fixes sign and the upper seven exponent bits (the low bit is free: significands of the larger
// exponent are shifted left by one); later passes fix the whole exponent.  `key_prefix`: any key of the bin.
__device__ __forceinline__ int bin_exponent(uint32_t key_prefix, int pass) {
  const uint32_t u = (key_prefix & 0x80000000u) ? (key_prefix & 0x7fffffffu) : ~key_prefix;   // back to float bits
  int e = (int)((u >> 23) & 255u);
  if (pass == 0) e &= ~1;
  return e < 1 ? 1 : e;
}
__device__ __forceinline__ double bin_mass(unsigned long long isum, uint32_t key_prefix, int pass) {
  const double m = ldexp((double)isum, bin_exponent(key_prefix, pass) - 150);     // isum < 2^53: exact
  return (key_prefix & 0x80000000u) ? m : -m;                                     // keys below 2^31 are negative scores
}

// s_l = sum over heads, fp32, in head order; also clears the histograms of the four passes
// Bound by memory latency (a few MB of scores): small workgroups, so that every CU has one from 16K tokens up, and the
// loads of eight heads requested together; the additions stay in head order.  12345 tokens x
// 32 heads: 11.2 -> 4.8 us (1024 threads, one load at a time before).
constexpr int kSumThreads = 64, kSumHeads = 8;
__global__ __launch_bounds__(kSumThreads) void head_sum_kernel(BudArgs a) {
  const long long b = blockIdx.y;
  const int t = blockIdx.x * kSumThreads + threadIdx.x;
  if (t < a.L) {
    const float* p = a.scores + b * a.Hq * a.L + t;
    float acc = 0.f;
    int h = 0;
    for (; h + kSumHeads <= a.Hq; h += kSumHeads) {
      float v[kSumHeads];
#pragma unroll
      for (int j = 0; j < kSumHeads; ++j) v[j] = p[(long long)(h + j) * a.L];
#pragma unroll
      for (int j = 0; j < kSumHeads; ++j) acc += v[j];
    }
    for (; h < a.Hq; ++h) acc += p[(long long)h * a.L];
    a.sl[b * a.L + t] = acc;
  }
  if (!a.rows) return;
  constexpr int n_words = (int)(sizeof(BudRow) / 4);
  uint32_t* row = (uint32_t*)(a.rows + b);
  for (int i = t; i < n_words; i += gridDim.x * kSumThreads) row[i] = 0u;
}

// Walks the 256 bins of one pass upwards (first wavefront): lane l owns bins 4l..4l+3.
// `total` (may be NULL): receives the mass of all bins of the pass (every lane gets the same value).
__device__ __forceinline__ BudState next_state(const BudRow* rw, int pass, BudState st, double tau, double* total, int shift,
                                               int lane) {
  double ms[4];
  uint32_t cn[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t key_prefix = st.prefix | ((uint32_t)(4 * lane + j) << shift);
    ms[j] = bin_mass(rw->isum[pass][4 * lane + j], key_prefix, pass);
    cn[j] = rw->count[pass][4 * lane + j];
  }
  const double mine = ms[0] + ms[1] + ms[2] + ms[3];
  const uint32_t minec = cn[0] + cn[1] + cn[2] + cn[3];
  double incl = mine;
  uint32_t inclc = minec;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double up = __shfl_up(incl, d);
    const uint32_t upc = __shfl_up(inclc, d);
    if (lane >= d) { incl += up; inclc += upc; }
  }
  double target;
  if (total) {                          // first pass: its bins hold every token, their mass is the total
    *total = __shfl(incl, 63);
    target = tau * *total;
  } else {
    target = tau * rw->total;
  }
  // first lane whose bins reach the target; if none does (tau >= 1 up to rounding), the last lane
  // that holds any token
  const unsigned long long reach = __ballot(minec > 0 && st.mass_below + incl >= target);
  const unsigned long long any = __ballot(minec > 0);
  const int who = reach ? __ffsll((long long)reach) - 1 : (any ? 63 - __clzll((long long)any) : 0);
  double mb = st.mass_below + (incl - mine);
  uint32_t cb = st.count_below + (inclc - minec);
  int bin = 4 * lane;
  int last_nonempty = -1;
  bool found = false;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (!found && cn[j] > 0) {
      if (mb + ms[j] >= target) { bin = 4 * lane + j; found = true; }
      else { mb += ms[j]; cb += cn[j]; last_nonempty = j; }
    }
  }
  if (!found) {
    // target not reached inside this lane: stay on its last non-empty bin
    bin = 4 * lane + (last_nonempty < 0 ? 0 : last_nonempty);
    if (last_nonempty >= 0) { mb -= ms[last_nonempty]; cb -= cn[last_nonempty]; }
  }
  BudState out;
  out.prefix = st.prefix | ((uint32_t)__shfl(bin, who) << shift);
  out.count_below = __shfl(cb, who);
  out.mass_below = __shfl(mb, who);
  return out;
}

template <int PASS>
__global__ __launch_bounds__(kThreads) void bud_hist_kernel(BudArgs a) {
  __shared__ unsigned long long hsum[256];
  __shared__ uint32_t hcount[256];
  __shared__ BudState sh_state;
  const int slice = blockIdx.x;
  const long long b = blockIdx.y;
  BudRow* rw = a.rows + b;
  const float* s = a.sl + b * a.L;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  constexpr int shift = 24 - 8 * PASS;
  if (wave == 0) {
    BudState st;
    if (PASS == 0) { st.prefix = 0u; st.count_below = 0u; st.mass_below = 0.0; }
    else {
      double total;
      st = next_state(rw, PASS - 1, rw->state[PASS - 1], a.tau, PASS == 1 ? &total : nullptr, shift + 8, lane);
      if (PASS == 1 && lane == 0 && slice == 0) rw->total = total;
    }
    if (lane == 0) {
      sh_state = st;
      if (slice == 0) rw->state[PASS] = st;
    }
  }
  if (tid < 256) { hsum[tid] = 0ull; hcount[tid] = 0u; }
  __syncthreads();
  const uint32_t prefix = sh_state.prefix;
  constexpr uint32_t himask = PASS == 0 ? 0u : (0xffffffffu << (shift + 8));
  const int t_end = min(a.L, (slice + 1) * kSlice);
  for (int t = slice * kSlice + tid; t < t_end; t += kThreads) {
    const float v = s[t];
    const uint32_t key = order_key(v);
    if ((key & himask) == prefix) {
      const uint32_t dg = (key >> shift) & 255u;
      uint32_t sig;
      int e;
      split_float(v, sig, e);
      atomicAdd(&hcount[dg], 1u);
      atomicAdd(&hsum[dg], (unsigned long long)sig << (e - bin_exponent(key, PASS)));   // shift is 0 or 1
    }
  }
  __syncthreads();
  if (tid < 256 && hcount[tid]) {
    atomicAdd(&rw->count[PASS][tid], hcount[tid]);
    atomicAdd(&rw->isum[PASS][tid], hsum[tid]);
  }
}

// The count from the value v at which the ascending mass crosses the target: n_eq tokens have it, count_below tokens
// with mass_below lie under it; of the n_eq, as many are dropped as are needed to reach the target.
__device__ __forceinline__ int32_t keep_of(const BudArgs& a, float value, uint32_t n_eq, uint32_t count_below, double mass_below,
                                           double target) {
  long long k_sparse = 0;
  if (a.tau > 0.0) {
    const double v = (double)value;
    long long j = n_eq;
    if (v > 0.0) {
      const double need = (target - mass_below) / v;
      j = (long long)ceil(need);
      if (j < 1) j = 1;
      if (j > (long long)n_eq) j = n_eq;
    }
    k_sparse = (long long)count_below + j;
  }
  long long keep = (long long)a.L - k_sparse;
  if (keep < a.k_min) keep = a.k_min;
  if (keep > a.k_max) keep = a.k_max;
  return (int32_t)keep;
}

__global__ void bud_final_kernel(BudArgs a) {
  const long long b = blockIdx.x;
  BudRow* rw = a.rows + b;
  const int lane = threadIdx.x;
  const double target = a.tau * rw->total;
  const BudState st = next_state(rw, 3, rw->state[3], a.tau, nullptr, 0, lane);
  if (lane == 0) {
    rw->state[4] = st;
    a.k_keep[b] = keep_of(a, key_value(st.prefix), rw->count[3][st.prefix & 255u], st.count_below, st.mass_below, target);
  }
}

// ---- rows of up to kRowTokens: the descent in one launch, one workgroup per row.
// The chain above is five launches of a few us each whose work is a few hundred ns: what they cost is the launches.  Here the
// row's keys stay in registers (J per thread), and the bins are cut from the RANGE the keys span (as the selection cuts
// them) instead of from the digits: 2048 bins of at most 2^21 consecutive keys, and the keys of a bin still differ by
// at most one step of the binary exponent, so that the bin's mass stays an exact integer sum.  Count and mass share one
// 64-bit LDS atomic per key: count in the upper 20 bits, the signed sum of the (at most 25-bit) shifted significands
// of up to 2^14 keys in the lower 44.  As soon as the bin that crosses the target holds at most 64 keys, one wavefront ranks
// them against each other (integer sums again, so the order in which they were collected does not matter): one
// pass in practice, three at most (2^32 -> 2^21 -> 2^10 -> 1).
// Bound by the chain of its steps on one CU: load, range, a pass (clear, count, scan), ranking.
constexpr int kRowBins = 2 * kThreads;
// 16 keys per thread are the most that is built; that, and not a crossing, is the line.  Whole budget with 32 heads, one launch /
// five: 4096 tokens 10.6 / 23.2 us, 8192 13.8 / 22.9, 12345 15.7 / 22.6, 16384 16.7 / 22.9; with more keys per thread 20000 20.4 / 23.7, 32768
// 26.1 / 23.8, so the two cross between these.
constexpr int kRowTokens = 16 * kThreads;
constexpr int kCountShift = 44;
constexpr int kHot = 16;                      // keys of a wavefront in one bin from which they are added up first
constexpr int kRank = 64;

__device__ __forceinline__ int key_exponent(uint32_t key) {
  const uint32_t u = (key & 0x80000000u) ? key : ~key;
  const int e = (int)((u >> 23) & 255u);
  return e < 1 ? 1 : e;
}
// smallest exponent field among the keys lo .. lo + last (see bin_exponent)
__device__ __forceinline__ int range_exponent(uint32_t lo, uint32_t last) {
  const uint32_t hi = lo > 0xffffffffu - last ? 0xffffffffu : lo + last;
  return min(key_exponent(lo), key_exponent(hi));
}
// a key's score as an integer, in units of 2^(base - 150)
__device__ __forceinline__ long long key_units(uint32_t key, int base) {
  uint32_t sig;
  int e;
  split_float(key_value(key), sig, e);
  const long long u = (long long)((unsigned long long)sig << ((e - base) & 1));   // e - base is 0 or 1
  return (key & 0x80000000u) ? u : -u;
}
__device__ __forceinline__ int lane_value(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

template <int J>
__global__ __launch_bounds__(kThreads) void bud_row_kernel(BudArgs a) {
  __shared__ unsigned long long bins[kRowBins];
  __shared__ double wmass[kWaves];
  __shared__ uint32_t wcount[kWaves], wmin[kWaves], wmax[kWaves];
  __shared__ uint32_t cand[kRank];
  __shared__ int sh_first, sh_last, n_cand;
  __shared__ double sh_mass;
  __shared__ uint32_t sh_below, sh_in;
  const long long b = blockIdx.x;
  const float* s = a.sl + b * a.L;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  uint32_t key[J];
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  float v[J];
#pragma unroll
  for (int j = 0; j < J; ++j) v[j] = s[min(tid + j * kThreads, a.L - 1)];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    key[j] = order_key(v[j]);                                // (past the end: the last key again)
    kmin = min(kmin, key[j]);
    kmax = max(kmax, key[j]);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, d));
    kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, d));
  }
  if (lane == 0) { wmin[wave] = kmin; wmax[wave] = kmax; }
  bins[tid] = 0ull;
  bins[tid + kThreads] = 0ull;
  if (tid == 0) { sh_first = INT_MAX; sh_last = -1; n_cand = 0; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) { kmin = min(kmin, wmin[w]); kmax = max(kmax, wmax[w]); }

  int n_mine = (a.L - tid + kThreads - 1) / kThreads;      // keys of this thread
  uint32_t lo = kmin, last = kmax - kmin;     // the keys still in question: [lo, lo + last]
  uint32_t count_below = 0, n_in = 0;
  double mass_below = 0.0, target = 0.0;
  for (bool first_pass = true;; first_pass = false) {
    const int shift = max(0, 32 - __clz((int)(last | 1u)) - 11);                   // last >> shift < kRowBins
    const uint32_t bin_last = (1u << shift) - 1u;
    asm volatile("" : "+v"(n_mine));            // (J comparisons per pass, not J lane masks kept across the passes)
#pragma unroll
    for (int j = 0; j < J; ++j) {
      asm volatile("" : "+v"(key[j]));                      // (nothing derived from a key lives across the passes: registers)
      const uint32_t off = key[j] - lo;                                            // keys below lo wrap beyond `last`
      const bool in = j < n_mine && off <= last;
      const unsigned long long act = __ballot(in);
      if (act == 0ull) continue;
      const uint32_t bin = in ? off >> shift : 0u;
      const unsigned long long add = (1ull << kCountShift) + (unsigned long long)key_units(key[j], range_exponent(lo + (bin << shift), bin_last));
      // additions to one address run one after the other: a wavefront whose keys crowd into one bin adds them up first
      const int leader = __ffsll((long long)act) - 1;
      const bool same = in && bin == (uint32_t)lane_value((int)bin, leader);
      const unsigned long long hot = __ballot(same);
      if (__popcll(hot) >= kHot) {
        unsigned long long sum = same ? add : 0ull;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
        if (lane == leader) atomicAdd(&bins[bin], sum);
        if (in && !same) atomicAdd(&bins[bin], add);
      } else if (in) {
        atomicAdd(&bins[bin], add);
      }
    }
    __syncthreads();
    // thread t owns bins 2 t and 2 t + 1; masses below them by a scan in a fixed order
    double ms[2] = {0.0, 0.0};
    uint32_t cn[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const unsigned long long w = bins[2 * tid + j];
      const long long sum = (long long)(w << (64 - kCountShift)) >> (64 - kCountShift);
      cn[j] = (uint32_t)((w - (unsigned long long)sum) >> kCountShift);
      if (cn[j]) ms[j] = ldexp((double)sum, range_exponent(lo + ((uint32_t)(2 * tid + j) << shift), bin_last) - 150);
    }
    const double mine = ms[0] + ms[1];
    const uint32_t minec = cn[0] + cn[1];
    double incl = mine;
    uint32_t inclc = minec;
    if (__ballot(minec != 0u)) {
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const double up = __shfl_up(incl, d);
        const uint32_t upc = __shfl_up(inclc, d);
        if (lane >= d) { incl += up; inclc += upc; }
      }
    }
    if (lane == 63) { wmass[wave] = incl; wcount[wave] = inclc; }
    __syncthreads();
    double base = 0.0, all = 0.0;
    uint32_t basec = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) { base += wmass[w]; basec += wcount[w]; }
      all += wmass[w];
    }
    if (first_pass) target = a.tau * all;                                          // the first pass's bins hold every token
    // the first bin whose keys reach the target; if none does (tau >= 1 up to rounding), the last bin with any token
    const double mb0 = mass_below + base + (incl - mine), mb1 = mb0 + ms[0];
    const uint32_t cb0 = count_below + basec + (inclc - minec), cb1 = cb0 + cn[0];
    const bool hit0 = cn[0] && mb0 + ms[0] >= target, hit1 = cn[1] && mb1 + ms[1] >= target;
    const unsigned long long reach = __ballot(hit0 || hit1), some = __ballot(minec != 0u);
    if (reach && lane == __ffsll((long long)reach) - 1) atomicMin(&sh_first, 2 * tid + (hit0 ? 0 : 1));
    if (some && lane == 63 - __clzll((long long)some)) atomicMax(&sh_last, 2 * tid + (cn[1] ? 1 : 0));
    __syncthreads();
    const int bin = sh_first != INT_MAX ? sh_first : sh_last;
    if (bin == 2 * tid) { sh_mass = mb0; sh_below = cb0; sh_in = cn[0]; }
    if (bin == 2 * tid + 1) { sh_mass = mb1; sh_below = cb1; sh_in = cn[1]; }
    bins[tid] = 0ull;                                      // for the next pass
    bins[tid + kThreads] = 0ull;
    __syncthreads();
    if (tid == 0) { sh_first = INT_MAX; sh_last = -1; }
    mass_below = sh_mass;
    count_below = sh_below;
    n_in = sh_in;
    lo += (uint32_t)bin << shift;
    last = bin_last;
    if (n_in <= kRank || shift == 0) break;
    __syncthreads();
  }
  if (last == 0) {                                         // a single value (as many keys as there may be)
    if (tid == 0) a.k_keep[b] = keep_of(a, key_value(lo), n_in, count_below, mass_below, target);
    return;
  }
  asm volatile("" : "+v"(n_mine));
#pragma unroll
  for (int j = 0; j < J; ++j)
    if (j < n_mine && key[j] - lo <= last) cand[atomicAdd(&n_cand, 1)] = key[j];     // n_in of them
  __syncthreads();
  if (wave) return;
  // lane i: the keys below candidate i, and those equal to it
  const int base = range_exponent(lo, last);
  const uint32_t mine = cand[min(lane, (int)n_in - 1)];
  const long long units = key_units(mine, base);
  long long below = 0;
  uint32_t n_less = 0, n_eq = 0;
  for (int i = 0; i < (int)n_in; ++i) {
    const uint32_t other = (uint32_t)lane_value((int)mine, i);
    const long long u = ((long long)lane_value((int)(units >> 32), i) << 32) | (uint32_t)lane_value((int)units, i);
    if (other < mine) { below += u; ++n_less; }
    n_eq += other == mine;
  }
  const double mb = mass_below + ldexp((double)below, base - 150);
  const bool reach = mb + ldexp((double)(units * (long long)n_eq), base - 150) >= target;
  // the smallest candidate that reaches the target, else the largest
  uint32_t pick = reach ? mine : 0xffffffffu, top = mine;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    pick = min(pick, (uint32_t)__shfl_xor((int)pick, d));
    top = max(top, (uint32_t)__shfl_xor((int)top, d));
  }
  if (!__ballot(reach)) pick = top;
  if (lane == __ffsll((long long)__ballot(mine == pick)) - 1)
    a.k_keep[b] = keep_of(a, key_value(mine), n_eq, count_below + n_less, mb, target);
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t budget_ws_bytes(const Dims& dm) {
  return align256((size_t)dm.B * sizeof(BudRow)) + align256((size_t)dm.B * dm.L * sizeof(float));
}

hipError_t launch_budget(const Dims& dm, const float* scores, double tau_cov, int32_t* k_keep, void* ws, hipStream_t st,
                         int k_max, int k_min) {
  BudArgs a;
  a.k_max = k_max > 0 ? k_max : dm.L;
  a.k_min = k_min > 1 ? k_min : 1;
  a.scores = scores;
  a.rows = (BudRow*)ws;
  a.sl = (float*)((char*)ws + align256((size_t)dm.B * sizeof(BudRow)));
  a.k_keep = k_keep;
  a.Hq = dm.Hq; a.L = dm.L; a.tau = tau_cov;
  if (dm.L <= kRowTokens) a.rows = nullptr;
  head_sum_kernel<<<dim3((dm.L + kSumThreads - 1) / kSumThreads, dm.B), kSumThreads, 0, st>>>(a);
  if (!a.rows) {
    const int per_thread = (dm.L + kThreads - 1) / kThreads;
    if (per_thread <= 4) bud_row_kernel<4><<<dm.B, kThreads, 0, st>>>(a);
    else bud_row_kernel<16><<<dm.B, kThreads, 0, st>>>(a);
    return hipGetLastError();
  }
  const dim3 grid((dm.L + kSlice - 1) / kSlice, dm.B);
  bud_hist_kernel<0><<<grid, kThreads, 0, st>>>(a);
  bud_hist_kernel<1><<<grid, kThreads, 0, st>>>(a);
  bud_hist_kernel<2><<<grid, kThreads, 0, st>>>(a);
  bud_hist_kernel<3><<<grid, kThreads, 0, st>>>(a);
  bud_final_kernel<<<dm.B, 64, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace tsa
