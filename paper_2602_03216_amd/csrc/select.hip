// Head-wise top-k selection: Algorithm 1 of the paper, S_h = TopK(s_h, k_keep).
// Exact: the k_keep largest scores, ties to the lowest token index, emitted in ascending
// token order together with the inverse map.  Integer work on the order-preserving uint32
// image of the fp32 score.  Rows of up to 32768 tokens (65536 if there are many) take one launch (select_row_kernel,
// below); longer ones:
//   1. radix select, 4 passes of 8 bits, most significant first: every pass histograms the
//      digit of the keys that still match the prefix found so far (LDS histograms per
//      wavefront), and the next kernel derives the digit of the k-th largest key from the
//      histogram.  The first pass writes one histogram per slice (nothing has to be cleared
//      beforehand; its first slice clears the row histograms of the later passes, which are
//      built with one global atomic per bin and workgroup); the last pass also leaves, per
//      slice, the number of keys above the 24-bit prefix and the histogram of the last digit;
//   2. write: the threshold key T from the last histogram; the per-slice figures of the last
//      pass give the number of keys above T / equal to T in the slices before this one,
//      per-wavefront counts inside the slice give every wavefront its output offset; a stable
//      ballot compaction writes idx ascending and inv.
// A head is cut into at most 64 slices (a power of two of tokens, at least 2048, one workgroup of 1024
// threads each), sized so that a launch has about 512 workgroups: each of the five small kernels
// is a chain of dependent steps per thread, so it pays to spread it over the whole chip, but not
// to go below a few tokens per thread.
#include <algorithm>

#include "v_tiles.h"

namespace tsa {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kMinSlice = 2048, kMaxSlice = 16384;   // tokens per workgroup (SelArgs::slice), unless a row needs more
constexpr int kMaxSlices = 64;                       // slices per row at most

struct SelState {
  uint32_t prefix;   // digits found so far, in place
  uint32_t krem;     // how many keys are still wanted among those that match the prefix
};

// Per selection row (batch, head or group) in the workspace:
struct RowWs {
  uint32_t hist[4][256];      // [0] is unused (the first pass keeps one histogram per slice)
  SelState state[5];          // state[p]: before pass p; state[4]: (T, number of keys equal to T to take)
  uint32_t pad[6];
};

// Per (row, slice) in the workspace:
struct SliceWs {
  uint32_t hist0[256];        // first pass: digit histogram of the slice
  uint32_t last[256];         // last pass: last digit of the slice's keys that match the 24-bit prefix
  uint32_t n_above;           // last pass: keys of the slice above the 24-bit prefix
  uint32_t pad[63];
};

struct SelArgs {
  const float* scores;
  int32_t* idx;
  int32_t* inv;
  RowWs* rows;
  SliceWs* slices;            // [row][nslices]
  int L, k, ff, fl, nslices;
  int slice;                  // tokens per workgroup; a wavefront owns slice / kWaves contiguous tokens
  // Count decided on the device (dynamic coverage budget): k_dev[b] replaces k for the rows of batch
  // entry b (NULL: every row takes k); a row of idx is k_stride entries long either way.
  const int32_t* k_dev;
  int k_stride;
  FastDiv by_b;               // batch entry of a row
  // select_row_kernel only: `parts` workgroups share a row; with tiles.Vt they also gather the row's V tiles
  int parts, n_rows;
  FastDiv by_parts;
  VTiles tiles;
  __device__ __forceinline__ uint32_t k_of(long long row) const {
    return (uint32_t)(k_dev ? k_dev[by_b.div((uint32_t)row)] : k);
  }
};

// fp32 -> uint32 with the same order (-0 and +0 map to the same key)
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u << 1) == 0u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ uint32_t key_at(const float* __restrict__ s, int t, int L, int ff, int fl) {
  if (t < ff || t >= L - fl) return 0xffffffffu;   // always-kept tokens rank above every score
  return order_key(s[t]);
}

// Digit of the krem-th largest key among those counted in `hist`, found by the first wavefront:
// lane l sums bins 255-4l .. 252-4l, a wave scan finds the lane where the running count from the
// top reaches krem, the lane then walks its four bins.
__device__ __forceinline__ SelState next_state(const uint32_t* __restrict__ hist, SelState st, int shift, int lane) {
  uint32_t c[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) c[j] = hist[255 - 4 * lane - j];
  const uint32_t mine = c[0] + c[1] + c[2] + c[3];
  uint32_t incl = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d);
    if (lane >= d) incl += up;
  }
  const unsigned long long reach = __ballot(incl >= st.krem);
  const int who = reach ? __ffsll((long long)reach) - 1 : 63;
  uint32_t above = incl - mine, bin = 255 - 4 * lane;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    if (above + c[j] < st.krem) { above += c[j]; bin = 255 - 4 * lane - (j + 1); }
    else break;
  }
  SelState out;
  out.prefix = st.prefix | (__shfl(bin, who) << shift);
  out.krem = st.krem - __shfl(above, who);
  return out;
}

template <int PASS>
__global__ __launch_bounds__(kThreads) void hist_kernel(SelArgs a) {
  __shared__ uint32_t hist[kWaves][256];
  __shared__ uint32_t tot[256];
  __shared__ SelState sh_state;
  __shared__ uint32_t sh_above;
  const int slice = blockIdx.x;
  const long long row = blockIdx.y;
  RowWs* rw = a.rows + row;
  SliceWs* sw = a.slices + row * a.nslices + slice;
  const float* s = a.scores + row * a.L;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  constexpr int shift = 24 - 8 * PASS;

  if (PASS == 0 && slice == 0) {                          // row histograms of the later passes start at zero
    for (int i = tid; i < 3 * 256; i += kThreads) rw->hist[1 + i / 256][i % 256] = 0u;
  }
  if (PASS == 1) {                                        // the first pass left one histogram per slice: add them up
    const SliceWs* row_slices = a.slices + row * a.nslices;
    uint32_t c = 0;
    for (int sl = tid >> 8; sl < a.nslices; sl += kThreads / 256) c += row_slices[sl].hist0[tid & 255];
    hist[tid >> 8][tid & 255] = c;
    __syncthreads();
    if (tid < 256) tot[tid] = hist[0][tid] + hist[1][tid] + hist[2][tid] + hist[3][tid];
    __syncthreads();
  }
  if (wave == 0) {
    SelState st;
    if (PASS == 0) { st.prefix = 0u; st.krem = a.k_of(row); }
    else st = next_state(PASS == 1 ? tot : rw->hist[PASS - 1], rw->state[PASS - 1], shift + 8, lane);
    if (lane == 0) {
      sh_state = st;
      if (slice == 0) rw->state[PASS] = st;
    }
  }
  for (int i = tid; i < kWaves * 256; i += kThreads) (&hist[0][0])[i] = 0u;
  if (tid == 0) sh_above = 0u;
  __syncthreads();
  const uint32_t prefix = sh_state.prefix;
  constexpr uint32_t himask = PASS == 0 ? 0u : (0xffffffffu << (shift + 8));
  const int t_end = min(a.L, (slice + 1) * a.slice);
  uint32_t above = 0;
  for (int base = slice * a.slice; base < t_end; base += kThreads) {
    const int t = base + tid;
    bool valid = false;
    uint32_t dg = 0;
    if (t < t_end) {
      const uint32_t key = key_at(s, t, a.L, a.ff, a.fl);
      valid = (key & himask) == prefix;
      dg = (key >> shift) & 255u;
      if (PASS == 3 && (key & himask) > prefix) ++above;
    }
    const unsigned long long act = __ballot(valid);
    if (act == 0ull) continue;
    // common case in the first pass: the whole wavefront falls into one bin
    const int leader = __ffsll((long long)act) - 1;
    const uint32_t dg0 = __shfl(dg, leader);
    const unsigned long long same = __ballot(valid && dg == dg0);
    if (same == act) {
      if (lane == leader) atomicAdd(&hist[wave][dg0], (uint32_t)__popcll(act));
    } else if (valid) {
      atomicAdd(&hist[wave][dg], 1u);
    }
  }
  if (PASS == 3) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) above += __shfl_xor(above, d);
    if (lane == 0 && above) atomicAdd(&sh_above, above);
  }
  __syncthreads();
  if (tid < 256) {
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) c += hist[w][tid];
    if (PASS == 0) sw->hist0[tid] = c;
    else if (c) atomicAdd(&rw->hist[PASS][tid], c);
    if (PASS == 3) sw->last[tid] = c;
  }
  if (PASS == 3 && tid == 0) sw->n_above = sh_above;
}

// Keys of a wavefront's segment held in registers between the counting and the compaction: segments of up
// to kRegKeys * 64 tokens (slices of up to 16384) are read once, longer ones are read again.
constexpr int kRegKeys = 16;

__global__ __launch_bounds__(kThreads) void write_kernel(SelArgs a) {
  __shared__ SelState sh_state;
  __shared__ uint32_t before_gt, before_eq;
  __shared__ uint2 cnt[kWaves];
  const int slice = blockIdx.x;
  const long long row = blockIdx.y;
  RowWs* rw = a.rows + row;
  const SliceWs* row_slices = a.slices + row * a.nslices;
  const float* s = a.scores + row * a.L;
  int32_t* out_idx = a.idx + row * a.k_stride;
  int32_t* out_inv = a.inv ? a.inv + row * a.L : nullptr;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // the keys of this wavefront's segment are requested first: their latency hides behind the threshold
  const int seg = a.slice / kWaves;
  const int t_lo = slice * a.slice + wave * seg;
  const int t_hi = min(a.L, t_lo + seg);
  const bool in_regs = seg <= kRegKeys * 64;
  uint32_t keys[kRegKeys];
  if (in_regs) {
#pragma unroll
    for (int j = 0; j < kRegKeys; ++j) {
      const int t = t_lo + 64 * j + lane;
      keys[j] = t < t_hi ? key_at(s, t, a.L, a.ff, a.fl) : 0u;
    }
  }
  if (tid == 0) { before_gt = 0u; before_eq = 0u; }
  if (wave == 0) {
    const SelState st = next_state(rw->hist[3], rw->state[3], 0, lane);
    if (lane == 0) {
      sh_state = st;
      if (slice == 0) rw->state[4] = st;
    }
  }
  __syncthreads();
  const uint32_t T = sh_state.prefix;
  const uint32_t need_eq = sh_state.krem;
  // keys above T / equal to T in the slices before this one, from what the last pass left per slice
  {
    const uint32_t dT = T & 255u;
    uint32_t gt = 0, eq = 0;
    if (tid < slice) gt = row_slices[tid].n_above;
    for (int i = tid; i < slice * 256; i += kThreads) {
      const uint32_t v = row_slices[i >> 8].last[i & 255];
      const uint32_t d = (uint32_t)(i & 255);
      gt += d > dT ? v : 0u;
      eq += d == dT ? v : 0u;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      gt += __shfl_xor(gt, d);
      eq += __shfl_xor(eq, d);
    }
    if (lane == 0) {
      if (gt) atomicAdd(&before_gt, gt);
      if (eq) atomicAdd(&before_eq, eq);
    }
  }
  // this slice: per-wavefront counts, then the stable compaction
  {
    uint32_t n_gt = 0, n_eq = 0;
    if (in_regs) {
#pragma unroll
      for (int j = 0; j < kRegKeys; ++j) {
        const bool in = t_lo + 64 * j + lane < t_hi;
        n_gt += (uint32_t)__popcll(__ballot(in && keys[j] > T));
        n_eq += (uint32_t)__popcll(__ballot(in && keys[j] == T));
      }
    } else {
      for (int base = t_lo; base < t_hi; base += 64) {
        const int t = base + lane;
        const bool in = t < t_hi;
        const uint32_t key = in ? key_at(s, t, a.L, a.ff, a.fl) : 0u;
        n_gt += (uint32_t)__popcll(__ballot(in && key > T));
        n_eq += (uint32_t)__popcll(__ballot(in && key == T));
      }
    }
    if (lane == 0) cnt[wave] = make_uint2(n_gt, n_eq);
  }
  __syncthreads();
  uint32_t gt_before = before_gt, eq_before = before_eq;
  for (int w = 0; w < wave; ++w) { gt_before += cnt[w].x; eq_before += cnt[w].y; }
  // ties are taken in token order until need_eq of them are used up
  uint32_t eq_run = eq_before, out_run = gt_before + min(need_eq, eq_before);
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  auto emit = [&](int t, uint32_t key) {
    const bool in = t < t_hi;
    const bool gt = in && key > T;
    const bool eq = in && key == T;
    const unsigned long long m_eq = __ballot(eq);
    const uint32_t eq_rank = eq_run + (uint32_t)__popcll(m_eq & lt_mask);
    const bool take = gt || (eq && eq_rank < need_eq);
    const unsigned long long m_take = __ballot(take);
    const uint32_t pos = out_run + (uint32_t)__popcll(m_take & lt_mask);
    if (take) out_idx[pos] = t;
    if (in && out_inv) out_inv[t] = take ? (int32_t)pos : -1;
    out_run += (uint32_t)__popcll(m_take);
    eq_run += (uint32_t)__popcll(m_eq);
  };
  if (in_regs) {
#pragma unroll
    for (int j = 0; j < kRegKeys; ++j)
      if (t_lo + 64 * j < t_hi) emit(t_lo + 64 * j + lane, keys[j]);
  } else {
    for (int base = t_lo; base < t_hi; base += 64) {
      const int t = base + lane;
      emit(t, t < t_hi ? key_at(s, t, a.L, a.ff, a.fl) : 0u);
    }
  }
}

// Rows of up to row_max_tokens: the whole selection of a row in ONE launch by one workgroup.  The keys of the row
// stay in registers (4 J per lane; a wavefront owns 256 J consecutive tokens, lane l of step j the four tokens
// 256 j + 4 l ..), and the threshold comes from a radix descent over the RANGE the row's keys span: the first
// pass cuts [smallest key, largest key] into kBins equal bins, so the keys spread over the bins whatever their
// magnitude (equal 8-bit digits of softmax scores fall into a handful of bins, and LDS atomics on one
// address run one after the other).  A pass narrows the range by 2^12; as soon as the bin with the k-th key
// holds at most kRank keys, they are ranked against each other directly.  At most three
// passes, one or two in practice.  With per-group sets the sum over the g heads happens in the key load or before it (kInlineSum).
// Bound: one CU's share of a row: 4 bytes per token into one CU and the vector instructions per key (at 32768 tokens
// of 15 us: 3 launch, 4 load, 3 keys and range, 3 histogram and ranking, 3 counting and compaction).
// Measured on softmax-like scores, 32 rows, against the former kernels (8-bit digits: one workgroup per row with the
// keys in LDS up to 16384 tokens, the five sliced launches above that): 3001 tokens 10.6 -> 6.9 us, 8192: 18.2 -> 8.1,
// 12345: 24.6 -> 10.1, 32768: 28.8 -> 15.3, 96 rows of 65536: 72 -> 32 us.
// A launch of few rows leaves most CUs idle, and the gather of the selected V rows that follows in the whole layer is
// a launch of its own that waits for the last row.  With up to 128 rows, `parts` workgroups therefore take the same row
// where the caller wants the V tiles: each of them finds the threshold (the scores come out of the L2 that the parts of
// a row share), writes its share of idx and inv, and builds the V tiles of its share of idx.  More rows fill the chip
// by themselves (one workgroup per CU is resident) and keep the separate gather.
// Selection + gather, 32 rows: 901 of 3001 tokens 14.0 -> 10.6 us, 4096 of 8192: 21.9 -> 20.4, 3277 of 32768: 27.4 -> 26.2,
// 16384 of 32768: 65.3 -> 63.7 (the last one and the second at the rate of HBM).
constexpr int kBins = 4096;
constexpr uint32_t kHotLanes = 16;  // keys of a wavefront in one bin from which they are counted by ballots
constexpr int kCrowd = 2048;        // keys left in a bin from which their range is taken anew
constexpr int kRank = 256;          // that many keys are ranked against each other instead of binned again
// One workgroup per row against the sliced kernels, which take 20 to 45 us, by the number of tokens and not by the scores (selection alone,
// softmax-like, sliced / one launch): 32768 tokens x 1 row 21.0 / 16.7, x 32 rows 28.5 / 17.9; 49152 x 1 22.5 / 23.0, x 8 23.6 / 23.8,
// x 16 28.5 / 23.9, x 64 41.8 / 25.4; in the layer 40000 x 8 110.0 / 114.3, x 16 146.3 / 140.0.  Beyond 49152 the 64 keys per lane no longer
// fit the registers (17 to 30 spill; 8 with 48 keys): 65536 x 8 25.0 / 30.9, x 28 33.5 / 32.7 and in the layer 240 / 240, x 64 43.4 / 33.1.
inline int row_max_tokens(int rows) { return rows > 32 ? 65536 : rows > 8 ? 49152 : 32768; }
// A row's workgroup can sum the g heads of its group while it loads them, but one CU then reads g rows, a head at a
// time (and in the layer every part of the row does).  Beyond that many extra scores the chip-wide sum in a launch of
// its own is faster, us without / with that launch: (g - 1) L = 24576 (4 x 8192) 9.7 / 11.4, 57344 (8 x 8192) 10.5 / 11.6 (whole layer
// 67.8 / 67.8), 98304 (4 x 32768) 19.8 / 19.9 (layer 156 / 154), 114688 (8 x 16384) 14.9 / 14.4 (layer 98.4 / 94.5), 229376 23.3 / 20.3,
// 1015808 (32 x 32768) 58 / 22; 32 heads.
constexpr long long kInlineSum = 65536;
constexpr int kCUs = 256;

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, d));
  return v;
}

__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// The order of order_key on other numbers, [1, 0xffffffff]: a negative value's bits are negated instead of inverted,
// which maps -0 to +0's key, leaves every other bit pattern a key of its own (NaNs among them) and key 0 to nothing.
__device__ __forceinline__ uint32_t row_key(uint32_t u) { return (int32_t)u < 0 ? 0u - u : u | 0x80000000u; }

// set bits of a ballot below this lane
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

typedef float __attribute__((ext_vector_type(4), aligned(4))) f32x4_a4;      // rows start at any multiple of 4 bytes

template <int J, bool TILES>
__global__ __launch_bounds__(kThreads) void select_row_kernel(SelArgs a, int g) {
  __shared__ __attribute__((aligned(16))) uint32_t hist[kBins];
  __shared__ __attribute__((aligned(16))) uint32_t cand[kRank];
  __shared__ uint32_t wtot[kWaves], wlo[kWaves];
  __shared__ uint32_t sh_bin, sh_rem, sh_cnt, sh_n, sh_T, sh_eq;
  // consecutive workgroup ids go to different XCDs: id % 8 picks a contiguous range of (row, part), so that the
  // workgroups of a row share an L2
  const unsigned at = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (at >= (unsigned)(a.n_rows * a.parts)) return;
  const unsigned row_ = a.by_parts.div(at);
  const long long row = row_;
  const int part = (int)(at - row_ * a.parts);
  const float* s = a.scores + row * g * a.L;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int t0 = wave * 256 * J + 4 * lane;
  uint32_t key[J][4];
  uint32_t kmax = 0u, kmin = 0xffffffffu;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int t = t0 + 256 * j;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (t + 3 < a.L) {
      v = *(const f32x4_a4*)(s + t);
      for (int h = 1; h < g; ++h) v += *(const f32x4_a4*)(s + (long long)h * a.L + t);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t + e < a.L) {
          v[e] = s[t + e];
          for (int h = 1; h < g; ++h) v[e] += s[(long long)h * a.L + t + e];
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) key[j][e] = __float_as_uint(v[e]);
  }
  // 0 = beyond the row, 0xffffffff = always kept (where there are such tokens, the one NaN with that key takes the key of
  // the NaN next to it): both stay outside the descent.  Few steps of a row hold such a token.
  const uint32_t n_forced = (uint32_t)(a.ff + a.fl);
  const uint32_t top = n_forced ? 0xfffffffeu : 0xffffffffu;
#pragma unroll
  for (int j = 0; j < J; ++j) {
#pragma unroll
    for (int e = 0; e < 4; ++e) key[j][e] = min(row_key(key[j][e]), top);
    const int first = wave * 256 * J + 256 * j;
    if (first < a.ff || first + 256 > a.L - a.fl) {        // the same for the whole wavefront
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int t = t0 + 256 * j + e;
        const bool special = t < a.ff || t >= a.L - a.fl;
        kmax = max(kmax, special ? 0u : key[j][e]);
        kmin = min(kmin, special ? 0xffffffffu : key[j][e]);
        if (special) key[j][e] = t < a.L ? 0xffffffffu : 0u;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        kmax = max(kmax, key[j][e]);
        kmin = min(kmin, key[j][e]);
      }
    }
  }
  kmax = wave_max(kmax);
  kmin = ~wave_max(~kmin);
  if (lane == 0) { wtot[wave] = kmax; wlo[wave] = kmin; }
  for (int i = tid; i < kBins; i += kThreads) hist[i] = 0u;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) { kmax = max(kmax, wtot[w]); kmin = min(kmin, wlo[w]); }
  kmax = uniform(kmax);
  kmin = uniform(kmin);

  const uint32_t k_row = uniform(a.k_of(row));
  uint32_t rem = k_row - n_forced;                                 // wanted among the keys in [lo, lo + 2^bits)
  uint32_t T = 0xfffffffeu, need_eq = 0u;                 // nothing but the always-kept tokens
  if (rem > 0u) {
    uint32_t lo = kmin, n_in = (uint32_t)a.L - n_forced;
    int bits = kmax > kmin ? 32 - __clz((int)(kmax - kmin)) : 0;
    while (true) {
      if (rem >= n_in) { T = lo - 1u; need_eq = 0u; break; }           // every key of the range
      if (bits == 0) { T = lo; need_eq = rem; break; }                 // one value
      // members: k - lo <= width (keys beyond the row and always-kept ones lie outside [kmin, kmax])
      const uint32_t width = min(bits >= 32 ? 0xffffffffu : (1u << bits) - 1u, kmax - lo);
      if (n_in <= (uint32_t)kRank) {
        // few keys: collect them and rank every one against all (0 in the places that stay empty ranks below them)
        if (tid == 0) sh_n = 0u;
        if (tid < kRank) cand[tid] = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t k = key[j][e];
            if (k - lo <= width) cand[atomicAdd(&sh_n, 1u)] = k;
          }
        __syncthreads();
        if (tid < (int)n_in) {
          const uint32_t mine = cand[tid];
          uint32_t above = 0u, same = 0u;
          for (uint32_t i = 0; i < n_in; i += 4) {
            const u32x4 o = *(const u32x4*)&cand[i];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              above += o[q] > mine ? 1u : 0u;
              same += o[q] == mine ? 1u : 0u;
            }
          }
          // equal keys write the same; where all of them are taken there is no tie to resolve: T just below them
          if (above < rem && rem <= above + same) {
            const bool all = rem == above + same;
            sh_T = all ? mine - 1u : mine;
            sh_eq = all ? 0u : rem - above;
          }
        }
        __syncthreads();
        T = uniform(sh_T);
        need_eq = uniform(sh_eq);
        break;
      }
      const int shift = bits > 12 ? bits - 12 : 0;
      // LDS atomics on one address run one after the other (0.85 ns each), and one bin takes most keys of a row where its far
      // tokens' probabilities underflow to 0 or an outlier stretches the range.  A wavefront looks for such a bin among
      // the keys of its first step and counts that bin's keys by ballots.  With the new range below, 32 rows of 32768: 60 %
      // zeros 33 -> 21 us, one value and an outlier 98 -> 20, a cluster and an outlier 51 -> 26, softmax-like scores
      // 17.6 -> 17.9.  Several crowded bins cost more: two values 65 -> 31, four 44 -> 29 (the sliced kernels: 28 to 31 us
      // on all of these).
      uint32_t hot = 0xffffffffu, hot_lanes = kHotLanes - 1;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t d = key[0][e] - lo, bin = d >> shift;
        const uint32_t cand = (uint32_t)__builtin_amdgcn_readlane((int)bin, 16 * e + 5);
        const uint32_t lanes = (uint32_t)__popcll(__ballot(d <= width && bin == cand));
        if (lanes > hot_lanes) { hot_lanes = lanes; hot = cand; }
      }
      if (hot == 0xffffffffu) {
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t k = key[j][e] - lo;
            if (k <= width) atomicAdd(&hist[k >> shift], 1u);
          }
      } else {
        uint32_t n_hot = 0;
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t k = key[j][e] - lo, bin = k >> shift;
            const bool in = k <= width;
            n_hot += (uint32_t)__popcll(__ballot(in && bin == hot));
            asm volatile("" : "+s"(n_hot));                // summed at once: the counts of all steps do not fit the scalar registers
            if (in && bin != hot) atomicAdd(&hist[bin], 1u);
          }
        if (lane == 0) atomicAdd(&hist[hot], n_hot);
      }
      __syncthreads();
      // bin of the rem-th largest: thread i owns the bins 4095 - 4 i .. 4092 - 4 i
      const u32x4 c = *(const u32x4*)&hist[kBins - 4 - 4 * tid];
      const uint32_t mine = c[0] + c[1] + c[2] + c[3];
      uint32_t incl = mine;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t up = __shfl_up(incl, d);
        if (lane >= d) incl += up;
      }
      if (lane == 63) wtot[wave] = incl;
      __syncthreads();
      *(u32x4*)&hist[kBins - 4 - 4 * tid] = u32x4{0u, 0u, 0u, 0u};     // clean for the next pass
      uint32_t above = incl - mine;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) above += w < wave ? wtot[w] : 0u;
      if (above < rem && rem <= above + mine) {
        uint32_t bin = kBins - 1 - 4 * tid;
#pragma unroll
        for (int q = 3; q >= 1; --q)
          if (bin == (uint32_t)(kBins - 4 - 4 * tid + q) && above + c[q] < rem) { above += c[q]; --bin; }
        sh_bin = bin;
        sh_rem = rem - above;
        sh_cnt = c[bin & 3u];
      }
      __syncthreads();
      lo += uniform(sh_bin) << shift;
      rem = uniform(sh_rem);
      n_in = uniform(sh_cnt);
      bits = shift;
      if (bits > 0 && n_in > (uint32_t)kCrowd) {
        // a bin with that many keys often holds one value or a narrow cluster: go on with the range they span
        const uint32_t w = min((1u << bits) - 1u, kmax - lo);
        uint32_t hi_k = 0u, lo_k = 0xffffffffu;
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool in = key[j][e] - lo <= w;
            hi_k = max(hi_k, in ? key[j][e] : 0u);
            lo_k = min(lo_k, in ? key[j][e] : 0xffffffffu);
          }
        hi_k = wave_max(hi_k);
        lo_k = ~wave_max(~lo_k);
        if (lane == 0) { wtot[wave] = hi_k; wlo[wave] = lo_k; }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kWaves; ++q) { hi_k = max(hi_k, wtot[q]); lo_k = min(lo_k, wlo[q]); }
        kmax = uniform(hi_k);
        lo = uniform(lo_k);
        bits = kmax > lo ? 32 - __clz((int)(kmax - lo)) : 0;
      }
    }
  }

  // stable compaction: keys above T, and the first need_eq keys equal to T, in token order
  uint32_t n_gt = 0, n_eq = 0;
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) n_gt += key[j][e] > T ? 1u : 0u;
  if (need_eq > 0u) {
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) n_eq += key[j][e] == T ? 1u : 0u;
  }
  uint32_t n_both = n_gt | (n_eq << 16);                   // at most 4096 tokens per wavefront
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) n_both += __shfl_xor(n_both, d);
  __syncthreads();                                         // wtot / wlo of the passes above are read
  if (lane == 0) { wtot[wave] = n_both & 0xffffu; wlo[wave] = n_both >> 16; }
  __syncthreads();
  uint32_t gt_before = 0, eq_run = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    gt_before += w < wave ? wtot[w] : 0u;
    eq_run += w < wave ? wlo[w] : 0u;
  }
  uint32_t out_run = gt_before + min(need_eq, eq_run);
  int32_t* out_idx = a.idx + row * a.k_stride;
  int32_t* out_inv = a.inv ? a.inv + row * a.L : nullptr;
  // this workgroup's share of the row: whole tiles of idx, every parts-th step of inv
  const uint32_t n_tiles = (k_row + kKeyTile - 1) / kKeyTile;
  const uint32_t tile_lo = a.by_parts.div(n_tiles * part), tile_hi = a.by_parts.div(n_tiles * (part + 1));
  const uint32_t pos_lo = tile_lo * kKeyTile, pos_n = (tile_hi - tile_lo) * kKeyTile;
  asm volatile("" : "+s"(T));                              // the comparisons below are made afresh: 8 J masks do not fit the scalar registers
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int t = t0 + 256 * j;
    if (wave * 256 * J + 256 * j >= a.L) break;            // the same for the whole wavefront
    // tokens of a step are in (lane, element) order: counts of the lanes below, then the lane's own elements
    bool take[4];
    uint32_t below = 0, total = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) take[e] = key[j][e] > T;
    if (need_eq > 0u) {                                    // ties are taken in token order until need_eq of them are used up
      bool eq[4];
      uint32_t er = eq_run;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        eq[e] = key[j][e] == T;
        const unsigned long long m = __ballot(eq[e]);
        er += lanes_below(m);
        eq_run += (uint32_t)__popcll(m);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        take[e] = take[e] || (eq[e] && er < need_eq);
        er += eq[e] ? 1u : 0u;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned long long m = __ballot(take[e]);
      below += lanes_below(m);
      total += (uint32_t)__popcll(m);
    }
    uint32_t pos = out_run + below;
    u32x4 iv;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      iv[e] = take[e] ? pos : 0xffffffffu;
      if (take[e]) {
        if (pos - pos_lo < pos_n) out_idx[pos] = t + e;
        ++pos;
      }
    }
    const uint32_t step = wave * J + j;
    if (out_inv && step - a.by_parts.div(step) * a.parts == (uint32_t)part) {
      if (t + 3 < a.L) *(u32x4_a4*)(out_inv + t) = iv;
      else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (t + e < a.L) out_inv[t + e] = (int32_t)iv[e];
      }
    }
    out_run += total;
  }
  if constexpr (!TILES) return;
  __shared__ __attribute__((aligned(16))) char vt_lds[TILES ? kWaves * kVtLds : 16];
  __syncthreads();                                         // the share of idx is written: all of this workgroup's wavefronts read it
  const uint32_t halves = (tile_hi - tile_lo) * a.tiles.halves;
  for (uint32_t i = wave; i < halves; i += kWaves)
    v_half_tile(a.tiles, row, tile_lo + (i >> (a.tiles.halves - 1)), i & (a.tiles.halves - 1), out_idx, (int)k_row, lane, vt_lds + wave * kVtLds);
}

// J with 4096 J >= L, from the built ones
template <int J = 1>
void run_select_row(const SelArgs& a, int g, hipStream_t st) {
  if constexpr (J < 16) {
    if (a.L > 4096 * J) return run_select_row<(J < 4 ? J + 1 : J < 8 ? J + 2 : J + 4)>(a, g, st);
  }
  const unsigned grid = 8u * (unsigned)((a.n_rows * a.parts + 7) / 8);
  if (a.tiles.Vt) select_row_kernel<J, true><<<grid, kThreads, 0, st>>>(a, g);
  else select_row_kernel<J, false><<<grid, kThreads, 0, st>>>(a, g);
}

// scores [B,Hq,L] -> [B,Hkv,L]: sum of the g heads of each KV group, in head order
__global__ void group_sum_kernel(const float* __restrict__ s, float* __restrict__ out, int g, int L, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const long long grp = i / L;
  const int t = (int)(i % L);
  float acc = 0.f;
  for (int j = 0; j < g; ++j) acc += s[(grp * g + j) * L + t];
  out[i] = acc;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
inline int n_rows(const Dims& dm) { return dm.B * (dm.group_mode ? dm.Hkv : dm.Hq); }
// tokens per workgroup: the power of two that gives the launch about 512 workgroups
inline int slice_for(const Dims& dm) {
  const long long want = (long long)n_rows(dm) * dm.L / 512;
  int s = kMinSlice;
  while (s < kMaxSlice && s < want) s *= 2;
  while ((dm.L + s - 1) / s > kMaxSlices) s *= 2;
  return s;
}
inline int n_slices(const Dims& dm) { return (dm.L + slice_for(dm) - 1) / slice_for(dm); }

}  // namespace

size_t select_ws_bytes(const Dims& dm) {
  size_t n = align256((size_t)n_rows(dm) * sizeof(RowWs));
  n += align256((size_t)n_rows(dm) * n_slices(dm) * sizeof(SliceWs));
  if (dm.group_mode) n += align256((size_t)dm.B * dm.Hkv * dm.L * sizeof(float));
  return n;
}

hipError_t launch_select(const Dims& dm, const float* scores, int k_keep, int32_t* idx, int32_t* inv,
                         void* ws, hipStream_t st, const int32_t* k_dev, const void* V, void* Vt) {
  const int rows = n_rows(dm);
  SelArgs a;
  a.rows = (RowWs*)ws;
  a.slices = (SliceWs*)((char*)ws + align256((size_t)rows * sizeof(RowWs)));
  a.scores = scores;
  a.idx = idx; a.inv = inv;
  a.L = dm.L; a.k = k_keep; a.ff = dm.force_first; a.fl = dm.force_last; a.nslices = n_slices(dm);
  a.k_dev = k_dev; a.k_stride = k_keep;
  a.by_b = FastDiv(rows / dm.B, rows);
  a.slice = slice_for(dm);
  int g = dm.group_mode ? dm.Hq / dm.Hkv : 1;
  const bool one_launch = dm.L <= row_max_tokens(rows);
  if (g > 1 && (!one_launch || (long long)(g - 1) * dm.L > kInlineSum)) {
    float* gs = (float*)((char*)a.slices + align256((size_t)rows * n_slices(dm) * sizeof(SliceWs)));
    const long long n = (long long)rows * dm.L;
    group_sum_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(scores, gs, g, dm.L, n);
    a.scores = gs;
    g = 1;
  }
  if (one_launch) {
    const bool with_tiles = Vt && 2 * rows <= kCUs;
    a.tiles = v_tiles_of(dm, k_keep, V, with_tiles ? Vt : nullptr);
    a.n_rows = rows;
    a.parts = with_tiles ? min(kCUs / rows, a.tiles.nk_tiles) : 1;
    a.by_parts = FastDiv(a.parts, (uint64_t)std::max(rows + 8, a.tiles.nk_tiles + 64) * a.parts);
    run_select_row(a, g, st);
    if (Vt && !with_tiles) return launch_compress_v_tiles(dm, V, idx, k_keep, Vt, st, k_dev);
    return hipGetLastError();
  }
  const dim3 grid(a.nslices, rows);
  hist_kernel<0><<<grid, kThreads, 0, st>>>(a);
  hist_kernel<1><<<grid, kThreads, 0, st>>>(a);
  hist_kernel<2><<<grid, kThreads, 0, st>>>(a);
  hist_kernel<3><<<grid, kThreads, 0, st>>>(a);
  write_kernel<<<grid, kThreads, 0, st>>>(a);
  if (Vt) return launch_compress_v_tiles(dm, V, idx, k_keep, Vt, st, k_dev);
  return hipGetLastError();
}

}  // namespace tsa
