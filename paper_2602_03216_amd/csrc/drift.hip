// Inter-Layer Representation Drift (Eq. 1 of the paper):
//   R = mean over tokens t of  ||h_out[t] - h_in[t]||_2 / (||h_in[t]||_2 + eps)
// for the hidden states entering and leaving one layer.  A streaming reduction bound by HBM
// bandwidth: one wavefront per token row, fp32 sums of squares, per-workgroup partial sums in a fixed
// order (the result is deterministic), a last small kernel adds the partials in fp64.
#include "tsa_internal.h"

#include <algorithm>

namespace tsa {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kRowsPerBlock = 64;     // rows per workgroup (4 per wavefront), fewer in short calls

// What it needs is bytes in flight: 256 CUs reach the HBM rate with about 64 KiB requested per CU.  Thirty-two
// wavefronts per CU (two workgroups) with two batches each (the next batch is requested before the sums of the
// current one, across row ends) keep at least that requested.  A row goes through a buffer descriptor of its own
// length, so the lanes past its end read zeros and add nothing.
// Both kernels, 16384 rows x 4096 from HBM: 91.5 us (2.9 TB/s, four wavefronts per CU, one pair of loads in flight
// each) -> 48.9 us (5.5 TB/s; 4 us of it the last kernel).
// kBatch = 16-byte pieces per lane and tensor in one request: 1 for rows of up to 512 values, whose batch is one row,
// 2 for wider ones.  Narrow rows pay for every piece they do not have (and for the wavefronts that the registers of more pieces keep
// out), us with 1 / 2 / 4 pieces (4: one workgroup per CU): 65536 x 64 17.2 / 19.7 / 33.6, x 512 24.0 / 24.6 / 35.4, x 1024 43.3 / 42.8 / 47.8,
// 300000 x 64 61 / 72 / 141, 16384 x 4096 (in the memory-side cache) 40.2 / 40.8 / 40.9, 20000 x 3584 53.6 / 52.5 / 54.1.
constexpr int kNarrow = 512;
constexpr int kResident = 512;        // workgroups of a launch that run at once (two per CU)

template <int kBatch>
__global__ __launch_bounds__(kThreads, 8) void drift_rows_kernel(const u32x4* __restrict__ hin, const u32x4* __restrict__ hout,
                                                              long long n_tokens, int rows_per_block, int width, float eps,
                                                              double* partial) {
  __shared__ double wsum[kWaves];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t row_bytes = (uint32_t)width * 2u;
  const long long row0 = (long long)blockIdx.x * rows_per_block;
  const int rows = (int)(n_tokens - row0 < rows_per_block ? n_tokens - row0 : rows_per_block);
  const int n_mine = wave < rows ? (rows - wave + kWaves - 1) / kWaves : 0;
  constexpr uint32_t kStep = kBatch * 64 * 16;        // bytes of a row per batch
  const uint32_t n_batches = row_bytes / kStep + (row_bytes % kStep ? 1u : 0u);
  u32x4 a[2][kBatch], b[2][kBatch];
  int lr = 0;                                         // next batch to request: row of this wavefront, batch in it
  uint32_t lb = 0;
  auto request = [&](u32x4 (&ra)[kBatch], u32x4 (&rb)[kBatch]) {
    if (lr >= n_mine) return;
    const long long at = (row0 + wave + (long long)lr * kWaves) * (width / 8);
    const __amdgpu_buffer_rsrc_t sa = __builtin_amdgcn_make_buffer_rsrc((void*)(hin + at), 0, (int)row_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t sb = __builtin_amdgcn_make_buffer_rsrc((void*)(hout + at), 0, (int)row_bytes, 0x00020000);
    const int off = (int)(lb * kStep) + 16 * lane;
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      ra[j] = __builtin_amdgcn_raw_buffer_load_b128(sa, off + 1024 * j, 0, 0);
      rb[j] = __builtin_amdgcn_raw_buffer_load_b128(sb, off + 1024 * j, 0, 0);
    }
    if (++lb == n_batches) { lb = 0; ++lr; }
  };
  double acc = 0.0;
  float d2[2] = {0.f, 0.f}, n2[2] = {0.f, 0.f};
  int cr = 0;                                         // the batch being summed
  uint32_t cb = 0;
  auto consume = [&](const u32x4 (&ra)[kBatch], const u32x4 (&rb)[kBatch]) {
#pragma unroll
    for (int q = 0; q < kBatch; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float a0 = __uint_as_float(ra[q][j] << 16), a1 = __uint_as_float(ra[q][j] & 0xffff0000u);
        const float b0 = __uint_as_float(rb[q][j] << 16), b1 = __uint_as_float(rb[q][j] & 0xffff0000u);
        const float e0 = b0 - a0, e1 = b1 - a1;
        d2[0] = fmaf(e0, e0, d2[0]); d2[1] = fmaf(e1, e1, d2[1]);
        n2[0] = fmaf(a0, a0, n2[0]); n2[1] = fmaf(a1, a1, n2[1]);
      }
    if (++cb < n_batches) return;
    float d = d2[0] + d2[1], n = n2[0] + n2[1];
#pragma unroll
    for (int x = 32; x >= 1; x >>= 1) { d += __shfl_xor(d, x); n += __shfl_xor(n, x); }
    acc += (double)(sqrtf(d) / (sqrtf(n) + eps));
    d2[0] = d2[1] = n2[0] = n2[1] = 0.f;
    cb = 0;
    ++cr;
  };
  request(a[0], b[0]);
  while (cr < n_mine) {
    request(a[1], b[1]);
    consume(a[0], b[0]);
    if (cr >= n_mine) break;
    request(a[0], b[0]);
    consume(a[1], b[1]);
  }
  if (lane == 0) wsum[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kWaves; ++w) s += wsum[w];
    partial[blockIdx.x] = s;
  }
}

__global__ void drift_final_kernel(const double* partial, int n_partial, long long n_tokens, float* out) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n_partial; i += 256) s += partial[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int d = 128; d >= 1; d >>= 1) {
    if ((int)threadIdx.x < d) sh[threadIdx.x] += sh[threadIdx.x + d];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = (float)(sh[0] / (double)n_tokens);
}

}  // namespace

// Partials of workgroups of kRowsPerBlock rows: what a workspace has to hold.
size_t drift_min_ws_bytes(long long n_tokens) {
  const size_t blocks = (size_t)((n_tokens + kRowsPerBlock - 1) / kRowsPerBlock);
  return (blocks * sizeof(double) + 255) & ~(size_t)255;
}
size_t drift_ws_bytes(long long n_tokens) {
  // Up to 8192 rows: one per wavefront, in up to 512 workgroups.  More than 16384: 512 equal shares (shares of 64 rows are a
  // second, nearly empty round on some CUs).  In between one workgroup of 64 rows per CU.  Both kernels, shares of 64 rows / these, inputs
  // from HBM: 1024 x 8192 16.7 / 12.2 us, 2048 x 4096 17.3 / 11.3, 4096 x 4096 27.4 / 16.1, 8192 x 4096 30.7 / 27.0, 20000 x 3584 60.8 / 52.0,
  // 30000 x 8192 167 / 166; in between 512 shares against 64 rows: 12000 x 4096 36.9 / 37.5 (in the memory-side cache 32.2 / 31.2),
  // 16384 x 4096 49.9 / 49.4 (47.1 / 42.6).
  const long long want = n_tokens <= (long long)kResident * kWaves ? (n_tokens + kWaves - 1) / kWaves
                         : n_tokens > (long long)kResident * kRowsPerBlock / 2 ? kResident : 0;
  return std::max(drift_min_ws_bytes(n_tokens), ((size_t)want * sizeof(double) + 255) & ~(size_t)255);
}

hipError_t launch_drift(const void* h_in, const void* h_out, long long n_tokens, int width, float eps, float* out,
                        void* ws, size_t ws_bytes, hipStream_t st) {
  // as many workgroups as the workspace has room for partials, and as there are rows for their wavefronts
  const long long slots = (long long)(std::min(ws_bytes, drift_ws_bytes(n_tokens)) / sizeof(double));
  const int rows = (int)((n_tokens + slots - 1) / slots);
  const int blocks = (int)((n_tokens + rows - 1) / rows);
  auto* kernel = width <= kNarrow ? drift_rows_kernel<1> : drift_rows_kernel<2>;
  kernel<<<blocks, kThreads, 0, st>>>((const u32x4*)h_in, (const u32x4*)h_out, n_tokens, rows, width, eps, (double*)ws);
  drift_final_kernel<<<1, 256, 0, st>>>((const double*)ws, blocks, n_tokens, out);
  return hipGetLastError();
}

}  // namespace tsa
