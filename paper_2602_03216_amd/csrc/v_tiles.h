// Building the tiled V^T that the attention kernels read (layout: tsa_internal.h) from rows of V, gathered through an
// index set or taken in order.
#pragma once

#include "tsa_internal.h"

namespace tsa {

typedef uint32_t __attribute__((ext_vector_type(4), aligned(4))) u32x4_a4;   // rows of index sets start at any multiple of 4 bytes

struct VTiles {
  const __bf16* V;
  __bf16* Vt;                 // [rows][nk_tiles][D][kKeyTile]; NULL: no tiles wanted
  Strides vs;                 // layout of V, in elements
  int rows_per_b;             // tile rows (index sets, or heads) per batch entry
  FastDiv by_b, by_kv;        // batch entry of a tile row; KV head of a tile row of its batch entry
  int nk_tiles, halves;       // tiles per row; halves = D / 64 (1 or 2)
};

// Tiles of the rows that an index set selects: one tile row per set.
inline VTiles v_tiles_of(const Dims& dm, int k_keep, const void* V, void* Vt) {
  VTiles t;
  t.V = (const __bf16*)V; t.Vt = (__bf16*)Vt; t.vs = dm.kv;
  t.rows_per_b = dm.group_mode ? dm.Hkv : dm.Hq;
  t.by_b = FastDiv(t.rows_per_b, (uint64_t)dm.B * t.rows_per_b);
  t.by_kv = FastDiv(dm.group_mode ? 1 : dm.Hq / dm.Hkv, t.rows_per_b);
  t.nk_tiles = (k_keep + kKeyTile - 1) / kKeyTile;
  t.halves = dm.d / 64;
  return t;
}

constexpr int kVtLds = 8192;   // bytes of LDS a wavefront uses in v_half_tile

// One wavefront builds 64 keys x 64 columns of a tile.  A lane loads 16 bytes (8 columns) of 8 consecutive keys (8 adjacent
// lanes cover 128 bytes of a row) and transposes its 8 x 8 block with 32 byte permutes; the blocks change places through
// 8 KiB of LDS of the wavefront's own, so that the stores write whole 128-byte columns of the tile (block o of
// column d sits at position o ^ (d / 8): free of bank conflicts, and a read still finds one whole column).
// Keys past `n` are zeros.  idx NULL: key r is row r.
__device__ __forceinline__ void v_half_tile(const VTiles& a, long long row, int tile, int half, const int32_t* idx, int n, int lane,
                                            char* lds) {
  const int col = lane & 7, oct = lane >> 3, r0 = tile * kKeyTile + 8 * oct;
  const int b = (int)a.by_b.div((uint32_t)row), kv = (int)a.by_kv.div((uint32_t)row - b * a.rows_per_b);
  const __bf16* head = a.V + a.vs.head(b, kv) + 64 * half + 8 * col;
  const bool whole = tile * kKeyTile + kKeyTile <= n;      // the same for the whole wavefront
  int tok[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) tok[j] = whole ? r0 + j : min(r0 + j, n - 1);
  if (idx && whole) {
    *(u32x4_a4*)&tok[0] = *(const u32x4_a4*)(idx + r0);
    *(u32x4_a4*)&tok[4] = *(const u32x4_a4*)(idx + r0 + 4);
  } else if (idx) {
#pragma unroll
    for (int j = 0; j < 8; ++j) tok[j] = idx[tok[j]];
  }
  u32x4 v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = *(const u32x4*)(head + tok[j] * a.vs.l);
  if (!whole) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (r0 + j >= n) v[j] = u32x4{0u, 0u, 0u, 0u};
  }
  char* put = lds + col * 1024 + ((oct ^ col) << 4);       // 128 bytes per column
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    u32x4 even, odd;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      even[i] = __builtin_amdgcn_perm(v[2 * i + 1][w], v[2 * i][w], 0x05040100u);
      odd[i] = __builtin_amdgcn_perm(v[2 * i + 1][w], v[2 * i][w], 0x07060302u);
    }
    *(u32x4*)(put + (2 * w) * 128) = even;
    *(u32x4*)(put + (2 * w + 1) * 128) = odd;
  }
  __builtin_amdgcn_wave_barrier();                         // LDS accesses of one wavefront complete in order
  __bf16* dst = a.Vt + ((row * a.nk_tiles + tile) * a.halves + half) * (64LL * kKeyTile);
#pragma unroll
  for (int i = 0; i < 8; ++i)
    *(u32x4*)(dst + 512 * i + (oct * kKeyTile) + 8 * (col ^ i)) = *(const u32x4*)(lds + 1024 * i + 16 * lane);
  __builtin_amdgcn_wave_barrier();
}

}  // namespace tsa
